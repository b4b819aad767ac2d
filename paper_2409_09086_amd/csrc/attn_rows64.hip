// Attention of up to a few hundred query rows per kv-head on bf16 MFMA for gfx950, head_dim 128: attn_rows
// (attn_rows.hip) with 64 query rows per workgroup.
//
// A workgroup of attn_rows takes the 128 KB of K and V of a pass of 256 keys at about 60 bytes a cycle, the rate of a CU's first
// level (1.12 us with 16 rows, 1.33 with 32; measured bytes into the CUs: 205 MB in a launch of 17 us by 192 workgroups), and
// its products take half of that.  Twice the rows per byte need twice the output accumulators (128 registers of
// a wavefront's 256, eight wavefronts on a CU); the query fragments then have no place in registers and are read from
// LDS, which all wavefronts share, beside the K fragments.  K and V have one buffer each per wavefront: a run's K
// buffer is refilled as soon as S has its fragments, its V buffer as soon as O has.  A pass of 256 keys takes 1.9 us, two
// workgroups of 32 rows 2.7.  No pipe is full in it: products 1.0 us (matrix pipes busy 30 % of the SIMD-cycles of a launch of
// 32 us, 32 x 128 heads, 512 rows on 2560 keys), LDS reads 0.7 (indexed reads 21 % of its CU-cycles, few conflicts),
// the bytes that come in 1.1; a wavefront goes through the three one after the other, and two share a SIMD.
#include "append_body.h"
#include "attn_rows.h"

namespace infmllm {

namespace {

template <int D>
struct Rows64Cfg {
    static constexpr int ROWB = D * 2, RUN = RW_RUN * ROWB, STAGE = 2 * RUN;
    static constexpr int NS = D / 32, NC = D / 16, NL = RUN / 1024, RPL = 1024 / ROWB;
    static constexpr int NX = 4, ROWS = 16 * NX;               // blocks of sixteen query rows
    static constexpr int QL = ROWS * ROWB / 1024 / RW_NW;      // direct loads of queries per wavefront
    static constexpr int MC = D / 2;                           // columns merged at once: a wavefront's share fits its stage
    static_assert(ROWS * MC * 4 <= STAGE, "the merge reuses the buffers of the tiles");
};

// Eight columns of a merged row (see leave_row).
template <int D>
__device__ __forceinline__ void leave_row8(const RowsArgs& a, int h, int sp, int rho, int d, float2 ml, f32x4 lo, f32x4 hi)
{
    if (a.nsplit == 1) {
        const int tok = rows_token(a, rho), gq = h * a.G + rho - tok * a.G;
        const float inv = 1.0f / ml.y;
        bf16x8 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) { w[e] = (__bf16)(lo[e] * inv); w[4 + e] = (__bf16)(hi[e] * inv); }
        *(bf16x8*)(a.out + ((size_t)tok * a.Hq + gq) * D + d) = w;
        if (a.lse && d == 0) a.lse[(size_t)gq * a.max_chunk + tok] = ml.x + __builtin_log2f(ml.y);
        return;
    }
    const size_t at = ((size_t)h * a.L * a.G + rho) * a.nsplit + sp;
    float* po = a.part_o + at * D + d;
    *(f32x4*)po = lo;
    *(f32x4*)(po + 4) = hi;
    if (d == 0) a.part_ml[at] = ml;
}

// The attention has no register left for a share of the append: the first half of the row groups of a launch
// with APPEND are workgroups that append and nothing else, which costs less than a launch of its own (us, 32 x 128 heads, 400 rows on 3500 keys / 32 on 8,
// 300 on 2000: shares after the loop, with a spilled register whose reload drained the loads in flight in every pass, 47.2 /
// 31.9; a launch of its own 48.2 / 34.0; workgroups of its own 45.7 / 30.0).
template <int D, bool APPEND>
__global__ void __launch_bounds__(RW_NT)
attn_rows64_kernel(RowsArgs a, AppendJob ap)
{
    using C = Rows64Cfg<D>;
    __shared__ __attribute__((aligned(1024))) char smem[RW_NW * C::STAGE];
    __shared__ __attribute__((aligned(1024))) char qmem[C::ROWS * C::ROWB];
    __shared__ __attribute__((aligned(16))) float s_m[C::ROWS][RW_NW], s_l[C::ROWS][RW_NW];
    __shared__ float2 s_tot[C::ROWS];                          // reference and sum of the merged rows

    const int sp = blockIdx.x, h = blockIdx.y;                 // piece, kv-head
    if constexpr (APPEND)
        if (blockIdx.z < gridDim.z / 2) {
            append_share(ap, sp + gridDim.x * (h + gridDim.y * blockIdx.z), gridDim.x * gridDim.y * (gridDim.z / 2), threadIdx.x, RW_NT);
            return;
        }
    const int rg = APPEND ? blockIdx.z - gridDim.z / 2 : blockIdx.z;               // row group (see attn_rows_kernel)
    const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.L * a.G, row0 = rg * C::ROWS, t = a.t;
    const int first_lim = t + rows_token(a, row0);             // last key the group's first row sees
    const int n_end = t + rows_token(a, min(row0 + C::ROWS, M) - 1) + 1;
    const int k_end = min((sp + 1) * a.ks, n_end);

    RunLoader<uint16_t, D, RW_RUN> runs(a, h, lane);
    char* const mine = smem + wave * C::STAGE;
    // queries: row r of the group in LDS row r, swizzled like K
#pragma unroll
    for (int u = 0; u < C::QL; ++u) {
        const int r = (wave * C::QL + u) * C::RPL + runs.lrow, rho = min(row0 + r, M - 1), tok = rows_token(a, rho);
        const uint16_t* src = a.q + ((size_t)tok * a.Hq + h * a.G + (rho - tok * a.G)) * D + (runs.lpos ^ swz_k<D>(r)) * 8;
        __builtin_amdgcn_global_load_lds((global_void*)src, (lds_void*)(qmem + (wave * C::QL + u) * 1024), 16, 0, 0);
    }
    const int k_first = sp * a.ks + wave * RW_RUN;
    const int np = k_end > k_first ? (k_end - k_first + RW_PASS - 1) / RW_PASS : 0;
    if (np > 0) {
        runs.template load<true, false>(k_first, mine);
        runs.template load<false, true>(k_first, mine);
        wait_loads<2 * C::NL>();                               // the queries have landed ...
    } else {
        wait_loads<0>();
    }

    f32x4 o[C::NX][C::NC];
    float m_ref[C::NX], m_use[C::NX], lsum[C::NX];
#pragma unroll
    for (int x = 0; x < C::NX; ++x) {
#pragma unroll
        for (int b = 0; b < C::NC; ++b) o[x][b] = f32x4{0.f, 0.f, 0.f, 0.f};
        m_ref[x] = -__builtin_inff(); m_use[x] = 0.f; lsum[x] = 0.f;
    }
    // Fragment addresses: K and Q as in attn_rows (lane (row c16, group g4), piece 4s + g4), V by the transpose read.  The
    // step or column block only flips address bits that are clear in the rest, so one address each is kept, in a form
    // that the compiler does not see through (it would keep all sixteen, and run out of registers); so is the lane's slot of a load.
    uint32_t k0addr, q0addr, v0addr;
    {
        const uint32_t base = (uint32_t)(uintptr_t)(lds_void*)mine, qbase = (uint32_t)(uintptr_t)(lds_void*)qmem;
        const int vkey = 4 * g4 + (c16 >> 2), q4 = c16 & 3;
        const uint32_t rel = c16 * C::ROWB + ((g4 ^ swz_k<D>(c16)) * 16);
        k0addr = base + rel;
        q0addr = qbase + rel;
        v0addr = base + C::RUN + vkey * C::ROWB + (((q4 >> 1) ^ swz_v<D>(vkey)) * 16) + 8 * (q4 & 1);
    }
    __builtin_amdgcn_s_barrier();                              // ... everybody's

    for (int p = 0; p < np; ++p) {
        const int k0 = k_first + p * RW_PASS;
        const bool more = p + 1 < np;
        // The SIMD prefers the older of its two wavefronts, which then leaves the other one 4 us of a launch of 33 to itself (7 of
        // 50): they take turns of four passes (one pass 32.8, two 32.5, four 32.3 us against 33.5; 50.1, 49.1, 48.7 against 50.5).
        if (((p >> 2) ^ (wave >> 2)) & 1) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
        asm volatile("" : "+v"(k0addr), "+v"(q0addr), "+v"(v0addr), "+v"(runs.lpos));
        wait_loads<C::NL>();                                   // this run's K has landed, its V may be on its way
        // ---- S^T = K.Q^T, the fragments of a step requested a step ahead
        bf16x8 kf[2][2], qf[2][C::NX];
        f32x4 S[C::NX][2];
        auto request = [&](auto step) {
            constexpr int s = decltype(step)::value, b = s & 1;
            const uint32_t ka = k0addr ^ (64 * s), qa = q0addr ^ (64 * s);
            kf[b][0] = rw_read_b128<0>(ka);
            kf[b][1] = rw_read_b128<16 * C::ROWB>(ka);
            qf[b][0] = rw_read_b128<0>(qa);
            qf[b][1] = rw_read_b128<16 * C::ROWB>(qa);
            qf[b][2] = rw_read_b128<32 * C::ROWB>(qa);
            qf[b][3] = rw_read_b128<48 * C::ROWB>(qa);
        };
        request(std::integral_constant<int, 0>{});
        static_for<0, C::NS>([&](auto step) {
            constexpr int s = decltype(step)::value, b = s & 1;
            if constexpr (s + 1 < C::NS) request(std::integral_constant<int, s + 1>{});
            asm volatile("s_waitcnt lgkmcnt(%6)"
                         : "+v"(kf[b][0]), "+v"(kf[b][1]), "+v"(qf[b][0]), "+v"(qf[b][1]), "+v"(qf[b][2]), "+v"(qf[b][3])
                         : "n"(s + 1 < C::NS ? 6 : 0));
            if constexpr (s + 1 == C::NS)
                if (more) runs.template load<true, false>(k0 + RW_PASS, mine);
#pragma unroll
            for (int x = 0; x < C::NX; ++x)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
                    S[x][kb] = mfma16(kf[b][kb], qf[b][x], s == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : S[x][kb]);
        });
        if (more) wait_loads<C::NL>();                         // this run's V has landed, the next one's K may be on its way
        else wait_loads<0>();
        // ---- V fragments of the lower columns, behind them mask and softmax
        constexpr int HC = C::NC / 2;
        bf16x4 vlo[2][HC], vhi[2][HC];
        auto request_v = [&](auto half) {
            constexpr int hf = decltype(half)::value;
#pragma unroll
            for (int b = 0; b < HC; ++b) {
                const uint32_t va = v0addr ^ (32 * (hf * HC + b));
                vlo[hf][b] = rw_read_tr16<0>(va);
                vhi[hf][b] = rw_read_tr16<16 * C::ROWB>(va);
            }
        };
        auto await_v = [&](auto half) {
            constexpr int hf = decltype(half)::value;
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(vlo[hf][0]), "+v"(vhi[hf][0]), "+v"(vlo[hf][1]), "+v"(vhi[hf][1]));
            if constexpr (HC == 4) asm volatile("" : "+v"(vlo[hf][2]), "+v"(vhi[hf][2]), "+v"(vlo[hf][3]), "+v"(vhi[hf][3]));
        };
        using I0 = std::integral_constant<int, 0>;
        using I1 = std::integral_constant<int, 1>;
        bf16x8 pf[C::NX];
        const bool masked = k0 + RW_RUN - 1 > first_lim;
#pragma unroll
        for (int x = 0; x < C::NX; ++x) {
            if (masked) {
                const int lim = t + rows_token(a, min(row0 + 16 * x + c16, M - 1));
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (k0 + 16 * kb + 4 * g4 + i > lim) S[x][kb][i] = -__builtin_inff();
            }
            float mx = fmaxf(fmaxf(fmaxf(S[x][0][0], S[x][0][1]), fmaxf(S[x][0][2], S[x][0][3])),
                             fmaxf(fmaxf(S[x][1][0], S[x][1][1]), fmaxf(S[x][1][2], S[x][1][3])));
            mx = groups_max(mx) * a.c;
            if (__any(mx > m_ref[x] + RESCALE_TAU)) {
                const float m_new = fmaxf(m_ref[x], mx);
                const float mu = (m_new == -__builtin_inff()) ? 0.f : m_new;
                const float alpha = fast_exp2(m_ref[x] - mu);  // m_ref = -inf gives 0
                m_ref[x] = m_new;
                m_use[x] = mu;
                lsum[x] *= alpha;
#pragma unroll
                for (int b = 0; b < C::NC; ++b) o[x][b] *= alpha;
            }
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float w = fast_exp2(__builtin_fmaf(S[x][kb][i], a.c, -m_use[x]));
                    lsum[x] += w;
                    pf[x][4 * kb + i] = (__bf16)w;
                }
        }
        // ---- O^T += V^T.P^T
        request_v(I0{});
        await_v(I0{});
        request_v(I1{});
        auto products = [&](auto half) {
            constexpr int hf = decltype(half)::value;
#pragma unroll
            for (int b = 0; b < HC; ++b) {
                const bf16x8 vf = __builtin_shufflevector(vlo[hf][b], vhi[hf][b], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                for (int x = 0; x < C::NX; ++x) o[x][hf * HC + b] = mfma16(vf, pf[x], o[x][hf * HC + b]);
            }
        };
        products(I0{});
        await_v(I1{});
        if (more) runs.template load<false, true>(k0 + RW_PASS, mine);
        products(I1{});
    }

    // ---- merge the wavefronts, half of the columns at a time: the tree of add_tree, whose products every wavefront takes
    // in its registers, so that the thread that adds eight columns of a row only adds.  Bound by 512 KB through the LDS,
    // 2 us; with a weight for each share of every four columns and two rounds of items per half a whole step took 58.6 us
    // instead of 58.1 (32 x 128 heads, 512 rows on 2560 keys), 95.1 instead of 94.4 (32 on 8, 512 rows on 4608 keys).
    int me = 64 * wave + 16 * g4 + c16;                        // tid, which needs no register in the loop
    asm volatile("" : "+v"(me));                               // nothing of this is made ready before the loop
#pragma unroll
    for (int x = 0; x < C::NX; ++x) {
        const float l = groups_sum(lsum[x]);
        if (g4 == 0) { s_m[16 * x + c16][wave] = m_ref[x]; s_l[16 * x + c16][wave] = l; }
    }
    __syncthreads();
    auto row_max = [&](int r) -> float {
        const f32x4 a4 = *(const f32x4*)s_m[r], b4 = *(const f32x4*)(s_m[r] + 4);
        return fmaxf(fmaxf(fmaxf(a4[0], a4[1]), fmaxf(a4[2], a4[3])), fmaxf(fmaxf(b4[0], b4[1]), fmaxf(b4[2], b4[3])));
    };
    auto finite = [](float m) -> float { return m == -__builtin_inff() ? 0.f : m; };
#pragma unroll
    for (int x = 0; x < C::NX; ++x) {
        const float w = fast_exp2(m_ref[x] - finite(row_max(16 * x + c16)));
#pragma unroll
        for (int b = 0; b < C::NC; ++b) o[x][b] *= w;
    }
    if (me < C::ROWS) {
#pragma clang fp contract(off)
        const float m = row_max(me), mz = finite(m);
        float wl[RW_NW];
#pragma unroll
        for (int w = 0; w < RW_NW; ++w) wl[w] = fast_exp2(s_m[me][w] - mz) * s_l[me][w];
        s_tot[me] = float2{m, ((wl[0] + wl[1]) + (wl[2] + wl[3])) + ((wl[4] + wl[5]) + (wl[6] + wl[7]))};
    }
    auto merged = [&](int w, int r, int p) -> char* {
        return smem + w * C::STAGE + r * (C::MC * 4) + ((p ^ ((r ^ w) & 7)) * 16);
    };
    static_assert(C::ROWS * C::MC == 8 * RW_NT, "eight columns of a row per thread");
    const int r = me / (C::MC / 8), rho = row0 + r;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
        if (hf > 0) __syncthreads();
        constexpr int CBH = C::NC / 2;
#pragma unroll
        for (int x = 0; x < C::NX; ++x)
#pragma unroll
            for (int b = 0; b < CBH; ++b) *(f32x4*)merged(wave, 16 * x + c16, 4 * b + g4) = o[x][hf * CBH + b];
        __syncthreads();
        if (rho < M) {
            const int p0 = 2 * (me % (C::MC / 8)), d = hf * C::MC + 4 * p0;
            f32x4 sum[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                f32x4 s[RW_NW];
#pragma unroll
                for (int w = 0; w < RW_NW; ++w) s[w] = *(const f32x4*)merged(w, r, p0 + u);
                sum[u] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
            }
            leave_row8<D>(a, h, sp, rho, d, s_tot[r], sum[0], sum[1]);
        }
    }
}

}  // namespace

void launch_rows64(const RowsArgs& a, const AppendJob& ap, hipStream_t st)
{
    const unsigned groups = (unsigned)((a.L * a.G + Rows64Cfg<128>::ROWS - 1) / Rows64Cfg<128>::ROWS);
    const dim3 grid((unsigned)a.nsplit, (unsigned)a.Hkv, groups), with_append((unsigned)a.nsplit, (unsigned)a.Hkv, 2 * groups);
    if (ap.k) hipLaunchKernelGGL((attn_rows64_kernel<128, true>), with_append, dim3(RW_NT), 0, st, a, ap);
    else hipLaunchKernelGGL((attn_rows64_kernel<128, false>), grid, dim3(RW_NT), 0, st, a, ap);
}

}  // namespace infmllm
