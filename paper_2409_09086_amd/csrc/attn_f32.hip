// Chunk attention and column scoring of fp32 streams on the fp32 matrix cores of gfx950 (v_mfma_f32_16x16x4_f32: fp32
// products and sums, 157 TFLOP/s).
//
//   attn_f32   row-stationary, as attn_rows (attn_rows.hip): a workgroup owns sixteen query rows (rows of a kv-head
//              numbered token * G + head) and a piece of the keys, each of its eight wavefronts every eighth run of 16 keys
//              through LDS buffers of its own, no barrier in the loop.  A lane's 16-byte reads of K and Q feed four
//              products: step e of piece j contracts head dimensions {16j + 4g + e} of lane group g, on both operands.
//              The weights of a run are the B operand of O^T += V^T.P^T as they stand (step i contracts keys 4g + i), and
//              a lane's 32 bytes of a V row are its operands of D/16 column blocks (block b is columns D/16 * c + b).
//              The matrix cores take 2048 cycles per run and wavefront at head_dim 128: busy 45 % of the SIMD-cycles of
//              a launch of 256 rows on 1280 keys, 8 x 128 heads (21 us, prologue, passes that only some wavefronts have and the
//              merge of the wavefronts included), 32 % where the cache is filling.
//   score_f32  column-stationary, as score_kernel (attn_mfma.hip): a wavefront keeps sixteen key columns as B operands,
//              the scored query rows go through LDS sixteen at a time, and S = Q.K^T leaves a column to a lane, so that a
//              column's weights are added without leaving it.  Where the columns do not fill the chip, the scored
//              rows are shared out over several workgroups, whose sums the last to finish adds in order.
//
// The kernels these replace kept K rows in registers and one query row per workgroup: 100 us against 13 for the attention of
// 256 rows over 1024 keys, 8 heads of 128.
#include <algorithm>

#include "append_body.h"
#include "attn_rows.h"

namespace infmllm {

namespace {

constexpr int F32_RUN = 16, F32_PASS = RW_NW * F32_RUN;        // keys of a wavefront's run, of a workgroup's pass
constexpr float F32_TAU = 5.5f;                                // the softmax reference moves when a logit exceeds it by this

__device__ __forceinline__ f32x4 mfma16_f32(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <int D, bool APPEND>
__global__ void __launch_bounds__(RW_NT)
attn_f32_kernel(RowsArgsT<float> a, AppendJob ap)
{
    typedef RunLoader<float, D, F32_RUN> Runs;
    constexpr int ROWB = Runs::ROWB, RUN = Runs::RUN, STAGE = 2 * RUN;
    constexpr int NJ = D / 16;                                 // 16-byte pieces of a row per lane group; also column blocks
    constexpr int VW = D / 16, VP = VW / 4;                    // columns, 16-byte pieces of a V row per lane
    __shared__ __attribute__((aligned(1024))) char smem[RW_NW * STAGE];
    __shared__ float s_m[RW_NW][16], s_l[RW_NW][16];

    const int sp = blockIdx.x, h = blockIdx.y, rg = a.rg0 + blockIdx.z;    // piece, kv-head, row group
    const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.L * a.G, row0 = 16 * rg, t = a.t;
    const int first_lim = t + rows_token(a, row0);             // last key the group's first row sees
    const int n_end = t + rows_token(a, min(row0 + 16, M) - 1) + 1;
    const int k_end = min((sp + 1) * a.ks, n_end);

    const Runs runs(a, h, lane);
    char* const mine = smem + wave * STAGE;
    const int k_first = sp * a.ks + wave * F32_RUN;
    const int np = k_end > k_first ? (k_end - k_first + F32_PASS - 1) / F32_PASS : 0;
    if (np > 0) runs.template load<true, true>(k_first, mine);
    f32x4 qf[NJ];                                              // lane (row c16, group g4): Q[row][16j + 4 g4 .. +4)
    const int my_rho = min(row0 + c16, M - 1), my_tok = rows_token(a, my_rho), lim = t + my_tok;
    {
        const float* qp = a.q + ((size_t)my_tok * a.Hq + h * a.G + (my_rho - my_tok * a.G)) * D + 4 * g4;
#pragma unroll
        for (int j = 0; j < NJ; ++j) qf[j] = *(const f32x4*)(qp + 16 * j);
    }
    if constexpr (APPEND)
        append_share(ap, sp + gridDim.x * (h + gridDim.y * blockIdx.z), gridDim.x * gridDim.y * gridDim.z, tid, RW_NT);
    f32x4 o[NJ];                                               // block b: lane (row c16, group g4) holds columns VW (4 g4 + i) + b
    float m_ref, m_use, lsum;

    const uint32_t base = (uint32_t)(uintptr_t)(lds_void*)mine;
    uint32_t kaddr[NJ], vaddr[VP];                             // K: row c16, piece 4j + g4; V: row 4 g4 (+ i), pieces VP c16 + x
#pragma unroll
    for (int j = 0; j < NJ; ++j) kaddr[j] = base + c16 * ROWB + Runs::Swz::k(c16, 4 * j + g4) * 16;
#pragma unroll
    for (int x = 0; x < VP; ++x) vaddr[x] = base + RUN + 4 * g4 * ROWB + Runs::Swz::v(0, VP * c16 + x) * 16;

    // A hidden key's weight is 0, but 0 times a value that is not finite is NaN, in every row of the group.  A wavefront
    // that finds its accumulators not finite goes through its keys again (CAREFUL), the rows that see the same number of a run's
    // keys at a time, hidden values replaced by 0.
    auto sweep = [&](auto careful) __attribute__((always_inline)) {
        constexpr bool CAREFUL = decltype(careful)::value;
#pragma unroll
        for (int b = 0; b < NJ; ++b) o[b] = f32x4{0.f, 0.f, 0.f, 0.f};
        m_ref = -__builtin_inff(); m_use = 0.f; lsum = 0.f;
        for (int p = 0; p < np; ++p) {
            const int k0 = k_first + p * F32_PASS;
            wait_loads<0>();
            f32x4 kf[NJ], vf[4][VP];
#pragma unroll
            for (int j = 0; j < NJ; ++j) kf[j] = rw_read_f32x4<0, CAREFUL>(kaddr[j]);
            static_for<0, 4>([&](auto I) {
                constexpr int i = decltype(I)::value;
#pragma unroll
                for (int x = 0; x < VP; ++x) vf[i][x] = rw_read_f32x4<i * ROWB, CAREFUL>(vaddr[x]);
            });
            // reads return in order: K has arrived when only the V reads are outstanding
            asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(kf[0]), "+v"(kf[1]), "+v"(kf[2]), "+v"(kf[3]) : "n"(4 * VP));
            if constexpr (NJ == 8) asm volatile("" : "+v"(kf[4]), "+v"(kf[5]), "+v"(kf[6]), "+v"(kf[7]));
            // ---- S^T = K.Q^T, in two chains
            f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NJ; j += 2)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    s0 = mfma16_f32(kf[j][e], qf[j][e], s0);
                    s1 = mfma16_f32(kf[j + 1][e], qf[j + 1][e], s1);
                }
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(vf[0][0]), "+v"(vf[1][0]), "+v"(vf[2][0]), "+v"(vf[3][0]));
            if constexpr (VP == 2) asm volatile("" : "+v"(vf[0][VP - 1]), "+v"(vf[1][VP - 1]), "+v"(vf[2][VP - 1]), "+v"(vf[3][VP - 1]));
            if (p + 1 < np) runs.template load<true, true>(k0 + F32_PASS, mine);   // this stage has been read
            // ---- mask, softmax
            float s[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = (s0[i] + s1[i]) * a.c;
            if (k0 + F32_RUN - 1 > first_lim) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (k0 + 4 * g4 + i > lim) s[i] = -__builtin_inff();
            }
            const float mx = groups_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
            if (__any(mx > m_ref + F32_TAU)) {
                const float m_new = fmaxf(m_ref, mx);
                const float mu = (m_new == -__builtin_inff()) ? 0.f : m_new;
                const float alpha = expf(m_ref - mu);              // m_ref = -inf gives 0
                m_ref = m_new;
                m_use = mu;
                lsum *= alpha;
#pragma unroll
                for (int b = 0; b < NJ; ++b) o[b] *= alpha;
            }
            float w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                w[i] = expf(s[i] - m_use);
                lsum += w[i];
            }
            // ---- O^T += V^T.P^T
            if constexpr (CAREFUL) {
                const int last = max(min(lim - k0, F32_RUN - 1), -1);      // last key of the run that the row sees, -1: none
#pragma nounroll
                for (int end = 0; end < F32_RUN; ++end) {
                    if (!__any(last == end)) continue;
#pragma unroll
                    for (int b = 0; b < NJ; ++b) {
                        f32x4 sum = o[b];
#pragma unroll
                        for (int i = 0; i < 4; ++i) sum = mfma16_f32(4 * g4 + i > end ? 0.f : vf[i][b / 4][b % 4], w[i], sum);
                        if (last == end) o[b] = sum;
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int b = 0; b < NJ; ++b) o[b] = mfma16_f32(vf[i][b / 4][b % 4], w[i], o[b]);
            }
        }
    };
    sweep(std::false_type{});
    float z = 0.f;
#pragma unroll
    for (int b = 0; b < NJ; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) z = __builtin_fmaf(o[b][i], 0.f, z);
    if (__builtin_expect(__any(z != 0.f), 0)) {
        runs.template load<true, true>(k_first, mine);         // np > 0
        sweep(std::true_type{});
    }

    // ---- merge the wavefronts (see attn_rows_kernel)
    {
        const float l = groups_sum(lsum);
        if (g4 == 0) { s_m[wave][c16] = m_ref; s_l[wave][c16] = l; }
    }
    auto merged = [&](int w, int r, int p) -> char* { return smem + w * STAGE + r * ROWB + ((p ^ ((r ^ w) & 7)) * 16); };
    const int rows = min(16, M - row0);
    if (c16 < rows) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int x = 0; x < VP; ++x)
                *(f32x4*)merged(wave, c16, VP * (4 * g4 + i) + x) = f32x4{o[4 * x][i], o[4 * x + 1][i], o[4 * x + 2][i], o[4 * x + 3][i]};
    }
    __syncthreads();
    for (int x = tid; x < rows * (D / 4); x += RW_NT) {
        const int r = x / (D / 4), d4 = x % (D / 4);
        PieceSumT<true> ps[RW_NW];
#pragma unroll
        for (int w = 0; w < RW_NW; ++w) ps[w] = PieceSumT<true>{s_m[w][r], s_l[w][r], *(const f32x4*)merged(w, r, d4)};
        leave_row<D>(a, h, sp, row0 + r, 4 * d4, add_tree(ps));
    }
}

// A column is a physical cache row (below tc; stream-order index rank[col]) or a chunk row read in place, as in score_kernel.
// 128 columns per workgroup, sixteen per wavefront; slice rs of rsplit of the group's scored rows.
template <int D>
__global__ void __launch_bounds__(RW_NT)
score_f32_kernel(const float* __restrict__ q, const float* __restrict__ K, const float* __restrict__ kc, int tc,
                 const float* __restrict__ lse, const float* __restrict__ carry, const int32_t* __restrict__ rank,
                 float* __restrict__ Wb, int L, int lq, int Hq, int Hkv, int G, int cap, int max_chunk, int cnd, int ncol,
                 float scale, float dstep /* b / c, Alg. 1 l.2 */, float* __restrict__ spart)
{
    constexpr int NJ = D / 16, QP = D * 4 + 16;                // pitch of a staged query row: sixteen rows, distinct banks
    constexpr int CPR = D / 4;                                 // 16-byte pieces of a query row
    __shared__ __attribute__((aligned(16))) char qs[2][16 * QP];
    __shared__ __attribute__((aligned(16))) float ls[2][16];
    __shared__ int s_ticket;

    const int bx = blockIdx.x, h = blockIdx.y, rs = blockIdx.z, nxb = gridDim.x, rsplit = gridDim.z;
    const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, g4 = lane >> 4, wave = tid >> 6;
    const int col = bx * 128 + wave * 16 + c16;
    f32x4 kf[NJ];                                              // lane (column c16, group g4): K[col][16j + 4 g4 .. +4)
    {
        const int cc = col < ncol ? col : 0;
        const float* kp = (cc < tc ? K + ((size_t)h * cap + cc) * D : kc + ((size_t)(cc - tc) * Hkv + h) * D) + 4 * g4;
#pragma unroll
        for (int j = 0; j < NJ; ++j) kf[j] = *(const f32x4*)(kp + 16 * j);
    }
    // blocks of sixteen scored rows, head after head of the group; this slice's share of them
    const int bph = (lq + 15) / 16, total = G * bph;
    const int b0 = (int)((long)rs * total / rsplit), b1 = (int)((long)(rs + 1) * total / rsplit);
    const int sr = tid / CPR, sc = tid % CPR;                  // this thread's row and piece of a staged block (if it has one)
    const bool stages = sr < 16;
    f32x4 nq = {0.f, 0.f, 0.f, 0.f};
    float nl = 0.f;
    auto request = [&](int b) {
        const int g = h * G + b / bph, i0 = L - lq + (b % bph) * 16;
        if (stages) nq = *(const f32x4*)(q + ((size_t)min(i0 + sr, L - 1) * Hq + g) * D + 4 * sc);
        if (tid < 16) nl = i0 + tid < L ? lse[(size_t)g * max_chunk + i0 + tid] : __builtin_inff();   // no row: weight 0
    };
    auto publish = [&](int buf) {
        if (stages) *(f32x4*)(qs[buf] + sr * QP + sc * 16) = nq;
        if (tid < 16) ls[buf][tid] = nl;
    };
    f32x4 part = {0.f, 0.f, 0.f, 0.f};
    if (b0 < b1) { request(b0); publish(0); }
    for (int b = b0; b < b1; ++b) {
        const int buf = (b - b0) & 1;
        if (b + 1 < b1) request(b + 1);
        __syncthreads();                                       // block b is complete, the other buffer no longer read
        const char* qp = qs[buf] + c16 * QP + 16 * g4;
        f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NJ; j += 2) {
            const f32x4 qa = *(const f32x4*)(qp + 64 * j), qb = *(const f32x4*)(qp + 64 * (j + 1));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                s0 = mfma16_f32(qa[e], kf[j][e], s0);
                s1 = mfma16_f32(qb[e], kf[j + 1][e], s1);
            }
        }
        const f32x4 lv = *(const f32x4*)(ls[buf] + 4 * g4);    // lane (column c16, group g4) holds rows 4 g4 + i
#pragma unroll
        for (int i = 0; i < 4; ++i) part[i] += expf((s0[i] + s1[i]) * scale - lv[i]);
        if (b + 1 < b1) publish(buf ^ 1);
    }
    float sum = groups_sum((part[0] + part[1]) + (part[2] + part[3]));
    float* my_part = nullptr;
    if (rsplit > 1) {
        // as in score_kernel: the sums go through to memory, the workgroup that arrives last adds the slices in order
        my_part = spart + ((size_t)(h * rsplit + rs) * nxb + bx) * 128 + wave * 16 + c16;
        if (g4 == 0) __hip_atomic_store(my_part, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int* arrived = (int*)(spart + (size_t)SCORE_SPLIT_WGS * 256) + h * nxb + bx;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) s_ticket = __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (s_ticket != rsplit - 1) return;
        if (tid == 0) __hip_atomic_store(arrived, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch
    }
    if (g4 != 0) return;
    const int j = col < tc ? (col < ncol ? rank[(size_t)h * cap + col] : cnd) : col;   // stream-order index
    if (j >= cnd) return;
    if (rsplit > 1) {
        sum = 0.f;
        for (int x = 0; x < rsplit; ++x)
            sum += __hip_atomic_load(my_part + (size_t)(x - rs) * nxb * 128, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const float S = lq > 0 ? sum / (float)(G * lq) : 0.f;      // Alg. 1 l.1, pooled over the group
    float w = S - (float)(cnd - 1 - j) * dstep;                // Alg. 1 l.3-4
    if (carry) {                                               // cumulative policy: total so far, no bias
        const float x = col < tc ? carry[(size_t)h * cap + col] : 0.f;
        w = S + (x < __builtin_inff() ? x : 0.f);              // +inf marks a row never ranked
    }
    Wb[(size_t)h * cap + j] = w;
}

}  // namespace

hipError_t launch_attn_f32(const Geometry& g, const CacheView& c, const KeySource& ks, const void* q, int t, int L,
                           void* out, float* lse, const RowsScratch& sc, const AppendJob& ap, hipStream_t st)
{
    RowsArgsT<float> a{};
    a.q = (const float*)q; a.K = (float*)c.K; a.V = (float*)c.V; a.kc = (const float*)ks.k; a.vc = (const float*)ks.v;
    a.out = (float*)out; a.lse = lse; a.part_o = sc.o; a.part_ml = sc.ml;
    a.t = t; a.L = L; a.tc = ks.rows; a.Hq = g.Hq; a.Hkv = g.Hkv; a.G = g.G; a.cap = g.cap; a.max_chunk = g.max_chunk;
    a.inv_g = rows_inv_g(L, g.G);
    a.c = (float)g.scale;
    // Pieces: as many as keep the chip's 256 CUs busy, of at least two passes.  Attention of evicting steps, us, with pieces of at
    // least one pass / two / three / four: 8 x 128 heads, 256 rows on 1280 keys 26.2 / 25.4 / 25.1 / 24.9, 64 on 664 15.5 /
    // 18.9 / 21.7 / 22.0, 16 on 3016 16.6 / 18.6 / 20.5 / 24.5; 8 on 2, 64 on 1564 17.6 / 18.2 / 19.4 / 21.6; 4 x 64 heads, 64 on
    // 1064 12.3 / 12.7 / 15.5 / 15.4, but 64 on 320 11.2 / 10.4 / 10.2 / 10.4: there the merging launch costs more than the
    // passes it takes away.
    const int n = t + L, units = g.Hkv * ((L * g.G + 15) / 16);
    const long most = std::min<long>(std::min(256 / units, n / (2 * F32_PASS)), sc.cap_rows / ((long)g.Hq * L));
    const int pieces = (int)std::max<long>(1, std::min<long>(most, RW_CLASSES));
    a.ks = ((n + pieces - 1) / pieces + F32_RUN - 1) / F32_RUN * F32_RUN;
    a.nsplit = (n + a.ks - 1) / a.ks;
    if (g.d != 64 && g.d != 128) return hipErrorInvalidValue;
    // one launch, but for the 65535 row groups that a grid dimension takes
    const int groups = (L * g.G + 15) / 16;
    for (a.rg0 = 0; a.rg0 < groups; a.rg0 += 65535) {
        const dim3 grid((unsigned)a.nsplit, (unsigned)g.Hkv, (unsigned)std::min(groups - a.rg0, 65535)), block(RW_NT);
        const bool append = ap.k && a.rg0 == 0;
        if (g.d == 128 && append) hipLaunchKernelGGL((attn_f32_kernel<128, true>), grid, block, 0, st, a, ap);
        else if (g.d == 128) hipLaunchKernelGGL((attn_f32_kernel<128, false>), grid, block, 0, st, a, ap);
        else if (append) hipLaunchKernelGGL((attn_f32_kernel<64, true>), grid, block, 0, st, a, ap);
        else hipLaunchKernelGGL((attn_f32_kernel<64, false>), grid, block, 0, st, a, ap);
    }
    if (a.nsplit > 1 && g.d == 128) launch_merge_rows<float, 128, true>(a, st);
    else if (a.nsplit > 1) launch_merge_rows<float, 64, true>(a, st);
    return hipGetLastError();
}

hipError_t launch_score_f32(const Geometry& g, const CacheView& c, const KeySource& ks, const void* q, const float* lse,
                            const FwdScratch& sc, int t, int L, float* Wb, hipStream_t st)
{
    const int n = t + L, cnd = n - g.R, lq = g.R < L ? g.R : L;
    if (cnd <= 0) return hipSuccess;
    const int ncol = ks.rows > cnd ? ks.rows : cnd;            // every cached row, and the chunk rows below cnd
    const int nxb = (ncol + 127) / 128, blocks = g.G * ((lq + 15) / 16);
    int rsplit = std::min(256 / (nxb * g.Hkv), blocks / 2);    // slices of at least two blocks, one workgroup per CU
    if (rsplit < 1 || !sc.score_part || nxb * g.Hkv * rsplit > SCORE_SPLIT_WGS) rsplit = 1;
    const dim3 grid((unsigned)nxb, (unsigned)g.Hkv, (unsigned)rsplit), block(RW_NT);
#define INFMLLM_SCORE(DD)                                                                                                 \
    hipLaunchKernelGGL(score_f32_kernel<DD>, grid, block, 0, st, (const float*)q, (const float*)c.K, (const float*)ks.k,      \
                       ks.rows, lse, g.policy == POLICY_CUMULATIVE ? c.score : nullptr, c.rank, Wb, L, lq, g.Hq, g.Hkv, g.G, \
                       g.cap, g.max_chunk, cnd, ncol, (float)g.scale, (float)(g.bias / (double)cnd), sc.score_part)
    if (g.d == 128) INFMLLM_SCORE(128);
    else if (g.d == 64) INFMLLM_SCORE(64);
    else return hipErrorInvalidValue;
#undef INFMLLM_SCORE
    return hipGetLastError();
}

}  // namespace infmllm
