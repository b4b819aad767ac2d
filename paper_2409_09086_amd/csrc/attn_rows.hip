// Attention of few query rows over many keys on bf16 MFMA for gfx950: decoding steps (one token or a run of
// known ones) and short chunks.
//
// attn_fwd and attn_fwd64 get their parallelism from the query rows; with a few dozen of them most of the chip
// would idle while each workgroup walks the whole cache.  Here the key range is cut into `nsplit` pieces of
// `ks` keys and a workgroup owns (kv-head, piece, 16 or 32 query rows of the head's group): the rows of a
// kv-head are numbered token-major (row = token * G + head in group), so grouped heads and consecutive tokens
// share every K and V byte.  Each of the eight wavefronts takes every eighth run of 32 keys and keeps its own
// online softmax; nothing is shared between them until the end, so the loop has no barrier:
//
// K and V go from memory to LDS without passing through registers, into a buffer only this wavefront uses (16 KB: 128 KB
// in flight per CU), and the next run is requested as soon as the fragments of a run are in registers; K is read in the
// layout of the MFMA's A operand, V with the LDS transpose read.
//
// S^T = K.Q^T on 16x16x32 MFMA leaves four consecutive keys of one query row in a lane; two such 16-key blocks
// are the B operand of O^T += V^T.P^T as they stand (the contraction runs over keys {4g..4g+3, 16+4g..+3} for lane
// group g, and V is read in that order).
//
// EXACT (decoding): a weight enters the product as three bf16 terms whose sum is the fp32 weight, so that the
// product is that of fp32 weights; the matrix cores have the time, the step is bound by the cache it reads.  Which
// keys a piece and a wavefront take depends on the row's absolute key index only, and every row decides for
// itself when its softmax reference moves: a token's output does not depend on how many tokens share the call.
//
// Pieces are merged by the workgroup that finishes last (a ticket per kv-head; decoding one token) or by a second
// launch where there are many rows.
#include <algorithm>

#include "launch.h"
#include "mfma_common.h"

namespace infmllm {

namespace {

constexpr int RW_NW = 8, RW_NT = 64 * RW_NW;        // wavefronts, threads
constexpr int RW_RUN = 32;                         // keys of a wavefront's run
constexpr int RW_PASS = RW_NW * RW_RUN;            // keys of a workgroup's pass

typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(1))) void global_void;

template <int D, int NRB>
struct RowsCfg {
    static constexpr int ROWB = D * 2;             // bytes of a K or V row
    static constexpr int RUN = RW_RUN * ROWB;      // bytes of a run of K or of V
    static constexpr int STAGE = 2 * RUN;          // ... of both
    static constexpr int NS = D / 32;              // MFMAs along head_dim of one 16-key block of S
    static constexpr int NC = D / 16;              // 16-column blocks of O
    static constexpr int NL = RUN / 1024;          // direct loads per run of K or V (1 KB each)
    static constexpr int RPL = 1024 / ROWB;        // rows per direct load
    static constexpr int ROWS = 16 * NRB;
    static constexpr int MB = ROWS * D * 4;        // bytes a wavefront leaves for the merge, in its own buffers
    static_assert(MB <= STAGE, "the merge reuses the buffers of the tiles");
};

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// maximum / sum over the four 16-lane groups of a wavefront (lanes l, l ^ 16, l ^ 32, l ^ 48), in every lane
__device__ __forceinline__ float groups_max(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return xhalf_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float groups_sum(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return xhalf_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}


// 16 bytes per lane, memory -> 1 KB of LDS at dst: lane's address base + off, base uniform, `bytes` = the extent of
// what base points at.  (A buffer load: the compiler counts it like any other load.  It takes global_load_lds for one
// that may also be an LDS access, and drains every load in flight at the next wait.)
// THROUGH: from where every XCD's agent-scope stores go (see part_load2).
template <bool THROUGH = false>
__device__ __forceinline__ void buffer_to_lds(const void* base, int bytes, char* dst, int off)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00020000),
                                             (lds_void*)dst, 16, off, 0, 0, THROUGH ? 16 /* sc1 */ : 0);
}

// sum / maximum over N = 8 or 16 consecutive lanes, the same bits in all of them: neighbours, pairs, quads, eights
template <int CTRL>
__device__ __forceinline__ float dpp(float x)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xF, 0xF, true));
}
template <int N>
__device__ __forceinline__ float lanes_sum(float x)
{
    x += dpp<0xB1>(x);                             // quad_perm [1,0,3,2]
    x += dpp<0x4E>(x);                             // quad_perm [2,3,0,1]
    x += dpp<0x141>(x);                            // row_half_mirror
    if (N == 16) x += dpp<0x140>(x);               // row_mirror
    return x;
}
template <int N>
__device__ __forceinline__ float lanes_max(float x)
{
    x = fmaxf(x, dpp<0xB1>(x));
    x = fmaxf(x, dpp<0x4E>(x));
    x = fmaxf(x, dpp<0x141>(x));
    if (N == 16) x = fmaxf(x, dpp<0x140>(x));
    return x;
}

template <int OFF>
__device__ __forceinline__ bf16x4 rw_read_tr16(uint32_t addr)
{
    bf16x4 v;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
template <int OFF>
__device__ __forceinline__ bf16x8 rw_read_b128(uint32_t addr)
{
    bf16x8 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
template <int N>
__device__ __forceinline__ void wait_loads()       // all but the N newest
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Partial results of a piece: un-normalised o[D], reference maximum and sum, per (kv-head, row, piece).
// THROUGH: read and written where every XCD sees them (the last workgroup of a launch merges), else plainly.
template <bool THROUGH>
__device__ __forceinline__ float2 part_load2(const float2* p)
{
    if constexpr (THROUGH) {
        const uint64_t a = __hip_atomic_load((const uint64_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return float2{__uint_as_float((uint32_t)a), __uint_as_float((uint32_t)(a >> 32))};
    } else {
        return *p;
    }
}

__device__ __forceinline__ void part_store2(float2* p, float2 v)
{
    __hip_atomic_store((uint64_t*)p, (uint64_t)__float_as_uint(v.x) | ((uint64_t)__float_as_uint(v.y) << 32), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// How the shares of a row are added, those of a workgroup's wavefronts as well as those of its pieces, and the same bits
// whoever does it: under their largest reference, products rounded before they are added, neighbours first, then pairs,
// and so on (a binary tree over the index; missing shares weigh 0).  Piece s belongs to class s % 16, and a class absorbs
// its pieces in ascending order before the tree.  A share in which the row saw no key has m = -inf and weight 0, so pieces
// past the row's last key change nothing.
constexpr int RW_CLASSES = 16;
constexpr int RW_TICKET_PARTS = 256;               // most (row, piece) pairs of a kv-head that its last workgroup merges
struct PieceSum {
    float m, l;
    f32x4 o;                   // four of the row's columns
    __device__ __forceinline__ void absorb(float2 ml, f32x4 x)
    {
        const float mn = fmaxf(m, ml.x), mz = (mn == -__builtin_inff()) ? 0.f : mn;
        const float wa = fast_exp2(m - mz), wb = fast_exp2(ml.x - mz);
        m = mn;
        l = __builtin_fmaf(wa, l, wb * ml.y);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = __builtin_fmaf(wa, o[e], wb * x[e]);
    }
    // the tree over N consecutive lanes: few instructions, for few rows
    template <int N>
    __device__ __forceinline__ void add_lanes()
    {
#pragma clang fp contract(off)
        const float mt = lanes_max<N>(m), mz = (mt == -__builtin_inff()) ? 0.f : mt;
        const float w = fast_exp2(m - mz);
        m = mt;
        l = lanes_sum<N>(w * l);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = lanes_sum<N>(w * o[e]);
    }
    __device__ __forceinline__ f32x4 out() const
    {
        const float inv = 1.0f / l;
        return f32x4{o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv};
    }
    __device__ __forceinline__ float lse() const { return m + __builtin_log2f(l); }
};
// the tree in one thread: no lane does another one's work, for many rows
template <int N>
__device__ __forceinline__ PieceSum add_tree(PieceSum (&p)[N])
{
#pragma clang fp contract(off)
    float mt = p[0].m;
#pragma unroll
    for (int i = 1; i < N; ++i) mt = fmaxf(mt, p[i].m);
    const float mz = (mt == -__builtin_inff()) ? 0.f : mt;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float w = fast_exp2(p[i].m - mz);
        p[i].l = w * p[i].l;
#pragma unroll
        for (int e = 0; e < 4; ++e) p[i].o[e] = w * p[i].o[e];
    }
#pragma unroll
    for (int st = 1; st < N; st *= 2)
#pragma unroll
        for (int i = 0; i < N; i += 2 * st) {
            p[i].l = p[i].l + p[i + st].l;
#pragma unroll
            for (int e = 0; e < 4; ++e) p[i].o[e] = p[i].o[e] + p[i + st].o[e];
        }
    p[0].m = mt;
    return p[0];
}

__device__ __forceinline__ void store_out4(uint16_t* p, f32x4 v)
{
    bf16x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = (__bf16)v[e];
    *(bf16x4*)p = w;
}

struct RowsArgs {
    const uint16_t* q;         // [L][Hq][D]
    uint16_t* K;               // cache
    uint16_t* V;
    const uint16_t* kc;        // keys and values from row tc on: chunk tensors [L][Hkv][D]
    const uint16_t* vc;
    uint16_t* out;             // [L][Hq][D]
    float* lse2;               // [Hq][max_chunk], or null (decoding)
    float* part_o;             // [Hkv][M][nsplit][D]
    float2* part_ml;           // [Hkv][M][nsplit]
    int* arrived;              // [Hkv] tickets, zero between launches; null: a second launch merges
    // decoding: the tokens become cache rows t .. t+L-1
    int32_t* pos;              // null: nothing is appended
    float* score;
    int32_t* rank;
    int32_t* row;
    int pos0;
    int t, L, tc, Hq, Hkv, G, cap, max_chunk, ks, nsplit;
    uint32_t inv_g;            // floor(2^32 / G) + 1
    float c;                   // scale * log2(e)
};

template <int D, int NRB, bool EXACT>
__global__ void __launch_bounds__(RW_NT)
attn_rows_kernel(RowsArgs a)
{
    using C = RowsCfg<D, NRB>;
    __shared__ __attribute__((aligned(1024))) char smem[(RW_NW + 1) * C::STAGE];   // a run of K and V per wavefront, two for the first one
    __shared__ float s_m[RW_NW][C::ROWS], s_l[RW_NW][C::ROWS];
    __shared__ int s_ticket;
    __shared__ float2 s_part[NRB == 1 ? RW_TICKET_PARTS : 1];

    // Workgroup = (piece, kv-head, row group), the piece fastest and the row group slowest: the row groups of a piece,
    // which read the same keys, land on one XCD where the number of (piece, head) pairs is a multiple of 8.
    const int sp = blockIdx.x, h = blockIdx.y, rg = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.L * a.G, row0 = rg * C::ROWS;
    const int t = a.t, tc = a.tc, n = t + a.L;
    // token of a row: row / G (inv_g = floor(2^32 / G) + 1 is exact for the at most 2^20 rows of a kv-head)
    auto token = [&](int rho) -> int { return a.G == 1 ? rho : (int)__umulhi((uint32_t)rho, a.inv_g); };
    const int first_lim = t + token(row0);                     // last key the group's first row sees
    const int n_end = t + token(min(row0 + C::ROWS, M) - 1) + 1;
    const int k_end = min((sp + 1) * a.ks, n_end);

    const uint16_t* Kh = a.K + (size_t)h * a.cap * D;
    const uint16_t* Vh = a.V + (size_t)h * a.cap * D;
    const uint16_t* kch = a.kc + (size_t)h * D;
    const uint16_t* vch = a.vc + (size_t)h * D;
    const size_t crs = (size_t)a.Hkv * D;                      // row stride of the chunk tensors

    // Tiles in LDS: rows are not padded; the 16-byte pieces of a row are permuted at load time instead (by choosing
    // which piece of its row a lane fetches), so that sixteen rows of K at one piece, and the sixteen rows of a
    // transpose read of V (32 bytes of each), spread over the banks.  Piece p of row r lies in slot p ^ swz(r).
    auto swz_k = [](int r) -> int { return D == 128 ? (r & 15) : ((r >> 1) & 7); };
    auto swz_v = [](int r) -> int { return D == 128 ? 2 * (r & 7) : 2 * ((r >> 1) & 3); };
    char* const mine = smem + wave * C::STAGE;
    const int lrow = lane / (C::ROWB / 16), lpos = lane % (C::ROWB / 16);   // this lane's row and slot of a direct load
    auto load_run = [&](int k0, char* dst) {
        // (past the last key the rows of a warm-up step's cache are read as they are: finite, and masked)
        const bool in_cache = k0 + RW_RUN <= (tc == n ? a.cap : tc), in_chunk = k0 >= tc && k0 + RW_RUN <= n;
        if (in_cache || in_chunk) {                            // rows a fixed stride apart
            const int stride = in_cache ? C::ROWB : (int)crs * 2, at = (in_cache ? k0 : k0 - tc) * stride;
            const int bytes = (in_cache ? a.cap : a.L) * stride - at;
            const char* kp = (const char*)(in_cache ? Kh : kch) + at;
            const char* vp = (const char*)(in_cache ? Vh : vch) + at;
#pragma unroll
            for (int u = 0; u < C::NL; ++u) {
                const int r = u * C::RPL + lrow;
                buffer_to_lds(kp, bytes, dst + u * 1024, r * stride + (lpos ^ swz_k(r)) * 16);
            }
#pragma unroll
            for (int u = 0; u < C::NL; ++u) {
                const int r = u * C::RPL + lrow;
                buffer_to_lds(vp, bytes, dst + C::RUN + u * 1024, r * stride + (lpos ^ swz_v(r)) * 16);
            }
        } else {                                               // where the cache or the chunk ends: row by row
#pragma nounroll
            for (int u = 0; u < C::NL; ++u) {
                const int r = u * C::RPL + lrow, key = min(k0 + r, n - 1);
                const bool cached = key < tc;
                const size_t off = cached ? (size_t)key * D : (size_t)(key - tc) * crs;
                const uint16_t* ks = (cached ? Kh : kch) + off;
                const uint16_t* vs = (cached ? Vh : vch) + off;
                __builtin_amdgcn_global_load_lds((global_void*)(ks + (lpos ^ swz_k(r)) * 8), (lds_void*)(dst + u * 1024), 16, 0, 0);
                __builtin_amdgcn_global_load_lds((global_void*)(vs + (lpos ^ swz_v(r)) * 8), (lds_void*)(dst + C::RUN + u * 1024), 16, 0, 0);
            }
        }
    };
    const int k_first = sp * a.ks + wave * RW_RUN;
    const int np = k_end > k_first ? (k_end - k_first + RW_PASS - 1) / RW_PASS : 0;
    // wavefront 0, which has a run more than the others if any has, has a second stage for its odd runs
    const int nst = wave == 0 ? 2 : 1;
    const uint32_t stage1 = wave == 0 ? RW_NW * C::STAGE : 0;
    if (np > 0) load_run(k_first, mine);
    if (nst == 2 && np > 1) load_run(k_first + RW_PASS, mine + stage1);
    // query fragments: B operand of S^T = K.Q^T, lane (row c16, group g4) holds Q[row][32s + 8 g4 .. +8)
    bf16x8 qf[NRB][C::NS];
    int lim[NRB];
#pragma unroll
    for (int x = 0; x < NRB; ++x) {
        const int rho = min(row0 + 16 * x + c16, M - 1), tok = token(rho);
        lim[x] = t + tok;
        const uint16_t* qp = a.q + ((size_t)tok * a.Hq + h * a.G + (rho - tok * a.G)) * D + 8 * g4;
#pragma unroll
        for (int s = 0; s < C::NS; ++s) qf[x][s] = as_bf16x8(*(const u32x4*)(qp + 32 * s));
    }

    f32x4 o[NRB][C::NC];
    float m_ref[NRB], m_use[NRB], lsum[NRB];
#pragma unroll
    for (int x = 0; x < NRB; ++x) {
#pragma unroll
        for (int b = 0; b < C::NC; ++b) o[x][b] = f32x4{0.f, 0.f, 0.f, 0.f};
        m_ref[x] = -__builtin_inff(); m_use[x] = 0.f; lsum[x] = 0.f;
    }

    // K fragments: lane (row c16, group g4) reads piece 4s + g4.  V: a 16-lane group reads keys 4 g4 .. +3 (then
    // 16 + 4 g4 .. +3) of sixteen columns; lane l of the group supplies the address of key l / 4, columns 4 (l % 4).
    uint32_t kaddr[C::NS], vaddr[C::NC];
    {
        const uint32_t base = (uint32_t)(uintptr_t)(lds_void*)mine;
        const int vkey = 4 * g4 + (c16 >> 2), q4 = c16 & 3;    // swz(key + 16) = swz(key)
#pragma unroll
        for (int s = 0; s < C::NS; ++s) kaddr[s] = base + c16 * C::ROWB + (((4 * s + g4) ^ swz_k(c16)) * 16);
#pragma unroll
        for (int b = 0; b < C::NC; ++b)
            vaddr[b] = base + C::RUN + vkey * C::ROWB + (((2 * b + (q4 >> 1)) ^ swz_v(vkey)) * 16) + 8 * (q4 & 1);
    }

    for (int p = 0; p < np; ++p) {
        const int k0 = k_first + p * RW_PASS;
        const uint32_t stage = (p & 1) ? stage1 : 0;
        if (nst == 2 && p + 1 < np) wait_loads<2 * C::NL>();   // this run has landed, the next one may be on its way
        else wait_loads<0>();
        // fragments: K, then V [column block] (keys 4 g4.. and 16 + 4 g4..), whose way through the LDS the products of
        // S hide
        bf16x8 kf[2][C::NS];
        bf16x4 vlo[C::NC], vhi[C::NC];
#pragma unroll
        for (int s = 0; s < C::NS; ++s) {
            kf[0][s] = rw_read_b128<0>(kaddr[s] + stage);
            kf[1][s] = rw_read_b128<16 * C::ROWB>(kaddr[s] + stage);
        }
#pragma unroll
        for (int b = 0; b < C::NC; ++b) {
            vlo[b] = rw_read_tr16<0>(vaddr[b] + stage);
            vhi[b] = rw_read_tr16<16 * C::ROWB>(vaddr[b] + stage);
        }
        // reads return in order: K has arrived when at most the V reads are outstanding (the counter ends at 15)
        asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(kf[0][0]), "+v"(kf[1][0]), "+v"(kf[0][1]), "+v"(kf[1][1])
                     : "n"(2 * C::NC < 15 ? 2 * C::NC : 15));
        if constexpr (C::NS == 4) asm volatile("" : "+v"(kf[0][2]), "+v"(kf[1][2]), "+v"(kf[0][3]), "+v"(kf[1][3]));
        // ---- S^T = K.Q^T
        f32x4 S[NRB][2];
#pragma unroll
        for (int s = 0; s < C::NS; ++s)
#pragma unroll
            for (int x = 0; x < NRB; ++x)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
                    S[x][kb] = mfma16(kf[kb][s], qf[x][s], s == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : S[x][kb]);
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(vlo[0]), "+v"(vhi[0]), "+v"(vlo[1]), "+v"(vhi[1]), "+v"(vlo[2]), "+v"(vhi[2]),
                     "+v"(vlo[3]), "+v"(vhi[3]));
        if constexpr (C::NC == 8)
            asm volatile("" : "+v"(vlo[4]), "+v"(vhi[4]), "+v"(vlo[5]), "+v"(vhi[5]), "+v"(vlo[6]), "+v"(vhi[6]), "+v"(vlo[7]), "+v"(vhi[7]));
        // this stage has been read: its next run goes there
        if (p + nst < np) load_run(k0 + nst * RW_PASS, mine + stage);
        // ---- mask, softmax
        bf16x8 pf[NRB][EXACT ? 3 : 1];
        const bool masked = k0 + RW_RUN - 1 > first_lim;
#pragma unroll
        for (int x = 0; x < NRB; ++x) {
            if (masked) {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (k0 + 16 * kb + 4 * g4 + i > lim[x]) S[x][kb][i] = -__builtin_inff();
            }
            float mx = fmaxf(fmaxf(fmaxf(S[x][0][0], S[x][0][1]), fmaxf(S[x][0][2], S[x][0][3])),
                             fmaxf(fmaxf(S[x][1][0], S[x][1][1]), fmaxf(S[x][1][2], S[x][1][3])));
            mx = groups_max(mx) * a.c;
            const bool moves = mx > m_ref[x] + RESCALE_TAU;    // each row for itself
            if (__any(moves)) {
                const float m_new = moves ? mx : m_ref[x];
                const float mu = (m_new == -__builtin_inff()) ? 0.f : m_new;
                const float alpha = moves ? fast_exp2(m_ref[x] - mu) : 1.f;   // m_ref = -inf gives 0
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
                    const float p = fast_exp2(__builtin_fmaf(S[x][kb][i], a.c, -m_use[x]));
                    lsum[x] += p;
                    const __bf16 hi = (__bf16)p;
                    pf[x][0][4 * kb + i] = hi;
                    if constexpr (EXACT) {
                        const float r1 = p - (float)hi;
                        const __bf16 mid = (__bf16)r1;
                        pf[x][1][4 * kb + i] = mid;
                        pf[x][2][4 * kb + i] = (__bf16)(r1 - (float)mid);
                    }
                }
        }
        // ---- O^T += V^T.P^T
#pragma unroll
        for (int b = 0; b < C::NC; ++b) {
            const bf16x8 vf = __builtin_shufflevector(vlo[b], vhi[b], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
            for (int term = 0; term < (EXACT ? 3 : 1); ++term)
#pragma unroll
                for (int x = 0; x < NRB; ++x) o[x][b] = mfma16(vf, pf[x][term], o[x][b]);
        }
    }

    // ---- decoding: tokens sp, sp + nsplit, .. become cache rows (read from the chunk tensors by everyone)
    if (a.pos && rg == 0 && sp < a.L) {
        constexpr int VPR = D / 8;
        for (int i = sp + a.nsplit * (tid / VPR); i < a.L; i += a.nsplit * (RW_NT / VPR)) {
            const int x = tid % VPR;
            const size_t dst = ((size_t)h * a.cap + t + i) * D + x * 8, src = (size_t)i * crs + x * 8;
            *(u32x4*)(a.K + dst) = *(const u32x4*)(kch + src);
            *(u32x4*)(a.V + dst) = *(const u32x4*)(vch + src);
            if (x == 0) {
                const size_t at = (size_t)h * a.cap + t + i;
                a.pos[at] = a.pos0 + i;
                a.score[at] = __builtin_inff();
                a.rank[at] = t + i;                            // the newest tokens, in the next free physical rows
                a.row[at] = t + i;
            }
        }
    }

    // ---- merge the wavefronts: lane (row c16, group g4) holds O[row][16b + 4 g4 + i]
#pragma unroll
    for (int x = 0; x < NRB; ++x) {
        const float l = groups_sum(lsum[x]);
        if (g4 == 0) { s_m[wave][16 * x + c16] = m_ref[x]; s_l[wave][16 * x + c16] = l; }
    }
    // wavefront w's share: 16-byte piece p of row r in slot p ^ ((r ^ w) & 7) of the row, which keeps both eight rows and
    // eight wavefronts apart in the banks; rows that do not exist are left out
    auto merged = [&](int w, int r, int p) -> char* {
        return smem + w * C::STAGE + r * (D * 4) + ((p ^ ((r ^ w) & 7)) * 16);
    };
    const int rows = min(C::ROWS, M - row0);
#pragma unroll
    for (int x = 0; x < NRB; ++x)
        if (16 * x + c16 < rows) {
#pragma unroll
            for (int b = 0; b < C::NC; ++b) *(f32x4*)merged(wave, 16 * x + c16, 4 * b + g4) = o[x][b];
        }
    __syncthreads();
    const bool single = a.nsplit == 1;
    auto leave = [&](const PieceSum& ps, int rho, int d) {     // a row's four columns: finished, or this piece's share
        if (single) {
            const int tok = token(rho), gq = h * a.G + rho - tok * a.G;
            store_out4(a.out + ((size_t)tok * a.Hq + gq) * D + d, ps.out());
            if (a.lse2 && d == 0) a.lse2[(size_t)gq * a.max_chunk + tok] = ps.lse();
        } else {
            const size_t at = ((size_t)h * M + rho) * a.nsplit + sp;
            float* po = a.part_o + at * D + d;
            if (a.arrived) {
                part_store2((float2*)po, float2{ps.o[0], ps.o[1]});
                part_store2((float2*)po + 1, float2{ps.o[2], ps.o[3]});
                if (d == 0) part_store2(a.part_ml + at, float2{ps.m, ps.l});
            } else {
                *(f32x4*)po = ps.o;
                if (d == 0) a.part_ml[at] = float2{ps.m, ps.l};
            }
        }
    };
    if (NRB == 1 && rows <= 4) {                               // eight lanes, one wavefront's share each
        for (int x = tid / RW_NW; x < rows * (D / 4); x += RW_NT / RW_NW) {
            const int r = x / (D / 4), d = 4 * (x % (D / 4)), w = tid % RW_NW;
            PieceSum ps{s_m[w][r], s_l[w][r], *(const f32x4*)merged(w, r, d / 4)};
            ps.add_lanes<RW_NW>();
            if (w == 0) leave(ps, row0 + r, d);
        }
    } else {
        for (int x = tid; x < rows * (D / 4); x += RW_NT) {
            const int r = x / (D / 4), d = 4 * (x % (D / 4));
            PieceSum ps[RW_NW];
#pragma unroll
            for (int w = 0; w < RW_NW; ++w) ps[w] = PieceSum{s_m[w][r], s_l[w][r], *(const f32x4*)merged(w, r, d / 4)};
            leave(add_tree(ps), row0 + r, d);
        }
    }
    if (single || !a.arrived) return;
    if constexpr (NRB == 1) {                                  // tickets are given out with a single row group only
        // Every workgroup waits until its own partials have been written through, then takes a ticket; the one of this
        // kv-head that arrives last merges the pieces.  No workgroup waits for another one.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) s_ticket = __hip_atomic_fetch_add(a.arrived + h, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (s_ticket != a.nsplit - 1) return;
        if (tid == 0) __hip_atomic_store(a.arrived + h, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch
        // The partials of all rows go to LDS (at most RW_TICKET_PARTS of them), one trip to memory; then sixteen lanes per
        // four columns of a row, one class of pieces each.
        const int parts = M * a.nsplit;
        const size_t at = (size_t)h * parts;
        static_assert(RW_TICKET_PARTS * D * 4 <= RW_NW * C::STAGE && RW_TICKET_PARTS <= RW_NT, "the partials reuse the buffers of the tiles");
        for (int x = wave * 1024; x < parts * D * 4; x += RW_NW * 1024)
            buffer_to_lds<true>((const char*)(a.part_o + at * D) + x, parts * D * 4 - x, smem + x, lane * 16);
        if (tid < parts) s_part[tid] = part_load2<true>(a.part_ml + at + tid);
        wait_loads<0>();
        __syncthreads();
        for (int x = tid / RW_CLASSES; x < M * (D / 4); x += RW_NT / RW_CLASSES) {
            const int r = x / (D / 4), d = 4 * (x % (D / 4)), c = tid % RW_CLASSES;
            const float* po = (const float*)smem + r * a.nsplit * D;
            PieceSum ps{-__builtin_inff(), 0.f, f32x4{0.f, 0.f, 0.f, 0.f}};
            for (int s = c; s < a.nsplit; s += RW_CLASSES) ps.absorb(s_part[r * a.nsplit + s], *(const f32x4*)(po + s * D + d));
            ps.add_lanes<RW_CLASSES>();
            if (c == 0) {
                const int tok = token(r), gq = h * a.G + r - tok * a.G;
                store_out4(a.out + ((size_t)tok * a.Hq + gq) * D + d, ps.out());
                if (a.lse2 && d == 0) a.lse2[(size_t)gq * a.max_chunk + tok] = ps.lse();
            }
        }
    }
}

// The second launch: one thread per four columns of a row.  N = classes that can have a piece (4, 8 or 16).
template <int D, int N>
__global__ void __launch_bounds__(256)
merge_rows_kernel(const float* __restrict__ part_o, const float2* __restrict__ part_ml, uint16_t* __restrict__ out,
                  float* __restrict__ lse2, int M, int Hq, int G, int max_chunk, int nsplit)
{
    const int h = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;
    if (i >= M * (D / 4)) return;
    const int rho = i / (D / 4), d = 4 * (i % (D / 4)), tok = rho / G, gq = h * G + rho - tok * G;
    const float2* pml = part_ml + ((size_t)h * M + rho) * nsplit;
    const float* po = part_o + ((size_t)h * M + rho) * nsplit * D + d;
    PieceSum ps[N];
#pragma unroll
    for (int c = 0; c < N; ++c) {                              // all requested before any is used
        const int s = min(c, nsplit - 1);
        const float2 ml = pml[s];
        ps[c] = PieceSum{c < nsplit ? ml.x : -__builtin_inff(), ml.y, *(const f32x4*)(po + (size_t)s * D)};
    }
    if (N == RW_CLASSES)
        for (int s0 = RW_CLASSES; s0 < nsplit; s0 += RW_CLASSES)
#pragma unroll
            for (int c = 0; c < N; ++c)
                if (s0 + c < nsplit) ps[c].absorb(pml[s0 + c], *(const f32x4*)(po + (size_t)(s0 + c) * D));
    const PieceSum tot = add_tree(ps);
    store_out4(out + ((size_t)tok * Hq + gq) * D + d, tot.out());
    if (lse2 && d == 0) lse2[(size_t)gq * max_chunk + tok] = tot.lse();
}

template <int D, int NRB, bool EXACT>
void launch_rows_cfg(const RowsArgs& a, hipStream_t st)
{
    constexpr int ROWS = 16 * NRB;
    const dim3 grid((unsigned)a.nsplit, (unsigned)a.Hkv, (unsigned)((a.L * a.G + ROWS - 1) / ROWS));
    hipLaunchKernelGGL((attn_rows_kernel<D, NRB, EXACT>), grid, dim3(RW_NT), 0, st, a);
}

template <int D, bool EXACT>
hipError_t launch_rows_d(const RowsArgs& args, int nrb, hipStream_t st)
{
    RowsArgs a = args;
    a.inv_g = (uint32_t)((1ull << 32) / (unsigned)a.G + 1);
    if (nrb == 1) launch_rows_cfg<D, 1, EXACT>(a, st);
    else launch_rows_cfg<D, 2, EXACT>(a, st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.nsplit == 1 || a.arrived) return e;
    const int M = a.L * a.G;
    const dim3 grid((unsigned)((M * (D / 4) + 255) / 256), (unsigned)a.Hkv), block(256);
#define INFMLLM_MERGE(N)                                                                                                \
    hipLaunchKernelGGL((merge_rows_kernel<D, N>), grid, block, 0, st, a.part_o, a.part_ml, a.out, a.lse2, M, a.Hq, a.G, \
                       a.max_chunk, a.nsplit)
    if (a.nsplit <= 4) INFMLLM_MERGE(4);
    else if (a.nsplit <= 8) INFMLLM_MERGE(8);
    else INFMLLM_MERGE(16);
#undef INFMLLM_MERGE
    return hipGetLastError();
}

}  // namespace

int rows_decode_keys_per_piece(const Geometry& g)
{
    // A function of the stream's geometry alone (see EXACT above): a whole number of runs, about 192 workgroups with
    // the cache at its fullest, a merge of at most sixteen pieces, and at least one run per wavefront.  Measured at 32 x 128
    // heads and 2048 + 48 rows: 13.2 us per token with 256 keys per piece, 11.8 with 288 (256 workgroups), 10.9 with 352
    // (192), 10.6 with 384, 11.6 with 576 (128); 4096 rows: 20.7 with 288, 17.1 with 544, 16.4 with 704 (192), 17.0 with
    // 1408; 8 kv-heads and 4096 rows: 12.3 with 256, 12.0 with 288, 13.3 with 704.
    const int pieces = std::max(1, std::min(192 / g.Hkv, RW_CLASSES));
    const int ks = ((g.B + g.max_decode + pieces - 1) / pieces + RW_RUN - 1) / RW_RUN * RW_RUN;
    return ks < 256 ? 256 : ks;
}

hipError_t launch_rows_decode(const Geometry& g, const CacheView& c, const void* q, const void* k, const void* v, int t,
                              int T, int64_t pos, void* out, const RowsScratch& sc, hipStream_t st)
{
    RowsArgs a{};
    a.q = (const uint16_t*)q; a.K = (uint16_t*)c.K; a.V = (uint16_t*)c.V;
    a.kc = (const uint16_t*)k; a.vc = (const uint16_t*)v; a.out = (uint16_t*)out; a.lse2 = nullptr;
    a.part_o = sc.o; a.part_ml = sc.ml;
    a.pos = c.pos; a.score = c.score; a.rank = c.rank; a.row = c.row; a.pos0 = (int)pos;
    a.t = t; a.L = T; a.tc = t; a.Hq = g.Hq; a.Hkv = g.Hkv; a.G = g.G; a.cap = g.cap; a.max_chunk = g.max_chunk;
    a.ks = rows_decode_keys_per_piece(g);
    a.nsplit = (t + T + a.ks - 1) / a.ks;
    a.c = (float)(g.scale * (double)LOG2E);
    if ((long)g.Hq * T * a.nsplit > sc.cap_rows) return hipErrorInvalidValue;
    const int M = T * g.G, nrb = M <= 16 ? 1 : 2;
    a.arrived = M <= 16 && M * a.nsplit <= RW_TICKET_PARTS ? sc.arrived : nullptr;
    if (g.d == 128) return launch_rows_d<128, true>(a, nrb, st);
    if (g.d == 64) return launch_rows_d<64, true>(a, nrb, st);
    return hipErrorInvalidValue;
}

// Time (us, between two events) that a chunk of L rows over n keys should take in this kernel, and the shape for it.
// Fitted to measurements at 500..8500 keys and 32..512 workgroups, within about 10 %: a part that does not depend on the
// keys, a pass of 256 keys per round of 256 workgroups, the partials and the merging launch of a cut key range, and
// never less than the cache takes to come in.  (32 heads of 128 on 4 kv-heads, measured / this: 16 rows per workgroup,
// 128 workgroups, 2064 keys 16.4 / 18.3; 256 workgroups, 8128 keys 45.4 / 44.0; 32 rows, 256 workgroups, 4256 keys
// 34.1 / 34.0; 512 workgroups, 4512 keys 63.7 / 63.3; four pieces, 256 workgroups, 8064 keys 25.2 / 25.0.)
float rows_chunk_plan(const Geometry& g, int n, int L, long cap_rows, RowsPlan& plan)
{
    struct Cost { float fixed, more_rounds, pass; };
    static constexpr Cost COST[2][2] = {{{6.5f, 1.f, 0.66f}, {8.7f, 1.f, 0.85f}},       // head_dim 64: 16, 32 rows
                                        {{8.2f, 4.f, 1.12f}, {11.4f, 4.f, 1.33f}}};     // 128
    const float floor_us = 6.f + (float)n * g.Hkv * g.d * 4.f / 5.5e6f;
    float best = 1e30f;
    for (int nrb = 1; nrb <= 2; ++nrb) {
        const Cost& c = COST[g.d == 128][nrb - 1];
        const long units = (long)g.Hkv * ((L * g.G + 16 * nrb - 1) / (16 * nrb));       // workgroups per piece
        const long most = std::min<long>(std::min<long>(256 / units, (n + 255) / 256), cap_rows / ((long)g.Hq * L));
        for (int pieces = 1; pieces == 1 || pieces <= std::min<long>(most, RW_CLASSES); ++pieces) {
            const int keys = ((n + pieces - 1) / pieces + RW_RUN - 1) / RW_RUN * RW_RUN;
            const float rounds = (float)((units * pieces + 255) / 256);
            float us = c.fixed + c.more_rounds * (rounds - 1.f) + rounds * c.pass * (float)((keys + RW_PASS - 1) / RW_PASS);
            if (us < floor_us) us = floor_us;
            if (pieces > 1) us += 1.2f + 0.45f * (float)pieces;
            if (us < best) { best = us; plan = RowsPlan{nrb, keys}; }
        }
    }
    return best;
}

hipError_t launch_rows_chunk(const Geometry& g, const CacheView& c, const KeySource& ks, const void* q, int t, int L,
                             void* out, float* lse, const RowsScratch& sc, const RowsPlan& plan, hipStream_t st)
{
    RowsArgs a{};
    a.q = (const uint16_t*)q; a.K = (uint16_t*)c.K; a.V = (uint16_t*)c.V;
    a.kc = (const uint16_t*)ks.k; a.vc = (const uint16_t*)ks.v; a.out = (uint16_t*)out; a.lse2 = lse;
    a.part_o = sc.o; a.part_ml = sc.ml;
    a.t = t; a.L = L; a.tc = ks.rows; a.Hq = g.Hq; a.Hkv = g.Hkv; a.G = g.G; a.cap = g.cap; a.max_chunk = g.max_chunk;
    a.ks = plan.keys;
    a.nsplit = (t + L + plan.keys - 1) / plan.keys;
    a.c = (float)(g.scale * (double)LOG2E);
    if (a.nsplit > 1 && (long)g.Hq * L * a.nsplit > sc.cap_rows) return hipErrorInvalidValue;
    a.arrived = plan.nrb == 1 && L * g.G <= 16 && L * g.G * a.nsplit <= RW_TICKET_PARTS ? sc.arrived : nullptr;
    if (g.d == 128) return launch_rows_d<128, false>(a, plan.nrb, st);
    if (g.d == 64) return launch_rows_d<64, false>(a, plan.nrb, st);
    return hipErrorInvalidValue;
}

}  // namespace infmllm
