// Device helpers shared by the attention kernels that cut the key range into pieces (attn_rows.hip, attn_rows64.hip).
#pragma once
#include "launch.h"
#include "mfma_common.h"

namespace infmllm {

template <typename T>
struct RowsArgsT {
    const T* q;                // [L][Hq][D]
    T* K;                      // cache
    T* V;
    const T* kc;               // keys and values from row tc on: chunk tensors [L][Hkv][D]
    const T* vc;
    T* out;                    // [L][Hq][D]
    float* lse;                // [Hq][max_chunk] row log-sum-exp (base 2; natural for fp32), or null (decoding)
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
    int rg0;                   // first row group of the launch (attn_f32)
    int beside;                // attn_rows: the row groups of a key are numbered beside each other, so many; 0: not
    uint32_t inv_g;            // see rows_token
    float c;                   // scale * log2(e); fp32: scale
};
typedef RowsArgsT<uint16_t> RowsArgs;

void launch_rows64(const RowsArgs& a, const AppendJob& ap, hipStream_t st);
inline uint32_t rows_inv_g(int L, int G) { return (uint64_t)L * G * G < (1ull << 32) ? (uint32_t)((1ull << 32) / (unsigned)G + 1) : 0u; }

namespace {

typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(1))) void global_void;

constexpr int RW_NW = 8, RW_NT = 64 * RW_NW;        // wavefronts, threads
constexpr int RW_RUN = 32;                         // keys of a wavefront's run
constexpr int RW_PASS = RW_NW * RW_RUN;            // keys of a workgroup's pass


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


// 16 bytes per lane, memory -> 1 KB of LDS at dst: lane's address base + off + soff, base and soff uniform, `bytes` =
// the extent of what base points at.  (A buffer load: the compiler counts it like any other load.  It takes global_load_lds for one
// that may also be an LDS access, and drains every load in flight at the next wait.)
// THROUGH: from where every XCD's agent-scope stores go (see part_load2).
template <bool THROUGH = false>
__device__ __forceinline__ void buffer_to_lds(const void* base, int bytes, char* dst, int off, int soff = 0)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00020000),
                                             (lds_void*)dst, 16, off, soff, 0, THROUGH ? 16 /* sc1 */ : 0);
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

// LDS reads as statements of their own: the compiler, which cannot tell one buffer from the other, would wait for
// every direct load in flight before each read it knows of.  They are waited for by hand, and the registers are
// first touched after that wait, which only holds where the compiler has no reason to move or spill them in between; WAITED:
// elsewhere, the wait is part of the read.
template <int OFF, bool WAITED = false>
__device__ __forceinline__ bf16x4 rw_read_tr16(uint32_t addr)
{
    bf16x4 v;
    if constexpr (WAITED) asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(addr), "n"(OFF));
    else asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
template <typename V, int OFF, bool WAITED>
__device__ __forceinline__ V rw_read16(uint32_t addr)
{
    V v;
    if constexpr (WAITED) asm volatile("ds_read_b128 %0, %1 offset:%2\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(addr), "n"(OFF));
    else asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
template <int OFF, bool WAITED = false>
__device__ __forceinline__ bf16x8 rw_read_b128(uint32_t addr) { return rw_read16<bf16x8, OFF, WAITED>(addr); }
template <int OFF, bool WAITED = false>
__device__ __forceinline__ f32x4 rw_read_f32x4(uint32_t addr) { return rw_read16<f32x4, OFF, WAITED>(addr); }
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
// NAT: references are natural logarithms (fp32 streams), else base 2
template <bool NAT>
struct PieceSumT {
    float m, l;
    f32x4 o;                   // four of the row's columns
    static __device__ __forceinline__ float power(float x) { return NAT ? expf(x) : fast_exp2(x); }
    __device__ __forceinline__ void absorb(float2 ml, f32x4 x)
    {
        const float mn = fmaxf(m, ml.x), mz = (mn == -__builtin_inff()) ? 0.f : mn;
        const float wa = power(m - mz), wb = power(ml.x - mz);
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
        const float w = power(m - mz);
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
    __device__ __forceinline__ float lse() const { return m + (NAT ? logf(l) : __builtin_log2f(l)); }
};
typedef PieceSumT<false> PieceSum;
// the tree in one thread: no lane does another one's work, for many rows
template <int N, bool NAT>
__device__ __forceinline__ PieceSumT<NAT> add_tree(PieceSumT<NAT> (&p)[N])
{
#pragma clang fp contract(off)
    float mt = p[0].m;
#pragma unroll
    for (int i = 1; i < N; ++i) mt = fmaxf(mt, p[i].m);
    const float mz = (mt == -__builtin_inff()) ? 0.f : mt;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float w = PieceSumT<NAT>::power(p[i].m - mz);
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
__device__ __forceinline__ void store_out4(float* p, f32x4 v) { *(f32x4*)p = v; }



// token of a row (row = token * G + head in group): row / G.  rho * inv_g / 2^32 exceeds rho / G by less than rho / 2^32, so it is
// exact while rho * G < 2^32.  Launches of fp32 streams may have more rows than that (inv_g = 0); those of bf16 streams have
// at most 2^20, and the division would cost attn_rows64 registers that it does not have.
template <typename T>
__device__ __forceinline__ int rows_token(const RowsArgsT<T>& a, int rho) 
{
    if (a.G == 1) return rho;
    if (sizeof(T) == 4 && a.inv_g == 0) return rho / a.G;
    return (int)__umulhi((uint32_t)rho, a.inv_g);
}

// Tiles in LDS: rows are not padded; the 16-byte pieces of a row are permuted at load time instead (by choosing which
// piece of its row a lane fetches), so that sixteen rows of K (or Q) at one piece, and the sixteen rows of a transpose
// read of V (32 bytes of each), spread over the banks.  Piece p of row r lies in slot p ^ swz(r).
template <int D> __device__ __forceinline__ int swz_k(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
template <int D> __device__ __forceinline__ int swz_v(int r) { return D == 128 ? 2 * (r & 7) : 2 * ((r >> 1) & 3); }
template <typename T, int D> struct Tile {
    static __device__ __forceinline__ int k(int r, int p) { return p ^ swz_k<D>(r); }      // slot of piece p; its own inverse
    static __device__ __forceinline__ int v(int r, int p) { return p ^ swz_v<D>(r); }
};
// fp32: sixteen rows of K at one piece; of V a row's pieces 2l (then 2l + 1) for the sixteen lanes l of a group
template <int D> struct Tile<float, D> {
    static __device__ __forceinline__ int k(int r, int p) { return p ^ (r & 15); }
    static __device__ __forceinline__ int v(int, int p) { return D == 128 ? p ^ ((p >> 4) & 1) : p; }
};

// A wavefront's direct loads of a run: KEYS rows of K and / or V from row k0 on, to `dst` (K) and `dst` + RUN (V).
template <typename T, int D, int KEYS>
struct RunLoader {
    static constexpr int ROWB = D * (int)sizeof(T), RUN = KEYS * ROWB, NL = RUN / 1024, RPL = 1024 / ROWB;
    typedef Tile<T, D> Swz;
    const T *Kh, *Vh, *kch, *vch;
    int tc, n, crs;                                // crs: row stride of the chunk tensors
    int lrow, lpos;                                // this lane's row and slot of a load
    __device__ __forceinline__ RunLoader(const RowsArgsT<T>& a, int h, int lane)
        : Kh(a.K + (size_t)h * a.cap * D), Vh(a.V + (size_t)h * a.cap * D), kch(a.kc + (size_t)h * D), vch(a.vc + (size_t)h * D),
          tc(a.tc), n(a.t + a.L), crs(a.Hkv * D), lrow(lane / (ROWB / 16)), lpos(lane % (ROWB / 16))
    {
    }
    template <bool K, bool V>
    __device__ __forceinline__ void load(int k0, char* dst) const
    {
        const bool in_cache = k0 + KEYS <= tc, in_chunk = k0 >= tc && k0 + KEYS <= n;
        if (in_cache || in_chunk) {                // rows a fixed stride apart
            const int stride = in_cache ? ROWB : crs * (int)sizeof(T), bytes = KEYS * stride;
            const size_t at = (size_t)(in_cache ? k0 : k0 - tc) * stride;
            const T *k_cache = Kh, *k_chunk = kch, *v_cache = Vh, *v_chunk = vch;
            const char* kp = (const char*)(in_cache ? k_cache : k_chunk) + at;
            const char* vp = (const char*)(in_cache ? v_cache : v_chunk) + at;
            if (K) {
#pragma unroll
                for (int u = 0; u < NL; ++u)
                    buffer_to_lds(kp, bytes, dst + u * 1024, lrow * stride + (Swz::k(u * RPL + lrow, lpos) * 16), u * RPL * stride);
            }
            if (V) {
#pragma unroll
                for (int u = 0; u < NL; ++u)
                    buffer_to_lds(vp, bytes, dst + RUN + u * 1024, lrow * stride + (Swz::v(u * RPL + lrow, lpos) * 16), u * RPL * stride);
            }
        } else {                                   // where the cache or the chunk ends: row by row, past it the last row again
#pragma nounroll
            for (int u = 0; u < NL; ++u) {
                const int r = u * RPL + lrow, key = min(k0 + r, n - 1);
                const bool cached = key < tc;
                const size_t off = cached ? (size_t)key * D : (size_t)(key - tc) * crs;
                const T *ka = Kh + off, *kb = kch + off, *va = Vh + off, *vb = vch + off;
                if (K) __builtin_amdgcn_global_load_lds((global_void*)((cached ? ka : kb) + Swz::k(r, lpos) * (16 / (int)sizeof(T))), (lds_void*)(dst + u * 1024), 16, 0, 0);
                if (V) __builtin_amdgcn_global_load_lds((global_void*)((cached ? va : vb) + Swz::v(r, lpos) * (16 / (int)sizeof(T))), (lds_void*)(dst + RUN + u * 1024), 16, 0, 0);
            }
        }
    }
};

// Four columns of a row, merged over the workgroup's wavefronts: the finished output, or this piece's share of it.
template <int D, typename T, bool NAT>
__device__ __forceinline__ void leave_row(const RowsArgsT<T>& a, int h, int sp, int rho, int d, const PieceSumT<NAT>& ps)
{
    if (a.nsplit == 1) {
        const int tok = rows_token(a, rho), gq = h * a.G + rho - tok * a.G;
        store_out4(a.out + ((size_t)tok * a.Hq + gq) * D + d, ps.out());
        if (a.lse && d == 0) a.lse[(size_t)gq * a.max_chunk + tok] = ps.lse();
        return;
    }
    const size_t at = ((size_t)h * a.L * a.G + rho) * a.nsplit + sp;
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

// The second launch: one thread per four columns of a row.  N = classes that can have a piece (4, 8 or 16).
template <typename T, int D, int N, bool NAT>
__global__ void __launch_bounds__(256)
merge_rows_kernel(const float* __restrict__ part_o, const float2* __restrict__ part_ml, T* __restrict__ out,
                  float* __restrict__ lse, int M, int Hq, int G, int max_chunk, int nsplit)
{
    const int h = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;
    if (i >= M * (D / 4)) return;
    const int rho = i / (D / 4), d = 4 * (i % (D / 4)), tok = rho / G, gq = h * G + rho - tok * G;
    const float2* pml = part_ml + ((size_t)h * M + rho) * nsplit;
    const float* po = part_o + ((size_t)h * M + rho) * nsplit * D + d;
    PieceSumT<NAT> ps[N];
#pragma unroll
    for (int c = 0; c < N; ++c) {                              // all requested before any is used
        const int s = min(c, nsplit - 1);
        const float2 ml = pml[s];
        ps[c] = PieceSumT<NAT>{ml.x, ml.y, *(const f32x4*)(po + (size_t)s * D)};
    }
#pragma unroll
    for (int c = 0; c < N; ++c)                                // no such piece (0 times an infinite output would not be 0)
        if (c >= nsplit) ps[c] = PieceSumT<NAT>{-__builtin_inff(), 0.f, f32x4{0.f, 0.f, 0.f, 0.f}};
    if (N == RW_CLASSES)
        for (int s0 = RW_CLASSES; s0 < nsplit; s0 += RW_CLASSES)
#pragma unroll
            for (int c = 0; c < N; ++c)
                if (s0 + c < nsplit) ps[c].absorb(pml[s0 + c], *(const f32x4*)(po + (size_t)(s0 + c) * D));
    const PieceSumT<NAT> tot = add_tree(ps);
    store_out4(out + ((size_t)tok * Hq + gq) * D + d, tot.out());
    if (lse && d == 0) lse[(size_t)gq * max_chunk + tok] = tot.lse();
}

template <typename T, int D, bool NAT>
void launch_merge_rows(const RowsArgsT<T>& a, hipStream_t st)
{
    const int M = a.L * a.G;
    const dim3 grid((unsigned)((M * (D / 4) + 255) / 256), (unsigned)a.Hkv), block(256);
#define INFMLLM_MERGE(N)                                                                                                    \
    hipLaunchKernelGGL((merge_rows_kernel<T, D, N, NAT>), grid, block, 0, st, a.part_o, a.part_ml, a.out, a.lse, M, a.Hq, a.G, \
                       a.max_chunk, a.nsplit)
    if (a.nsplit <= 4) INFMLLM_MERGE(4);
    else if (a.nsplit <= 8) INFMLLM_MERGE(8);
    else INFMLLM_MERGE(16);
#undef INFMLLM_MERGE
}

}  // namespace
}  // namespace infmllm
