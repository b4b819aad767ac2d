// Device code of the per-head top-r selection (Alg. 1 l.5-7) and of the placement plan that follows it
// (which retained rows stay where they are, which move where), templated on TPB, the threads of the
// calling workgroup.
#pragma once
#include "launch.h"

namespace infmllm {
namespace {

__device__ __forceinline__ uint32_t order_key(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);    // larger float <=> larger key
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }
// lanes of a ballot below this one
__device__ __forceinline__ uint32_t lanes_below(uint64_t b)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
}

// Workgroup barrier for data handed over through LDS only.  `__syncthreads` also waits for every global store
// and load of the wavefront to complete (about a microsecond for a store on its way to memory), which the
// selection and the plan never need: nothing they write to memory is read again before the kernel ends.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Adds 1 to hist[digit] for every active lane whose `on` is true, one LDS atomic per distinct
// digit per wavefront.
__device__ __forceinline__ void wave_histogram(uint32_t* hist, uint32_t digit, bool on)
{
    uint64_t todo = __ballot(on);
    while (todo) {
        const int leader = __ffsll((long long)todo) - 1;      // wavefront-uniform
        const uint32_t dl = (uint32_t)__builtin_amdgcn_readlane((int)digit, leader);
        const uint64_t same = __ballot(on && digit == dl);
        if (lane_id() == leader) atomicAdd(&hist[dl], (uint32_t)__popcll(same));
        todo &= ~same;
    }
}

// Histogram of 256 bins in LDS.  An atomic on one address is as many operations as it has lanes, and the leading digit of
// scores tends to be the same for most keys of a head (8K cache: 10 us of counting in such a head, 4 in others): every
// eighth lane has counters of its own (4 us and 2.6).  The copies of a bin lie in different banks, and a lane that reads four neighbouring
// bins of a copy reads 16 bytes.  (Counting the lanes that share the first one's digit as one took 1.1 us longer
// where digits differ.)
constexpr int HIST_COPIES = 8, HIST_PITCH = 256 + 8, HIST_WORDS = HIST_COPIES * HIST_PITCH;
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void count_digit(uint32_t* hist, uint32_t digit)
{
    atomicAdd(&hist[(lane_id() & (HIST_COPIES - 1)) * HIST_PITCH + digit], 1u);
}
__device__ __forceinline__ u32x4_t four_bins(const uint32_t* hist, int bin)      // counts of bins bin .. bin + 3
{
    u32x4_t v = *(const u32x4_t*)&hist[bin];
#pragma unroll
    for (int c = 1; c < HIST_COPIES; ++c) v += *(const u32x4_t*)&hist[c * HIST_PITCH + bin];
    return v;
}
__device__ __forceinline__ void clear_hist(uint32_t* hist, int thread)           // by HIST_WORDS / 4 threads
{
    if (thread >= 0 && thread < HIST_WORDS / 4) *(u32x4_t*)&hist[4 * thread] = u32x4_t{0u, 0u, 0u, 0u};
}

// p[i] for i < 2^30, addressed as a uniform base and a 32-bit offset: one instruction where a signed or 64-bit index
// costs four
template <typename T>
__device__ __forceinline__ T& at32(T* p, uint32_t i)
{
    static_assert(sizeof(T) == 4, "");
    return *(T*)((char*)p + (uint32_t)(i * 4u));
}

// Inclusive prefix sum over the 64 lanes of a wavefront whose lanes are all active, through the
// data-parallel-primitive lane shifts (no LDS round trip): shifts by 1, 2, 4, 8 inside each row
// of 16 lanes, then the last lane of rows 0 and 2 added to rows 1 and 3, then lane 31 to rows 2, 3.
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);   // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);   // row_bcast:15
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);   // row_bcast:31
    return x;
}

// Exclusive prefix sums of tab[0 .. count) in place, by one whole wavefront.
__device__ __forceinline__ void wave_exclusive_table(uint32_t* tab, int count)
{
    const int l = lane_id();
    uint32_t run = 0;
    for (int base = 0; base < count; base += 64) {
        const int idx = base + l;
        const uint32_t v = idx < count ? tab[idx] : 0u;
        const uint32_t incl = wave_inclusive_sum(v);
        if (idx < count) tab[idx] = run + incl - v;
        run += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    }
}

// Minimum / maximum over the 64 lanes of a wavefront whose lanes are all active; lane 63 holds the result.
template <bool MAX>
__device__ __forceinline__ uint32_t wave_extreme_to_last_lane(uint32_t x)
{
    constexpr int ID = MAX ? 0 : -1;                          // identity, read where a shift has no source lane
#define INFMLLM_STEP(ctrl, rows)                                                             \
    {                                                                                        \
        const uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp(ID, (int)x, ctrl, rows, 0xf, false); \
        x = MAX ? (x > y ? x : y) : (x < y ? x : y);                                         \
    }
    INFMLLM_STEP(0x111, 0xf) INFMLLM_STEP(0x112, 0xf) INFMLLM_STEP(0x114, 0xf) INFMLLM_STEP(0x118, 0xf)
    INFMLLM_STEP(0x142, 0xa) INFMLLM_STEP(0x143, 0xc)
#undef INFMLLM_STEP
    return x;
}

// What the selection of candidates left in memory leaves in LDS for the placement plan: for every segment of 64 candidates (stream-order
// indices 64 s .. 64 s + 63) which of them are retained, and how many retained candidates precede the
// segment.  The new stream-order index of a retained candidate j is base[j / 64] plus the retained ones below
// it in its segment; a token of the recent window (j >= c) is retained with index r + (j - c).
constexpr int PLAN_MAX_C = 131072;                            // most candidates (n - R) a step may have
struct KeptMap {
    uint64_t bits[PLAN_MAX_C / 64];
    uint32_t base[PLAN_MAX_C / 64];
};

// The tables of one kv-head that the placement plan reads and writes (see CacheView, MoveList).
struct PlanTables {
    int32_t* rank;             // [cap] stream-order index of each physical row: read, and rewritten for the rows that stay
    int32_t* row;              // [cap] physical row of each stream-order index: written for the rows that stay
    float* score;              // [cap]
    int32_t* mv_src;           // [mv_max] move list of this head
    int32_t* mv_dst;
    int32_t* mv_x;
    float* mv_score;
    int32_t* mv_count;         // one int
};

// Alg. 1 l.8 without moving the rows that stay.  Every physical row below max(tc, B) and every chunk row is
// looked at once, 64 consecutive ones per wavefront, so that all table traffic is coalesced and the two lists
// are compacted with ballots: a cached row whose token is retained and that lies below B keeps its place (its
// new index goes into rank / row, its score entry becomes W'[j], +inf inside the recent window); a retained
// token in a row at or above B, or in the chunk, is a mover; a row below B whose token is evicted (or that is
// empty) is free.  There are exactly as many movers as free rows, and the k-th mover is paired with the k-th
// free row, both in ascending order, which makes the layout a function of the retained set alone.  The K/V
// copies and the movers' table entries are left to the placement launch.
// What the plan reads from memory does not depend on the selection: the stream-order index of every physical
// row.  The first PLAN_PRE items of every thread are therefore requested before
// the selection starts and have long arrived when the plan wants them; a plan with more items (more than
// PLAN_PRE * 1024 rows) loads the rest pass by pass.  Candidates that
// were in registers leave their fate, new index and score by token, in LDS: one 8-byte read per item.  (The plan is bound by
// its vector instructions, one workgroup's on one CU: 1.5 us per 4096 items, 1.9 with the new index from a bit map and
// a prefix count and the score gathered from memory.  Selection and plan, from the first workgroup's start to the last one's end:
// 10.7 -> 9.6 us at 8 heads, 4096 + 1024 rows; 22.6 -> 14.4 at 32 heads, 8192 + 2048 rows; 11.8 -> 9.5 at 4096 + 37 rows with a
// steep ramp.  Putting `row` together in LDS, so that its stores are coalesced, gained nothing.)
constexpr int PLAN_PRE = 12;
struct PlanPre {
    int jj[PLAN_PRE];
    float w[PLAN_PRE];         // KPT = 0 only
};
// What the selection leaves for the plan.  KPT = candidates per thread that it holds in registers (0: in memory).
struct Candidate {
    int x;                     // new stream-order index, -1: evicted
    float w;                   // W'
};
template <int KPT, int TPB>
struct PlanLds {
    Candidate cand[KPT * TPB];
};
template <int TPB>
struct PlanLds<0, TPB> {
    KeptMap km;
};
// item q of the plan: a physical row below max(tc, B), then the chunk rows read in place; its token, or -1
__device__ __forceinline__ int plan_item_token(const int32_t* __restrict__ rank, int q, int tc, int P1, int nitems)
{
    return q < tc ? at32(rank, q) : (q >= P1 && q < nitems ? tc + (q - P1) : -1);
}
// The prefetch: the tokens of the items (table reads), and, with the candidates in memory, once those have arrived,
// their scores.
template <int TPB>
__device__ __forceinline__ void plan_prefetch_tokens(PlanPre& pre, const int32_t* __restrict__ rank, int n, int tc, int B)
{
    const int P1 = tc > B ? tc : B, nitems = P1 + (n - tc);
#pragma unroll
    for (int g = 0; g < PLAN_PRE; ++g) pre.jj[g] = plan_item_token(rank, g * TPB + (int)threadIdx.x, tc, P1, nitems);
}
template <int TPB>
__device__ __forceinline__ void plan_prefetch_scores(PlanPre& pre, const float* __restrict__ W, int cnd)
{
#pragma unroll
    for (int g = 0; g < PLAN_PRE; ++g) pre.w[g] = (uint32_t)pre.jj[g] < (uint32_t)cnd ? at32(W, pre.jj[g]) : __builtin_inff();
}

// The placement of a short move list by the workgroup that made it (Alg. 1 l.8), instead of a launch of its own: see
// place_in_select.
struct PlaceHere {
    bool on;
    int vec_shift, Hkv, h, cap, pos0;              // 2^vec_shift 16-byte vectors per row
    const u32x4_t *kc, *vc;                        // chunk tensors
    u32x4_t *K, *V;                                // the cache (all heads)
    int32_t* pos;                                  // of this head
};
struct Mover {
    int src, dst, x;
    float score;
};
template <int TPB>
__device__ __forceinline__ void place_movers(const Mover* mv, int count, int tc, const PlanTables& pt, const PlaceHere& ph)
{
    const size_t hb = (size_t)ph.h * ph.cap;
    const int total = count << ph.vec_shift, xmask = (1 << ph.vec_shift) - 1;
    constexpr int U = 2;                           // vectors in flight per thread and tensor
    for (int i0 = threadIdx.x; i0 < total; i0 += U * TPB) {
        u32x4_t kk[U], vv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = min(i0 + u * TPB, total - 1), src = mv[i >> ph.vec_shift].src;
            const bool cached = src < tc;
            const size_t row = cached ? hb + src : (size_t)(src - tc) * ph.Hkv + ph.h;
            const size_t at = (row << ph.vec_shift) + (i & xmask);
            kk[u] = __builtin_nontemporal_load((cached ? (const u32x4_t*)ph.K : ph.kc) + at);
            vv[u] = __builtin_nontemporal_load((cached ? (const u32x4_t*)ph.V : ph.vc) + at);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * TPB;
            if (i >= total) break;
            const Mover m = mv[i >> ph.vec_shift];
            const size_t at = ((hb + m.dst) << ph.vec_shift) + (i & xmask);
            ph.K[at] = kk[u];
            ph.V[at] = vv[u];
            if ((i & xmask) == 0) {
                ph.pos[m.dst] = m.src < tc ? ph.pos[m.src] : ph.pos0 + (m.src - tc);
                pt.rank[m.dst] = m.x;
                pt.row[m.x] = m.dst;
                pt.score[m.dst] = m.score;
            }
        }
    }
}

template <int KPT, int TPB>
__device__ __forceinline__ void plan_moves(const PlanLds<KPT, TPB>& pl, const float* __restrict__ W, int n, int tc, int cnd,
                                           int B, int r, const PlanTables& pt, const PlanPre& pre, const PlaceHere& ph)
{
    __shared__ Mover movers[PLACE_HERE_ROWS];
    constexpr int NW = TPB / 64, CH = 64 / NW;                 // CH passes of TPB items share one table of 64 counts
    __shared__ uint32_t cnt_free[64], cnt_mov[64];
    __shared__ uint32_t tot_free, tot_mov;
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
    const int P1 = tc > B ? tc : B;                           // physical rows looked at
    const int nitems = P1 + (n - tc);                         // ... then the chunk rows read in place
    // new index of token j, or -1 if it is evicted (or there is none, j < 0), and its score entry: W' (pre_w if the
    // candidates are in memory), +inf inside the recent window
    auto fate = [&](int j, float pre_w) -> Candidate {
        const bool ranked = (uint32_t)j < (uint32_t)cnd;
        if constexpr (KPT > 0) {
            const Candidate c = pl.cand[ranked ? j : 0];
            return Candidate{ranked ? c.x : (j < 0 ? -1 : j + (r - cnd)), ranked ? c.w : __builtin_inff()};
        } else {
            if (!ranked) return Candidate{j < 0 ? -1 : j + (r - cnd), __builtin_inff()};
            const uint64_t bits = pl.km.bits[j >> 6];
            const bool kept = (bits >> (j & 63)) & 1ull;
            return Candidate{kept ? (int)(pl.km.base[j >> 6] + (uint32_t)__popcll(bits & ((1ull << (j & 63)) - 1ull))) : -1, pre_w};
        }
    };
    const int stay_end = tc < B ? tc : B;                     // rows below it keep the tokens that are retained
    uint32_t fbase = 0, mbase = 0;                            // free rows / movers listed so far (uniform)
    lds_barrier();                                          // the kept map is complete
    static_assert(PLAN_PRE % CH == 0, "prefetched items are consumed in whole passes");
    auto pass = [&](int q0, const int (&jj)[CH], const float (&wv)[CH]) {
        int xs[CH], src[CH];
        uint64_t bfree[CH], bmov[CH];
        float sc[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const Candidate f = fate(jj[u], wv[u]);
            xs[u] = f.x;
            sc[u] = f.w;
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int q = q0 + u * TPB + tid;
            const bool kept = xs[u] >= 0;
            const bool stays = kept && q < stay_end;
            const bool moves = kept && !stays;
            const bool is_free = !kept && q < B;
            src[u] = q < P1 ? q : jj[u];                      // a cache row below tc, or tc + chunk row
            if (stays) {
                at32(pt.rank, q) = xs[u];
                at32(pt.row, xs[u]) = q;
                at32(pt.score, q) = sc[u];
            }
            bfree[u] = __ballot(is_free);
            bmov[u] = __ballot(moves);
            if (l == 0) {
                cnt_free[u * NW + w] = (uint32_t)__popcll(bfree[u]);
                cnt_mov[u * NW + w] = (uint32_t)__popcll(bmov[u]);
            }
        }
        lds_barrier();
        if (w == 0) {
            const uint32_t v = cnt_free[l], incl = wave_inclusive_sum(v);
            cnt_free[l] = incl - v;
            if (l == 63) tot_free = incl;
        } else if (w == 1) {
            const uint32_t v = cnt_mov[l], incl = wave_inclusive_sum(v);
            cnt_mov[l] = incl - v;
            if (l == 63) tot_mov = incl;
        }
        lds_barrier();
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int q = q0 + u * TPB + tid;
            if ((bfree[u] >> l) & 1ull) {
                const uint32_t k = fbase + cnt_free[u * NW + w] + lanes_below(bfree[u]);
                if (ph.on) movers[k].dst = q;
                else at32(pt.mv_dst, k) = q;
            }
            if ((bmov[u] >> l) & 1ull) {
                const uint32_t k = mbase + cnt_mov[u * NW + w] + lanes_below(bmov[u]);
                if (ph.on) {
                    movers[k].src = src[u];
                    movers[k].x = xs[u];
                    movers[k].score = sc[u];
                } else {
                    at32(pt.mv_src, k) = src[u];
                    at32(pt.mv_x, k) = xs[u];
                    at32(pt.mv_score, k) = sc[u];
                }
            }
        }
        fbase += tot_free;
        mbase += tot_mov;
        lds_barrier();                                      // the count tables are rewritten by the next pass
    };
#pragma unroll
    for (int p = 0; p < PLAN_PRE / CH; ++p) {                 // the passes whose loads were requested up front
        if (p * CH * TPB < nitems) {
            int jj[CH];
            float wv[CH];
#pragma unroll
            for (int u = 0; u < CH; ++u) { jj[u] = pre.jj[p * CH + u]; wv[u] = KPT == 0 ? pre.w[p * CH + u] : 0.f; }
            pass(p * CH * TPB, jj, wv);
        }
    }
    for (int q0 = PLAN_PRE * TPB; q0 < nitems; q0 += CH * TPB) {
        int jj[CH];
        float wv[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u) jj[u] = plan_item_token(pt.rank, q0 + u * TPB + tid, tc, P1, nitems);
#pragma unroll
        for (int u = 0; u < CH; ++u)
            wv[u] = KPT == 0 && (uint32_t)jj[u] < (uint32_t)cnd ? at32(W, jj[u]) : 0.f;
        pass(q0, jj, wv);
    }
    if (ph.on) place_movers<TPB>(movers, (int)mbase, tc, pt, ph);   // the last pass ended with a barrier
    else if (tid == 0) *pt.mv_count = (int32_t)mbase;               // = fbase: B tokens are retained, B rows lie below B
}

// Same selection with the candidates of a head held in registers (KPT keys per thread, key
// k*TPB + tid in slot k): the scores are read from memory once.  The leading bits that every key
// shares (sign and most of the exponent, as a rule) are found from the smallest and the largest
// key and skipped, so that the 8-bit digits that follow are spread over their bins and can be
// counted with plain LDS atomics, into one of two histograms: the other is cleared beside the
// bin search and a pass costs two barriers.  The digits stop as soon as the bin that holds the
// r-th largest key is wanted whole (as a rule after the second: few of a few thousand candidates
// share 16 bits), and the ordered write needs two more barriers.
template <int KPT, int TPB>
__device__ __forceinline__ void select_reg_body(const float* __restrict__ Wb, int32_t* __restrict__ userI, int32_t* __restrict__ user_count,
                                                int h, int cnd, int r, int R, int B, int cap, PlanLds<KPT, TPB>& pl)
{
    constexpr int NW = TPB / 64;
    static_assert(TPB >= 640 && HIST_WORDS / 4 <= 576, "one wavefront searches the bins while nine others clear the next histogram");
    __shared__ __attribute__((aligned(16))) uint32_t hist[2][HIST_WORDS];
    __shared__ uint32_t s_min, s_max, s_prefix, s_remaining, s_ties, s_done;
    __shared__ uint32_t tab_eq[KPT * NW], tab_gt[KPT * NW];

    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
    const float* W = Wb + (size_t)h * cap;
    int32_t* Uh = userI ? userI + (size_t)h * B : nullptr;

    if (r > 0) {
        if (tid == 0) { s_min = 0xffffffffu; s_max = 0u; s_remaining = (uint32_t)r; s_ties = (uint32_t)cnd; s_done = 0; }
        clear_hist(hist[0], tid);
        uint32_t key[KPT];
        float wj[KPT];
        uint32_t lo_key = 0xffffffffu, hi_key = 0u;
#pragma unroll
        for (int k = 0; k < KPT; ++k) wj[k] = at32(W, k * TPB + tid < cnd ? k * TPB + tid : 0);   // cnd >= 1 here
#pragma unroll
        for (int k = 0; k < KPT; ++k) {
            const int j = k * TPB + tid;
            key[k] = 0u;
            if (j < cnd) {
                key[k] = order_key(wj[k]);
                lo_key = key[k] < lo_key ? key[k] : lo_key;
                hi_key = key[k] > hi_key ? key[k] : hi_key;
            }
        }
        lo_key = wave_extreme_to_last_lane<false>(lo_key);
        hi_key = wave_extreme_to_last_lane<true>(hi_key);
        lds_barrier();
        if (l == 63) { atomicMin(&s_min, lo_key); atomicMax(&s_max, hi_key); }
        lds_barrier();
        // bits [top, 32) are the same in every key; the digits cover bits [0, top) from the top down
        const uint32_t spread = s_min ^ s_max;
        int hi = spread ? 32 - __builtin_clz(spread) : 0;
        uint32_t T = hi >= 32 ? 0u : (s_min >> hi << hi);      // the r-th largest key, as far as it is known
        for (int pass = 0; hi > 0; ++pass) {
            const int lo = hi > 8 ? hi - 8 : 0;
            uint32_t* hp = hist[pass & 1];
            const uint32_t himask = hi >= 32 ? 0u : (0xffffffffu << hi), dmask = (1u << (hi - lo)) - 1u;
#pragma unroll
            for (int k = 0; k < KPT; ++k)
                if ((k * TPB + tid < cnd) && ((key[k] & himask) == T)) count_digit(hp, (key[k] >> lo) & dmask);
            lds_barrier();
            if (tid < 64) {
                // wavefront 0 walks the bins from the top; lane l owns bins 255-4l .. 252-4l
                const u32x4_t four = four_bins(hp, 252 - 4 * l);
                const uint32_t c0 = four[3], c1 = four[2], c2 = four[1], c3 = four[0];
                const uint32_t mine = c0 + c1 + c2 + c3, incl = wave_inclusive_sum(mine);
                const uint32_t before = incl - mine, need = s_remaining;
                if (before < need && need <= incl) {          // the r-th largest falls in my bins
                    uint32_t acc = before;
                    int bin = 255 - 4 * l;
                    uint32_t cnt = c0;
                    if (acc + cnt < need) { acc += cnt; --bin; cnt = c1;
                        if (acc + cnt < need) { acc += cnt; --bin; cnt = c2;
                            if (acc + cnt < need) { acc += cnt; --bin; cnt = c3; } } }
                    s_prefix = T | ((uint32_t)bin << lo);
                    s_remaining = need - acc;                 // still to take inside that bin
                    s_ties = cnt;                             // keys in that bin
                    // the whole bin is wanted: every key >= the bin's lowest is kept, the later digits
                    // decide nothing (T = that lowest key, no tie dropped)
                    if (need - acc == cnt) s_done = 1;
                }
            } else if (tid >= TPB - 576) {
                clear_hist(hist[(pass + 1) & 1], tid - (TPB - 576));
            }
            lds_barrier();
            T = s_prefix;
            hi = s_done ? 0 : lo;
        }
        const uint32_t skip_eq = s_ties - s_remaining;        // oldest ties that are dropped

        // kept = {key > T} U {ties of rank >= skip_eq in index order}; a segment is the 64 keys of
        // slot k in wavefront w, and segments follow index order
        uint64_t beq[KPT], bgt[KPT];
#pragma unroll
        for (int k = 0; k < KPT; ++k) {
            const bool in = k * TPB + tid < cnd;
            beq[k] = __ballot(in && key[k] == T);
            bgt[k] = __ballot(in && key[k] > T);
            if (l == 0) {
                tab_eq[k * NW + w] = (uint32_t)__popcll(beq[k]);
                tab_gt[k * NW + w] = (uint32_t)__popcll(bgt[k]);
            }
        }
        lds_barrier();
        if (w == 0) wave_exclusive_table(tab_eq, KPT * NW);
        else if (w == 1) wave_exclusive_table(tab_gt, KPT * NW);
        lds_barrier();
#pragma unroll
        for (int k = 0; k < KPT; ++k) {
            const uint32_t eq_before = tab_eq[k * NW + w];
            const uint32_t eq_rank = eq_before + lanes_below(beq[k]);
            const bool keep_eq = ((beq[k] >> l) & 1ull) && eq_rank >= skip_eq;
            const int j = k * TPB + tid;
            const uint64_t bke = __ballot(keep_eq);
            // kept before this segment: every greater key, and the ties past the dropped ones
            const uint32_t seg_base = tab_gt[k * NW + w] + (eq_before > skip_eq ? eq_before - skip_eq : 0u);
            const bool keep = keep_eq || ((bgt[k] >> l) & 1ull);
            const uint32_t dst = seg_base + lanes_below(bgt[k] | bke);
            pl.cand[j] = Candidate{keep ? (int)dst : -1, wj[k]};      // for the placement plan
            if (keep && Uh) at32(Uh, dst) = j;
        }
    }
    else {
        for (int j = tid; j < cnd; j += TPB) pl.cand[j] = Candidate{-1, 0.f};     // nothing ranked
    }
    for (int x = Uh ? tid : R; x < R; x += TPB) {             // recent window: [c, n)
        at32(Uh, r + x) = cnd + x;
    }
    if (user_count && h == 0 && tid == 0) *user_count = B;
}

}  // namespace
}  // namespace infmllm
