// Internal launch interface between the C-ABI host code and the gfx950 kernels.
// Everything here is asynchronous on the given HIP stream; nothing allocates.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace infmllm {

// Every K and V buffer of the cache is followed by this many rows of padding, and the whole
// workspace is zeroed when it is attached: the matrix-core attention kernel reads whole key
// tiles and may run this far past the last cached row (into finite data it then masks).
constexpr int CACHE_PAD_ROWS = 256;

// Geometry of one stream, fixed at attach time.
struct Geometry {
    int B;        // budget (rows kept after a step)
    int R;        // recent window (newest rows always kept)
    int Hq;       // query heads
    int Hkv;      // key/value heads
    int G;        // Hq / Hkv
    int d;        // head_dim (64 or 128)
    int cap;      // physical cache rows per kv-head = B + max_decode + max_chunk
    int max_chunk;
    int max_decode;
    int elt;      // bytes per element (2 = bf16, 4 = fp32)
    double scale; // softmax scale (kernels take it, times log2(e) where they work in base 2, rounded once to float)
    double bias;  // b of Alg. 1 (the ramp step b / c is formed in double and rounded once to float)
    int policy;   // score ranked by the selection: 0 Alg. 1, 1 window, 2 initial + recent, 3 cumulative
    int attn_tile;// test hook: 0 = the matrix-core attention picks its tile shape, 1..5 = forces one
    int cut_hold; // test hook: see INFMLLM_PARAM_CUT_HOLD
};
enum { POLICY_INFMLLM = 0, POLICY_WINDOW = 1, POLICY_INITIAL_RECENT = 2, POLICY_CUMULATIVE = 3 };

// The cache of one stream.  Rows are kept where they are: an eviction does not compact K and V, it
// frees the physical rows of the evicted tokens and hands them to the retained rows that lie outside
// rows 0..B-1 (the chunk's survivors, tokens decoded since the last chunk).  Softmax attention over the
// cached keys does not depend on their order, so the attention kernels sweep physical rows 0..len-1 as
// they are; what needs the stream order (Alg. 1's slot index: the bias ramp, the tie rule, the index
// list) goes through two small tables.  The cached rows always occupy physical rows 0..len-1.
struct CacheView {
    void* K;            // [Hkv][cap][d]   by physical row
    void* V;            // [Hkv][cap][d]
    int32_t* pos;       // [Hkv][cap]      stream position of the token in each physical row
    float* score;       // [Hkv][cap]      W' the row was last retained with (+inf: never ranked)
    int32_t* rank;      // [Hkv][cap]      stream-order index (0 = oldest cached token) of each physical row
    int32_t* row;       // [Hkv][cap]      physical row of each stream-order index (inverse of rank)
};

// Retained rows an eviction has to move, per kv-head: entry k says that the token in src[k] (physical
// cache row src[k] if src[k] < tc, the rows in the cache; else row src[k] - tc of the chunk tensors)
// becomes physical row dst[k] with the new stream-order index x[k] and the score entry score[k].
// Written by the selection launch, read by the placement launch.  max = max_chunk + max_decode entries
// per head.
struct MoveList {
    int32_t* src;       // [Hkv][max]
    int32_t* dst;       // [Hkv][max]
    int32_t* x;         // [Hkv][max]
    float* score;       // [Hkv][max]
    int32_t* count;     // [Hkv]
    int max;
};

// a1 and the list of a step that evicts nothing: physical rows t..t+L-1 <- chunk; pos <- pos0..pos0+L-1; score <- +inf;
// rank and row <- identity there; list[h][j] = j for j < n (list and count may be null).  The attention kernels that
// read the chunk in place take the job along (append_share in append_body.h), else launch_append does it.
// k == nullptr: nothing to do.
struct AppendJob {
    const void *k, *v;  // chunk tensors [L][Hkv][d]
    CacheView c;
    int32_t* list;      // [Hkv][B]
    int32_t* count;
    int t, L, pos0, Hkv, cap, B, n, vec_shift;      // 2^vec_shift 16-byte vectors per row
};
AppendJob append_job(const Geometry& g, const CacheView& c, const void* k, const void* v, int t, int L, int64_t T,
                     int32_t* list, int32_t* count);
hipError_t launch_append(const AppendJob& job, hipStream_t st);

// a2 (plain fp32 arithmetic on bf16 streams, the debug override): out and per-row log-sum-exp (natural).
hipError_t launch_attn_simple(const Geometry& g, const CacheView& c, const void* q, int t, int L,
                              void* out, float* lse, hipStream_t st);

// a3+a4 (plain fp32 arithmetic on bf16 streams, the debug override): W'[h][j] for j < cnd = n - R, j = the stream-order index of a
// column (c.rank of its physical row); all n rows are in the cache here.
// With g.policy == POLICY_CUMULATIVE the score is S plus the score the row carries in c.score
// (a row never ranked carries +inf there and counts as 0) and no bias is applied.
hipError_t launch_score_simple(const Geometry& g, const CacheView& c, const void* q, const float* lse,
                               int t, int L, float* Wb, hipStream_t st);

// Scratch of the matrix-core scoring launches.
struct FwdScratch {
    // Row-split scoring: raw column sums of each split, [SCORE_SPLIT_WGS][256] fp32 (at most), followed by one
    // arrival counter per (kv-head, column block), [SCORE_SPLIT_WGS] int32, zero between launches.
    float* score_part;
};
// most workgroups a row-split scoring launch may have
constexpr int SCORE_SPLIT_WGS = 512;

// Where the keys and values of a step live.  Rows below `rows` come from the cache; rows from
// `rows` on are taken straight from the chunk tensors k, v ([L][Hkv][d]) as chunk row j - rows.
// With rows = n (after an append) the chunk pointers are never used.
struct KeySource {
    int rows;
    const void* k;
    const void* v;
};

// Partial results of attention launches whose key range is cut into pieces (attn_rows.hip): for every
// (query row, piece) the un-normalised output, the softmax reference and the sum.
struct RowsScratch {
    float* o;           // [cap_rows][d]
    float2* ml;         // [cap_rows]
    int* arrived;       // [Hkv] tickets, zero between launches
    long cap_rows;      // most (query row, piece) pairs of a launch
};

// The same of attn_fwd64 launches whose key ranges are cut in two.
constexpr int CUT_MAX_UNITS = 128;   // 256 workgroups: one round
constexpr int CUT_MIN_KEYS = 512;    // of the rows in the middle of a chunk: every piece of every unit has a tile then
struct CutScratch {
    float* part;
    int* arrived;       // [units] tickets, zero between launches; with the test hook then [units] who merged: 1 the first piece, 2 the
                        // last piece, 3 the last piece without having written its own results
    int units;          // 0: none
};

// a2 on bf16 MFMA (bf16 streams only): out and the row log-sum-exp (base 2).  With a job (ap.k set) the chunk also
// enters the cache, beside the attention.
hipError_t launch_attn_mfma(const Geometry& g, const CacheView& c, const KeySource& ks, const void* q, int t, int L,
                            void* out, float* lse, const RowsScratch& sc, const CutScratch& cut, const AppendJob& ap, hipStream_t st);

// Which kernel that is for a chunk of L rows that makes n keys (tensors aligned to 16 bytes).
const char* attn_mfma_kernel(const Geometry& g, int n, int L, long cap_rows, int cut_units);
int attn_cut_units(const Geometry& g);   // most units that a chunk's launch may cut: what a workspace should hold scratch for

// a2 and a3+a4 of fp32 streams, on the fp32 matrix cores; lse is the natural log-sum-exp.
hipError_t launch_attn_f32(const Geometry& g, const CacheView& c, const KeySource& ks, const void* q, int t, int L,
                           void* out, float* lse, const RowsScratch& sc, const AppendJob& ap, hipStream_t st);
hipError_t launch_score_f32(const Geometry& g, const CacheView& c, const KeySource& ks, const void* q, const float* lse,
                            const FwdScratch& sc, int t, int L, float* Wb, hipStream_t st);

// The same for head_dim 128 with 64 query rows per wavefront (one wavefront per SIMD, 256-row workgroups):
// the shape for long key ranges and grids that fill the chip; launch_attn_mfma picks it by itself.
// With two pieces every workgroup's key range is shared by two workgroups, at most sc.units workgroups' worth of rows, and
// the chunk enters the cache with ap.
hipError_t launch_attn_mfma64(const Geometry& g, const CacheView& c, const KeySource& ks, const void* q, int t, int L,
                              void* out, float* lse, const CutScratch& sc, int pieces, const AppendJob& ap, hipStream_t st);
int attn_mfma64_units(const Geometry& g, int L);                     // its workgroups of uncut key ranges
size_t attn_mfma64_piece_bytes();                                    // what a piece leaves for its merge

constexpr long ROWS_MAX_PARTS = 16384;
constexpr int DECODE_MAX_TOKENS = 64;    // most tokens a launch decodes
// Decoding on bf16 MFMA: T tokens in one launch (and a merging one where there are many rows); the tokens' keys and
// values become cache rows t .. t+T-1 (stream positions pos ..).  Needs Hq * T * pieces <= sc.cap_rows unless there is one piece.
// k, v null: the tokens are in the cache already.
// `keys` per piece, a constant of the stream; rows_decode_keys_per_piece proposes one that makes at most `most` pieces of the
// fullest cache.
int rows_decode_keys_per_piece(const Geometry& g, int most);
inline int rows_decode_pieces(const Geometry& g, int keys) { return (g.B + g.max_decode + keys - 1) / keys; }
hipError_t launch_rows_decode(const Geometry& g, const CacheView& c, const void* q, const void* k, const void* v, int t,
                              int T, int64_t pos, int keys, void* out, const RowsScratch& sc, hipStream_t st);
// Chunk attention (a2) with few query rows, the key range cut into pieces of plan.keys keys, workgroups of 16 * plan.nrb
// query rows, nrb <= max_nrb.  rows_chunk_plan fills the plan in and returns the time it should take, in us.
struct RowsPlan { int nrb, keys; };
float rows_chunk_plan(const Geometry& g, int n, int L, long cap_rows, int max_nrb, RowsPlan& plan);
hipError_t launch_rows_chunk(const Geometry& g, const CacheView& c, const KeySource& ks, const void* q, int t, int L,
                             void* out, float* lse, const RowsScratch& sc, const RowsPlan& plan, const AppendJob& ap,
                             hipStream_t st);

// a3+a4 on bf16 MFMA (bf16 streams only).
hipError_t launch_score_mfma(const Geometry& g, const CacheView& c, const KeySource& ks, const void* q,
                             const float* lse, const FwdScratch& sc, int t, int L, float* Wb, hipStream_t st);

// Which kernel that is for ncol columns (candidates) and lq scored rows per head.
const char* score_mfma_kernel(const Geometry& g, int ncol, int lq);

// a5+a6: user_I[h] = sort_asc(top-r of W'[h][0..cnd)) ++ [cnd, n), in stream-order indices, row stride B.  user_I
// and user_count may be null.  The same workgroup then plans the
// placement (Alg. 1 l.8 without moving the rows that stay): a retained token whose physical row is
// below B keeps it and gets its new rank, row and score entries here; the others go into the move
// list, paired in order with the physical rows the eviction frees.  tc = rows in the cache (stream-order
// indices from tc on are chunk rows read in place).  With `place` it moves them as well (ks, T as in launch_place).
hipError_t launch_select(const Geometry& g, const float* Wb, int n, int tc, int32_t* user_I,
                         int32_t* user_count, const CacheView& c, const MoveList& mv, const KeySource& ks, int64_t T, bool place,
                         hipStream_t st);
// Whether the selection also places (a7) when at most nmax rows of a head have to move; launch_place is not called then.
constexpr int PLACE_HERE_ROWS = 512;
bool place_in_select(const Geometry& g, int nmax);

// a7: copies the K and V rows of the move list to their new physical rows and writes their pos, rank,
// row and score entries.  nmax = most entries a head's list can hold in this step.
hipError_t launch_place(const Geometry& g, const CacheView& c, const KeySource& ks, int64_t T, const MoveList& mv,
                        int nmax, hipStream_t st);

// One stream's share of a batched eviction (a5-a7 for the layers of a model in one launch each,
// Alg. 1 Input note).  All streams of a batch have the same geometry.
struct EvictJob {
    const float* Wb;          // [Hkv][cap] biased scores of this stream
    int32_t* user_I;          // [Hkv][B] or null
    int32_t* user_count;      // one int or null
    CacheView c;
    MoveList mv;
    const void* kc;           // chunk tensors, stream-order indices >= tc
    const void* vc;
    int tc, pos0, n, pad_;
};
constexpr int EVICT_MAX_JOBS = 16;
struct EvictBatch {
    int count, pad_;
    EvictJob job[EVICT_MAX_JOBS];
};
hipError_t launch_select_batch(const Geometry& g, const EvictBatch& eb, bool place, hipStream_t st);
hipError_t launch_place_batch(const Geometry& g, const EvictBatch& eb, int nmax, hipStream_t st);

// Comparison policies that rank by age: W'[h][j] = sign * j for j < cnd (sign +1 keeps the newest,
// -1 the oldest).
hipError_t launch_rank_scores(const Geometry& g, float* Wb, int cnd, float sign, hipStream_t st);

// Cache-relative rotary encoding pre-pass: Krot[h][p] <- K[h][p] turned to position rank[h][p] (the row's
// stream-order index in the cache) for physical rows p in [j0, j1);
// kcrot[i][h] <- kc[i][h] and qrot[i][h] <- q[i][h] turned to position t + i for i < L (kc and q may each
// be null).  tab = [cap][d/2] pairs (cos, sin) of doubles; within a position, the entry of pair 8a + e is at
// index e * (d/16) + a, so that the threads of a row (one per a) read consecutive entries.
hipError_t launch_rope(const Geometry& g, const void* K, void* Krot, const int32_t* rank, int j0, int j1,
                       const void* kc, void* kcrot, const void* q, void* qrot, int t, int L, const double* tab,
                       hipStream_t st);

// Clears `bytes` bytes (a multiple of 16) at p (16-byte aligned) with a fill kernel, which, unlike a
// memset node, may be recorded into a HIP graph.
hipError_t launch_zero(void* p, size_t bytes, hipStream_t st);

// Decoding step in plain fp32 arithmetic (fp32 streams, bf16 ones with the plain-arithmetic override): appends the
// token's k, v as cache row t and attends all t + 1 keys with q (one
// row per query head).  The keys are cut into at most max_split pieces (decode_pieces: what the fullest cache is worth).  With
// max_split > 1 part is scratch of [Hq][max_split][d + 2] floats followed by Hkv ints that are zero
// between launches (ticket counters; the last workgroup of a kv-head to finish merges its splits), else it is not used.
constexpr int DECODE_MAX_SPLIT = 64;
int decode_pieces(const Geometry& g);
hipError_t launch_decode(const Geometry& g, const CacheView& c, const void* q, const void* k, const void* v, int t,
                         int64_t T, void* out, float* part, int max_split, hipStream_t st);

// After an import: score[h][0..len) <- +inf, rank and row <- identity.
hipError_t launch_reset_tables(const Geometry& g, const CacheView& c, int len, hipStream_t st);

// The cache in stream order (Alg. 1's K_s, V_s and their positions): out row j <- physical row c.row[h][j],
// j < len.  Kout / Vout [Hkv][len][d], pos_out / score_out [Hkv][pitch]; any of them may be null.
hipError_t launch_export(const Geometry& g, const CacheView& c, int len, void* Kout, void* Vout, int32_t* pos_out,
                         float* score_out, int pitch, hipStream_t st);

}  // namespace infmllm
