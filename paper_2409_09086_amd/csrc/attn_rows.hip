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

#include "append_body.h"
#include "attn_rows.h"

namespace infmllm {

namespace {

template <int D, int NRB, bool EXACT, bool APPEND>
__global__ void __launch_bounds__(RW_NT, D == 64 ? 4 : 2)       // head_dim 64: two workgroups per CU (CAREFUL spills then)
attn_rows_kernel(RowsArgs a, AppendJob ap)
{
    using C = RowsCfg<D, NRB>;
    __shared__ __attribute__((aligned(1024))) char smem[(RW_NW + 1) * C::STAGE];   // a run of K and V per wavefront, two for the first one
    __shared__ float s_m[RW_NW][C::ROWS], s_l[RW_NW][C::ROWS];
    __shared__ int s_ticket;
    __shared__ float2 s_part[NRB == 1 ? RW_TICKET_PARTS : 1];

    // Workgroup = (piece, kv-head, row group), the piece fastest and the row group slowest: the row groups of a piece, which
    // read the same keys, land on one XCD where the number of (piece, head) pairs is a multiple of 8.  Groups of 32 rows may take
    // several rounds of the chip, over more keys and values than the L2s hold (32 MB); they then get neighbouring ids of one residue
    // class mod 8, i.e. one XCD at one time, so that a key comes into its L2 once.  us with the merge: 64 tokens over 8256 rows of 32
    // heads, 134 MB, 384 workgroups 48.0 -> 43.5; 40 over 8232 46.1 -> 42.9; not where they fit: 64 over 2112 of 32 heads 26.6 / 26.9, 34
    // tokens of 32 heads on 8 over 4130 30.1 / 31.4.  (The host says so: the grid's size is a trip to memory ahead of the first keys.)
    const int t = a.t;
    int sp = blockIdx.x, h = blockIdx.y, rg = blockIdx.z;
    if constexpr (NRB == 2) {
        if (a.beside) {                                        // row groups of the launch
            const unsigned ns = (unsigned)a.nsplit, groups = (unsigned)a.beside;
            const unsigned id = blockIdx.x + ns * (blockIdx.y + (unsigned)a.Hkv * blockIdx.z), li = id >> 3;
            const unsigned pair = li / groups * 8 + (id & 7);
            rg = (int)(li % groups);
            h = (int)(pair / ns);
            sp = (int)(pair % ns);
        }
    }
    const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.L * a.G, row0 = rg * C::ROWS;
    auto token = [&](int rho) -> int { return rows_token(a, rho); };
    const int first_lim = t + token(row0);                     // last key the group's first row sees
    const int n_end = t + token(min(row0 + C::ROWS, M) - 1) + 1;
    const int k_end = min((sp + 1) * a.ks, n_end);

    const RunLoader<uint16_t, D, RW_RUN> runs(a, h, lane);
    char* const mine = smem + wave * C::STAGE;
    auto load_run = [&](int k0, char* dst) { runs.template load<true, true>(k0, dst); };
    const int k_first = sp * a.ks + wave * RW_RUN;
    const int np = k_end > k_first ? (k_end - k_first + RW_PASS - 1) / RW_PASS : 0;
    // wavefront 0, which has a run more than the others if any has, has a second stage for its odd runs
    const int nst = wave == 0 ? 2 : 1;
    const uint32_t stage1 = wave == 0 ? RW_NW * C::STAGE : 0;
    auto load_first = [&]() {
        if (np > 0) load_run(k_first, mine);
        if (nst == 2 && np > 1) load_run(k_first + RW_PASS, mine + stage1);
    };
    load_first();
    // query fragments: B operand of S^T = K.Q^T, lane (row c16, group g4) holds Q[row][32s + 8 g4 .. +8)
    bf16x8 qf[NRB][C::NS];
    int lim[NRB];
    auto query_row = [&](int x, int& tok) -> const uint16_t* {
        const int rho = min(row0 + 16 * x + c16, M - 1);
        tok = token(rho);
        return a.q + ((size_t)tok * a.Hq + h * a.G + (rho - tok * a.G)) * D + 8 * g4;
    };
#pragma unroll
    for (int x = 0; x < NRB; ++x) {
        int tok;
        const uint16_t* qp = query_row(x, tok);
        lim[x] = t + tok;
#pragma unroll
        for (int s = 0; s < C::NS; ++s) qf[x][s] = as_bf16x8(*(const u32x4*)(qp + 32 * s));
    }

    f32x4 o[NRB][C::NC];
    float m_ref[NRB], m_use[NRB], lsum[NRB];
    // K fragments: lane (row c16, group g4) reads piece 4s + g4.  V: a 16-lane group reads keys 4 g4 .. +3 (then
    // 16 + 4 g4 .. +3) of sixteen columns; lane l of the group supplies the address of key l / 4, columns 4 (l % 4).
    uint32_t kaddr[C::NS], vaddr[C::NC];
    {
        const uint32_t base = (uint32_t)(uintptr_t)(lds_void*)mine;
        const int vkey = 4 * g4 + (c16 >> 2), q4 = c16 & 3;    // swz(key + 16) = swz(key)
#pragma unroll
        for (int s = 0; s < C::NS; ++s) kaddr[s] = base + c16 * C::ROWB + (((4 * s + g4) ^ swz_k<D>(c16)) * 16);
#pragma unroll
        for (int b = 0; b < C::NC; ++b)
            vaddr[b] = base + C::RUN + vkey * C::ROWB + (((2 * b + (q4 >> 1)) ^ swz_v<D>(vkey)) * 16) + 8 * (q4 & 1);
    }

    // A hidden key's weight is 0, but 0 times a value that is not finite is NaN, in every row of the group; and such a value
    // times a weight's three terms is not its product with the weight.  Both show in the accumulators.  A wavefront of a
    // decoding launch that finds them not finite goes through its keys again (CAREFUL): the rows that see the same number
    // of a run's keys at a time, hidden values replaced by 0, values that are not finite taken by a weight's first term alone.  What
    // is finite comes out with the same bits, so that a token's output does not depend on the tokens decoded with it.
    auto sweep = [&](auto careful) __attribute__((always_inline)) {
        constexpr bool CAREFUL = decltype(careful)::value;
#pragma unroll
        for (int x = 0; x < NRB; ++x) {
#pragma unroll
            for (int b = 0; b < C::NC; ++b) o[x][b] = f32x4{0.f, 0.f, 0.f, 0.f};
            m_ref[x] = -__builtin_inff(); m_use[x] = 0.f; lsum[x] = 0.f;
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
                kf[0][s] = rw_read_b128<0, CAREFUL>(kaddr[s] + stage);
                kf[1][s] = rw_read_b128<16 * C::ROWB, CAREFUL>(kaddr[s] + stage);
            }
#pragma unroll
            for (int b = 0; b < C::NC; ++b) {
                vlo[b] = rw_read_tr16<0, CAREFUL>(vaddr[b] + stage);
                vhi[b] = rw_read_tr16<16 * C::ROWB, CAREFUL>(vaddr[b] + stage);
            }
            // reads return in order: K has arrived when at most the V reads are outstanding (the counter ends at 15)
            asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(kf[0][0]), "+v"(kf[1][0]), "+v"(kf[0][1]), "+v"(kf[1][1])
                         : "n"(2 * C::NC < 15 ? 2 * C::NC : 15));
            if constexpr (C::NS == 4) asm volatile("" : "+v"(kf[0][2]), "+v"(kf[1][2]), "+v"(kf[0][3]), "+v"(kf[1][3]));
            // ---- S^T = K.Q^T
            f32x4 S[NRB][2];
            if constexpr (CAREFUL) {                           // the registers are wanted below
#pragma unroll
                for (int x = 0; x < NRB; ++x) {
                    int tok;
                    const uint16_t* qp = query_row(x, tok);
#pragma unroll
                    for (int s = 0; s < C::NS; ++s) qf[x][s] = as_bf16x8(*(const u32x4*)(qp + 32 * s));
                }
            }
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
                if constexpr (CAREFUL) {                       // ---- O^T += V^T.P^T, see above
                    const int last = max(min(lim[x] - k0, RW_RUN - 1), -1);    // last key of the run that the row sees, -1: none
#pragma nounroll
                    for (int end = 0; end < RW_RUN; ++end) {
                        if (!__any(last == end)) continue;
#pragma unroll
                        for (int b = 0; b < C::NC; ++b) {
                            const bf16x8 v = __builtin_shufflevector(vlo[b], vhi[b], 0, 1, 2, 3, 4, 5, 6, 7);
                            u32x4 vis = __builtin_bit_cast(u32x4, v), fin;
#pragma unroll
                            for (int e = 0; e < 4; ++e) {      // elements 2e and 2e + 1: two consecutive keys
                                const int key = 4 * g4 + (e < 2 ? 2 * e : 2 * e + 12);
                                vis[e] &= key + 1 <= end ? ~0u : (key <= end ? 0xffffu : 0u);
                                const uint32_t inf = 0x7f80u;
                                fin[e] = vis[e] & (((vis[e] & inf) == inf ? 0u : 0xffffu) | (((vis[e] >> 16) & inf) == inf ? 0u : 0xffff0000u));
                            }
                            f32x4 sum = mfma16(as_bf16x8(vis), pf[x][0], o[x][b]);
#pragma unroll
                            for (int term = 1; term < (EXACT ? 3 : 1); ++term) sum = mfma16(as_bf16x8(fin), pf[x][term], sum);
                            if (last == end) o[x][b] = sum;
                        }
                    }
                }
            }
            // ---- O^T += V^T.P^T
            if constexpr (!CAREFUL) {
#pragma unroll
                for (int b = 0; b < C::NC; ++b) {
                    const bf16x8 vf = __builtin_shufflevector(vlo[b], vhi[b], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                    for (int term = 0; term < (EXACT ? 3 : 1); ++term)
#pragma unroll
                        for (int x = 0; x < NRB; ++x) o[x][b] = mfma16(vf, pf[x][term], o[x][b]);
                }
            }
        }
    };
    sweep(std::false_type{});
    if constexpr (APPEND)
        append_share(ap, sp + gridDim.x * (h + gridDim.y * rg), gridDim.x * gridDim.y * gridDim.z, tid, RW_NT);
    // ---- decoding: tokens sp, sp + nsplit, .. become cache rows (read from the chunk tensors by everyone).  Where the last workgroup
    // of a kv-head merges the pieces there is time for it while the partials are on their way, and the wavefront with the fewest
    // keys does it first (ahead of the merge of the wavefronts 24 tokens after a prompt took 234.2 instead of 230.7 us); whole rows
    // have gone to out by then, and the caller keeps out off k and v where the keys make one piece.  Groups of 32 rows are merged
    // by a second launch, which waits for all of it: there it comes ahead (29 tokens of 8 x 64 heads on 2 over 3829 rows 12.9 against 13.2 us).
    auto append_tokens = [&]() __attribute__((always_inline)) {
        if (!a.pos || rg != 0 || sp >= a.L) return;
        constexpr int VPR = D / 8;
        const int from_last = NRB == 1 ? tid ^ (RW_NT - 64) : tid;
        for (int i = sp + a.nsplit * (from_last / VPR); i < a.L; i += a.nsplit * (RW_NT / VPR)) {
            const int x = from_last % VPR;
            const size_t dst = ((size_t)h * a.cap + t + i) * D + x * 8, src = (size_t)i * runs.crs + x * 8;
            *(u32x4*)(a.K + dst) = *(const u32x4*)(runs.kch + src);
            *(u32x4*)(a.V + dst) = *(const u32x4*)(runs.vch + src);
            if (x == 0) {
                const size_t at = (size_t)h * a.cap + t + i;
                a.pos[at] = a.pos0 + i;
                a.score[at] = __builtin_inff();
                a.rank[at] = t + i;                            // the newest tokens, in the next free physical rows
                a.row[at] = t + i;
            }
        }
    };
    if constexpr (NRB == 2) append_tokens();
    // ---- merge the wavefronts: lane (row c16, group g4) holds O[row][16b + 4 g4 + i]
    // wavefront w's share: 16-byte piece p of row r in slot p ^ ((r ^ w) & 7) of the row, which keeps both eight rows and
    // eight wavefronts apart in the banks; rows that do not exist are left out
    auto merged = [&](int w, int r, int p) -> char* {
        return smem + w * C::STAGE + r * (D * 4) + ((p ^ ((r ^ w) & 7)) * 16);
    };
    const int rows = min(C::ROWS, M - row0);
    auto leave_share = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < NRB; ++x) {
            const float l = groups_sum(lsum[x]);
            if (g4 == 0) { s_m[wave][16 * x + c16] = m_ref[x]; s_l[wave][16 * x + c16] = l; }
        }
#pragma unroll
        for (int x = 0; x < NRB; ++x)
            if (16 * x + c16 < rows) {
#pragma unroll
                for (int b = 0; b < C::NC; ++b) *(f32x4*)merged(wave, 16 * x + c16, 4 * b + g4) = o[x][b];
            }
    };
    leave_share();
    if constexpr (EXACT) {
        float z = 0.f;                                         // beside the stores (0.08 us less than ahead of them): see sweep
#pragma unroll
        for (int x = 0; x < NRB; ++x)
#pragma unroll
            for (int b = 0; b < C::NC; ++b)
#pragma unroll
                for (int i = 0; i < 4; ++i) z = __builtin_fmaf(o[x][b][i], 0.f, z);
        if (__builtin_expect(__any(z != 0.f), 0)) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // the share lies where the first runs go
            load_first();
            sweep(std::true_type{});
            leave_share();
        }
    }
    __syncthreads();
    if (NRB == 1 && rows <= 4) {                               // eight lanes, one wavefront's share each
        for (int x = tid / RW_NW; x < rows * (D / 4); x += RW_NT / RW_NW) {
            const int r = x / (D / 4), d = 4 * (x % (D / 4)), w = tid % RW_NW;
            PieceSum ps{s_m[w][r], s_l[w][r], *(const f32x4*)merged(w, r, d / 4)};
            ps.add_lanes<RW_NW>();
            if (w == 0) leave_row<D>(a, h, sp, row0 + r, d, ps);
        }
    } else {
        for (int x = tid; x < rows * (D / 4); x += RW_NT) {
            const int r = x / (D / 4), d = 4 * (x % (D / 4));
            PieceSum ps[RW_NW];
#pragma unroll
            for (int w = 0; w < RW_NW; ++w) ps[w] = PieceSum{s_m[w][r], s_l[w][r], *(const f32x4*)merged(w, r, d / 4)};
            leave_row<D>(a, h, sp, row0 + r, d, add_tree(ps));
        }
    }
    if constexpr (NRB == 1) append_tokens();
    if (a.nsplit == 1 || !a.arrived) return;
    if constexpr (NRB == 1) {                                  // tickets are given out with a single row group only
        // Every workgroup waits until its own partials have been written through, then takes a ticket; the one of this
        // kv-head that arrives last merges the pieces.  No workgroup waits for another one.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) s_ticket = __hip_atomic_fetch_add(a.arrived + h, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (s_ticket != a.nsplit - 1) return;
        if (tid == 0) __hip_atomic_store(a.arrived + h, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch
        // One trip to memory for the partials of all rows (at most RW_TICKET_PARTS of them); then sixteen lanes per four
        // columns of a row, one class of pieces each.  With a piece to a class and up to four rows every thread takes what it
        // adds straight into its registers, else they go through LDS (32 heads on 8, 4096 rows 9.7 instead of 9.4 us a token;
        // 16 x 64 heads, 2048 rows 6.7 / 6.5).
        const int parts = M * a.nsplit;
        const size_t at = (size_t)h * parts;
        auto store_row = [&](int r, int d, const PieceSum& ps) {
            const int tok = token(r), gq = h * a.G + r - tok * a.G;
            store_out4(a.out + ((size_t)tok * a.Hq + gq) * D + d, ps.out());
            if (a.lse && d == 0) a.lse[(size_t)gq * a.max_chunk + tok] = ps.lse();
        };
        constexpr int DIRECT = 4, PER_ROW = D / 4 * RW_CLASSES;
        static_assert(PER_ROW % RW_NT == 0 || RW_NT % PER_ROW == 0, "a row takes whole rounds of the threads, or a round whole rows");
        auto direct = [&](auto rounds) __attribute__((always_inline)) {   // of the threads over the rows
            constexpr int U = decltype(rounds)::value;
            const int c = tid % RW_CLASSES, cc = min(c, a.nsplit - 1);
            const auto src = __builtin_amdgcn_make_buffer_rsrc((void*)(a.part_o + at * D), 0, parts * D * 4, 0x00020000);
            float2 ml[U];
            u32x4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int x = tid / RW_CLASSES + u * (RW_NT / RW_CLASSES), r = min(x / (D / 4), M - 1), d4 = x % (D / 4);
                ml[u] = part_load2<true>(a.part_ml + at + r * a.nsplit + cc);
                v[u] = __builtin_amdgcn_raw_buffer_load_b128(src, ((r * a.nsplit + cc) * (D / 4) + d4) * 16, 0, 16 /* sc1 */);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int x = tid / RW_CLASSES + u * (RW_NT / RW_CLASSES), r = x / (D / 4);
                if (r >= M) break;                             // uniform over the sixteen lanes
                PieceSum ps{-__builtin_inff(), 0.f, f32x4{0.f, 0.f, 0.f, 0.f}};
                if (c < a.nsplit) ps.absorb(ml[u], __builtin_bit_cast(f32x4, v[u]));
                ps.add_lanes<RW_CLASSES>();
                if (c == 0) store_row(r, 4 * (x % (D / 4)), ps);
            }
        };
        if (a.nsplit <= RW_CLASSES && M <= DIRECT) {
            constexpr int ALL = DIRECT * PER_ROW / RW_NT;
            if (M * PER_ROW <= RW_NT) direct(std::integral_constant<int, 1>{});
            else if (ALL > 2 && M * PER_ROW <= 2 * RW_NT) direct(std::integral_constant<int, 2>{});
            else direct(std::integral_constant<int, ALL>{});
            return;
        }
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
            if (c == 0) store_row(r, d, ps);
        }
    }
}

template <int D, int NRB, bool EXACT>
void launch_rows_cfg(RowsArgs a, const AppendJob& ap, hipStream_t st)
{
    constexpr int ROWS = 16 * NRB;
    const dim3 grid((unsigned)a.nsplit, (unsigned)a.Hkv, (unsigned)((a.L * a.G + ROWS - 1) / ROWS));
    const unsigned pairs = grid.x * grid.y;
    a.beside = NRB == 2 && pairs * grid.z > (D == 64 ? 512u : 256u) && pairs % 8 == 0 && (uint64_t)(a.t + a.L) * a.Hkv * (D * 4) > (48u << 20)
                   ? (int)grid.z : 0;
    if constexpr (!EXACT)
        if (ap.k) {
            hipLaunchKernelGGL((attn_rows_kernel<D, NRB, false, true>), grid, dim3(RW_NT), 0, st, a, ap);
            return;
        }
    hipLaunchKernelGGL((attn_rows_kernel<D, NRB, EXACT, false>), grid, dim3(RW_NT), 0, st, a, ap);
}

template <int D, bool EXACT>
hipError_t launch_rows_d(const RowsArgs& args, int nrb, const AppendJob& ap, hipStream_t st)
{
    RowsArgs a = args;
    a.inv_g = rows_inv_g(a.L, a.G);
    if (nrb == 1) launch_rows_cfg<D, 1, EXACT>(a, ap, st);
    else if (EXACT || nrb == 2) launch_rows_cfg<D, 2, EXACT>(a, ap, st);
    else if constexpr (D == 128) launch_rows64(a, ap, st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.nsplit == 1 || a.arrived) return e;
    launch_merge_rows<uint16_t, D, false>(a, st);
    return hipGetLastError();
}

}  // namespace

int rows_decode_keys_per_piece(const Geometry& g, int most)
{
    // A function of the stream's geometry alone (see EXACT above): a whole number of runs, about 192 workgroups with
    // the cache at its fullest, as a rule a merge of at most sixteen pieces, and at least one run per wavefront.  Measured at 32 x 128
    // heads and 2048 + 48 rows: 13.2 us per token with 256 keys per piece, 11.8 with 288 (256 workgroups), 10.9 with 352
    // (192), 10.6 with 384, 11.6 with 576 (128); 4096 rows: 20.7 with 288, 17.1 with 544, 16.4 with 704 (192), 17.0 with
    // 1408; 8 kv-heads and 4096 rows: 12.3 with 256, 12.0 with 288, 13.3 with 704.
    // Few kv-heads leave CUs without a piece, which long caches show.  Where a token's rows fill a row group four times over at
    // most, they are cut into up to 64 pieces of 768 keys or more, as long as two row groups of each fit on the chip.  One token
    // (16 together), us, with sixteen pieces / 32 / 64: 1 kv-head, 1 x 128 heads, 32768 rows 14.9 (27) / 10.7 (21) / 8.7 (28),
    // 130000 rows 45 (57) / 27 (36) / 18 (35); 4 heads on 1, 130000 rows 47 (68) / 29 (47) / 21 (44); 16 on 4, 32768 rows
    // 19.2 (28) / 17.1 (28) / 48 pieces 18.0 (46).  Not with more heads to a kv-head: 8 on 1, 32768 rows 18.9 (27) / 16.0 (27),
    // but 32 on 4, 16384 rows 15.3 (22) and with 21 pieces 15.2 (34).
    const int rows = g.B + g.max_decode, longs = g.G <= 4 ? std::min({rows / 768, 128 / g.Hkv, 4 * RW_CLASSES}) : 1;
    const int pieces = std::max(1, std::min(std::max(std::min(192 / g.Hkv, RW_CLASSES), longs), most));
    const int ks = ((rows + pieces - 1) / pieces + RW_RUN - 1) / RW_RUN * RW_RUN;
    return ks < 256 ? 256 : ks;
}

hipError_t launch_rows_decode(const Geometry& g, const CacheView& c, const void* q, const void* k, const void* v, int t,
                              int T, int64_t pos, int keys, void* out, const RowsScratch& sc, hipStream_t st)
{
    RowsArgs a{};
    a.q = (const uint16_t*)q; a.K = (uint16_t*)c.K; a.V = (uint16_t*)c.V;
    a.kc = (const uint16_t*)k; a.vc = (const uint16_t*)v; a.out = (uint16_t*)out; a.lse = nullptr;
    a.part_o = sc.o; a.part_ml = sc.ml;
    a.pos = k ? c.pos : nullptr; a.score = c.score; a.rank = c.rank; a.row = c.row; a.pos0 = (int)pos;
    a.t = t; a.L = T; a.tc = k ? t : t + T; a.Hq = g.Hq; a.Hkv = g.Hkv; a.G = g.G; a.cap = g.cap; a.max_chunk = g.max_chunk;
    a.ks = keys;
    a.nsplit = (t + T + a.ks - 1) / a.ks;
    a.c = (float)(g.scale * (double)LOG2E);
    if (a.nsplit > 1 && (long)g.Hq * T * a.nsplit > sc.cap_rows) return hipErrorInvalidValue;
    const int M = T * g.G, nrb = M <= 16 ? 1 : 2;
    a.arrived = M <= 16 && M * a.nsplit <= RW_TICKET_PARTS ? sc.arrived : nullptr;
    if (g.d == 128) return launch_rows_d<128, true>(a, nrb, AppendJob{}, st);
    if (g.d == 64) return launch_rows_d<64, true>(a, nrb, AppendJob{}, st);
    return hipErrorInvalidValue;
}

// Time (us, between two events) that a chunk of L rows over n keys should take in this kernel, and the shape for it.
// Fitted to measurements at 500..8500 keys and 32..512 workgroups, within about 10 %: a part that does not depend on the
// keys, a pass of 256 keys per round of 256 workgroups, the partials and the merging launch of a cut key range, and
// never less than the cache takes to come in.  (32 heads of 128 on 4 kv-heads, measured / this: 16 rows per workgroup,
// 128 workgroups, 2064 keys 16.4 / 18.3; 256 workgroups, 8128 keys 45.4 / 44.0; 32 rows, 256 workgroups, 4256 keys
// 34.1 / 34.0; 512 workgroups, 4512 keys 63.7 / 63.3; four pieces, 256 workgroups, 8064 keys 25.2 / 25.0; 64 rows,
// 256 workgroups, 4608 keys 51.7 / 49.3, 2560 keys 36.6 / 34.3; at head_dim 64 rows of 64 gain nothing over 32: 24.9 and
// 24.8 us for 32 heads, 512 rows, 2560 keys.)
float rows_chunk_plan(const Geometry& g, int n, int L, long cap_rows, int max_nrb, RowsPlan& plan)
{
    struct Cost { float fixed, more_rounds, pass; };
    static constexpr Cost COST[2][3] = {{{6.5f, 1.f, 0.66f}, {8.7f, 1.f, 0.85f}, {}},                      // head_dim 64: 16, 32 rows
                                        {{8.2f, 4.f, 1.12f}, {11.4f, 4.f, 1.33f}, {15.5f, 8.f, 1.88f}}};   // 128: 16, 32, 64
    const float floor_us = 6.f + (float)n * g.Hkv * g.d * 4.f / 5.5e6f;
    float best = 1e30f;
    for (int i = 0; i < (g.d == 128 ? 3 : 2); ++i) {
        const int nrb = 1 << i;
        if (nrb > max_nrb) break;
        const Cost& c = COST[g.d == 128][i];
        const long units = (long)g.Hkv * ((L * g.G + 16 * nrb - 1) / (16 * nrb));       // workgroups per piece
        const long most = std::min<long>(std::min<long>(256 / units, (n + 255) / 256), cap_rows / ((long)g.Hq * L));
        for (int pieces = 1; pieces == 1 || pieces <= std::min<long>(most, RW_CLASSES); ++pieces) {
            const int keys = ((n + pieces - 1) / pieces + RW_RUN - 1) / RW_RUN * RW_RUN;
            const float rounds = (float)((units * pieces + 255) / 256);
            if (nrb == 4 && rounds > 1.f) continue;            // attn_fwd is as good or better: 100 / 109 us at 4 x 8 heads, 1077 rows
            float us = c.fixed + c.more_rounds * (rounds - 1.f) + rounds * c.pass * (float)((keys + RW_PASS - 1) / RW_PASS);
            if (us < floor_us) us = floor_us;
            if (pieces > 1) us += 1.2f + 0.45f * (float)pieces;
            if (us < best) { best = us; plan = RowsPlan{nrb, keys}; }
        }
    }
    return best;
}

hipError_t launch_rows_chunk(const Geometry& g, const CacheView& c, const KeySource& ks, const void* q, int t, int L,
                             void* out, float* lse, const RowsScratch& sc, const RowsPlan& plan, const AppendJob& ap,
                             hipStream_t st)
{
    RowsArgs a{};
    a.q = (const uint16_t*)q; a.K = (uint16_t*)c.K; a.V = (uint16_t*)c.V;
    a.kc = (const uint16_t*)ks.k; a.vc = (const uint16_t*)ks.v; a.out = (uint16_t*)out; a.lse = lse;
    a.part_o = sc.o; a.part_ml = sc.ml;
    a.t = t; a.L = L; a.tc = ks.rows; a.Hq = g.Hq; a.Hkv = g.Hkv; a.G = g.G; a.cap = g.cap; a.max_chunk = g.max_chunk;
    a.ks = plan.keys;
    a.nsplit = (t + L + plan.keys - 1) / plan.keys;
    a.c = (float)(g.scale * (double)LOG2E);
    if (a.nsplit > 1 && (long)g.Hq * L * a.nsplit > sc.cap_rows) return hipErrorInvalidValue;
    a.arrived = plan.nrb == 1 && L * g.G <= 16 && L * g.G * a.nsplit <= RW_TICKET_PARTS ? sc.arrived : nullptr;
    if (g.d == 128) return launch_rows_d<128, false>(a, plan.nrb, ap, st);
    if (g.d == 64) return launch_rows_d<64, false>(a, plan.nrb, ap, st);
    return hipErrorInvalidValue;
}

}  // namespace infmllm
