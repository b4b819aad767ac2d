// Device side of AppendJob (launch.h): the chunk enters the cache, and the list of a step that evicts nothing is written.
//
// A launch of its own for this took 5 us and the list another 4.5 us, for 4 MB that take 1 us (1024 tokens of 8 x 128
// heads): launch, one trip to memory, drain.  The attention kernels that read the chunk in place therefore do a share each:
// attn_fwd and attn_f32 before their loop, where the trip overlaps with that of their first keys, attn_rows after it, because it has
// no registers left for it earlier, attn_rows64 in workgroups of its own, attn_fwd64 with cut key ranges by the one of two
// workgroups that does not merge.  Measured, same box: small fp32 document (4 x 64 heads, four chunks of 64 that fit, four that
// evict) 143.5 -> 121 us; fp32 document of 1280 tokens (8 x 128) 122 -> 110; bf16 document of 4500 tokens (32 heads of 128
// on 8) 303 -> 285.
#pragma once
#include "launch.h"

namespace infmllm {
namespace {

typedef uint32_t append_vec __attribute__((ext_vector_type(4)));

// Share `part` of `parts`, by nt threads of which this is number tid.  The rows written (t and up) are not read by a
// launch that reads the chunk in place.
__device__ __forceinline__ void append_share(const AppendJob& a, int part, int parts, int tid, int nt)
{
    const append_vec *k = (const append_vec*)a.k, *v = (const append_vec*)a.v;
    append_vec *K = (append_vec*)a.c.K, *V = (append_vec*)a.c.V;
    const size_t total = (size_t)a.L * a.Hkv << a.vec_shift, step = (size_t)parts * nt;
    auto row_of = [&](size_t idx, uint32_t& i) -> size_t {     // chunk row and cache row of a vector
        const uint32_t ih = (uint32_t)(idx >> a.vec_shift), h = ih % (uint32_t)a.Hkv;
        i = ih / (uint32_t)a.Hkv;
        return (size_t)h * a.cap + a.t + i;
    };
    const uint32_t xmask = (1u << a.vec_shift) - 1;
    auto put = [&](size_t idx, append_vec kx, append_vec vx) {
        uint32_t i;
        const uint32_t x = (uint32_t)idx & xmask;
        const size_t at = row_of(idx, i);
        K[(at << a.vec_shift) + x] = kx;
        V[(at << a.vec_shift) + x] = vx;
        if (x == 0) {
            a.c.pos[at] = a.pos0 + (int)i;
            a.c.score[at] = __builtin_inff();
            a.c.rank[at] = a.t + (int)i;                       // the cached rows fill physical rows 0..t-1, so the
            a.c.row[at] = a.t + (int)i;                        // next stream-order index and the next free row agree
        }
    };
    for (size_t idx = (size_t)part * nt + tid; idx < total; idx += 2 * step) {     // two rows' trips to memory at once
        const bool two = idx + step < total;
        const size_t idx1 = two ? idx + step : idx;
        const append_vec k0 = k[idx], v0 = v[idx], k1 = k[idx1], v1 = v[idx1];
        put(idx, k0, v0);
        if (two) put(idx1, k1, v1);
    }
    if (a.list) {
        const size_t entries = (size_t)a.n * a.Hkv;
        for (size_t idx = (size_t)part * nt + tid; idx < entries; idx += step) {
            const uint32_t h = (uint32_t)idx / (uint32_t)a.n, j = (uint32_t)idx - h * a.n;   // entries <= Hkv * 131072
            a.list[(size_t)h * a.B + j] = (int)j;
        }
    }
    if (a.count && part == 0 && tid == 0) *a.count = a.n;
}

}  // namespace
}  // namespace infmllm
