"""Tensors that start anywhere an element can: the same outputs and cache as from aligned copies."""
import pytest
import torch

from paper_2409_09086_amd import binding as B
from paper_2409_09086_amd.workloads import random_chunk

pytestmark = pytest.mark.gpu
DT = {"fp32": torch.float32, "bf16": torch.bfloat16}


def shifted(x, by):
    """Copy of x that starts `by` elements into an allocation."""
    buf = torch.empty(x.numel() + by, dtype=x.dtype, device="cuda")
    y = buf[by:].view(x.shape)
    y.copy_(x)
    assert y.data_ptr() % 16 == by * x.element_size() % 16
    return y


@pytest.mark.parametrize("by", [1, 4])
@pytest.mark.parametrize("dtype,heads,kv,d,budget,chunks,tokens,rope", [
    ("bf16", 4, 2, 128, 300, [300, 33, 130], (1, 9), None),
    ("bf16", 4, 4, 64, 300, [200, 100, 40], (1, 40), None),
    ("bf16", 16, 2, 128, 1700, [1000, 700, 867], (3,), None),          # aligned: 64 rows per workgroup, queries loaded into LDS
    ("bf16", 32, 32, 128, 2048, [1024, 1024, 2048], (), None),         # attn_fwd64
    ("bf16", 4, 2, 64, 200, [150, 50, 40], (1, 5), 10000.0),
    ("fp32", 4, 2, 64, 300, [200, 100, 70], (1, 3), None),
])
def test_tensors_need_no_alignment_beyond_their_elements(dtype, heads, kv, d, budget, chunks, tokens, rope, by):
    """Outputs within the rounding of one product (another kernel may run): 2^-7 relative and 4e-3 absolute in bf16, whose weights are
    rounded to 2^-9 of each and add up to 1 with values of size up to 4; 1e-5 in fp32.  Cache: the same bits."""
    if dtype == "fp32" and by == 4:
        by = 3
    a, b = (B.Stream(budget, budget // 4, heads, kv, d, dtype=DT[dtype], bias=1.0, max_chunk=max(chunks), max_decode=64,
                     rope_base=rope) for _ in range(2))
    tol = dict(rtol=2.0 ** -7, atol=4e-3) if dtype == "bf16" else dict(rtol=0, atol=1e-5)
    calls = [("step", L) for L in chunks] + [("decode_n", n) for n in tokens] + [("step", chunks[-1])]
    for i, (call, n) in enumerate(calls):
        print("alignment", (dtype, heads, kv, d, budget, rope, by), call, n, flush=True)
        q, k, v = (x.cuda() for x in random_chunk(4500 + i, n, heads, kv, d, dtype))
        out = shifted(torch.zeros_like(q), by)
        getattr(a, call)(shifted(q, by), shifted(k, by), shifted(v, by), out=out)
        want = getattr(b, call)(q, k, v)
        want = want[0] if call == "step" else want
        assert torch.allclose(out.float(), want.float(), **tol), (out.float() - want.float()).abs().max()
    # a bias of 1 ranks by age but for ties of no weight: both keep the same rows
    for x, y in zip(a.export()[:3], b.export()[:3]):
        assert torch.equal(x, y)
