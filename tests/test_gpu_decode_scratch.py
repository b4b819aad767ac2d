"""Decoding and the scratch it is given: the workspace holds what every call that is accepted needs."""
import numpy as np
import pytest
import torch

from oracle import OracleStream
from paper_2409_09086_amd import binding as B
from paper_2409_09086_amd.workloads import random_chunk
from _parity import LockStep

pytestmark = pytest.mark.gpu
DT = {"fp32": torch.float32, "bf16": torch.bfloat16}


def load_both(ls, n, seed):
    """A cache of n rows on both sides."""
    s = ls.gpu
    g = torch.Generator().manual_seed(seed)
    K, V = (torch.randn((s.kv_heads, n, s.head_dim), generator=g).to(s.dtype) for _ in range(2))
    pos = torch.arange(n, dtype=torch.int32).repeat(s.kv_heads, 1).contiguous()
    s.load(K.cuda(), V.cuda(), pos.cuda(), n)
    ls.oracle.load(K.double().numpy(), V.double().numpy(), pos.numpy(), n)


@pytest.mark.parametrize("dtype,impl,heads,kv,d,budget,held", [
    ("fp32", 0, 4, 2, 64, 2000, 1500),        # five pieces, after a chunk that left partials of its own
    ("fp32", 0, 2, 2, 128, 200, 60),          # one piece: nothing to merge
    ("bf16", 1, 6, 2, 64, 1500, 1200),
    ("bf16", 1, 1, 1, 128, 300, 100),
    ("bf16", 0, 8, 2, 128, 2000, 1500),
])
def test_decoding_below_the_budget_without_max_decode(dtype, impl, heads, kv, d, budget, held):
    """Accepted while the cache is below its budget.  What lies behind the workspace stays as it is."""
    s = B.Stream(budget, budget // 4, heads, kv, d, dtype=DT[dtype], impl=impl, max_chunk=16)
    assert s.workspace.data_ptr() % 256 == 0
    tail = s.workspace[-256:]                  # the binding allocates 256 bytes more than it hands over
    tail.fill_(0xA5)
    ls = LockStep(s, OracleStream(budget, budget // 4, heads, kv, d))
    load_both(ls, held, 29)
    print("decode without max_decode", (dtype, impl, heads, kv, d, budget, held), flush=True)
    ls.step(*random_chunk(4400, 5, heads, kv, d, dtype))
    for i in range(4):
        ls.decode(*random_chunk(4410 + i, 1, heads, kv, d, dtype))
    ls.step(*random_chunk(4420, 7, heads, kv, d, dtype), check_state=True)
    assert (tail == 0xA5).all()


def largest_static_budget(heads, kv, d, elt, max_chunk):
    """Largest budget whose cache, tables, move lists, scores, one index list and (bf16) row-split scoring sums, max_decode =
    0, fit the library's array."""
    up = lambda x: (x + 255) // 256 * 256

    def need(b):
        rows = b + max_chunk
        return (2 * up((kv * rows + 256) * d * elt) + 5 * up(kv * rows * 4) + up(heads * max_chunk * 4) + 4 * up(kv * max_chunk * 4) +
                up(kv * 4) + up(kv * b * 4) + (up(512 * 257 * 4) if elt == 2 else 0))
    return max(b for b in range(1, 131072 - max_chunk) if need(b) <= 64 << 20)


@pytest.mark.parametrize("dtype,heads,kv,d", [
    ("fp32", 4, 4, 128),                      # partials for all pieces fit
    ("bf16", 64, 1, 128),                     # for fourteen of sixteen
    ("bf16", 512, 1, 128),                    # for none: one piece
    ("bf16", 32, 8, 128),
])
def test_streams_that_fill_the_static_workspace_decode(dtype, heads, kv, d):
    """Such a stream is accepted, and its tokens are those of a twin with a workspace of its own, whose keys are cut
    otherwise, to the rounding of an output (2^-8, both sides) and of sums of weights that add up to 1 (2e-5)."""
    budget = largest_static_budget(heads, kv, d, 4 if dtype == "fp32" else 2, 16)
    a, b = (B.Stream(budget, budget // 4, heads, kv, d, dtype=DT[dtype], max_chunk=16, static_workspace=x) for x in (True, False))
    g = torch.Generator(device="cuda").manual_seed(31)
    K, V = (torch.randn((kv, budget - 10, d), generator=g, device="cuda").to(a.dtype) for _ in range(2))
    pos = torch.arange(budget - 10, dtype=torch.int32, device="cuda").repeat(kv, 1).contiguous()
    for s in (a, b):
        s.load(K, V, pos, budget - 10)
    print("full static workspace", (dtype, heads, kv, d, budget), flush=True)
    for call, n in enumerate((1, 9)):
        x = [y.cuda() for y in random_chunk(4430 + call, n, heads, kv, d, dtype)]
        assert torch.allclose(a.decode_n(*x).double(), b.decode_n(*x).double(), rtol=2.0 ** -7 if dtype == "bf16" else 0, atol=2e-5)
    for x, y in zip(a.export(), b.export()):
        assert torch.equal(x, y)
    x = [y.cuda() for y in random_chunk(4440, 16, heads, kv, d, dtype)]
    assert torch.allclose(a.step(*x)[0].double(), b.step(*x)[0].double(), rtol=2.0 ** -6 if dtype == "bf16" else 0, atol=2e-4)
    torch.cuda.synchronize()
    a.close()


@pytest.mark.parametrize("heads,kv,d,budget", [(1, 1, 128, 50000), (4, 1, 64, 20000), (2, 2, 64, 25000), (4, 4, 128, 20000)])
def test_long_caches_of_few_heads_are_cut_into_more_than_sixteen_pieces(heads, kv, d, budget):
    """Tokens one by one (a ticketed merge) and together (a merging launch): the same bits, and the oracle's values to a
    rounding of the output and 2e-5 for the sums (see test_tokens_do_not_depend_on_how_many_share_a_call)."""
    a, b = (B.Stream(budget, budget // 4, heads, kv, d, dtype=torch.bfloat16, max_chunk=16, max_decode=24) for _ in range(2))
    ls = LockStep(a, OracleStream(budget, budget // 4, heads, kv, d))
    load_both(ls, budget, 37)
    b.load(*a.export()[:3], budget)
    for call, n in enumerate((1, 6, 17)):
        print("long cache", (heads, kv, d, budget), "tokens", n, flush=True)
        x = random_chunk(4450 + call, n, heads, kv, d, "bf16")
        out = a.decode_n(*(y.cuda() for y in x))
        one = torch.cat([b.decode(*(y[i:i + 1].contiguous().cuda() for y in x)) for i in range(n)])
        assert torch.equal(out.view(torch.int16), one.view(torch.int16))
        ref = np.concatenate([ls.oracle.decode(*(y[i:i + 1].double().numpy() for y in x)) for i in range(n)])
        err = np.abs(out.double().cpu().numpy() - ref)
        assert (err <= 2.0 ** -8 * np.abs(ref) + 2e-5).all(), err.max()
