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
    tail = s.workspace[-((s.workspace.data_ptr() + s.workspace.numel() - 1) % 256 + 1):] if s.workspace.data_ptr() % 256 else s.workspace[-256:]
    tail = tail[-64:]                          # past the last byte the library was given, whatever the alignment
    tail.fill_(0xA5)
    ls = LockStep(s, OracleStream(budget, budget // 4, heads, kv, d))
    load_both(ls, held, 29)
    print("decode without max_decode", (dtype, impl, heads, kv, d, budget, held), flush=True)
    ls.step(*random_chunk(4400, 5, heads, kv, d, dtype))
    for i in range(4):
        ls.decode(*random_chunk(4410 + i, 1, heads, kv, d, dtype))
    ls.step(*random_chunk(4420, 7, heads, kv, d, dtype), check_state=True)
    assert (tail == 0xA5).all()


