"""Kernels that only larger shapes reach, at the smallest ones that do; each test asserts which kernel runs."""
import numpy as np
import pytest
import torch

from oracle import OracleStream
from paper_2409_09086_amd import binding as B
from paper_2409_09086_amd.workloads import random_chunk
from _parity import LockStep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,kv,budget,chunks,tile", [
    (4, 2, 300, [100, 37, 163, 129, 300, 1], 1),              # forced: ragged chunks that fit, then evicting ones
    (8, 8, 200, [1, 130, 69, 129, 64], 1),
    (6, 2, 257, [257, 128, 3], 1),                            # three heads to a group
    (32, 8, 1024, [1024, 1024, 777], None),                   # by the launch's own rule
])
def test_attn_fwd_of_head_dim_64(heads, kv, budget, chunks, tile):
    recent, d = budget // 4, 64
    gpu = B.Stream(budget, recent, heads, kv, d, dtype=torch.bfloat16, bias=1e-3, max_chunk=max(chunks), attn_tile=tile)
    ls = LockStep(gpu, OracleStream(budget, recent, heads, kv, d, bias=1e-3))
    for step, L in enumerate(chunks):
        print("attn_fwd d64", (heads, kv, budget, tile), "step", step, "L", L, flush=True)
        if tile or L > 1000:
            assert gpu.kernel("attn", len(gpu), L) == "attn_fwd"
        ls.step(*random_chunk(4600 + step, L, heads, kv, d, "bf16"), check_state=True)


@pytest.mark.parametrize("heads,kv,d,budget,L,kernel", [
    (24, 24, 64, 1300, 159, "score_kernel"),                  # 256 columns per workgroup
    (24, 24, 128, 1300, 159, "score_kernel"),
    (40, 40, 128, 2560, 159, "score_kernel"),                 # 512 columns
    (16, 4, 64, 9000, 1055, "score_kernel"),                  # more scored rows than it keeps log-sum-exps of in LDS (4096)
    (3, 3, 64, 9000, 543, "score_kernel, sliced"),            # two slices
    (3, 3, 128, 9000, 543, "score_kernel, sliced"),
    (48, 12, 64, 1300, 255, "score_kernel, sliced"),          # three
    (32, 16, 128, 1300, 383, "score_kernel, sliced"),
    (48, 6, 64, 1300, 255, "score_kernel, sliced"),           # four
    (48, 6, 128, 1300, 255, "score_kernel, sliced"),
    (8, 1, 64, 4096, 543, "score_kernel, sliced"),            # four, and more than 4096 scored rows
    (8, 1, 128, 4096, 543, "score_kernel, sliced"),
])
def test_score_kernel_matches_oracle(heads, kv, d, budget, L, kernel):
    """W' without bias (bound as in test_scores_of_few_rows_match_oracle), and the same bits on every run."""
    g = torch.Generator().manual_seed(41)
    K, V = (torch.randn((kv, budget, d), generator=g).bfloat16() for _ in range(2))
    pos = torch.arange(budget, dtype=torch.int32).repeat(kv, 1).contiguous()
    q, k, v = random_chunk(4700, L, heads, kv, d, "bf16")
    got = []
    for run in range(3):
        s = B.Stream(budget, L, heads, kv, d, dtype=torch.bfloat16, bias=0.0, max_chunk=L)
        assert s.kernel("score", budget, L) == kernel
        s.load(K.cuda(), V.cuda(), pos.cuda(), budget)
        print("score_kernel", (heads, kv, d, budget, L), "run", run, flush=True)
        s.step(q.cuda(), k.cuda(), v.cuda())
        got.append(s.last_scores())
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
    orc = OracleStream(budget, L, heads, kv, d, bias=0.0)
    orc.load(K.double().numpy(), V.double().numpy(), pos.numpy(), budget)
    orc.attend(*(x.double().numpy() for x in (q, k, v)))
    want = orc.scores()[1]
    assert np.allclose(got[0].double().cpu().numpy(), want, rtol=2e-5, atol=1e-12), np.abs(got[0].double().cpu().numpy() - want).max()


@pytest.mark.parametrize("heads,kv,d,budget,n,launches", [
    (4, 4, 64, 300, 130, 3),                                  # 64 tokens to a launch at most
    (32, 8, 128, 4096, 64, 2),                                # as many as the scratch holds partials for: 34
    (8, 2, 128, 1000, 200, 4),
])
def test_calls_of_more_tokens_than_share_a_launch(heads, kv, d, budget, n, launches):
    """Outputs and cache bit for bit those of a twin that decodes one token at a time."""
    a, b = (B.Stream(budget, budget // 4, heads, kv, d, dtype=torch.bfloat16, max_chunk=16, max_decode=n) for _ in range(2))
    g = torch.Generator(device="cuda").manual_seed(43)
    K, V = (torch.randn((kv, budget, d), generator=g, device="cuda").bfloat16() for _ in range(2))
    pos = torch.arange(budget, dtype=torch.int32, device="cuda").repeat(kv, 1).contiguous()
    for s in (a, b):
        s.load(K, V, pos, budget)
    q, k, v = (x.cuda() for x in random_chunk(4800, n, heads, kv, d, "bf16"))
    print("many tokens", (heads, kv, d, budget, n), flush=True)
    a.profile(16)
    out = a.decode_n(q, k, v)
    assert a.profile_read()["decode"][1] == launches
    one = torch.cat([b.decode(*(x[i:i + 1].contiguous() for x in (q, k, v))) for i in range(n)])
    assert torch.equal(out.view(torch.int16), one.view(torch.int16))
    for x, y in zip(a.export(), b.export()):
        assert torch.equal(x, y)


@pytest.mark.parametrize("L,placed", [(64, True), (300, False)])
def test_profile_has_a_placement_interval_only_where_there_is_a_launch(L, placed):
    heads, kv, d, budget = 4, 4, 128, 600
    s = B.Stream(budget, 100, heads, kv, d, dtype=torch.bfloat16, max_chunk=300)
    assert (s.kernel("compact", budget, L) == "") == placed
    chunks = [[x.cuda() for x in random_chunk(4900 + i, n, heads, kv, d, "bf16")] for i, n in enumerate((300, 300, L))]
    for c in chunks:
        s.step(*c)
    for names in (B.KERNELS, ["evict"], ["select", "evict"], ["compact", "evict"]):
        s.profile_select(names)
        s.profile(8)
        for _ in range(3):
            s.step(*chunks[2])
        s.step_attend(*chunks[2])
        B.evict_batched([s])
        p = s.profile_read()
        want = {"select": 4, "compact": 0 if placed else 4, "evict": 4}
        assert all(p[k][1] == (want[k] if k in names else 0) for k in want), (names, p)
        if len(names) > 2:
            assert p["evict"][0] >= p["select"][0] + p["compact"][0] - 1e-3


def test_row_groups_of_a_key_beside_each_other():
    """Launches of several rounds over more keys than the L2s hold number their workgroups in another order: tokens decoded
    together bit for bit as one at a time."""
    heads, kv, d, budget, n = 32, 32, 128, 3200, 64
    a, b = (B.Stream(budget, budget // 4, heads, kv, d, dtype=torch.bfloat16, max_chunk=16, max_decode=n) for _ in range(2))
    g = torch.Generator(device="cuda").manual_seed(53)
    K, V = (torch.randn((kv, budget, d), generator=g, device="cuda").bfloat16() for _ in range(2))
    pos = torch.arange(budget, dtype=torch.int32, device="cuda").repeat(kv, 1).contiguous()
    for s in (a, b):
        s.load(K, V, pos, budget)
    q, k, v = (x.cuda() for x in random_chunk(4950, n, heads, kv, d, "bf16"))
    print("row groups", flush=True)
    out = a.decode_n(q, k, v)
    one = torch.cat([b.decode(*(x[i:i + 1].contiguous() for x in (q, k, v))) for i in range(n)])
    assert torch.equal(out.view(torch.int16), one.view(torch.int16))
    for x, y in zip(a.export(), b.export()):
        assert torch.equal(x, y)
