"""Scores where some cached rows are no candidates (the recent window is longer than the chunk): the scoring kernels then go
through the candidates in stream order, whatever cache rows they lie in."""
import numpy as np
import pytest
import torch

from oracle import OracleStream
from paper_2409_09086_amd import binding as B
from paper_2409_09086_amd.workloads import random_chunk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,kv,d,budget,recent,L,decoded,kernel", [
    (4, 4, 128, 512, 290, 33, 0, "score_once"),               # 255 candidates: one short of a workgroup's columns
    (4, 2, 64, 512, 289, 33, 0, "score_once"),                # 256
    (4, 4, 128, 512, 285, 30, 0, "score_once"),               # 257
    (8, 2, 128, 300, 299, 1, 3, "score_once"),                # five
    (2, 2, 64, 300, 300, 7, 0, "score_once"),                 # none of the budget is theirs
    (8, 1, 128, 700, 300, 65, 4, "score_once, sliced"),
    (24, 24, 64, 1500, 300, 159, 4, "score_kernel"),          # five blocks of rows: the last iteration has one
    (24, 24, 128, 1500, 300, 191, 0, "score_kernel"),         # six: two
    (24, 24, 128, 1500, 300, 223, 0, "score_kernel"),         # seven: three
    (40, 40, 128, 2900, 400, 159, 0, "score_kernel"),         # 512 columns per workgroup
    (32, 32, 128, 2300, 500, 208, 0, "score_kernel"),         # 288 blocks of 256 columns are more than a round: 512 here too
    (3, 3, 128, 9000, 700, 543, 2, "score_kernel, sliced"),   # the last slice ends with one block
])
def test_scores_of_candidates_in_stream_order(heads, kv, d, budget, recent, L, decoded, kernel):
    """W' without bias against the oracle (bound as in test_score_kernel_matches_oracle), with the carry of the cumulative
    policy beside it: a row's carry is looked up where the row lies."""
    for policy in ("infmllm", "cumulative"):
        s = B.Stream(budget, recent, heads, kv, d, dtype=torch.bfloat16, bias=0.0, max_chunk=max(L, 64), max_decode=decoded, policy=policy)
        orc = OracleStream(budget, recent, heads, kv, d, bias=0.0)
        g = torch.Generator().manual_seed(47)
        K, V = (torch.randn((kv, budget, d), generator=g).bfloat16() for _ in range(2))
        s.load(K.cuda(), V.cuda(), torch.arange(budget, dtype=torch.int32).repeat(kv, 1).contiguous().cuda(), budget)
        print("score columns", (heads, kv, d, budget, recent, L, decoded), policy, flush=True)
        for i, n in enumerate((64, 17, 64)):                  # evictions: cache rows out of stream order
            s.step(*(x.cuda() for x in random_chunk(5100 + i, min(n, max(L, 64)), heads, kv, d, "bf16")))
        Ke, Ve, pos, _ = s.export()
        orc.load(Ke.double().cpu().numpy(), Ve.double().cpu().numpy(), pos.cpu().numpy(), s.streamed)
        for i in range(decoded):
            tok = random_chunk(5200 + i, 1, heads, kv, d, "bf16")
            s.decode(*(x.cuda() for x in tok))
            orc.decode(*(x.double().numpy() for x in tok))
        assert s.kernel("score", budget + decoded, L) == kernel
        score = s.export()[3]
        q, k, v = random_chunk(5300, L, heads, kv, d, "bf16")
        s.step(q.cuda(), k.cuda(), v.cuda())
        got = s.last_scores().double().cpu().numpy()
        orc.attend(*(x.double().numpy() for x in (q, k, v)))
        want = np.array(orc.scores()[1])
        cnd = budget + decoded + L - recent
        assert got.shape == want.shape == (kv, cnd) and cnd < budget + decoded
        if policy == "cumulative":
            a = score.double().cpu().numpy()[:, :cnd]
            want = want + np.where(np.isfinite(a), a, 0.0)
        assert np.allclose(got, want, rtol=2e-5, atol=1e-12), np.abs(got - want).max()
