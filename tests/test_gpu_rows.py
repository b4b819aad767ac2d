"""attn_rows: attention of few query rows with the key range cut into pieces, against the fp64 oracle.  Chunks whose
rows, pieces and key runs end in every way the kernel distinguishes, decoding of several tokens per launch, and that
a token's output does not depend on how many tokens share the call."""
import numpy as np
import pytest
import torch

from oracle import OracleStream
from paper_2409_09086_amd import binding as B
from paper_2409_09086_amd.workloads import random_chunk
from _parity import LockStep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,kv,d,budget,recent,chunks", [
    (4, 4, 128, 900, 200, [900, 1, 16, 17, 33, 300]),     # four pieces; 1, 16 and 17 rows (tickets, then a merging launch)
    (8, 2, 128, 1500, 300, [800, 700, 5, 37, 64]),        # grouped heads: a row group holds several tokens
    (6, 2, 64, 777, 100, [777, 3, 11, 50]),               # three heads per group, runs that straddle the cache's end
    (2, 1, 64, 5000, 500, [2500, 2500, 2, 40]),           # more than sixteen pieces' worth of keys
    (16, 16, 64, 600, 150, [300, 300, 128, 31]),          # many heads: few pieces or one
    (1, 1, 128, 31, 8, [31, 7, 20]),                      # fewer keys than a run
    (4, 2, 64, 96, 96, [96, 33, 96]),                     # the whole budget is recent window: nothing is ranked
    (2, 2, 64, 900, 100, [900, 511, 512, 513]),           # as many moved rows as the selection places itself, and one more
    (2, 1, 128, 600, 50, [600, 255, 256, 257]),
    (16, 2, 128, 2600, 300, [1300, 1300, 270, 301]),      # 64 rows per workgroup, three pieces, ragged rows and keys
])
def test_short_chunks_match_oracle(heads, kv, d, budget, recent, chunks):
    gpu = B.Stream(budget, recent, heads, kv, d, dtype=torch.bfloat16, bias=1e-3, max_chunk=max(chunks))
    ls = LockStep(gpu, OracleStream(budget, recent, heads, kv, d, bias=1e-3))
    for step, L in enumerate(chunks):
        print("rows", (heads, kv, d, budget), "step", step, "L", L, flush=True)
        ls.step(*random_chunk(3100 + step, L, heads, kv, d, "bf16"), check_state=True)


@pytest.mark.parametrize("heads,kv,d,budget,rope", [(4, 4, 128, 1300, None), (8, 2, 128, 1300, None), (6, 2, 64, 700, None),
                                                    (4, 1, 64, 5000, None), (8, 2, 128, 600, 10000.0)])
def test_tokens_do_not_depend_on_how_many_share_a_call(heads, kv, d, budget, rope):
    """decode_n in calls of 1, 2, 17 and 40 tokens against a twin that decodes one at a time: outputs and cache bit for
    bit; and against the oracle with the error of one rounding to bf16 (eight significant bits: at most 2^-8 relative) plus 2e-5 for the fp32 sums of
    a few thousand terms of size |v| <= 5 (2^-24 * 5 * sqrt(5000)): the weights enter the product unrounded."""
    max_chunk, nd = 64, 60
    mk = lambda: B.Stream(budget, budget // 4, heads, kv, d, dtype=torch.bfloat16, max_chunk=max_chunk, max_decode=nd,
                          rope_base=rope)
    a, b = mk(), mk()
    orc = OracleStream(budget, budget // 4, heads, kv, d, rope_base=rope or 0.0, rope_round="bf16" if rope else None)
    g = torch.Generator().manual_seed(17)
    K, V = torch.randn((kv, budget, d), generator=g).bfloat16(), torch.randn((kv, budget, d), generator=g).bfloat16()
    pos = torch.arange(budget, dtype=torch.int32).repeat(kv, 1).contiguous()
    for s in (a, b):
        s.load(K.cuda(), V.cuda(), pos.cuda(), budget)
    orc.load(K.double().numpy(), V.double().numpy(), pos.numpy(), budget)
    for key, n in enumerate((1, 2, 17, 40)):
        print("tokens", (heads, kv, d, budget, rope), "n", n, flush=True)
        q, k, v = random_chunk(3200 + key, n, heads, kv, d, "bf16")
        out = a.decode_n(q.cuda(), k.cuda(), v.cuda())
        one = torch.cat([b.decode(*(x[i:i + 1].contiguous().cuda() for x in (q, k, v))) for i in range(n)])
        assert torch.equal(out.view(torch.int16), one.view(torch.int16)), "%d tokens per call" % n
        ref = np.concatenate([orc.decode(*(x[i:i + 1].double().numpy() for x in (q, k, v))) for i in range(n)])
        err = np.abs(out.double().cpu().numpy() - ref)
        assert (err <= 2.0 ** -8 * np.abs(ref) + 2e-5).all(), err.max()
    for x, y in zip(a.export(), b.export()):
        assert torch.equal(x, y)


@pytest.mark.parametrize("heads,kv,d,budget,recent,chunks", [
    (4, 4, 128, 512, 128, [512, 1, 31, 32, 33, 128]),     # one slice of one to four blocks, ragged last block
    (4, 4, 128, 511, 160, [511, 129, 160, 300]),          # slices of 3 and 2 blocks; 160 rows scored of 300
    (8, 2, 128, 300, 64, [257, 43, 1, 5, 33, 64]),        # grouped heads: slices that cross from head to head
    (6, 2, 64, 255, 0, [255, 16, 256]),                   # no scored row at all: selection by age
    (16, 1, 64, 700, 512, [512, 188, 512, 100]),          # 256 blocks: 64 slices of a column block; columns past a tile's end
])
def test_scores_of_few_rows_match_oracle(heads, kv, d, budget, recent, chunks):
    """score_once: W' against the oracle's, without bias.  p = exp2(s c - lse) with s, lse of size up to 8 in fp32 is off by
    8 * 2^-23 * ln 2 < 1e-6 relative and the sums of positive terms by as much again: well inside 2e-5."""
    gpu = B.Stream(budget, recent, heads, kv, d, dtype=torch.bfloat16, bias=0.0, max_chunk=max(chunks))
    orc = OracleStream(budget, recent, heads, kv, d, bias=0.0)
    for step, L in enumerate(chunks):
        print("scores", (heads, kv, d, budget, recent), "step", step, "L", L, flush=True)
        q, k, v = random_chunk(3300 + step, L, heads, kv, d, "bf16")
        _, ret, cnt = gpu.step(q.cuda(), k.cuda(), v.cuda())
        orc.attend(*(x.double().numpy() for x in (q, k, v)))
        sc = orc.scores()
        got = gpu.last_scores()
        assert (got is None) == (sc is None)
        if sc is not None:
            assert np.allclose(got.double().cpu().numpy(), sc[1], rtol=2e-5, atol=1e-12), np.abs(got.double().cpu().numpy() - sc[1]).max()
        orc.select()
        orc.commit(ret.cpu().numpy()[:, : int(cnt.item())])


@pytest.mark.parametrize("heads,kv,d,dtype,budget,chunks,report", [
    (8, 2, 128, "bf16", 700, [300, 1, 17, 333, 49], True),          # attn_rows with 16 and 32 rows, cut and uncut
    (16, 2, 128, "bf16", 1700, [333, 500, 867], True),              # 64 rows per workgroup
    (32, 8, 128, "bf16", 2400, [1100, 1300], True),                 # attn_fwd: more keys than the first wave of shares copies
    (32, 32, 128, "bf16", 3100, [2048, 1024], False),               # attn_fwd64: appended by a launch of its own; no lists wanted
    (16, 4, 64, "bf16", 2100, [1024, 1030], True),
    (6, 3, 64, "fp32", 300, [5, 128, 130], True),
    (2, 1, 128, "fp32", 600, [333, 267], False),
])
def test_chunks_that_fit_enter_the_cache_as_given(heads, kv, d, dtype, budget, chunks, report):
    """Steps that evict nothing: the cache is the concatenation of the chunks, bit for bit, with its positions and tables
    (the export goes through them), and the list counts up.  A chunk whose output overwrites its own values included."""
    dt = {"bf16": torch.bfloat16, "fp32": torch.float32}[dtype]
    s = B.Stream(budget, budget // 4, heads, kv, d, dtype=dt, max_chunk=max(chunks))
    twin = B.Stream(budget, budget // 4, heads, kv, d, dtype=dt, max_chunk=max(chunks))
    Ks, Vs, n = [], [], 0
    for step, L in enumerate(chunks):
        print("fits", (heads, kv, d, dtype, budget), "step", step, "L", L, flush=True)
        q, k, v = (x.cuda() for x in random_chunk(3400 + step, L, heads, kv, d, dtype))
        if heads == 32 and kv == 8:
            assert s.kernel("attn", len(s), L) == "attn_fwd"
        out, ret, cnt = s.step(q, k, v, report=report)
        Ks.append(k.transpose(0, 1)); Vs.append(v.transpose(0, 1)); n += L
        K, V, pos, score = s.export()
        assert torch.equal(K, torch.cat(Ks, 1)) and torch.equal(V, torch.cat(Vs, 1))
        want = torch.arange(n, dtype=torch.int32, device="cuda").expand(kv, n)
        assert torch.equal(pos, want) and torch.isinf(score).all()
        if report:
            assert int(cnt.item()) == n and torch.equal(ret[:, :n], want)
        if heads == kv:                                       # out and v have the same shape
            over = v.clone()
            twin.step(q, k, over, out=over)
            assert torch.equal(over, out)
    if heads == kv:
        for x, y in zip(s.export(), twin.export()):
            assert torch.equal(x, y)
