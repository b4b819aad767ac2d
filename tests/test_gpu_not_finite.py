"""Values that are not finite reach the rows that see them, as their product with a positive weight, and no other row."""
import pytest
import torch

from paper_2409_09086_amd import binding as B
from paper_2409_09086_amd.workloads import random_chunk

pytestmark = pytest.mark.gpu
INF, NAN = float("inf"), float("nan")


def spoil(v, at):
    """Copy of v [n, kv, d] with values of tokens `at` replaced: an infinity, the other one, a NaN, in three columns."""
    w = v.clone()
    for i in at:
        w[i, :, 3], w[i, :, 17], w[i, :, v.shape[2] - 1] = INF, -INF, NAN
    return w


def reference(q, K, V, t):
    """64-bit softmax attention in which a row multiplies only what it sees; q [L,Hq,d], K, V [Hkv,n,d]."""
    q, K, V = q.double().cpu(), K.double().cpu(), V.double().cpu()
    out = torch.empty_like(q)
    for h in range(q.shape[1]):
        kh, vh = K[h * K.shape[0] // q.shape[1]], V[h * K.shape[0] // q.shape[1]]
        for i in range(q.shape[0]):
            n = t + i + 1
            p = torch.softmax(kh[:n] @ q[i, h] / q.shape[2] ** 0.5, 0)
            out[i, h] = (p[:, None] * vh[:n]).sum(0)
    return out


@pytest.mark.parametrize("heads,kv,d,chunks,at", [
    (4, 4, 64, [70, 50], (5, 33)),
    (6, 2, 128, [100, 33], (0, 17, 32)),          # three rows per token: a block of rows ends inside a token
    (2, 1, 64, [300, 1], (0,)),
    (1, 1, 128, [1500, 40], (20, 39)),            # pieces and a merging launch
])
def test_fp32_rows_that_do_not_see_a_value_are_as_without_it(heads, kv, d, chunks, at):
    mk = lambda: B.Stream(2000, 100, heads, kv, d, dtype=torch.float32, max_chunk=max(chunks))
    a, b = mk(), mk()
    Ks, Vs, t = [], [], 0
    for step, L in enumerate(chunks):
        print("not finite fp32", (heads, kv, d, chunks, at), "step", step, flush=True)
        q, k, v = (x.cuda() for x in random_chunk(4300 + step, L, heads, kv, d, "fp32"))
        w = spoil(v, at) if step == len(chunks) - 1 else v
        out, clean = a.step(q, k, w)[0], b.step(q, k, v)[0]
        Ks.append(k.transpose(0, 1)); Vs.append(w.transpose(0, 1))
        if w is not v:
            assert torch.equal(out[: at[0]], clean[: at[0]])
            ref = reference(q, torch.cat(Ks, 1), torch.cat(Vs, 1), t).float()
            assert torch.allclose(out.cpu(), ref, rtol=0, atol=1e-4, equal_nan=True)
        t += L


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_rows_past_the_cache_are_not_multiplied(dtype):
    """With the position encoding a step that fits reads the chunk from the cache, whose next rows are left from before."""
    dt = {"fp32": torch.float32, "bf16": torch.bfloat16}[dtype]
    q, k, v = (x.cuda() for x in random_chunk(4310, 40, 2, 2, 64, dtype))
    w = spoil(v, range(22, 40))
    outs = []
    for old in (v, w):
        s = B.Stream(100, 20, 2, 2, 64, dtype=dt, max_chunk=40, rope_base=10000.0)
        assert dtype == "fp32" or s.kernel("attn", 20, 2) == "attn_rows"
        s.step(q, k, old)
        K, V, pos = (x.transpose(0, 1)[:, :20].contiguous() for x in (k, v, torch.arange(40, dtype=torch.int32, device="cuda")[:, None].repeat(1, 2)))
        s.load(K, V, pos, 20)
        outs.append(s.step(q[:2].contiguous(), k[:2].contiguous(), v[:2].contiguous())[0])
    assert torch.isfinite(outs[0]).all() and torch.equal(*outs)


@pytest.mark.parametrize("heads,kv,d,held,n,at,rope", [
    (4, 4, 128, 50, 40, (3, 20, 39), None),
    (8, 2, 128, 900, 17, (0, 9), None),
    (6, 2, 64, 700, 9, (8,), None),
    (2, 2, 64, 120, 64, (40, 41), 10000.0),
])
def test_tokens_decoded_together_do_not_see_later_values(heads, kv, d, held, n, at, rope):
    """decode_n against one token at a time, bit for bit, and the values that are not finite against 64-bit arithmetic."""
    mk = lambda: B.Stream(1000, 100, heads, kv, d, dtype=torch.bfloat16, max_chunk=1000, max_decode=64, rope_base=rope)
    a, b = mk(), mk()
    chunk = [x.cuda() for x in random_chunk(4320, held, heads, kv, d, "bf16")]
    a.step(*chunk)
    b.step(*chunk)
    q, k, v = (x.cuda() for x in random_chunk(4321, n, heads, kv, d, "bf16"))
    w = spoil(v, at)
    print("not finite tokens", (heads, kv, d, held, n, at, rope), flush=True)
    out = a.decode_n(q, k, w)
    one = torch.cat([b.decode(*(x[i:i + 1].contiguous() for x in (q, k, w))) for i in range(n)])
    bits = lambda x: torch.where(x.isnan(), torch.full_like(x, NAN), x).view(torch.int16)    # the sign of a NaN is nobody's
    assert torch.equal(bits(out), bits(one))
    ref = reference(q, torch.cat([chunk[1], k]).transpose(0, 1), torch.cat([chunk[2], w]).transpose(0, 1), held)
    if rope is None:
        assert torch.allclose(out.double().cpu(), ref, rtol=2 ** -8, atol=2e-5, equal_nan=True)
    else:
        assert torch.equal(torch.isfinite(out.cpu()), torch.isfinite(ref))
