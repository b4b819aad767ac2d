"""Calls whose output overwrites their own inputs: the values before the call count."""
import pytest
import torch

from paper_2409_09086_amd import binding as B
from paper_2409_09086_amd.workloads import random_chunk

pytestmark = pytest.mark.gpu
DT = {"fp32": torch.float32, "bf16": torch.bfloat16}



@pytest.mark.parametrize("over", ["k", "v"])
@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("dtype,impl,heads,kv,d,budget,chunks,rope", [
    ("fp32", 0, 4, 4, 64, 200, [120, 80, 130, 33, 7], None),
    ("fp32", 0, 2, 2, 128, 640, [340, 300, 300, 256], None),           # moves more rows than the selection places itself
    ("fp32", 0, 2, 2, 64, 200, [200, 70, 33], 10000.0),
    ("bf16", 0, 4, 4, 128, 300, [300, 129, 40, 1], None),
    ("bf16", 0, 4, 4, 64, 300, [300, 129, 40], 10000.0),
    ("bf16", 1, 4, 4, 128, 200, [200, 100, 33], None),
    ("bf16", 0, 8, 2, 128, 300, [300, 130, 40], None),            # grouped heads: out is larger than k and covers it
])
def test_evicting_steps_whose_output_overwrites_the_chunk(dtype, impl, heads, kv, d, budget, chunks, rope, batched, over):
    """Against a twin with an output of its own.  The twin reads the chunk in place, this stream from the cache, the same
    keys in the same order: outputs, lists and cache agree bit for bit."""
    a, b = (B.Stream(budget, budget // 4, heads, kv, d, dtype=DT[dtype], bias=1e-3, max_chunk=max(chunks), impl=impl,
                     rope_base=rope) for _ in range(2))
    for step, L in enumerate(chunks):
        print("overlap", (dtype, impl, heads, kv, d, budget, rope, batched, over), "step", step, "L", L, flush=True)
        q, k, v = (x.cuda() for x in random_chunk(4100 + step, L, heads, kv, d, dtype))
        n = k.numel()
        buf = torch.empty(q.numel() + 64, dtype=q.dtype, device="cuda")
        out = buf[: q.numel()].view(q.shape)                      # the chunk's tensor lies at the start of the output
        mine = buf[:n].view(k.shape)
        mine.copy_(k if over == "k" else v)
        args = (q, mine, v) if over == "k" else (q, k, mine)
        if batched:
            r = a.step_attend(*args, out=out)
            w = b.step_attend(q, k, v)
            if a.pending:
                B.evict_batched([a])
                B.evict_batched([b])
        else:
            r = a.step(*args, out=out)
            w = b.step(q, k, v)
        cnt = int(w[2].item())
        assert int(r[2].item()) == cnt
        assert torch.equal(r[0], w[0]) and torch.equal(r[1][:, :cnt], w[1][:, :cnt])
        for x, y in zip(a.export(), b.export()):
            assert torch.equal(x, y)


TOKENS = [
    ("bf16", 4, 4, 128, 30, 60, None),        # one piece, two row groups
    ("bf16", 2, 2, 64, 100, 64, None),
    ("bf16", 4, 4, 128, 900, 40, None),       # several pieces, a merging launch
    ("bf16", 8, 2, 128, 100, 40, None),       # only tensors of one shape may coincide: q alone
    ("bf16", 4, 4, 64, 100, 40, 10000.0),
    ("fp32", 2, 2, 64, 100, 5, None),
]


@pytest.mark.parametrize("dtype,heads,kv,d,held,n,rope,over",
                         [t + (over,) for t in TOKENS for over in (("q", "k", "v") if t[1] == t[2] else ("q",))])
def test_tokens_whose_output_overwrites_their_inputs(dtype, heads, kv, d, held, n, rope, over):
    """decode_n against a twin with an output of its own: outputs and cache bit for bit."""
    a, b = (B.Stream(1000, 100, heads, kv, d, dtype=DT[dtype], max_chunk=max(held, 64), max_decode=64, rope_base=rope) for _ in range(2))
    for s in (a, b):
        s.step(*(x.cuda() for x in random_chunk(4200, held, heads, kv, d, dtype)))
    for call in range(2):
        print("overlap", (dtype, heads, kv, d, held, n, rope, over), "call", call, flush=True)
        q, k, v = (x.cuda() for x in random_chunk(4201 + call, n, heads, kv, d, dtype))
        want = b.decode_n(q, k, v)
        args = {"q": q.clone(), "k": k.clone(), "v": v.clone()}
        out = a.decode_n(args["q"], args["k"], args["v"], out=args[over])
        assert torch.equal(out, want)
        for x, y in zip(a.export(), b.export()):
            assert torch.equal(x, y)


@pytest.mark.parametrize("heads,kv,d,held,at_k,at_v", [
    (8, 2, 128, 900, 2, 5),                   # several pieces: rows of out that are another kv-head's key and value
    (32, 8, 128, 900, 20, 1),
    (32, 32, 128, 900, 1, None),              # the keys a head further
    (16, 16, 64, 900, None, -1),              # the values a head before
    (8, 2, 128, 100, 2, 5),                   # one piece
])
def test_tokens_whose_output_overlaps_other_keys(heads, kv, d, held, at_k, at_v):
    """Output rows of one kv-head that lie over the key or value of another: a token enters the cache, and is read from there,
    before any row is stored.  Against a twin with an output of its own, bit for bit."""
    a, b = (B.Stream(1000, 100, heads, kv, d, dtype=torch.bfloat16, max_chunk=held, max_decode=64) for _ in range(2))
    for s in (a, b):
        s.step(*(x.cuda() for x in random_chunk(4300, held, heads, kv, d, "bf16")))
    for call in range(24):
        print("overlap", (heads, kv, d, held, at_k, at_v), "call", call, flush=True)
        q, k, v = (x.cuda() for x in random_chunk(4301 + call, 1, heads, kv, d, "bf16"))
        want = b.decode(q, k, v)
        buf = torch.empty(3 * heads * d, dtype=torch.bfloat16, device="cuda")
        out = buf[heads * d: 2 * heads * d].view(q.shape)
        put = lambda x, at: x if at is None else buf[(heads + at) * d:][: x.numel()].view(x.shape).copy_(x)
        assert torch.equal(a.decode(q, put(k, at_k), put(v, at_v), out=out), want)
        for x, y in zip(a.export(), b.export()):
            assert torch.equal(x, y)
