"""Host-side checks of the C ABI that need no GPU: the shared library loads, exports every
symbol the header declares, and rejects bad arguments with the documented codes."""
import ctypes
import os
import re

import pytest

from paper_2409_09086_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "infmllm.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(infmllm_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    L = B.lib()
    names = declared_functions()
    assert len(names) >= 13
    for name in names:
        assert hasattr(L, name), name
    assert sorted(B.EXPORTS) == names


def make(budget=16, recent=4, heads=4, kv=2, d=64, dtype=B.BF16):
    h = ctypes.c_void_p()
    rc = B.lib().infmllm_stream_create(budget, recent, heads, kv, d, dtype, ctypes.byref(h))
    return rc, h


@pytest.mark.parametrize("args", [
    dict(budget=0), dict(budget=-3), dict(recent=-1), dict(recent=17), dict(heads=3, kv=2), dict(heads=0),
    dict(kv=0), dict(d=96), dict(d=0), dict(dtype=7),
])
def test_create_rejects_bad_arguments(args):
    rc, h = make(**args)
    assert rc == B.EINVAL and not h.value
    assert B.last_error() != ""


def test_create_null_out_pointer():
    assert B.lib().infmllm_stream_create(16, 4, 4, 2, 64, 0, None) == B.EINVAL


def test_host_state_machine_without_a_device():
    L = B.lib()
    rc, h = make()
    assert rc == B.OK and h.value
    assert L.infmllm_stream_len(h) == 0 and L.infmllm_stream_streamed(h) == 0
    base = L.infmllm_stream_workspace_bytes(h)
    assert base > 2 * 2 * 2 * 32 * 64 * 2                       # two copies of K and V at capacity 2B
    assert L.infmllm_stream_set_param(h, B.PARAM_MAX_CHUNK, 4.0) == B.OK
    assert L.infmllm_stream_workspace_bytes(h) < base          # capacity is budget + max_chunk
    assert L.infmllm_stream_set_param(h, B.PARAM_BIAS, -1.0) == B.EINVAL
    assert L.infmllm_stream_set_param(h, B.PARAM_BIAS, float("nan")) == B.EINVAL
    assert L.infmllm_stream_set_param(h, B.PARAM_SCALE, 0.0) == B.EINVAL
    assert L.infmllm_stream_set_param(h, B.PARAM_MAX_CHUNK, 0.0) == B.EINVAL
    assert L.infmllm_stream_set_param(h, B.PARAM_IMPL, 2.0) == B.EINVAL
    assert [L.infmllm_stream_set_param(h, B.PARAM_CUT_HOLD, v) for v in (-1.0, 8.0, 2.5, 7.0, 0.0)] == [B.EINVAL] * 3 + [B.OK] * 2
    assert L.infmllm_stream_set_param(h, 99, 1.0) == B.EINVAL
    assert L.infmllm_stream_set_param(h, B.PARAM_BIAS, 0.5) == B.OK
    # nothing below reaches a device: every call is refused on the host
    one = ctypes.c_void_p(256)
    assert L.infmllm_step(h, one, one, one, 4, one, None, None) == B.ESTATE
    assert "attach" in B.last_error()
    assert L.infmllm_stream_positions(h, one) == B.ESTATE
    assert L.infmllm_stream_export(h, None, None, None, None) == B.ESTATE
    assert L.infmllm_stream_import(h, None, None, None, 0, 0) == B.ESTATE
    assert L.infmllm_stream_attach(h, None, 1 << 30, None) == B.EINVAL
    assert L.infmllm_stream_attach(h, ctypes.c_void_p(257), 1 << 30, None) == B.EINVAL     # misaligned
    assert L.infmllm_stream_attach(h, ctypes.c_void_p(256), 16, None) == B.ENOMEM
    L.infmllm_stream_destroy(h)
    L.infmllm_stream_destroy(None)
    assert L.infmllm_stream_len(None) == -1 and L.infmllm_stream_workspace_bytes(None) == 0


def test_optional_modes_are_checked_and_sized_on_the_host():
    """decoding room, comparison policies, position encoding, batched eviction: parameter checks and the
    workspace they ask for, all without a device"""
    L = B.lib()
    rc, h = make(budget=64, recent=16, heads=4, kv=2, d=128)
    assert rc == B.OK
    assert L.infmllm_stream_set_param(h, B.PARAM_MAX_CHUNK, 32.0) == B.OK
    base = L.infmllm_stream_workspace_bytes(h)
    assert L.infmllm_stream_max_len(h) == 64
    assert L.infmllm_stream_set_param(h, B.PARAM_MAX_DECODE, -1.0) == B.EINVAL
    assert L.infmllm_stream_set_param(h, B.PARAM_MAX_DECODE, 2.5) == B.EINVAL
    assert L.infmllm_stream_set_param(h, B.PARAM_MAX_DECODE, 8.0) == B.OK
    with_decode = L.infmllm_stream_workspace_bytes(h)
    assert with_decode > base and L.infmllm_stream_max_len(h) == 72           # 8 more rows per head + partials
    for bad in (-1.0, 4.0, 1.5):
        assert L.infmllm_stream_set_param(h, B.PARAM_POLICY, bad) == B.EINVAL
    for ok in (1.0, 2.0, 3.0, 0.0):
        assert L.infmllm_stream_set_param(h, B.PARAM_POLICY, ok) == B.OK
    assert L.infmllm_stream_workspace_bytes(h) == with_decode                 # policies need no memory
    for bad in (1.0, 0.5, -10000.0, float("inf")):
        assert L.infmllm_stream_set_param(h, B.PARAM_ROPE_BASE, bad) == B.EINVAL
    assert L.infmllm_stream_set_param(h, B.PARAM_ROPE_BASE, 10000.0) == B.OK
    with_rope = L.infmllm_stream_workspace_bytes(h)
    cap, d, elt = 64 + 8 + 32, 128, 2
    assert with_rope - with_decode >= 2 * cap * d * elt + cap * (d // 2) * 16   # turned keys of 2 heads + the table
    assert L.infmllm_stream_set_param(h, B.PARAM_ROPE_BASE, 0.0) == B.OK
    assert L.infmllm_stream_workspace_bytes(h) == with_decode
    # calls that need an attached stream are refused on the host
    one = ctypes.c_void_p(256)
    assert L.infmllm_decode(h, one, one, one, one) == B.ESTATE
    assert L.infmllm_decode_n(h, one, one, one, one, 3) == B.ESTATE
    assert L.infmllm_decode_n(None, one, one, one, one, 3) == B.EINVAL
    assert L.infmllm_step_attend(h, one, one, one, 4, one, None, None) == B.ESTATE
    assert L.infmllm_stream_pending(h) == 0 and L.infmllm_stream_pending(None) == -1
    arr = (ctypes.c_void_p * 1)(h)
    assert L.infmllm_evict_batched(arr, 1, None, None) == B.ESTATE
    assert L.infmllm_evict_batched(arr, 0, None, None) == B.EINVAL
    assert L.infmllm_evict_batched(None, 1, None, None) == B.EINVAL
    assert L.infmllm_stream_profile_select(h, 0) == B.EINVAL
    assert L.infmllm_stream_profile_select(h, 1 << 20) == B.EINVAL
    assert L.infmllm_stream_profile_select(h, 0xFF) == B.OK
    L.infmllm_stream_destroy(h)


@pytest.mark.gpu
def test_step_argument_checks_after_attach():
    """host-side checks of step on an attached stream: every call is refused before any launch"""
    import torch
    ws = torch.empty(1 << 22, dtype=torch.uint8, device="cuda:0")
    addr = (ws.data_ptr() + 255) // 256 * 256
    L = B.lib()
    rc, h = make()
    assert L.infmllm_stream_set_param(h, B.PARAM_MAX_CHUNK, 8.0) == B.OK
    need = L.infmllm_stream_workspace_bytes(h)
    assert need < (1 << 22) - 256
    assert L.infmllm_stream_attach(h, ctypes.c_void_p(addr), need, None) == B.OK
    assert L.infmllm_stream_attach(h, ctypes.c_void_p(addr), need, None) == B.ESTATE
    assert L.infmllm_stream_set_param(h, B.PARAM_BIAS, 0.1) == B.ESTATE
    one = ctypes.c_void_p(256)
    assert L.infmllm_step(h, None, one, one, 4, one, None, None) == B.EINVAL
    assert L.infmllm_step(h, one, one, one, 0, one, None, None) == B.EINVAL
    assert L.infmllm_step(h, one, one, one, 9, one, None, None) == B.ECAPACITY
    assert L.infmllm_stream_import(h, None, None, None, 17, 17) == B.EINVAL
    assert L.infmllm_stream_len(h) == 0
    L.infmllm_stream_destroy(h)


@pytest.mark.parametrize("heads,kv,d,dtype", [(32, 8, 128, B.BF16), (64, 1, 128, B.BF16), (512, 1, 128, B.BF16),
                                              (32, 32, 64, B.BF16), (4, 4, 128, B.FP32), (8, 1, 64, B.FP32)])
def test_static_workspace_takes_every_stream_whose_cache_and_tables_fit(heads, kv, d, dtype):
    """Scratch that launches can do without is not a reason to refuse a stream: accepted as far as the device call, which
    fails here if there is no GPU."""
    up = lambda x: (x + 255) // 256 * 256
    elt = 4 if dtype == B.FP32 else 2

    def need(b):                               # see largest_static_budget in test_gpu_decode_scratch.py
        rows = b + 16
        return (2 * up((kv * rows + 256) * d * elt) + 5 * up(kv * rows * 4) + up(heads * 16 * 4) + 4 * up(kv * 16 * 4) +
                up(kv * 4) + up(kv * b * 4) + (up(512 * 257 * 4) if elt == 2 else 0))
    budget = max(b for b in range(1, 131072 - 16) if need(b) <= 64 << 20)
    if elt == 4:
        budget = min(budget, 38400 - 16)       # what fp32 streams are limited to
    L = B.lib()
    rc, h = make(budget, 0, heads, kv, d, dtype)
    assert rc == B.OK and L.infmllm_stream_set_param(h, B.PARAM_MAX_CHUNK, 16.0) == B.OK
    rc = L.infmllm_stream_attach_static(h, None)
    assert rc in (B.OK, B.EHIP), B.last_error()
    L.infmllm_stream_destroy(h)


def test_kernel_names_on_the_host():
    """infmllm_stream_kernel: what the launches' rules choose, without a device."""
    L = B.lib()
    kernel = lambda h, name, cached, n: L.infmllm_stream_kernel(h, B.KERNELS.index(name), cached, n)

    def stream(chunk, *args, **params):
        rc, h = make(*args)
        assert rc == B.OK and L.infmllm_stream_set_param(h, B.PARAM_MAX_CHUNK, float(chunk)) == B.OK
        for k, v in params.items():
            assert L.infmllm_stream_set_param(h, getattr(B, "PARAM_" + k), v) == B.OK
        return h
    for chunk, args, want in [(512, (2048, 512, 32, 32, 128, B.BF16), (b"attn_rows64", b"score_kernel", b"place")),
                              (1024, (4096, 1024, 32, 8, 128, B.BF16), (b"attn_fwd64, cut", b"score_kernel, sliced", b"place")),
                              (2048, (8192, 2048, 32, 32, 128, B.BF16), (b"attn_fwd64", b"score_kernel", b"place")),
                              (37, (4096, 1152, 32, 32, 128, B.BF16), (b"attn_rows", b"score_once", b"")),
                              (64, (256, 64, 4, 4, 64, B.FP32), (b"attn_f32", b"score_f32", b""))]:
        h = stream(chunk, *args)
        assert tuple(kernel(h, n, args[0], chunk) for n in ("attn", "score", "compact")) == want
        assert kernel(h, "score", 0, 1) == b"" and kernel(h, "compact", 0, 1) == b""        # nothing is evicted
        assert kernel(h, "attn", args[0], chunk + 1) is None and kernel(h, "attn", args[0] + 1, 1) is None
        assert kernel(h, "attn", 0, 0) is None and kernel(h, "rope", 0, 1) is None
        L.infmllm_stream_destroy(h)
    h = stream(37, 4096, 1152, 32, 32, 128, B.BF16, IMPL=1.0)
    assert kernel(h, "attn", 4096, 37) == b"attn_simple" and kernel(h, "score", 4096, 37) == b"score_simple"
    assert kernel(h, "decode", 10, 1) == b"decode"
    L.infmllm_stream_destroy(h)
    h = stream(37, 4096, 1152, 32, 32, 128, B.BF16, POLICY=1.0)
    assert kernel(h, "score", 4096, 37) == b"rank_score"
    L.infmllm_stream_destroy(h)
    assert kernel(None, "attn", 0, 1) is None
    # Where attn_fwd64 does not fill the chip it takes no other kernel's place but that of attn_fwd's 128-row workgroups, with cut key
    # ranges: rows have one softmax reference in it, eight in attn_rows.  What is cut does not depend on max_chunk.
    for heads, kv, budget, n, want in [(32, 32, 4096, 1155, b"attn_rows"), (40, 5, 2451, 876, b"attn_rows"), (32, 16, 3164, 1077, b"attn_rows"),
                                       (32, 8, 2309, 1108, b"attn_rows"), (16, 4, 1041, 1041, b"attn_rows"), (32, 8, 5508, 1299, b"attn_fwd"),
                                       (32, 4, 1850, 1418, b"attn_fwd"), (32, 32, 16384, 512, b"attn_rows64"), (32, 32, 8192, 2048, b"attn_fwd64"),
                                       (40, 20, 4028, 1549, b"attn_fwd64"), (32, 32, 4096, 576, b"attn_fwd64, cut"),
                                       (32, 8, 4096, 1024, b"attn_fwd64, cut"), (16, 16, 2053, 1756, b"attn_fwd64, cut")]:
        for more in (0, 1500):
            h = stream(n + more, budget, budget // 4, heads, kv, 128, B.BF16)
            assert kernel(h, "attn", budget, n) == want, (heads, kv, budget, n, more)
            L.infmllm_stream_destroy(h)
