"""The layer as one call (moe_layer_forward): the buffers of the separate calls,
bit for bit, on both sides of its small-batch rule; refusals."""
import ctypes

import numpy as np
import pytest
import torch

import synth
from tests import gpu_common as gc
from tests.gpu_common import log


@pytest.fixture(scope="module")
def m():
    from paper_2609_15627_amd import moe
    return moe


def _args(m, **kw):
    p = 1 << 20  # never dereferenced: every refusal comes before a launch
    d = dict(T=4, H=256, E=8, k=2, n_shared=1, I=128, n_experts_total=9, f=0, fused=0,
             perm_ws_bytes=1 << 20, gemm_ws_bytes=1 << 30)
    d.update({n: p for n, t in m._LayerArgs._fields_ if t is ctypes.c_void_p})
    d["w_router"] = None
    d.update(kw)
    return m._LayerArgs(**d)


@pytest.mark.parametrize("kw,status", [
    (dict(T=-1), 1), (dict(k=9), 1), (dict(n_shared=2), 1), (dict(H=200), 1), (dict(I=100), 1),
    (dict(logits=None), 1), (dict(out=None), 1), (dict(partials=None), 1), (dict(w13=None), 1),
    (dict(sorted=None), 1), (dict(f=7), 1), (dict(x=(1 << 20) + 8), 1),
    (dict(w_router=1 << 20, logits_buf=None), 1), (dict(gemm_ws_bytes=64), 3),
    (dict(gemm_ws=None), 3), (dict(T=600, perm_ws=None), 3), (dict(fused=1, f=1), 2),
])
def test_layer_forward_rejects(m, kw, status):
    a = _args(m, **kw)
    assert m.lib.moe_layer_forward(ctypes.byref(a), None) == status
    assert m.lib.moe_layer_forward(None, None) == 1


@pytest.mark.gpu
@pytest.mark.parametrize("T,H,I,E,k,S,fmt,routing,fused", [
    (1, 256, 128, 8, 2, 0, "e4m3", "router", False),
    (1, 512, 256, 300, 8, 1, "bf16", "normal", False),
    (16, 256, 128, 511, 8, 1, "e2m1", "normal", False),     # NE = 512, a token per wave
    (16, 256, 128, 512, 8, 1, "e4m3", "normal", False),     # NE = 513: separate launches
    (17, 256, 128, 40, 3, 1, "e2m3", "router", False),      # routed by its own launch
    (16, 512, 512, 64, 31, 1, "e4m3", "normal", True),      # k_total = 32, fused
    (64, 256, 256, 100, 16, 0, "e4m3", "zipf", False),      # 1024 assignments, empty experts
    (128, 256, 128, 130, 8, 0, "bf16", "zipf", False),      # 1024 assignments
    (129, 256, 128, 130, 8, 0, "e4m3", "normal", False),    # more: three launches, two chunks
    (3000, 256, 128, 511, 31, 1, "e2m1", "zipf", False),    # 94 chunks, NE = 512, k_total = 32
    (3073, 256, 128, 100, 32, 0, "e4m3", "normal", False),  # 97 chunks: separate launches
    (2050, 256, 256, 40, 3, 1, "e2m3", "router", False),    # two lists (short-K stage 2)
    (300, 512, 512, 4, 2, 1, "bf16", "normal", False),      # LDS-tiled bf16, 128-row tiles
    (300, 512, 512, 4, 2, 1, "e4m3", "normal", False),      # LDS-tiled: separate launches
    (1100, 512, 512, 3, 2, 1, "e4m3", "normal", False),     # LDS-tiled, three launches
    (400, 512, 256, 6, 2, 0, "e4m3", "normal", False),      # tiled stage 1, short-K stage 2
])
def test_layer_forward_is_the_separate_calls(m, T, H, I, E, k, S, fmt, routing, fused):
    cfg = synth.LayerConfig("call", T, H, E, k, I, S, routing, T + E, zipf_empty=3)
    inp = synth.make_inputs(cfg)
    log(f"layer call {(T, H, I, E, k, S, fmt, routing, fused)}")
    w = gc.dev_expert_weights(inp.weights)
    x = gc.to_dev_bf16(inp.x)
    lg = None if inp.logits is None else torch.from_numpy(inp.logits).cuda()
    wr = None if inp.wr is None else gc.to_dev_bf16(inp.wr)
    one, sep = (m.MoELayer(T, H, E, k, I, S, fmt, fused=fused) for _ in range(2))
    for _ in range(2):  # the second call finds the first one's buffers
        one.forward(x, w, logits=lg, w_router=wr)
    v = m.moe_last_variant()
    sep.forward(x, w, logits=lg, w_router=wr,
                events=[torch.cuda.Event(enable_timing=True) for _ in range(7)])
    torch.cuda.synchronize()
    assert m.moe_last_variant() == v
    names = ["out", "ids", "w"] + ([] if fused else ["partials"])
    for n in names:
        a, b = getattr(one, n), getattr(sep, n)
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), n
    for n, a, b in zip(("counts", "offsets", "sorted", "pos"), one.perm, sep.perm):
        assert torch.equal(a, b), n
    if wr is not None:
        assert torch.equal(one.logits, sep.logits)
    for r, n in ((0, T * m.ws_code_bytes(H, fmt)), (1, T * H // 32)):
        if fmt not in ("bf16", "e2m3"):
            assert torch.equal(one.workspace_view(r)[:n], sep.workspace_view(r)[:n])


@pytest.mark.gpu
def test_empty_batch(m):
    """No token: nothing but the empty expert lists, in every format."""
    log("layer call, no token")
    cfg = synth.LayerConfig("none", 1, 256, 8, 2, 128, 1, "normal", 3)
    w = gc.dev_expert_weights(synth.gen_all_experts(cfg))
    for fmt in ("e4m3", "e2m3", "e2m1", "bf16"):
        layer = m.MoELayer(0, 256, 8, 2, 128, 1, fmt)
        out = layer.forward(torch.empty((0, 256), dtype=torch.bfloat16, device="cuda"), w,
                            logits=torch.empty((0, 8), device="cuda"))
        torch.cuda.synchronize()
        assert out.shape == (0, 256) and not layer.perm[1].any()


@pytest.mark.gpu
@pytest.mark.parametrize("T", [4, 600])
def test_more_router_columns_than_experts(m, T):
    """600 logits for 9 experts: ids past the last expert are left out alike."""
    log(f"layer call, 600 router columns, {T} tokens")
    cfg = synth.LayerConfig("wide", T, 256, 8, 2, 128, 1, "normal", 5)
    inp = synth.make_inputs(cfg)
    w, x = gc.dev_expert_weights(inp.weights), gc.to_dev_bf16(inp.x)
    lg = np.random.default_rng(T).standard_normal((T, 600)).astype(np.float32)
    lg[::2, 599] = 9.0  # a choice past column 512
    lg[1::2, 3] = 9.0
    lg = torch.from_numpy(lg).cuda()
    one, sep = (m.MoELayer(T, 256, 8, 2, 128, 1, "e4m3") for _ in range(2))
    for layer in (one, sep):
        layer.partials.zero_()  # rows of the left-out ids stay as they are
    one.forward(x, w, logits=lg)
    sep.forward(x, w, logits=lg, events=[torch.cuda.Event(enable_timing=True) for _ in range(7)])
    torch.cuda.synchronize()
    assert (one.ids[::2] == 599).any(1).all()
    for n in ("ids", "w", "out"):
        assert torch.equal(getattr(one, n), getattr(sep, n)), n
    for i in (0, 1):
        assert torch.equal(one.perm[i], sep.perm[i])
