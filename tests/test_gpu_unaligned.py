"""The bf16 kernels on tensors and frames that 16-byte accesses do not fit:
odd widths (against the oracle) and tensors at odd element addresses, whose
results must be the aligned call's bit for bit: the tile and the order of
every sum are the same, only the loads and stores differ.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_31938_amd import c3c, inputs
from paper_2609_31938_amd.inputs import spec

from gpu_util import as_f64, check, chunk, guarded, guards_intact, host, layer, oracle_args, say
from test_gpu_fused import _check_cache

pytestmark = pytest.mark.gpu

PIN = c3c.MODE_CHANNEL_TILES
# (mode, tile, shape): every tile of the 3x3 kernel
TILES = [
    (PIN, (16, 8, 64), dict(Co=12, H=11, W=72)),
    (0, (32, 8, 64), dict(Co=20, T=6, H=95, W=136)),
    (0, (48, 8, 64), dict(Co=41, T=6, H=95, W=136)),
    (0, (96, 6, 64), dict(Co=90, H=9, W=72)),
    (PIN, (128, 4, 80), dict(Co=256, H=9, W=88)),
    (PIN, (128, 10, 32), dict(Co=256, T=4, H=153, W=40)),
    (PIN, (160, 4, 80), dict(Co=150, H=9, W=88)),
    (PIN, (160, 10, 32), dict(Co=150, T=4, H=333, W=32)),
    (PIN, (192, 4, 64), dict(Co=192, H=9, W=72)),
    (0, (192, 4, 64), dict(Co=528, T=4, H=65, W=64)),
    (0, (64, 4, 64), dict(Co=192, H=9, W=72)),
    # one frame a source: the element after the last real channel is the
    # first of the padding channels (NaN here), and must not be read as one
    (0, (96, 6, 64), dict(Co=90, T=1, Tc=1, H=9, W=72)),
]


def _at(t, offset):
    """The same values ``offset`` elements past a 16-byte address."""
    buf = torch.full((t.numel() + 16,), float("nan"), dtype=t.dtype, device=t.device)
    v = buf[offset:offset + t.numel()].view(t.shape)
    v.copy_(t)
    return v


def _call(sp, mode, offset, form, ws):
    ctx = c3c.Context(mode)
    w, b = layer(sp, "bf16", 917)
    x, cache = chunk(sp, "bf16", 917, 0, 0), chunk(dict(sp, T=sp["Tc"]), "bf16", 917, 0, 1)
    To, Ho, Wo, L = c3c.output_dims(sp, "bf16")
    y = torch.full((sp["N"], sp["Co"], To, Ho, Wo), float("nan"), dtype=torch.bfloat16, device="cuda")
    co = torch.full((sp["N"], sp["Ci"], L, Ho, Wo), float("nan"), dtype=torch.bfloat16, device="cuda")
    need = c3c.workspace_bytes(sp, "bf16") if ws else 0
    if ws:
        assert need > 0
        ctx.set_workspace(torch.empty(need, dtype=torch.uint8, device="cuda"))
    x, cache, y, co = (_at(t, offset) for t in (x, cache, y, co))
    args = (ctx, sp, x, cache, w, c3c.weight_repack(ctx, sp, w), b)
    if form == "plain":
        c3c.conv3d_causal_cached(*args, y, co)
    else:
        res = _at(inputs.residual_input(tuple(y.shape), "bf16", 917, 0, 0, "cuda"), offset)
        sc, sh = inputs.affine_inputs(sp, 917, 0, 0, "cuda") if form == "prologue" else (None, None)
        c3c.conv3d_causal_cached_fused(*args, sc, sh, res, y, co)
    torch.cuda.synchronize()
    return y, co


@pytest.mark.parametrize("form", ["plain", "residual", "prologue"])
@pytest.mark.parametrize("mode,tile,over", TILES)
def test_odd_addresses_give_the_aligned_result(mode, tile, over, form):
    sp = spec(**dict(dict(Ci=40, T=2, Tc=2), **over))
    plan = c3c.plan_query(c3c.Context(mode), sp, "bf16")
    say(f"unaligned case {sp} {form} plan={plan}")
    assert (plan["tile_co"], plan["tile_h"], plan["tile_w"]) == tile, plan
    want = _call(sp, mode, 0, form, False)
    for offset in (1, 2):
        got = _call(sp, mode, offset, form, False)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), offset


@pytest.mark.parametrize("form", ["plain", "residual"])
def test_odd_addresses_under_split_k(form):
    sp = spec(Ci=256, Co=192, T=1, Tc=2, H=9, W=72)
    say(f"unaligned split-K case {sp} {form}")
    want = _call(sp, 0, 0, form, True)
    for offset in (1, 2):
        got = _call(sp, 0, offset, form, True)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), offset


# an unaligned residual is read four elements at a time, the tensor's last ones
# from its last four, and one by one where it has fewer than four
@pytest.mark.parametrize("N,Co,T,H,W", [(1, 1, 1, 1, 1), (1, 1, 1, 1, 3), (3, 1, 1, 1, 1), (1, 2, 1, 1, 2),
                                        (1, 1, 1, 1, 5), (1, 1, 1, 3, 3), (2, 17, 2, 5, 7), (1, 50, 1, 7, 66),
                                        (1, 180, 1, 4, 67)])
def test_unaligned_residual_to_its_last_element(N, Co, T, H, W):
    sp = spec(N=N, Ci=8, Co=Co, T=T, Tc=2, H=H, W=W)
    say(f"unaligned residual case {sp}")
    w, b = layer(sp, "bf16", 917)
    x, cache = chunk(sp, "bf16", 917, 0, 0), chunk(dict(sp, T=2), "bf16", 917, 0, 1)
    shape = (N, Co) + c3c.output_dims(sp, "bf16")[:3]
    # NaN on both sides: a value from outside the tensor would show
    res = _at(inputs.residual_input(shape, "bf16", 917, 0, 0, "cuda"), 3)
    ctx = c3c.Context(c3c.MODE_STRICT)
    y, ybuf = guarded(shape, "bf16")
    c3c.conv3d_causal_cached_fused(ctx, sp, x, cache, w, c3c.weight_repack(ctx, sp, w), b, None, None, res, y)
    torch.cuda.synchronize()
    assert guards_intact(ybuf), "a write outside the output"
    ref, _ = oracle.conv3d_fused(sp, *oracle_args(sp, x, cache, w, b), None, None, res.cpu())
    check(as_f64(y), ref, "bf16", str(sp))


@pytest.mark.parametrize("over", [
    dict(Ci=40, Co=192, H=9, W=67), dict(Ci=33, Co=256, T=4, H=153, W=37), dict(Ci=31, Co=96, H=13, W=65),
    dict(Ci=40, Co=150, H=5, W=81), dict(N=2, Ci=35, Co=20, H=7, W=3), dict(Ci=256, Co=192, T=1, H=9, W=71),
    dict(Ci=40, Co=60, H=1, W=1),
])
@pytest.mark.parametrize("ws", [False, True])
def test_odd_widths_match_the_oracle(over, ws):
    sp = spec(**dict(dict(T=2, Tc=2), **over))
    ctx = c3c.Context(c3c.MODE_STRICT)
    need = c3c.workspace_bytes(sp, "bf16") if ws else 0
    if ws and need == 0:
        pytest.skip("runs unsplit")
    say(f"odd width case {sp} ws={ws} plan={c3c.plan_query(ctx, sp, 'bf16', need)}")
    if need:
        ctx.set_workspace(torch.empty(need, dtype=torch.uint8, device="cuda"))
    w, b = layer(sp, "bf16", 917)
    x, cache = chunk(sp, "bf16", 917, 0, 0), chunk(dict(sp, T=2), "bf16", 917, 0, 1)
    To, Ho, Wo, L = c3c.output_dims(sp, "bf16")
    y, ybuf = guarded((sp["N"], sp["Co"], To, Ho, Wo), "bf16")
    co, cbuf = guarded((sp["N"], sp["Ci"], L, Ho, Wo), "bf16")
    c3c.conv3d_causal_cached(ctx, sp, x, cache, w, c3c.weight_repack(ctx, sp, w), b, y, co)
    torch.cuda.synchronize()
    assert guards_intact(ybuf) and guards_intact(cbuf), "a write outside the outputs"
    args = oracle_args(sp, x, cache, w, b)
    check(as_f64(y), oracle.conv3d(sp, "bf16", *args), "bf16", str(sp))
    got = host(co).contiguous().view(torch.int16).numpy().view(np.uint16)
    assert np.array_equal(got, oracle.cache_update(sp, "bf16", args[0], args[1]))


@pytest.mark.parametrize("tile_co,splits,over", [(32, 1, dict(Ci=23, Co=20, T=2, H=195, W=263)),
                                                 (48, 1, dict(Ci=23, Co=43, T=2, H=195, W=263)),
                                                 (48, 4, dict(Ci=464, Co=41, T=1, H=127, W=255))])
def test_odd_widths_on_the_narrow_tiles(tile_co, splits, over):
    sp = spec(**dict(over, Tc=2))
    need = c3c.workspace_bytes(sp, "bf16")
    plan = c3c.plan_query(None, sp, "bf16", need)
    assert (plan["tile_co"], plan["splits"]) == (tile_co, splits), plan
    test_odd_widths_match_the_oracle(over, splits > 1)


# the 1x1 kernels: 192 x 128-pixel tiles and the
# 160 x 256 pointwise tiles, with ragged channels and pixel tiles, stride
# 2, one source frame a tensor, new-cache frames in and out of the kernel
TEMPORAL = [
    ("tap1x1", "bf16", dict(Ci=40, Co=192, T=4, Tc=2, H=63, W=67)),
    ("tap1x1", "bf16", dict(N=2, Ci=33, Co=180, T=8, Tc=1, H=59, W=37, s_t=2, p_base=1)),
    ("tap1x1", "bf16", dict(Ci=72, Co=384, T=1, Tc=1, H=95, W=91)),
    ("tap1x1", "bf16", dict(Ci=31, Co=768, T=3, Tc=0, H=43, W=31, p_base=2)),
    ("pointwise", "bf16", dict(Ci=40, Co=150, T=2, Tc=2, H=21, W=27)),
    ("pointwise", "bf16", dict(N=2, Ci=33, Co=330, T=1, Tc=1, H=17, W=19)),
    ("pointwise", "bf16", dict(Ci=100, Co=16, T=2, Tc=2, H=1, W=3)),
    # 1x1x1: resident weights (Co <= 160, several tiles a workgroup), and not
    ("pointwise", "bf16", dict(Ci=72, Co=96, T=4, Tc=0, H=131, W=137, Kt=1)),
    ("pointwise", "f16", dict(N=2, Ci=40, Co=160, T=1, Tc=0, H=9, W=31, Kt=1)),
    ("pointwise", "bf16", dict(Ci=136, Co=170, T=1, Tc=1, H=23, W=21, Kt=1, p_base=1)),
    ("pointwise", "f16", dict(Ci=400, Co=33, T=3, Tc=0, H=1, W=5, Kt=1)),
]


@pytest.mark.parametrize("form", ["plain", "residual", "prologue"])
@pytest.mark.parametrize("kernel,dtype,over", TEMPORAL)
def test_1x1_odd_planes_match_the_oracle(kernel, dtype, over, form):
    if dtype == "f16" and form != "plain":
        pytest.skip("the fused form is bf16")
    sp = spec(Kh=1, Kw=1, **over)
    fast = sp["Kt"] > 1
    ctx = c3c.Context(c3c.MODE_STRICT if fast else 0)
    say(f"1x1 odd plane case {sp} {form} plan={c3c.plan_query(ctx, sp, dtype)}")
    w, b = layer(sp, dtype, 917)
    x = chunk(sp, dtype, 917, 0, 0)
    cache = chunk(dict(sp, T=sp["Tc"]), dtype, 917, 0, 1) if sp["Tc"] else None
    To, Ho, Wo, L = c3c.output_dims(sp, dtype)
    shape = (sp["N"], sp["Co"], To, Ho, Wo)
    fused = {}
    if form != "plain":
        fused["residual"] = _at(inputs.residual_input(shape, "bf16", 917, 0, 0, "cuda"), 1)
        if form == "prologue":
            fused["scale"], fused["shift"] = inputs.affine_inputs(sp, 917, 0, 0, "cuda")
    sc, sh, res = fused.get("scale"), fused.get("shift"), fused.get("residual")
    # at odd addresses too, NaN on both sides
    xo, co_ = _at(x, 1), _at(cache, 3) if cache is not None else None
    y, ybuf = guarded(shape, dtype)
    co, cbuf = guarded((sp["N"], sp["Ci"], L, Ho, Wo), dtype)
    wp = c3c.weight_repack(ctx, sp, w) if fast else None
    if form == "plain":
        assert c3c.plan_query(ctx, sp, dtype)["kernel"] == kernel
        c3c.conv3d_causal_cached(ctx, sp, xo, co_, w, wp, b, y, co)
    else:
        c3c.conv3d_causal_cached_fused(ctx, sp, xo, co_, w, wp, b, sc, sh, res, y, co)
    torch.cuda.synchronize()
    assert guards_intact(ybuf) and guards_intact(cbuf), "a write outside the outputs"
    args = oracle_args(sp, x, cache, w, b)
    if form == "plain":
        ref, ref_c = oracle.conv3d(sp, dtype, *args), oracle.cache_update(sp, dtype, args[0], args[1])
    else:
        sch, shh = (t.cpu() if t is not None else None for t in (sc, sh))
        ref, ref_c = oracle.conv3d_fused(sp, *args, sch, shh, res.cpu())
    check(as_f64(y), ref, dtype, str(sp))
    got = host(co).contiguous().view(torch.int16).numpy().view(np.uint16).reshape(ref_c.shape)
    ref_c = ref_c.view(np.uint16)
    _check_cache(got, ref_c, sp) if form == "prologue" else np.testing.assert_array_equal(got, ref_c)
