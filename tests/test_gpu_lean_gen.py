"""The lean kernel's mask-testing form (plan ids 66-69: any pattern library)
against the CPU oracle and the channel-chunk kernel it takes layers from."""
import numpy as np
import pytest

import workloads
from oracle import bf16 as obf16
from oracle import conv as oconv
from tests.tolerance import check

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pp = pytest.importorskip("paper_2004_11250_amd")

MIXED = [0x010, 0x003, 0x007, 0x01F, 0x155, 0x1EF, 0x1FF]   # 1, 2, 3, 5, 5, 8 and 9 taps
WIDE = list(range(1, 256))                                  # masks in both of the kernel's registers


def _params(kind, seed, c_out, c_in):
    if kind == "column":   # one mask per channel, all filters; some channels with all nine taps, some pruned
        L = workloads.random_layer(seed, c_out, c_in, lib=[0x1FF])
        col = pp.project_columns(L["w"], 9 * c_in // 2)
        col[0], col[1] = 0x1FF, 0
        L["lib"], L["pid"], L["conn"] = pp.column_library(col, c_out)
        return L
    L = workloads.random_layer(seed, c_out, c_in, lib=MIXED if kind != "wide" else WIDE, keep=1.0 if kind == "full9" else 0.5)
    if kind == "full9":    # nine taps everywhere: the last slot's weights lie past the 64th dword
        L["pid"][:] = 6
    return L


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("recipe", [66, 67, 68, 69])
@pytest.mark.parametrize("kind", ["column", "mixed", "wide", "full9"])
def test_any_library(kind, recipe, dtype, monkeypatch):
    wd = pp.PP_BF16 if dtype == "bf16" else pp.PP_F32
    # a ragged last tile and slot group; the 4-byte staging tilings on widths the 16-byte ones cannot take
    n, c_out, c_in, h, w = (2, 13, 33, 19, 40) if recipe in (66, 68) else (1, 24, 17, 35, 38 if dtype == "bf16" else 37)
    seed = 2100 + recipe
    L = _params(kind, seed, c_out, c_in)
    layer = pp.PackedLayer.from_weights(L["w"], L["b"], L["pid"], L["conn"], L["lib"], wdtype=wd)
    x = workloads.random_input(seed, (n, c_in, h, w))
    wt = L["w"]
    if dtype == "bf16":
        x, wt = obf16.round_f32(x), obf16.round_f32(wt)
    args = (x, wt, L["b"], L["pid"], L["conn"], L["lib"])
    ref, bound = oconv.conv3x3_pruned(*args, 1, 1, 1, True), oconv.conv3x3_bound(*args, 1, 1, 1)
    xd = torch.from_numpy(x).cuda().to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    print("any library", kind, recipe, dtype, (n, c_out, c_in, h, w), "seed", seed, flush=True)
    monkeypatch.setenv("PP_RECIPE", str(recipe))
    assert pp.conv2d_recipe(layer.h_blob, n, h, w, wd) == recipe
    y = pp.conv2d_fwd(layer, xd, relu=True)
    check(y.float().cpu().numpy().astype(np.float64), ref, bound, dtype, f"{kind} {recipe}")
    monkeypatch.setenv("PP_RECIPE", "13")   # the channel-chunk kernel
    assert pp.conv2d_recipe(layer.h_blob, n, h, w, wd) == 13
    old = pp.conv2d_fwd(layer, xd, relu=True)
    check(old.float().cpu().numpy().astype(np.float64), ref, bound, dtype, f"{kind} 13")
    # an infinity reaches the outputs whose kept taps see it and no others, as there
    monkeypatch.setenv("PP_RECIPE", str(recipe))
    xd[0, 2, 5, 7] = float("inf")
    new_inf = pp.conv2d_fwd(layer, xd)
    monkeypatch.setenv("PP_RECIPE", "13")
    assert torch.equal(torch.isfinite(new_inf), torch.isfinite(pp.conv2d_fwd(layer, xd)))


def test_planned_and_unaligned(monkeypatch):
    monkeypatch.delenv("PP_RECIPE", raising=False)
    L = _params("column", 2200, 16, 32)
    layer = pp.PackedLayer.from_weights(L["w"], L["b"], L["pid"], L["conn"], L["lib"])
    assert pp.conv2d_recipe(layer.h_blob, 1, 72, 72, pp.PP_F32) == 66
    assert pp.conv2d_recipe(layer.h_blob, 1, 72, 71, pp.PP_F32) == 67
    assert pp.conv2d_recipe(layer.h_blob, 1, 24, 24, pp.PP_F32) == 68
    x = torch.from_numpy(workloads.random_input(2200, (1, 32, 72, 72))).cuda()
    y = pp.conv2d_fwd(layer, x)
    off = torch.empty(x.numel() + 1, device="cuda")[1:].view(x.shape)   # 4-byte aligned: 4-byte staging, same sums
    off.copy_(x)
    assert torch.equal(pp.conv2d_fwd(layer, off), y)


def _offset(t):
    """a copy of t that starts one element past an aligned address"""
    v = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:].view(t.shape)
    v.copy_(t)
    return v


@pytest.mark.parametrize("c_out,c_in,h,w,kind", [
    (16, 32, 72, 72, "column"),      # the mask-testing tilings: 16-byte and 4-byte staging, large and small maps
    (13, 33, 71, 70, "mixed"),
    (24, 17, 24, 32, "wide"),
    (24, 24, 19, 38, "column"),
    (24, 48, 64, 64, "canon"),       # the lean kernel's own library
    (24, 48, 100, 90, "canon"),
])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("which", ["x", "y", "both"])
def test_tensors_that_start_on_one_element(c_out, c_in, h, w, kind, dtype, which, monkeypatch):
    # bf16 tensors on a 2-byte boundary, fp32 ones on a 4-byte boundary
    monkeypatch.delenv("PP_RECIPE", raising=False)
    wd = pp.PP_BF16 if dtype == "bf16" else pp.PP_F32
    L = workloads.random_layer(2300, c_out, c_in) if kind == "canon" else _params(kind, 2300, c_out, c_in)
    layer = pp.PackedLayer.from_weights(L["w"], L["b"], L["pid"], L["conn"], L["lib"], wdtype=wd)
    x = workloads.random_input(2300, (2, c_in, h, w))
    wt = L["w"]
    if dtype == "bf16":
        x, wt = obf16.round_f32(x), obf16.round_f32(wt)
    args = (x, wt, L["b"], L["pid"], L["conn"], L["lib"])
    ref, bound = oconv.conv3x3_pruned(*args, 1, 1, 1, True), oconv.conv3x3_bound(*args, 1, 1, 1)
    xd = torch.from_numpy(x).cuda().to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    print("one element past", kind, dtype, which, (c_out, c_in, h, w), "plan", pp.conv2d_plan(layer.h_blob, 2, h, w, wd), flush=True)
    out = torch.full((2, c_out, h, w), float("nan"), dtype=xd.dtype, device="cuda")
    if which != "y":
        xd = _offset(xd)
    if which != "x":
        out = _offset(out)
    y = pp.conv2d_fwd(layer, xd, relu=True, out=out)
    assert torch.isfinite(y).all()
    check(y.float().cpu().numpy().astype(np.float64), ref, bound, dtype, f"one element past {kind} {which}")
