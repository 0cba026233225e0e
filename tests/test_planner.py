"""Planner choices that need no GPU (pp_conv2d_recipe is host-only): where
the bf16 matrix-core form (plan id 64) is taken and where it cannot be."""
import numpy as np
import pytest

import workloads

pp = pytest.importorskip("paper_2004_11250_amd")
MFMA = 64


def _blob(seed, c_out, c_in, dt, keep=0.5, s=1, p=1, d=1, lib=None):
    lib = np.array(workloads.CANON8 if lib is None else lib, np.uint16)
    L = workloads.random_layer(seed, c_out, c_in, lib=lib, keep=keep)
    return pp.pack(L["w"], L["b"], L["pid"], L["conn"], lib, s, p, d, dt)


@pytest.fixture(autouse=True)
def _no_forced_plan(monkeypatch):
    monkeypatch.delenv("PP_RECIPE", raising=False)
    monkeypatch.delenv("PP_KSPLIT", raising=False)


def test_large_bf16_layers_take_the_matrix_cores():
    assert pp.conv2d_recipe(_blob(1, 64, 64, pp.PP_BF16), 1, 270, 480, pp.PP_BF16) == MFMA      # super-resolution body
    assert pp.conv2d_recipe(_blob(2, 512, 512, pp.PP_BF16), 8, 32, 32, pp.PP_BF16) == MFMA     # colourization
    # the style network's 128 -> 128 at 128 x 128: the lean kernel (24 us with
    # prepared weights; 12 on the matrix cores, which the planner leaves out here)
    assert pp.conv2d_recipe(_blob(3, 128, 128, pp.PP_BF16), 1, 128, 128, pp.PP_BF16) == 46
    # any library: the form reads the blob's own masks
    other = [0x00F, 0x0B2, 0x1C8, 0x055, 0x113, 0x0A9]
    assert pp.conv2d_recipe(_blob(4, 64, 64, pp.PP_BF16, lib=other), 1, 270, 480, pp.PP_BF16) == MFMA


def test_small_or_ineligible_layers_stay_on_the_vector_kernels():
    b = _blob(5, 512, 512, pp.PP_BF16, keep=1 / 3)
    assert pp.conv2d_recipe(b, 1, 14, 14, pp.PP_BF16) != MFMA           # few tiles, long reduction
    assert pp.conv2d_recipe(b, 1, 28, 28, pp.PP_BF16) != MFMA
    assert pp.conv2d_recipe(_blob(6, 3, 64, pp.PP_BF16), 1, 1080, 1920, pp.PP_BF16) != MFMA   # 3 filters
    sr = _blob(7, 64, 64, pp.PP_BF16)
    assert pp.conv2d_recipe(sr, 1, 270, 480, pp.PP_BF16, with_workspace=False) != MFMA        # needs scratch
    assert pp.conv2d_recipe(_blob(8, 64, 48, pp.PP_BF16), 1, 270, 480, pp.PP_BF16) != MFMA    # c_in % 32
    assert pp.conv2d_recipe(_blob(9, 64, 64, pp.PP_F32), 1, 270, 480, pp.PP_F32) != MFMA       # fp32


def test_forced_matrix_core_plan(monkeypatch):
    monkeypatch.setenv("PP_RECIPE", str(MFMA))
    assert pp.conv2d_recipe(_blob(10, 40, 32, pp.PP_BF16), 2, 19, 23, pp.PP_BF16) == MFMA
    assert pp.conv2d_recipe(_blob(11, 40, 24, pp.PP_BF16), 2, 19, 23, pp.PP_BF16) != MFMA   # cannot run: ignored


def test_workspace_covers_the_matrix_core_form():
    b = _blob(12, 64, 64, pp.PP_BF16)
    ws = pp.conv2d_workspace(b, 1, 270, 480, pp.PP_BF16)
    assert ws >= 64 * 9 * 64 * 2 + 64 * 4   # the expanded weights and the bias


def test_large_fp32_image_layers_take_the_few_output_kernel():
    full = _blob(13, 3, 64, pp.PP_F32, keep=1.0, lib=workloads.DENSE9)
    assert pp.conv2d_recipe(full, 1, 1080, 1920, pp.PP_F32) == 61
    assert pp.conv2d_recipe(full, 1, 540, 960, pp.PP_F32) != 61     # small: the wave kernel
    assert pp.conv2d_recipe(full, 2, 1080, 1920, pp.PP_F32) != 61   # a batch
    some = _blob(14, 3, 64, pp.PP_F32, keep=0.9, lib=workloads.DENSE9)
    assert pp.conv2d_recipe(some, 1, 1080, 1920, pp.PP_F32) != 61   # a pruned kernel


@pytest.mark.parametrize("c_out,c_in,s,d,n,h,w,keep,mfma", [
    (64, 64, 1, 1, 1, 224, 224, 1 / 3, True),      # VGG-16, one image (12 us, lean 26)
    (512, 512, 2, 1, 1, 32, 32, 0.4, True),        # stride 2 (42 us, wave 108)
    (256, 256, 2, 1, 8, 32, 32, 0.3, True),
    (64, 128, 1, 2, 2, 40, 40, 0.4, True),         # dilation 2 (10 us, wave 32)
    (96, 64, 1, 1, 1, 119, 191, 0.3, True),        # odd width
    (512, 512, 1, 1, 1, 4, 15, 1 / 3, False),      # the smallest maps: split over the channels there
    (512, 512, 1, 1, 1, 10, 12, 0.6, False),
    (32, 32, 1, 1, 1, 32, 32, 0.5, False),
])
def test_matrix_core_choice_over_the_range(c_out, c_in, s, d, n, h, w, keep, mfma):
    b = _blob(15, c_out, c_in, pp.PP_BF16, keep=keep, s=s, p=d, d=d)
    assert (pp.conv2d_recipe(b, n, h, w, pp.PP_BF16) == MFMA) is mfma
    # without scratch for the expansion: another plan, never a refusal
    assert pp.conv2d_recipe(b, n, h, w, pp.PP_BF16, with_workspace=False) not in (MFMA, -1)


def test_fused_pool_runs_the_form_of_the_plain_conv():
    # a network's fused pool gives bitwise the conv and the pool apart, so both run one form
    conv = dict(op="conv3", src=0, dst=2, c_in=64, c_out=64, stride=1, pad=1, dil=1, lib="canon8")
    for c_out, c_in, hw in ((64, 64, 224), (256, 256, 56), (64, 64, 40), (64, 48, 100)):
        L = workloads.random_layer(16, c_out, c_in, keep=1 / 3)
        ops = [dict(conv, c_in=c_in, c_out=c_out), dict(op="maxpool2", src=2, dst=1)]
        plan = pp.net_plan(ops, [L, {}], 1, c_in, hw, hw, "bf16")
        alone = pp.conv2d_recipe(_blob(16, c_out, c_in, pp.PP_BF16, keep=1 / 3), 1, hw, hw, pp.PP_BF16)
        assert plan["fused"] == {1: "maxpool2"} and plan["recipe"][0] == alone, (c_out, c_in, hw)
    other = [0x00F, 0x0B2, 0x1C8, 0x055, 0x113, 0x0A9]   # any other library: no fused pool, as on the vector kernels
    L = workloads.random_layer(17, 64, 64, lib=np.array(other, np.uint16))
    assert pp.net_plan([conv, dict(op="maxpool2", src=2, dst=1)], [L, {}], 1, 64, 224, 224, "bf16")["fused"] == {}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("op", ["maxpool2", "pshuf2"])
def test_no_fusion_takes_a_conv_off_the_few_channel_kernels(op, dtype):
    # (they take no fused op, and the kernel that does sums in another order)
    def plan(c_in, c_out, hw, lib):
        conv = dict(op="conv3", src=0, dst=2, c_in=c_in, c_out=c_out, stride=1, pad=1, dil=1)
        L = workloads.random_layer(18, c_out, c_in, lib=lib, keep=1.0)
        return pp.net_plan([conv, dict(op=op, src=2, dst=1)], [L, {}], 1, c_in, *hw, dtype)

    assert plan(64, 4, (960, 1024), workloads.DENSE9)["fused"] == {}
    assert plan(64, 4, (960, 1024), workloads.DENSE9)["recipe"][0] == 61
    assert plan(3, 16, (64, 64), workloads.DENSE9)["fused"] == {}
    # layers of the other kernels fuse as before
    assert plan(64, 4, (64, 64), workloads.DENSE9)["fused"] == ({1: op} if dtype == "f32" else {})
    assert plan(64, 16, (960, 1024), workloads.DENSE9)["fused"] == {1: op}


@pytest.mark.parametrize("c_out,c_in", [(128, 128), (64, 256), (64, 64), (256, 64)])
@pytest.mark.parametrize("dtype", [0, 1])
def test_workspace_covers_every_fused_call(c_out, c_in, dtype):
    import ctypes
    lib = pp.load_library()
    b = _blob(19, c_out, c_in, dtype, keep=1 / 3)
    grown = 0
    for h, w in ((14, 14), (28, 28), (40, 56), (56, 56), (128, 128), (120, 200)):
        ws, plain = pp.conv2d_workspace(b, 1, h, w, dtype), 0
        for flags in (0, pp.PP_MAXPOOL2, pp.PP_ACCUMULATE, pp.PP_PIXSHUF2, pp.PP_UPSAMPLE2, pp.PP_UPSAMPLE2 | pp.PP_PIXSHUF2):
            up = 2 if flags & pp.PP_UPSAMPLE2 else 1
            nb = ctypes.c_size_t(0)
            assert lib.pp_conv2d_scratch(b.ctypes.data, b.nbytes, 1, h // up, w // up, dtype, flags, ctypes.byref(nb)) == pp.PP_OK
            assert nb.value <= ws
            plain = nb.value if not flags else plain
        grown += ws > plain
    if (c_out, c_in, dtype) == (128, 128, 1):
        assert grown   # 128 x 128: lean alone, on the matrix cores with a shuffle
