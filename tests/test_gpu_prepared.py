"""Prepared weights are read where pp_conv2d_prepare wrote them, by calls on
any stream: bitwise the result of the call that expands them itself, right
after prepare(), after a second prepare() with other weights, and where the
first prepared call of a shape is recorded in a graph."""
import numpy as np
import pytest

import workloads
from oracle import bf16 as obf16

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
pp = pytest.importorskip("paper_2004_11250_amd")

SHAPES = [  # dtype, (n, c_out, c_in, h, w): the matrix-core form, and the lean kernel with and without a channel split
    ("bf16", (1, 256, 256, 56, 56)),
    ("bf16", (1, 512, 512, 14, 14)),
    ("f32", (1, 512, 512, 14, 14)),
    ("f32", (1, 64, 64, 60, 44)),
]


def _pair(seed, dtype, shape):
    """(packed layer, input)"""
    n, c_out, c_in, h, w = shape
    L = workloads.random_layer(seed, c_out, c_in, keep=1 / 3)
    wd = pp.PP_BF16 if dtype == "bf16" else pp.PP_F32
    layer = pp.PackedLayer.from_weights(L["w"], L["b"], L["pid"], L["conn"], L["lib"], wdtype=wd)
    x = torch.from_numpy(obf16.round_f32(workloads.random_input(seed, (n, c_in, h, w)))).cuda()
    return layer, x.to(torch.bfloat16) if dtype == "bf16" else x


@pytest.mark.parametrize("dtype,shape", SHAPES)
def test_another_stream_right_after_prepare(dtype, shape):
    layer, x = _pair(3100, dtype, shape)
    print("prepared, another stream", dtype, shape, flush=True)
    want = pp.conv2d_fwd(layer, x, relu=True)
    out = torch.empty_like(want)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    layer.scratch.clear()
    layer.prepare()
    pp.conv2d_fwd(layer, x, relu=True, prepared=True, stream=side, out=out)
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    if pp.conv2d_recipe(layer.h_blob, shape[0], *shape[3:], layer.info["wdtype"]) == 64:
        assert not layer.scratch   # no copy of the weights


@pytest.mark.parametrize("dtype,shape", SHAPES)
def test_second_prepare_with_other_weights(dtype, shape):
    layer, x = _pair(3200, dtype, shape)
    other, _ = _pair(3201, dtype, shape)
    print("prepared twice", dtype, shape, flush=True)
    layer.prepare()
    first = pp.conv2d_fwd(layer, x, prepared=True)
    layer.h_blob, layer.d_blob, layer.info = other.h_blob, other.d_blob, other.info
    layer.prepare()
    got, want = pp.conv2d_fwd(layer, x, prepared=True), pp.conv2d_fwd(other, x)
    assert torch.equal(got, want) and not torch.equal(got, first)


@pytest.mark.parametrize("dtype,shape", SHAPES)
def test_first_prepared_call_in_a_graph(dtype, shape):
    layer, x = _pair(3300, dtype, shape)
    print("prepared, first call recorded", dtype, shape, flush=True)
    layer.prepare()
    out = torch.empty_like(pp.conv2d_fwd(layer, x))
    layer.scratch.clear()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pp.conv2d_fwd(layer, x, out=out, prepared=True)
    eager = pp.conv2d_fwd(layer, x, prepared=True)   # before the graph has run
    want = pp.conv2d_fwd(layer, x)
    assert torch.equal(eager, want)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert torch.equal(pp.conv2d_fwd(layer, x, prepared=True), want)


@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("dtype,shape", [("f32", (1, 512, 512, 14, 14)), ("bf16", (2, 128, 256, 40, 40))])
def test_two_streams_have_scratch_of_their_own(dtype, shape, prepared):
    # a channel split's partial sums (or the expanded weights) of calls that overlap
    layer, x = _pair(3600, dtype, shape)
    print("two streams", dtype, shape, prepared, flush=True)
    layer.prepare()
    xs = [x, (x * 0.5 + 1).contiguous()]
    want = [pp.conv2d_fwd(layer, v, prepared=prepared) for v in xs]
    outs = [[torch.empty_like(want[0]) for _ in range(20)] for _ in xs]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in xs]
    for k in range(20):
        for v, o, s in zip(xs, outs, streams):
            pp.conv2d_fwd(layer, v, out=o[k], prepared=prepared, stream=s)
    torch.cuda.synchronize()
    for w, o in zip(want, outs):
        assert all(torch.equal(y, w) for y in o)
    bufs = [b.data_ptr() for b in layer.scratch.values()]
    assert len(set(bufs)) == len(bufs) and (not bufs or len(bufs) == 3)   # the current stream's and theirs


@pytest.mark.parametrize("how", ["deepcopy", "pickle", "saved by another build"])
@pytest.mark.parametrize("dtype,shape", SHAPES[:3])
def test_copied_and_saved_layers_prepare_their_own(dtype, shape, how):
    import copy
    import io
    layer, x = _pair(3700, dtype, shape)
    print("prepared layer", how, dtype, shape, flush=True)
    layer.prepare()
    want = pp.conv2d_fwd(layer, x, prepared=True)
    if how == "deepcopy":
        other = copy.deepcopy(layer)
    else:
        if how != "pickle":   # as whole attributes, the prepared bytes in another order
            state = dict(h_blob=layer.h_blob, info=layer.info, d_blob=layer.d_blob, scratch={},
                         prepared=layer.prepared.view(-1, 2).flip(0).reshape(-1).contiguous())
            other = pp.PackedLayer.__new__(pp.PackedLayer)
            other.__setstate__(state)
        else:
            buf = io.BytesIO()
            torch.save(layer, buf)
            buf.seek(0)
            other = torch.load(buf, weights_only=False)
    assert other.prepared.data_ptr() != layer.prepared.data_ptr()
    assert torch.equal(pp.conv2d_fwd(other, x, prepared=True), want)


@pytest.mark.parametrize("mode", ["pixshuf2", "upsample2"])
def test_fused_call_takes_one_form_prepared_or_not(mode):
    # lean alone (no scratch), on the matrix cores with the op fused: the same
    # bits with the weights expanded per call, prepared, and in the call
    # without an allocation
    layer, x = _pair(3900, "bf16", (1, 128, 128, 128, 128))
    print("one form", mode, flush=True)
    if mode == "upsample2":
        x = x[:, :, :64, :64].contiguous()
    h, w = x.shape[2:]
    layer.prepare()
    want = pp.conv2d_fwd(layer, x, prepared=True, **{mode: True})
    assert torch.equal(pp.conv2d_fwd(layer, x, **{mode: True}), want)
    out = torch.empty_like(want)
    lib, flag = pp.load_library(), pp.PP_PIXSHUF2 if mode == "pixshuf2" else pp.PP_UPSAMPLE2
    assert lib.pp_conv2d_fwd_noalloc(layer.h_blob.ctypes.data, layer.h_blob.nbytes, layer.d_blob.data_ptr(), x.data_ptr(),
                                     out.data_ptr(), 1, h, w, pp.PP_BF16, flag, None) == pp.PP_OK
    torch.cuda.synchronize()
    assert torch.equal(out, want)


@pytest.mark.parametrize("dtype,shape", SHAPES)
def test_prepared_weights_at_the_head_of_a_workspace(dtype, shape):
    # pp_conv2d_fwd with PP_PREPARED: the weights, then scratch from the next
    # 256-byte boundary; and without that scratch
    layer, x = _pair(4000, dtype, shape)
    n, c_out, c_in, h, w = shape
    wd = layer.info["wdtype"]
    print("prepared head", dtype, shape, flush=True)
    head = layer.prepare()
    tail = pp.conv2d_workspace(layer.h_blob, n, h, w, wd)
    size = -(-head.numel() // 256) * 256 + tail
    ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")
    ws[:head.numel()] = head
    lib = pp.load_library()
    for nbytes, want in ((size, pp.conv2d_fwd(layer, x, relu=True, prepared=True)),
                         (head.numel(), None if tail else pp.conv2d_fwd(layer, x, relu=True, workspace=None))):
        y = torch.full((n, c_out, h, w), float("nan"), dtype=x.dtype, device="cuda")
        st = lib.pp_conv2d_fwd(layer.h_blob.ctypes.data, layer.h_blob.nbytes, layer.d_blob.data_ptr(), x.data_ptr(),
                               y.data_ptr(), n, h, w, wd, pp.PP_RELU | pp.PP_PREPARED, ws.data_ptr(), nbytes, None)
        assert st == pp.PP_OK, lib.pp_last_error()
        torch.cuda.synchronize()
        assert torch.isfinite(y).all() and (want is None or torch.equal(y, want))
    assert torch.equal(ws[:head.numel()], head)   # read only
