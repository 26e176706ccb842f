"""The entry point for callers that cannot allocate (sparq_conv_gemm_static_ws): called through the C ABI with
ctypes, its int32 and fp32 results must equal those of sparq_conv_gemm with a caller workspace, bit for bit, on
calls in a row that share the library's one scratch array -- the second with a smaller input than the first."""
import ctypes

import numpy as np
import pytest
import torch

import sparq_synth as S

pytestmark = pytest.mark.gpu

LIMIT = 64 << 20      # SPARQ_STATIC_WORKSPACE_BYTES of include/sparq.h


@pytest.fixture(scope="module")
def sq():
    assert torch.cuda.is_available(), "GPU tests need a device"
    import paper_2105_11010_amd as sq_
    return sq_


def _both(sq, layer, seed):
    """(acc, out) of sparq_conv_gemm with a caller workspace, and of the static-scratch entry point via raw ctypes."""
    dev = torch.device("cuda:0")
    from dataclasses import replace
    x, w, sc = S.gen_layer(7, replace(layer, index=seed))
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    m = sq.mode(*layer.mode.astuple())
    xd, wd, sd = (torch.from_numpy(a).to(dev) for a in (x, w, sc))
    packed = torch.empty(sq.sparq_packed_bytes(d), dtype=torch.uint8, device=dev)
    sq.sparq_pack_weights(wd, d, packed)
    wsb = sq.sparq_workspace_bytes(d, m)
    ws = torch.empty(wsb, dtype=torch.uint8, device=dev) if wsb else None
    acc0 = torch.empty((layer.M, layer.N), dtype=torch.int32, device=dev)
    out0 = torch.empty((layer.M, layer.N), dtype=torch.float32, device=dev)
    sq.sparq_conv_gemm(xd, packed, d, m, acc=acc0, scale=sd, out=out0, workspace=ws)
    acc1 = torch.full((layer.M, layer.N), -7, dtype=torch.int32, device=dev)
    out1 = torch.full((layer.M, layer.N), -7.0, dtype=torch.float32, device=dev)
    torch.cuda.synchronize()
    vp = ctypes.c_void_p
    st = sq.lib.sparq_conv_gemm_static_ws(vp(xd.data_ptr()), vp(packed.data_ptr()), ctypes.byref(d), ctypes.byref(m),
                                          vp(acc1.data_ptr()), vp(sd.data_ptr()), vp(out1.data_ptr()),
                                          vp(torch.cuda.current_stream().cuda_stream))
    assert st == 0, sq.strerror(st)
    torch.cuda.synchronize()
    return wsb, (x, w, sc), acc0, out0, acc1, out1


def test_two_calls_in_a_row_the_second_smaller(sq, oracle):
    m5 = S.Mode(4, S.OPT5, 1, 1)
    # first: a layer with an odd channel count (trimmed, channel-padded copy in the scratch), 6.4 MB of scratch;
    # second: a smaller such layer (in the same scratch, among what the first left there);
    # third: a layer that needs no scratch at all
    layers = [S.ConvLayer("first_3x3_63", 2, 223, 223, 63, 64, 3, 3, (2, 2), (1, 1), 0.3, m5),
              S.ConvLayer("odd_3x3_65", 2, 17, 17, 65, 48, 3, 3, (1, 1), (1, 1), 0.5, S.Mode(4, S.OPT3, 0, 1)),
              S.ConvLayer("plain_1x1_128", 2, 14, 14, 128, 96, 1, 1, (1, 1), (0, 0), 0.5, m5)]
    used = []
    for i, layer in enumerate(layers):
        d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
        assert ("padded_copy" in sq.sparq_conv_plan(d, sq.mode(*layer.mode.astuple()))) == (i < 2)      # (written, not only asked for)
        wsb, (x, w, sc), acc0, out0, acc1, out1 = _both(sq, layer, i)
        used.append(wsb)
        assert torch.equal(acc0, acc1), f"{layer.name}: int32 results differ from sparq_conv_gemm"
        assert torch.equal(out0, out1), f"{layer.name}: fp32 results differ from sparq_conv_gemm"
        if i > 0:     # and the small ones against the oracle itself
            ref_acc, ref_out = oracle.conv_gemm(x, w, layer.stride, layer.pad, scale=sc, **layer.mode.kwargs())
            assert np.array_equal(acc1.cpu().numpy(), ref_acc)
            assert np.all(np.abs(out1.cpu().numpy().astype(np.float64) - ref_out) <= 1e-6 * np.abs(ref_out))
    assert used[0] > used[1] > 0 and used[2] == 0, used


def test_a_layer_past_the_scratch_limit_is_refused_before_any_launch(sq):
    """102 MB of padded copy: SPARQ_EWORKSPACE, nothing launched (the pointers are never dereferenced)."""
    d = sq.conv_desc(512, 224, 224, 3, 64, 7, 7, (2, 2), (3, 3))
    m = sq.mode(4, S.OPT5, 1, 1)
    assert sq.sparq_workspace_bytes(d, m) > LIMIT
    vp = ctypes.c_void_p
    dummy = torch.empty(256, dtype=torch.uint8, device="cuda:0")
    st = sq.lib.sparq_conv_gemm_static_ws(vp(dummy.data_ptr()), vp(dummy.data_ptr()), ctypes.byref(d), ctypes.byref(m),
                                          vp(dummy.data_ptr()), None, None, None)
    assert st == 3, sq.strerror(st)
