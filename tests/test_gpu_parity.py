"""GPU parity: libsparq (HIP, through the C ABI) against the CPU oracle, element by element."""
import numpy as np
import pytest
import torch

import sparq_synth as S

pytestmark = pytest.mark.gpu

MODES_N4 = [S.Mode(4, m, r, p) for m in (S.OPT5, S.OPT3, S.OPT2) for r in (0, 1) for p in (0, 1)]
MODES_LOW = [S.Mode(2, S.OPT7_2B, r, p) for r in (0, 1) for p in (0, 1)] + \
            [S.Mode(3, S.OPT6_3B, r, p) for r in (0, 1) for p in (0, 1)]
MODES_ODD = [S.Mode(4, 0x1B, 1, 1), S.Mode(4, 0x13, 0, 1), S.Mode(3, 0x2D, 1, 1), S.Mode(2, 0x5F, 1, 1), S.PLAIN8]


@pytest.fixture(scope="module")
def sq():
    assert torch.cuda.is_available(), "GPU tests need a device"
    import paper_2105_11010_amd as sq_
    return sq_


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def run_conv(sq, x, w, sc, layer, mode, want_acc=True, want_out=True):
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    m = sq.mode(*mode.astuple())
    xd, wd, sd = dev(x), dev(w), dev(sc)
    packed = torch.empty(sq.sparq_packed_bytes(d), dtype=torch.uint8, device="cuda:0")
    sq.sparq_pack_weights(wd, d, packed)
    wsb = sq.sparq_workspace_bytes(d, m)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda:0") if wsb else None
    acc = torch.full((layer.M, layer.N), -7, dtype=torch.int32, device="cuda:0") if want_acc else None
    out = torch.full((layer.M, layer.N), -7.0, dtype=torch.float32, device="cuda:0") if want_out else None
    sq.sparq_conv_gemm(xd, packed, d, m, acc=acc, scale=sd if want_out else None, out=out, workspace=ws)
    torch.cuda.synchronize()
    return (acc.cpu().numpy() if want_acc else None), (out.cpu().numpy() if want_out else None)


def check_layer(sq, oracle, layer, mode, seed_cfg=8, rows=None):
    x, w, sc = S.gen_layer(seed_cfg, layer)
    acc, out = run_conv(sq, x, w, sc, layer, mode)
    ref_acc, ref_out = oracle.conv_gemm(x, w, layer.stride, layer.pad, scale=sc, rows=rows, **mode.kwargs())
    if rows is not None:
        acc, out = acc[rows], out[rows]
    assert np.array_equal(acc, ref_acc), f"{layer.name} {mode.label}: int32 mismatch"
    # fp32 dequantised output within 1e-6 relative of the fp64 oracle
    err = np.abs(out.astype(np.float64) - ref_out)
    assert np.all(err <= 1e-6 * np.abs(ref_out)), f"{layer.name} {mode.label}: fp32 output off"


# ---------------------------------------------------------------- trim ------

@pytest.mark.parametrize("mode", MODES_N4 + MODES_LOW + MODES_ODD, ids=lambda m: m.label + f"-{m.shift_mask:#x}")
def test_trim_all_pairs(sq, oracle, mode):
    """All 256 x 256 activation pairs, in both byte lanes of the packed word."""
    a, b = np.meshgrid(np.arange(256, dtype=np.uint8), np.arange(256, dtype=np.uint8), indexing="ij")
    x = np.stack([a, b, b, a], axis=-1).reshape(-1, 4)
    xd = dev(x)
    y = torch.empty_like(xd)
    sq.sparq_trim(xd, y, sq.mode(*mode.astuple()))
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy(), oracle.trim(x, **mode.kwargs()))


@pytest.mark.parametrize("C", [1, 2, 3, 6, 7, 16, 30, 33, 64, 159])
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.Mode(4, S.OPT3, 0, 1), S.Mode(2, S.OPT7_2B, 1, 1)],
                         ids=lambda m: m.label)
def test_trim_row_lengths(sq, oracle, C, mode):
    """Odd and ragged channel counts: the last channel of an odd row has no partner."""
    rng = S.rng_for(8, 100 + C)
    for rows in (1, 5, 1031):
        x = S.gen_activations((rows, C), 0.5, rng)
        xd = dev(x)
        y = torch.empty_like(xd)
        sq.sparq_trim(xd, y, sq.mode(*mode.astuple()))
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), oracle.trim(x, **mode.kwargs())), (rows, C)


def test_trim_in_place_large_and_empty(sq, oracle):
    mode = S.Mode(4, S.OPT5, 1, 1)
    x = S.gen_activations((4099, 96), 0.5, S.rng_for(8, 200))
    xd = dev(x)
    sq.sparq_trim(xd, xd, sq.mode(*mode.astuple()))
    torch.cuda.synchronize()
    assert np.array_equal(xd.cpu().numpy(), oracle.trim(x, **mode.kwargs()))
    e = torch.empty((0, 8), dtype=torch.uint8, device="cuda:0")
    sq.sparq_trim(e, e, sq.mode(*mode.astuple()))


def test_trim_streamed_form(sq, oracle):
    """A call that moves 256 MiB or more out of place takes the kernel with non-temporal accesses: every byte
    against the oracle on a 136 MB tensor with a ragged tail (one 16-byte word plus a few pairs left over)."""
    mode = S.Mode(4, S.OPT3, 1, 1)
    block = S.gen_activations((1 << 22,), 0.5, S.rng_for(8, 210))
    x = np.resize(block, (1, (136 << 20) + 22))
    xd, yd = dev(x), torch.zeros(x.shape, dtype=torch.uint8, device="cuda:0")
    sq.sparq_trim(xd, yd, sq.mode(*mode.astuple()))
    torch.cuda.synchronize()
    assert np.array_equal(yd.cpu().numpy(), oracle.trim(x, **mode.kwargs()))


@pytest.mark.parametrize("C", [17, 19, 31, 1023])
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.Mode(4, S.OPT3, 0, 1), S.Mode(3, S.OPT6_3B, 1, 1),
                                  S.Mode(2, S.OPT7_2B, 0, 1), S.Mode(4, S.OPT5, 1, 0)], ids=lambda m: m.label)
def test_trim_odd_rows_as_one_stream(sq, oracle, C, mode):
    """Odd channel counts of at least 16: pairs across words, wavefronts and workgroups, row ends at every place of a
    word, tensors that end inside a word; more than one round per wavefront."""
    rng = S.rng_for(8, 220 + C)
    for rows in (1, 2, 61, 64, 999, 1 + (18 << 20) // C):
        x = S.gen_activations((rows, C), 0.5, rng)
        y = torch.full((rows * C + 16,), 77, dtype=torch.uint8, device="cuda:0")
        sq.sparq_trim(dev(x), y[:rows * C].view(rows, C), sq.mode(*mode.astuple()))
        torch.cuda.synchronize()
        got = y.cpu().numpy()
        assert np.array_equal(got[:rows * C].reshape(rows, C), oracle.trim(x, **mode.kwargs())), (rows, C)
        assert np.all(got[rows * C:] == 77), "bytes past the tensor were written"


@pytest.mark.parametrize("C", [35, 36, 7, 16])
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.Mode(4, S.OPT3, 0, 0)], ids=lambda m: m.label)
def test_trim_is_one_launch(sq, oracle, C, mode):
    """Also where the tensor ends inside a 16-byte word: captured calls hold one node, and replays give the oracle's bytes."""
    import ctypes
    x = S.gen_activations((333, C), 0.5, S.rng_for(8, 240 + C))
    m = sq.mode(*mode.astuple())
    xd = dev(x)
    y = torch.zeros_like(xd)
    sq.sparq_trim(xd, y, m)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        sq.sparq_trim(xd, y, m)
    nodes = ctypes.c_size_t(0)
    assert sq.lib.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(nodes)) == 0
    assert nodes.value == 1
    for _ in range(2):
        y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), oracle.trim(x, **mode.kwargs()))


# ------------------------------------------------------------- dequant ------

@pytest.mark.parametrize("M,N", [(1, 1), (37, 19), (513, 64), (1000, 160)])
def test_dequant(sq, oracle, M, N):
    rng = S.rng_for(8, 300 + N)
    acc = rng.integers(-2 ** 31, 2 ** 31, size=(M, N), dtype=np.int64).astype(np.int32)
    sc = S.gen_scales(N, rng)
    out = torch.empty((M, N), dtype=torch.float32, device="cuda:0")
    sq.sparq_dequant(dev(acc), dev(sc), out)
    torch.cuda.synchronize()
    ref = oracle.dequant(acc, sc)
    err = np.abs(out.cpu().numpy().astype(np.float64) - ref)
    assert np.all(err <= 1e-6 * np.abs(ref))


def test_dequant_streamed_form(sq, oracle):
    """8 * M * N >= 256 MiB: the dequantisation kernel with non-temporal accesses, every element."""
    M, N = 65537, 512
    rng = S.rng_for(8, 310)
    acc = np.resize(rng.integers(-2 ** 31, 2 ** 31, size=(1 << 20,), dtype=np.int64).astype(np.int32), (M, N))
    sc = S.gen_scales(N, rng)
    out = torch.empty((M, N), dtype=torch.float32, device="cuda:0")
    sq.sparq_dequant(dev(acc), dev(sc), out)
    torch.cuda.synchronize()
    ref = oracle.dequant(acc, sc)
    err = np.abs(out.cpu().numpy().astype(np.float64) - ref)
    assert np.all(err <= 1e-6 * np.abs(ref))


# ------------------------------------------------------------- requant ------

@pytest.mark.parametrize("M,N", [(1, 1), (37, 19), (513, 64), (1000, 160), (0, 8)])
def test_requant(sq, oracle, M, N):
    """The standalone requantisation pass: bit-exact bytes, ties and both clamps included."""
    rng = S.rng_for(8, 400 + N)
    acc = rng.integers(-60000, 200000, size=(M, N), dtype=np.int64).astype(np.int32)
    if M:
        acc[0, 0] = 5                       # 2.5 with factor 0.5: the tie
    f = rng.uniform(5e-4, 3e-3, size=N).astype(np.float32)
    f[0] = 0.5
    y = torch.full((M, N), 7, dtype=torch.uint8, device="cuda:0")
    sq.sparq_requant(dev(acc), dev(f), y)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy(), oracle.requant(acc, f))


# Widths that are no multiple of four and factors off 16 bytes: words that end a row and begin the next, results past the last
# word, the table's smallest and largest widths (and one past them), calls of less than and more than one workgroup.
@pytest.mark.parametrize("M,N,skew", [(3, 1, 0), (1031, 2, 0), (5, 3, 0), (4099, 5, 0), (37, 161, 0), (2051, 161, 0), (513, 64, 1),
                                      (33, 1023, 0), (2050, 2047, 0), (2048, 2049, 0), (2050, 2048, 1), (524289, 65, 0),
                                      # ... and the line below which there is no table, by results and by rows
                                      (2047, 1, 0), (2050, 1, 0), (682, 3, 0), (683, 3, 0), (120, 161, 0), (121, 161, 0), (767, 1023, 0),
                                      (768, 1023, 0), (767, 1024, 1), (769, 1024, 1)])
def test_per_channel_any_width(sq, oracle, M, N, skew):
    rng = S.rng_for(8, 500 + N)
    acc = np.resize(rng.integers(-60000, 200000, size=min(M * N, 1 << 18), dtype=np.int64).astype(np.int32), (M, N))
    f = np.concatenate([np.zeros(skew), rng.uniform(5e-4, 3e-3, size=N)]).astype(np.float32)
    accd, fd = dev(acc), dev(f)[skew:]
    y = torch.full((M, N), 7, dtype=torch.uint8, device="cuda:0")
    out = torch.full((M, N), -7.0, dtype=torch.float32, device="cuda:0")
    sq.sparq_requant(accd, fd, y)
    sq.sparq_dequant(accd, fd, out)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy(), oracle.requant(acc, f[skew:]))
    assert np.array_equal(out.cpu().numpy(), acc.astype(np.float32) * f[skew:])      # two roundings to nearest, as defined


def run_conv_u8(sq, x, w, f, layer, mode, out_mode=None):
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    m = sq.mode(*mode.astuple())
    packed = torch.empty(sq.sparq_packed_bytes(d), dtype=torch.uint8, device="cuda:0")
    sq.sparq_pack_weights(dev(w), d, packed)
    wsb = sq.sparq_workspace_bytes(d, m)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda:0") if wsb else None
    y = torch.full((layer.M, layer.N), 7, dtype=torch.uint8, device="cuda:0")
    sq.sparq_conv_gemm_u8(dev(x), packed, d, m, dev(f), y, workspace=ws,
                          out_mode=sq.mode(*out_mode.astuple()) if out_mode else None)
    torch.cuda.synchronize()
    return y.cpu().numpy()


def check_layer_u8(sq, oracle, layer, mode, seed_cfg=8, out_mode=None):
    """Requantised uint8 output of the fused convolution (optionally trimmed for the next layer): every byte
    equals the oracle's."""
    x, w, _ = S.gen_layer(seed_cfg, layer)
    f = S.gen_requant(layer, S.rng_for(seed_cfg, 900 + layer.index))
    y = run_conv_u8(sq, x, w, f, layer, mode, out_mode)
    ref = oracle.conv_gemm_u8(x, w, f, layer.stride, layer.pad, out_mode=out_mode.kwargs() if out_mode else None,
                              **mode.kwargs())
    assert np.array_equal(y, ref), f"{layer.name} {mode.label}: uint8 mismatch"
    assert (ref == 0).any() and ref.max() > 60, "degenerate test case"


@pytest.mark.parametrize("N", [4, 3])
def test_requant_every_tie_and_both_clamps(sq, oracle, N):
    """Factors 0.5 and 0.25 over a run of consecutive accumulators: every second / fourth product is a tie;
    negative products clamp to 0, large ones to 255 (N = 4: the vector kernel, N = 3: the scalar one)."""
    acc = np.arange(-600, 600 + 1200 * N, dtype=np.int32)[:1200 * N].reshape(1200, N)
    f = np.array([0.5, 0.25, 0.5, 0.125][:N], dtype=np.float32)
    y = torch.full((1200, N), 7, dtype=torch.uint8, device="cuda:0")
    sq.sparq_requant(dev(acc), dev(f), y)
    torch.cuda.synchronize()
    ref = oracle.requant(acc, f)
    assert np.array_equal(y.cpu().numpy(), ref)
    assert (ref == 0).any() and (ref == 255).any()


# ---------------------------------------------------------- conv / gemm -----

def test_config0_full(sq, oracle):
    (layer,) = S.config0()
    x, w, sc = S.gen_layer(0, layer)
    acc, out = run_conv(sq, x, w, sc, layer, layer.mode)
    ref_acc, ref_out = oracle.conv_gemm(x, w, layer.stride, layer.pad, scale=sc, **layer.mode.kwargs())
    assert np.array_equal(acc, ref_acc)
    assert np.all(np.abs(out.astype(np.float64) - ref_out) <= 1e-6 * np.abs(ref_out))


SHAPES = [
    # name, B, H, W, C, N, KH, KW, stride, pad
    S.ConvLayer("gemm_small", 1, 300, 1, 64, 32),
    S.ConvLayer("gemm_ragged", 1, 777, 1, 208, 100),
    S.ConvLayer("gemm_k16", 1, 130, 1, 16, 8),
    S.ConvLayer("gemm_k48_n3", 1, 129, 1, 48, 3),
    S.ConvLayer("1x1_s2", 3, 15, 13, 32, 40, 1, 1, (2, 2), (0, 0)),
    S.ConvLayer("3x3_p1", 2, 13, 11, 32, 24, 3, 3, (1, 1), (1, 1)),
    S.ConvLayer("3x3_s2_p1", 2, 17, 19, 48, 36, 3, 3, (2, 2), (1, 1)),
    S.ConvLayer("3x3_s2_p0", 1, 17, 17, 96, 20, 3, 3, (2, 2), (0, 0)),
    S.ConvLayer("5x5_p2", 1, 12, 12, 48, 64, 5, 5, (1, 1), (2, 2)),
    S.ConvLayer("1x7", 2, 9, 17, 32, 33, 1, 7, (1, 1), (0, 3)),
    S.ConvLayer("7x1", 2, 17, 9, 160, 17, 7, 1, (1, 1), (3, 0)),
    S.ConvLayer("odd_c65", 1, 10, 10, 65, 12, 3, 3, (1, 1), (1, 1)),
    S.ConvLayer("odd_c3_7x7", 2, 20, 20, 3, 16, 7, 7, (2, 2), (3, 3)),
    S.ConvLayer("odd_c159_n161", 1, 6, 17, 159, 161, 1, 7, (1, 1), (0, 3)),
    S.ConvLayer("wide_n", 1, 140, 1, 128, 520),
    # at most 4 channels: the pixel-folded first-layer path (and shapes that cannot fold)
    S.ConvLayer("thin_3x3_s1_c3", 2, 9, 16, 3, 10, 3, 3, (1, 1), (1, 1)),
    S.ConvLayer("thin_5x5_s2_c4", 1, 12, 24, 4, 7, 5, 5, (2, 2), (2, 2)),
    S.ConvLayer("thin_7x7_s2_c1", 3, 16, 32, 1, 64, 7, 7, (2, 2), (3, 3)),
    S.ConvLayer("thin_3x3_s2_c2_n130", 2, 10, 40, 2, 130, 3, 3, (2, 2), (1, 1)),
    S.ConvLayer("thin_s4_no_fold", 1, 16, 32, 1, 5, 3, 3, (4, 4), (1, 1)),
    S.ConvLayer("thin_w18_no_fold", 1, 7, 18, 3, 9, 3, 3, (1, 1), (1, 1)),
]


# The library holds two convolution kernels (an im2col-gather form and an input-patch form) and
# picks one per layer; the tuning hook (sparq_set_tuning) forces either where the layer is eligible,
# so both are compared with the oracle on every shape.
@pytest.fixture
def tuning(sq):
    """tuning("path=patch,patch_tn=128") forces the kernel choice for the rest of the test."""
    yield sq.sparq_set_tuning
    sq.sparq_set_tuning(None)


@pytest.fixture(params=["auto", "gather", "patch", "patch-ws"])
def path(request, tuning):
    if request.param == "patch-ws":      # the wave-specialised form of the patch kernel
        tuning("path=patch,patch_ws=1")
    elif request.param != "auto":
        tuning(f"path={request.param},patch_ws=0")
    return request.param


@pytest.mark.parametrize("layer", SHAPES, ids=lambda l: l.name)
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.Mode(4, S.OPT3, 0, 1), S.Mode(2, S.OPT7_2B, 1, 1), S.PLAIN8],
                         ids=lambda m: m.label)
def test_conv_shapes(sq, oracle, layer, mode, path):
    check_layer(sq, oracle, layer, mode, seed_cfg=8)


# The kernel of layers with at most four channels: every channel count, row stride and filter height it is compiled for (and
# one in between), filters that need one or two groups of four pixels a row, an odd number of rows beside a half-empty last
# step, tiles of several images, of several rows and of a part of one row, output channels that fill no 64, ragged last tiles.
FEW_SHAPES = [
    S.ConvLayer("f_7x7_s2_c3_n64", 3, 40, 36, 3, 64, 7, 7, (2, 2), (3, 3)),
    S.ConvLayer("f_7x7_s2_c3_w224", 1, 30, 224, 3, 64, 7, 7, (2, 2), (3, 3)),
    S.ConvLayer("f_3x3_s1_c3_n48", 2, 9, 16, 3, 48, 3, 3, (1, 1), (1, 1)),
    S.ConvLayer("f_3x3_s1_c3_w1200", 1, 3, 1200, 3, 32, 3, 3, (1, 1), (1, 1)),
    S.ConvLayer("f_5x5_s1_c1_n16", 2, 11, 20, 1, 16, 5, 5, (1, 1), (2, 2)),
    S.ConvLayer("f_5x5_s2_c4_n80", 5, 7, 24, 4, 80, 5, 5, (2, 2), (2, 2)),
    S.ConvLayer("f_6x6_s2_c2_n130", 2, 10, 40, 2, 130, 6, 6, (2, 2), (2, 2)),
    S.ConvLayer("f_4x4_s4_c3_n96", 2, 16, 32, 3, 96, 4, 4, (4, 4), (0, 0)),
    S.ConvLayer("f_7x4_s4_c4_n16", 1, 30, 16, 4, 16, 7, 4, (4, 4), (3, 0)),
    S.ConvLayer("f_2x2_s2_c1_n17", 40, 2, 8, 1, 17, 2, 2, (2, 2), (0, 0)),
    S.ConvLayer("f_8x7_s1_c3_n33", 1, 16, 12, 3, 33, 8, 7, (1, 1), (3, 3)),
    S.ConvLayer("f_1x3_s1_c2_n64_m8", 1, 1, 8, 2, 64, 1, 3, (1, 1), (0, 1)),
]


@pytest.mark.parametrize("layer", FEW_SHAPES, ids=lambda l: l.name)
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.Mode(4, S.OPT5, 1, 0), S.Mode(4, S.OPT3, 0, 1), S.Mode(4, S.OPT3, 0, 0),
                                  S.Mode(3, S.OPT6_3B, 1, 0), S.Mode(2, S.OPT7_2B, 1, 1), S.Mode(2, S.OPT7_2B, 0, 1), S.PLAIN8],
                         ids=lambda m: m.label)
def test_conv_few_channels(sq, oracle, layer, mode):
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    text = sq.sparq_conv_plan(d, sq.mode(*mode.astuple()))
    assert " kernel=conv_few_kernel" in text and ("u8_kernel=conv_few_kernel" in text) == (layer.N % 16 == 0), text
    check_layer(sq, oracle, layer, mode, seed_cfg=8)
    check_layer_u8(sq, oracle, layer, mode, seed_cfg=8, out_mode=mode if layer.N == 64 else None)


def exact_sums(oracle, x, w, layer, mode):
    """int32 sums of the trimmed input on the GPU, in double precision (every product and sum exact), a few images at a time."""
    xt, wd = dev(oracle.trim(x, **mode.kwargs())), dev(w).double().permute(0, 3, 1, 2).reshape(layer.N, -1).T.contiguous()
    step = max(1, (1 << 19) * layer.B // layer.M)
    for b in range(0, layer.B, step):
        rows = torch.nn.functional.unfold(xt[b:b + step].double().permute(0, 3, 1, 2), (layer.KH, layer.KW), padding=layer.pad, stride=layer.stride)
        yield rows.transpose(1, 2).reshape(-1, layer.K).contiguous().mm(wd).to(torch.int32)


# Workgroups that do several tiles one after the other -- their two patches in turn, the next tile's input on its way -- at every tile
# height (tm: of the results named) and row stride, with one, two and four channels, several column blocks and ragged last tiles.
FEW_MANY_TILES = [
    (128, "fp32", S.ConvLayer("f_many_3x3_c2_n96", 5, 111, 112, 2, 96, 3, 3, (1, 1), (1, 1))),
    (256, "fp32", S.ConvLayer("f_many_7x7_c4_n96", 31, 121, 116, 4, 96, 7, 7, (1, 1), (3, 3))),
    (512, "fp32", S.ConvLayer("f_many_7x7s2_c3_n80", 67, 219, 224, 3, 80, 7, 7, (2, 2), (3, 3))),
    (1024, "fp32", S.ConvLayer("f_many_3x1s2_c1_n18", 259, 223, 224, 1, 18, 3, 1, (2, 2), (1, 0))),
    (256, "bytes", S.ConvLayer("f_many_4x4s4_c2_n272", 9, 232, 240, 2, 272, 4, 4, (4, 4), (0, 0))),
    (512, "bytes", S.ConvLayer("f_many_5x7s2_c1_n144", 9, 213, 216, 1, 144, 5, 7, (2, 2), (2, 3))),
    (1024, "bytes", S.ConvLayer("f_many_3x3_c4_n48", 341, 40, 40, 4, 48, 3, 3, (1, 1), (1, 1))),
]


@pytest.mark.parametrize("tm,results,layer", FEW_MANY_TILES, ids=lambda v: v.name if isinstance(v, S.ConvLayer) else str(v))
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.Mode(2, S.OPT7_2B, 0, 1), S.PLAIN8], ids=lambda m: m.label)
def test_few_channels_many_tiles(sq, oracle, tm, results, layer, mode):
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    m = sq.mode(*mode.astuple())
    text, columns = sq.sparq_conv_plan(d, m), (layer.N + 63) // 64
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    slots = 2 * cus // columns
    assert layer.M > slots * tm and layer.M % tm != 0                # more tiles than workgroups, a ragged one at the end
    if results == "fp32":
        assert f"few_channels tile={tm}x64" in text, text
    else:                                                            # (the text names four-byte tiles: three tiles for two CUs decide for bytes)
        assert "u8_kernel=conv_few_kernel" in text, text
        assert (tm == 1024 or -(-layer.M // (2 * tm)) * columns * 2 < 3 * cus) and -(-layer.M // tm) * columns * 2 >= 3 * cus
    x, w, sc = S.gen_layer(8, layer)
    wd, sd = dev(w), dev(sc if results == "fp32" else S.rng_for(8, 900).uniform(2e-4, 4e-4, size=layer.N).astype(np.float32))
    packed = torch.empty(sq.sparq_packed_bytes(d), dtype=torch.uint8, device="cuda:0")
    sq.sparq_pack_weights(wd, d, packed)
    ws = torch.empty(sq.sparq_workspace_bytes(d, m), dtype=torch.uint8, device="cuda:0")
    acc = out = y = None
    if results == "fp32":
        acc = torch.full((layer.M, layer.N), -7, dtype=torch.int32, device="cuda:0")
        out = torch.full((layer.M, layer.N), -7.0, dtype=torch.float32, device="cuda:0")
        sq.sparq_conv_gemm(dev(x), packed, d, m, acc=acc, scale=sd, out=out, workspace=ws)
    else:
        y = torch.full((layer.M, layer.N), 7, dtype=torch.uint8, device="cuda:0")
        sq.sparq_conv_gemm_u8(dev(x), packed, d, m, sd, y, workspace=ws)
    torch.cuda.synchronize()
    at = 0
    for ref in exact_sums(oracle, x, w, layer, mode):
        here = slice(at, at + ref.shape[0])
        if results == "fp32":
            assert torch.equal(acc[here], ref), at
            assert torch.equal(out[here], ref.float() * sd), at      # two roundings to nearest, as defined
        else:
            assert torch.equal(y[here], (ref.float() * sd).round().clamp(0, 255).to(torch.uint8)), at
        at += ref.shape[0]
    assert at == layer.M


def test_few_channels_beside_half_a_million_outputs(sq, oracle):
    """The widest results: 1024 of these rows are 2^31 bytes and more, so tiles of 1024 pixels would store what is past N inside the
    tensor.  Every int32 and fp32 result against exact sums in double precision of the oracle's trimmed input."""
    layer, mode = S.ConvLayer("f_5x3_c2_n524304", 1, 32, 32, 2, 524304, 5, 3, (1, 1), (2, 1)), S.Mode(4, S.OPT5, 1, 1)
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    m = sq.mode(*mode.astuple())
    text = sq.sparq_conv_plan(d, m)
    assert "few_channels tile=512x64" in text, text
    x, w, sc = S.gen_layer(8, layer)
    wd, sd = dev(w), dev(sc)
    packed = torch.empty(sq.sparq_packed_bytes(d), dtype=torch.uint8, device="cuda:0")
    sq.sparq_pack_weights(wd, d, packed)
    ws = torch.empty(sq.sparq_workspace_bytes(d, m), dtype=torch.uint8, device="cuda:0")
    acc = torch.full((layer.M, layer.N), -7, dtype=torch.int32, device="cuda:0")
    out = torch.full((layer.M, layer.N), -7.0, dtype=torch.float32, device="cuda:0")
    sq.sparq_conv_gemm(dev(x), packed, d, m, acc=acc, scale=sd, out=out, workspace=ws)
    torch.cuda.synchronize()
    (ref,) = exact_sums(oracle, x, w, layer, mode)
    assert torch.equal(acc, ref)
    assert torch.equal(out, ref.float() * sd)                            # two roundings to nearest, as defined


# The split-reduction form (small layers): its three tiles; fewer reduction steps than wavefronts, shares of unequal
# length, ragged tiles, padded channels, images that share a tile, a patch that fills most of LDS.
SPLIT_SHAPES = [
    ("32x32", S.ConvLayer("s_1x3_c64", 1, 5, 5, 64, 33, 1, 3, (1, 1), (0, 1))),
    ("32x32", S.ConvLayer("s_1x1_c320", 1, 33, 1, 320, 70)),
    ("32x32", S.ConvLayer("s_1x1_c528_m1", 1, 1, 1, 528, 33)),
    ("32x32", S.ConvLayer("s_3x3_7x7_c512", 1, 7, 7, 512, 96, 3, 3, (1, 1), (1, 1))),
    ("32x32", S.ConvLayer("s_3x3_3x3_c80", 9, 3, 3, 80, 50, 3, 3, (1, 1), (1, 1))),
    ("32x32", S.ConvLayer("s_1x1_c4608", 1, 40, 1, 4608, 40)),
    ("32x32", S.ConvLayer("s_2x2_c72", 2, 10, 10, 72, 16, 2, 2, (1, 1), (0, 0))),
    ("32x32", S.ConvLayer("s_1x1_s2_c320", 3, 9, 9, 320, 40, 1, 1, (2, 2), (0, 0))),       # pixels of a strided 1x1 layer
    ("32x32", S.ConvLayer("s_3x3_s2_8x8_c96", 2, 8, 8, 96, 48, 3, 3, (2, 2), (1, 1))),     # many short patch rows
    ("32x64", S.ConvLayer("s_3x3_28_c64_n130", 3, 28, 28, 64, 130, 3, 3, (1, 1), (1, 1))),
    ("64x64", S.ConvLayer("s_3x3_56_c64", 4, 56, 56, 64, 64, 3, 3, (1, 1), (1, 1))),
    ("64x64", S.ConvLayer("s_3x3_s2_c96_n70", 6, 60, 60, 96, 70, 3, 3, (2, 2), (1, 1))),
]


@pytest.mark.parametrize("tile,layer", SPLIT_SHAPES, ids=lambda v: v if isinstance(v, str) else v.name)
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.Mode(4, S.OPT5, 1, 0), S.Mode(4, S.OPT3, 0, 1), S.Mode(4, S.OPT3, 0, 0),
                                  S.Mode(3, S.OPT6_3B, 1, 0), S.Mode(2, S.OPT7_2B, 1, 1), S.Mode(2, S.OPT7_2B, 0, 1), S.PLAIN8],
                         ids=lambda m: m.label)
def test_conv_split_reduction(sq, oracle, tile, layer, mode):
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    assert f"split_reduction tile={tile}" in sq.sparq_conv_plan(d, sq.mode(*mode.astuple()))
    check_layer(sq, oracle, layer, mode, seed_cfg=8)
    check_layer_u8(sq, oracle, layer, mode, seed_cfg=8)


# ... and patches whose rows are far from whole pieces of 64 chunks: one output column, strides that leave rows and columns out, many
# images to a tile, tiles inside one output row beside tiles of several, channel padding, each tile.
SPLIT_SHORT_ROWS = [
    ("32x32", S.ConvLayer("u_7x1_s2_2x2_c148", 57, 2, 2, 148, 36, 7, 1, (2, 2), (3, 0))), ("32x32", S.ConvLayer("u_3x3_s3_5x5_c112", 59, 5, 5, 112, 17, 3, 3, (3, 3), (1, 0))),
    ("32x32", S.ConvLayer("u_2x2_s3_88x4_c48", 5, 88, 4, 48, 60, 2, 2, (3, 3), (1, 0))), ("32x32", S.ConvLayer("u_1x3_5x40_c64", 2, 5, 40, 64, 50, 1, 3, (1, 1), (0, 1))),
    ("32x32", S.ConvLayer("u_5x5_s2_6x6_c96_m9", 1, 6, 6, 96, 80, 5, 5, (2, 2), (2, 2))), ("32x64", S.ConvLayer("u_3x3_5x5_c64_n96", 131, 5, 5, 64, 96, 3, 3, (1, 1), (1, 1))),
    ("64x64", S.ConvLayer("u_3x3_5x5_c60_n130", 121, 5, 5, 60, 130, 3, 3, (1, 1), (1, 1))),
]


@pytest.mark.parametrize("tile,layer", SPLIT_SHORT_ROWS, ids=lambda v: v if isinstance(v, str) else v.name)
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.Mode(4, S.OPT5, 1, 0), S.Mode(4, S.OPT3, 0, 1), S.Mode(4, S.OPT3, 0, 0),
                                  S.Mode(3, S.OPT6_3B, 1, 0), S.Mode(2, S.OPT7_2B, 1, 1), S.Mode(2, S.OPT7_2B, 0, 1), S.PLAIN8],
                         ids=lambda m: m.label)
def test_conv_split_reduction_of_short_patch_rows(sq, oracle, tile, layer, mode):
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    assert f"split_reduction tile={tile}" in sq.sparq_conv_plan(d, sq.mode(*mode.astuple()))
    check_layer(sq, oracle, layer, mode, seed_cfg=8)
    check_layer_u8(sq, oracle, layer, mode, seed_cfg=8, out_mode=mode)


# The form with the activations in registers (1x1 layers): every number of reduction steps it holds and numbers in between,
# pixels and channels that fill no fragment, strides, odd channel counts, runs of fewer than 128 result bytes, shares of the
# output channels, 64 pixels per wavefront (many pixels and channels).
ROWS_SHAPES = [
    S.ConvLayer("r_c64_m3", 1, 3, 1, 64, 64), S.ConvLayer("r_c64_n33", 1, 65, 1, 64, 33), S.ConvLayer("r_c48_n48", 1, 9, 7, 48, 48),
    S.ConvLayer("r_c128_n80_s2", 3, 15, 13, 128, 80, 1, 1, (2, 2), (0, 0)), S.ConvLayer("r_c65_n144", 2, 11, 11, 65, 144),
    S.ConvLayer("r_c192_n272", 5, 20, 20, 192, 272), S.ConvLayer("r_c176_n400", 1, 3000, 1, 176, 400),
    S.ConvLayer("r_c256_n1024_s3x2", 4, 17, 19, 256, 1024, 1, 1, (3, 2), (0, 0)), S.ConvLayer("r_c288_n96", 20, 35, 35, 288, 96),
    S.ConvLayer("r_c384_n160", 1, 9001, 1, 384, 160), S.ConvLayer("r_c512_n144", 1, 12555, 1, 512, 144),
    S.ConvLayer("r_c192_n512_wide", 1, 49169, 1, 192, 512), S.ConvLayer("r_c448_n528_wide", 1, 49169, 1, 448, 528),
]


@pytest.mark.parametrize("layer", ROWS_SHAPES, ids=lambda l: l.name)
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.Mode(3, S.OPT6_3B, 0, 1), S.PLAIN8], ids=lambda m: m.label)
def test_conv_activations_in_registers(sq, oracle, layer, mode):
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    assert "in_registers" in sq.sparq_conv_plan(d, sq.mode(*mode.astuple()))
    check_layer(sq, oracle, layer, mode, seed_cfg=8)
    check_layer_u8(sq, oracle, layer, mode, seed_cfg=8, out_mode=S.Mode(4, S.OPT5, 1, 1))


# Its kernel by name, for both results; asked for where the rule holds the weights instead.
@pytest.mark.parametrize("layer", ROWS_SHAPES, ids=lambda l: l.name)
def test_conv_activations_in_registers_by_name(sq, oracle, tuning, layer):
    mode = S.Mode(4, S.OPT5, 1, 1)
    if layer.name.endswith("_wide"):
        tuning("form=rows")
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    words = sq.sparq_conv_plan(d, sq.mode(*mode.astuple())).split()
    assert "kernel=conv_rows_kernel" in words and (layer.N % 16 or "u8_kernel=conv_rows_kernel" in words), words
    if layer.name.endswith("_wide"):
        check_layer(sq, oracle, layer, mode, seed_cfg=8)
        check_layer_u8(sq, oracle, layer, mode, seed_cfg=8, out_mode=mode)


# The same with the weights in LDS (pixels for every wavefront slot of 256 CUs, 98304 or 131072, and 1.1 to 2 times that for four-byte
# results): steps past the layer's own, ragged pixels and channels, a stride, layers on either side of that rule.
ROWS_HELD_SHAPES = [
    S.ConvLayer("rh_c40_n33", 1, 144193, 1, 40, 33), S.ConvLayer("rh_c64_n208", 1, 131103, 1, 64, 208), S.ConvLayer("rh_c64_n64_s2", 6, 299, 301, 64, 64, 1, 1, (2, 2), (0, 0)),
    S.ConvLayer("rh_c96_n96", 1, 196641, 1, 96, 96), S.ConvLayer("rh_c160_n128", 1, 262175, 1, 160, 128), S.ConvLayer("rh_c256_n64", 1, 144224, 1, 256, 64),
    S.ConvLayer("rh_c260_n16", 1, 147457, 1, 260, 16), S.ConvLayer("rh_c384_n224", 1, 98305, 1, 384, 224), S.ConvLayer("rh_c448_n48", 1, 98335, 1, 448, 48),
    S.ConvLayer("rh_c512_n208", 1, 98304, 1, 512, 208), S.ConvLayer("rh_c512_n224", 1, 196609, 1, 512, 224),
]


@pytest.mark.parametrize("layer", ROWS_HELD_SHAPES, ids=lambda l: l.name)
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.PLAIN8], ids=lambda m: m.label)
def test_conv_activations_in_registers_weights_in_lds(sq, oracle, layer, mode):
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    if layer.N % 16 == 0:
        assert "u8_kernel=conv_rows_kernel" in sq.sparq_conv_plan(d, sq.mode(*mode.astuple()))
        check_layer_u8(sq, oracle, layer, mode, seed_cfg=8, out_mode=S.Mode(4, S.OPT5, 1, 1))
    check_layer(sq, oracle, layer, mode, seed_cfg=8)


# Each kernel of that kind, by the plan: every number of steps for four-byte results and for bytes, at the fewest pixels and one more (256 CUs:
# 32 pixels for 1.1 to 2 times the wavefront slots, or for all of them), and the rows of 64 result bytes that leave room for more weights.
ROWS_HELD_FORMS = [
    (True, 128, S.ConvLayer("rf_c40_n48", 1, 144193, 1, 40, 48)), (True, 128, S.ConvLayer("rf_c100_n64", 1, 144193, 1, 100, 64)), (True, 128, S.ConvLayer("rf_c192_n64", 1, 144193, 1, 192, 64)),
    (True, 128, S.ConvLayer("rf_c256_n64", 1, 144193, 1, 256, 64)), (True, 128, S.ConvLayer("rf_c300_n16", 1, 137633, 1, 300, 16)), (True, 128, S.ConvLayer("rf_c384_n48", 1, 137633, 1, 384, 48)),
    (True, 128, S.ConvLayer("rf_c512_n80", 1, 147457, 1, 512, 80)), (True, 128, S.ConvLayer("rf_c128_n112", 1, 262177, 1, 128, 112)),
    (False, 128, S.ConvLayer("rf_c64_n80", 1, 131073, 1, 64, 80)), (False, 128, S.ConvLayer("rf_c100_n96", 1, 98305, 1, 100, 96)), (False, 128, S.ConvLayer("rf_c192_n32", 1, 98305, 1, 192, 32)),
    (False, 128, S.ConvLayer("rf_c256_n112", 1, 98305, 1, 256, 112)), (False, 128, S.ConvLayer("rf_c320_n144", 1, 98305, 1, 320, 144)), (False, 128, S.ConvLayer("rf_c384_n224", 1, 98305, 1, 384, 224)),
    (False, 64, S.ConvLayer("rf_c384_n288", 1, 196577, 1, 384, 288)), (False, 64, S.ConvLayer("rf_c330_n304", 1, 196609, 1, 330, 304)), (False, 64, S.ConvLayer("rf_c512_n224", 1, 196609, 1, 512, 224)),
    (None, 64, S.ConvLayer("rf_c320_n384", 1, 196577, 1, 320, 384)), (False, 0, S.ConvLayer("rf_c512_n208_l2", 1, 196576, 1, 512, 208)),
]


@pytest.mark.parametrize("held,run,layer", ROWS_HELD_FORMS, ids=lambda v: v.name if hasattr(v, "name") else str(v))
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.PLAIN8], ids=lambda m: m.label)
def test_conv_weights_in_lds_by_plan(sq, oracle, held, run, layer, mode):
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    words = sq.sparq_conv_plan(d, sq.mode(*mode.astuple())).split()
    assert "u8_kernel=conv_rows_kernel" in words and [w[len("u8_weights_in_lds="):] for w in words if w.startswith("u8_weights_in_lds=")] == [str(run)] * (run != 0), words
    assert ("weights_in_lds" in words) == bool(held) and ("kernel=conv_rows_kernel" in words or held is None), words      # (None: not this form)
    check_layer_u8(sq, oracle, layer, mode, seed_cfg=8, out_mode=S.Mode(4, S.OPT5, 1, 1))
    if held:
        check_layer(sq, oracle, layer, mode, seed_cfg=8)


# Eight wavefronts per tile (1x1 layers with long reductions): steps that are padded to a multiple of four, an odd channel
# count, strides, ragged pixels and channels, one tile, more tiles than CUs with two tiles of channels each.
WIDE_SHAPES = [
    ("128x256", S.ConvLayer("w_c520_n112", 1, 19999, 1, 520, 112)), ("128x256", S.ConvLayer("w_c575_n272_s2", 3, 99, 101, 575, 272, 1, 1, (2, 2), (0, 0))),
    ("128x256", S.ConvLayer("w_c512_n512", 1, 12544, 1, 512, 512)), ("128x256", S.ConvLayer("w_c528_n528", 1, 33001, 1, 528, 528)),
    ("128x512", S.ConvLayer("w_c1024_n320", 1, 32769, 1, 1024, 320)), ("128x256", S.ConvLayer("w_c4608_n130", 1, 9000, 1, 4608, 130)),
]


@pytest.mark.parametrize("tile,layer", WIDE_SHAPES, ids=lambda v: v if isinstance(v, str) else v.name)
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.Mode(3, S.OPT6_3B, 0, 1), S.PLAIN8], ids=lambda m: m.label)
def test_conv_eight_wavefronts(sq, oracle, tuning, tile, layer, mode):
    tuning("form=wide")                    # (the rules give some of these to the tile kernels: few tiles, mostly padding)
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    assert f"tile={tile} eight_wavefronts" in sq.sparq_conv_plan(d, sq.mode(*mode.astuple()))
    check_layer(sq, oracle, layer, mode, seed_cfg=8)
    check_layer_u8(sq, oracle, layer, mode, seed_cfg=8, out_mode=S.Mode(4, S.OPT5, 1, 1))


# Small workgroups (multi-tap layers with many tiles): several 64-channel blocks, padded channels, an odd channel count, ragged
# pixels and outputs, images that share a tile, wide rows, patches the tile kernel cannot stage.
BLOCK_SHAPES = [
    S.ConvLayer("b_3x3_56_c64", 25, 56, 56, 64, 64, 3, 3, (1, 1), (1, 1)), S.ConvLayer("b_3x3_p0_c48_n32", 105, 30, 29, 48, 32, 3, 3),
    S.ConvLayer("b_3x3_17_c128_n272", 61, 17, 17, 128, 272, 3, 3, (1, 1), (1, 1)), S.ConvLayer("b_3x3_28_c120_n80", 53, 28, 28, 120, 80, 3, 3, (1, 1), (1, 1)),
    S.ConvLayer("b_5x5_57_c130_n33", 25, 57, 55, 130, 33, 5, 5, (1, 1), (2, 2)), S.ConvLayer("b_2x2_c40_n96", 33, 36, 36, 40, 96, 2, 2, (1, 1), (0, 0)),
    S.ConvLayer("b_3x3_wide_rows_c60_n33", 7, 112, 111, 60, 33, 3, 3, (1, 1), (1, 1)),
]


@pytest.mark.parametrize("layer", BLOCK_SHAPES, ids=lambda l: l.name)
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.Mode(3, S.OPT6_3B, 0, 1), S.PLAIN8], ids=lambda m: m.label)
def test_conv_small_workgroups(sq, oracle, layer, mode):
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    # (113 to 128 channels: requantised results only, which the plan line does not speak of)
    assert ("small_workgroups" in sq.sparq_conv_plan(d, sq.mode(*mode.astuple()))) == (layer.C <= 64 or layer.KH == 5)
    check_layer(sq, oracle, layer, mode, seed_cfg=8)
    check_layer_u8(sq, oracle, layer, mode, seed_cfg=8, out_mode=S.Mode(4, S.OPT5, 1, 1))


# Channel counts that are a multiple of four and not of 16, read where they are: words that start off a 16-byte border, run into
# the next pixel and past the tensor's end, in every form; and the layers that keep the channel-padded copy (`copy`).
@pytest.mark.parametrize("kernel,copy,layer", [
    ("split", False, S.ConvLayer("a_split_3x3_c36", 2, 9, 11, 36, 48, 3, 3, (1, 1), (1, 1))), ("split", False, S.ConvLayer("a_split_1x1_c364", 1, 97, 1, 364, 80)),
    ("rows", False, S.ConvLayer("a_rows_c60", 1, 71, 1, 60, 64)), ("rows", False, S.ConvLayer("a_rows_c188_s2", 3, 15, 13, 188, 96, 1, 1, (2, 2), (0, 0))),
    ("rows", False, S.ConvLayer("a_rows_c492", 1, 6003, 1, 492, 144)), ("wide", False, S.ConvLayer("a_wide_c516", 1, 20011, 1, 516, 256)),
    ("wide", False, S.ConvLayer("a_wide_c1004", 1, 32801, 1, 1004, 320)), ("block", False, S.ConvLayer("a_block_3x3_c52", 25, 56, 56, 52, 64, 3, 3, (1, 1), (1, 1))),
    ("patch", False, S.ConvLayer("a_patch_3x3_c100", 21, 35, 35, 100, 96, 3, 3, (1, 1), (1, 1))), ("patch", False, S.ConvLayer("a_patch_1x7_c132", 33, 17, 17, 132, 272, 1, 7, (1, 1), (0, 3))),
    ("gemm", False, S.ConvLayer("a_gather_1x1_c20", 3, 13, 11, 20, 48)), ("gemm", False, S.ConvLayer("a_gather_1x1_c4", 2, 9, 7, 4, 33)),
    ("gemm", True, S.ConvLayer("a_gather_3x3_c28", 2, 13, 11, 28, 48, 3, 3, (1, 1), (1, 1))), ("wide", True, S.ConvLayer("a_few_tiles_c4108", 1, 2978, 1, 4108, 304)),
], ids=lambda v: v.name if hasattr(v, "name") else str(v))
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.Mode(4, S.OPT3, 0, 0), S.Mode(2, S.OPT7_2B, 1, 1), S.PLAIN8], ids=lambda m: m.label)
def test_conv_channels_in_words(sq, oracle, kernel, copy, layer, mode):
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    m = sq.mode(*mode.astuple())
    text = sq.sparq_conv_plan(d, m)
    assert sq.sparq_workspace_bytes(d, m) > 0                    # (asked for whether or not the copy is made)
    assert ("padded_copy" in text) == (copy and mode.window_bits != 8), text
    if not copy:
        assert f" kernel=conv_{kernel}_kernel" in text, text
    check_layer(sq, oracle, layer, mode, seed_cfg=8)
    check_layer_u8(sq, oracle, layer, mode, seed_cfg=8)
    check_layer_u8(sq, oracle, layer, mode, seed_cfg=8, out_mode=mode if layer.N % 16 == 0 else S.Mode(4, S.OPT5, 1, 1))


# The tile kernels' layers of that kind which keep the copy because their staging would be the longer side.
@pytest.mark.parametrize("layer", [S.ConvLayer("a_copy_1x7_c1396", 3, 15, 15, 1396, 96, 1, 7, (2, 2), (0, 3)), S.ConvLayer("a_copy_3x3_c1016", 2, 31, 5, 1016, 18, 3, 3, (2, 2))],
                         ids=lambda l: l.name)
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.Mode(2, S.OPT7_2B, 1, 1)], ids=lambda m: m.label)
def test_conv_channels_in_words_copied(sq, oracle, layer, mode):
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    text = sq.sparq_conv_plan(d, sq.mode(*mode.astuple()))
    assert "padded_copy" in text and " kernel=conv_patch_kernel" in text, text
    check_layer(sq, oracle, layer, mode, seed_cfg=8)
    check_layer_u8(sq, oracle, layer, mode, seed_cfg=8, out_mode=mode)


# 1x1 layers of several column tiles: bytes of the gather kernel, and the eight-wavefront form, in place and from the copy by their trims.
@pytest.mark.parametrize("layer", [S.ConvLayer("a_columns_c772_n1001", 1, 20003, 1, 772, 1001)], ids=lambda l: l.name)
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.Mode(4, S.OPT3, 0, 1), S.Mode(2, S.OPT7_2B, 1, 1), S.Mode(3, S.OPT6_3B, 1, 0)], ids=lambda m: m.label)
def test_conv_channels_in_words_over_column_tiles(sq, oracle, layer, mode):
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    assert " u8_kernel=conv_gemm_kernel" in sq.sparq_conv_plan(d, sq.mode(*mode.astuple()))
    check_layer(sq, oracle, layer, mode, seed_cfg=8)
    check_layer_u8(sq, oracle, layer, mode, seed_cfg=8, out_mode=mode)


FORM_MODES = [S.Mode(4, S.OPT5, 1, 1), S.Mode(4, S.OPT5, 1, 0), S.Mode(4, S.OPT3, 0, 1), S.Mode(4, S.OPT3, 0, 0),
              S.Mode(3, S.OPT6_3B, 1, 0), S.Mode(2, S.OPT7_2B, 1, 1), S.Mode(2, S.OPT7_2B, 0, 1), S.PLAIN8]


# The 128 x 128 tile of the small workgroups: outputs that fill no 128 (and no wavefront's 64), ragged pixels, several 64-channel
# blocks, images that share a tile, the layers of the gather kernel it takes; `takes`: for four-byte results, for bytes.
SQUARE_SHAPES = [
    ((True, True), S.ConvLayer("q_3x3_c64_n80", 27, 35, 35, 64, 80, 3, 3, (1, 1), (1, 1))), ((True, True), S.ConvLayer("q_3x3_c52_n144", 150, 11, 10, 52, 144, 3, 3, (1, 1), (1, 1))),
    ((True, True), S.ConvLayer("q_1x7_c160_n176", 115, 17, 17, 160, 176, 1, 7, (1, 1), (0, 3))), ((False, True), S.ConvLayer("q_3x3_c128_n272", 61, 17, 17, 128, 272, 3, 3, (1, 1), (1, 1))),
    ((True, True), S.ConvLayer("q_3x3_s2_c96_n112", 115, 35, 35, 96, 112, 3, 3, (2, 2))), ((True, True), S.ConvLayer("q_5x5_c112_n48", 6, 78, 77, 112, 48, 5, 5, (1, 1), (2, 2))),
]


@pytest.mark.parametrize("takes,layer", SQUARE_SHAPES, ids=lambda v: v.name if hasattr(v, "name") else "")
@pytest.mark.parametrize("mode", FORM_MODES, ids=lambda m: m.label)
def test_conv_square_tiles(sq, oracle, takes, layer, mode):
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    text = sq.sparq_conv_plan(d, sq.mode(*mode.astuple()))
    gather = layer.stride != (1, 1) or layer.KH == 5                # (what is not trimmed stays with the gather kernel)
    assert ("small_workgroups tile=128x128" in text) == (takes[0] and not (gather and mode.window_bits == 8)), text
    assert ("u8_kernel=conv_block_kernel" in text) == (takes[1] and not (gather and mode.window_bits == 8)), text
    check_layer(sq, oracle, layer, mode, seed_cfg=8)
    check_layer_u8(sq, oracle, layer, mode, seed_cfg=8, out_mode=mode)


# The small workgroups on either side of where the tile kernel hands a layer over: its tiles one above and one below the rounds that the
# rule names for three and for five 64-channel blocks and for tiles 64 wide, 192 outputs in three columns of 64, ragged outputs and channels.
HANDED_OVER = [
    ("128x128", S.ConvLayer("q_1x7_c160_n96", 114, 17, 17, 160, 96, 1, 7, (1, 1), (0, 3))), (None, S.ConvLayer("q_1x7_c160_n96_less", 113, 17, 17, 160, 96, 1, 7, (1, 1), (0, 3))),
    ("128x128", S.ConvLayer("q_1x7_c272_n80", 228, 17, 17, 272, 80, 1, 7, (1, 1), (0, 3))), (None, S.ConvLayer("q_1x7_c272_n80_less", 226, 17, 17, 272, 80, 1, 7, (1, 1), (0, 3))),
    ("256x64", S.ConvLayer("q_1x7_c160_n48", 341, 17, 17, 160, 48, 1, 7, (1, 1), (0, 3))), (None, S.ConvLayer("q_1x7_c160_n48_less", 340, 17, 17, 160, 48, 1, 7, (1, 1), (0, 3))),
    ("256x64", S.ConvLayer("q_3x3_c52_n192", 115, 17, 17, 52, 192, 3, 3, (1, 1), (1, 1))), ("256x64", S.ConvLayer("q_7x1_c160_n192", 115, 17, 17, 160, 192, 7, 1, (1, 1), (3, 0))),
]


@pytest.mark.parametrize("tile,layer", HANDED_OVER, ids=lambda v: v.name if hasattr(v, "name") else str(v))
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.PLAIN8], ids=lambda m: m.label)
def test_conv_tile_kernel_hands_over(sq, oracle, tile, layer, mode):
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    text = sq.sparq_conv_plan(d, sq.mode(*mode.astuple()))
    assert (f"small_workgroups tile={tile}" in text) if tile else (" kernel=conv_patch_kernel" in text), text
    check_layer(sq, oracle, layer, mode, seed_cfg=8)
    check_layer_u8(sq, oracle, layer, mode, seed_cfg=8, out_mode=mode)


# Each of these forms, forced by the tuning hook, in every trim variant it is built for and every form of its results: int32
# alone, fp32 alone, both, bytes, bytes trimmed with the layer's own mode, and bytes trimmed where the input already is.
FORM_SHAPES = [
    ("split", S.ConvLayer("f_3x3_c80_n32", 2, 9, 11, 80, 32, 3, 3, (1, 1), (1, 1))),
    ("split", S.ConvLayer("f_1x1_c208_n48_s2", 2, 9, 11, 208, 48, 1, 1, (2, 2), (0, 0))),
    ("rows", S.ConvLayer("f_c64_n48", 1, 71, 1, 64, 48)), ("rows", S.ConvLayer("f_c128_n80", 3, 9, 7, 128, 80)),
    ("rows", S.ConvLayer("f_c176_n144_s2", 3, 15, 13, 176, 144, 1, 1, (2, 2), (0, 0))), ("rows", S.ConvLayer("f_c256_n272", 1, 100, 1, 256, 272)),
    ("rows", S.ConvLayer("f_c304_n64", 1, 333, 1, 304, 64)), ("rows", S.ConvLayer("f_c384_n160", 1, 130, 1, 384, 160)),
    ("rows", S.ConvLayer("f_c512_n16", 1, 67, 1, 512, 16)), ("rows", S.ConvLayer("f_c192_n512_wide", 1, 49169, 1, 192, 512)),
    ("wide", S.ConvLayer("f_c336_n48", 1, 200, 1, 336, 48)), ("wide", S.ConvLayer("f_c576_n272_s2", 3, 21, 19, 576, 272, 1, 1, (2, 2), (0, 0))),
    ("wide", S.ConvLayer("f_c528_n320", 1, 16500, 1, 528, 320)),          # the 512-wide tile
    ("block", S.ConvLayer("f_3x3_c80_n80", 2, 13, 11, 80, 80, 3, 3, (1, 1), (1, 1))), ("block", S.ConvLayer("f_5x5_c144_n48", 1, 20, 20, 144, 48, 5, 5, (1, 1), (2, 2))),
]


@pytest.mark.parametrize("form,layer", FORM_SHAPES, ids=lambda v: v if isinstance(v, str) else v.name)
@pytest.mark.parametrize("mode", FORM_MODES, ids=lambda m: m.label)
def test_conv_every_variant_of_a_form(sq, oracle, tuning, form, layer, mode):
    tuning(f"form={form}")
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    words = sq.sparq_conv_plan(d, sq.mode(*mode.astuple())).split()
    assert f"kernel=conv_{form}_kernel" in words and any(w.startswith(f"u8_kernel=conv_{form}_kernel") for w in words), words
    x, w, sc = S.gen_layer(8, layer)
    ref_acc, ref_out = oracle.conv_gemm(x, w, layer.stride, layer.pad, scale=sc, **mode.kwargs())
    for want_acc, want_out in ((True, False), (False, True), (True, True)):
        acc, out = run_conv(sq, x, w, sc, layer, mode, want_acc, want_out)
        assert acc is None or np.array_equal(acc, ref_acc)
        assert out is None or np.all(np.abs(out.astype(np.float64) - ref_out) <= 1e-6 * np.abs(ref_out))
    f = S.gen_requant(layer, S.rng_for(8, 900 + layer.index))
    ref = oracle.requant(ref_acc, f)
    assert np.array_equal(run_conv_u8(sq, x, w, f, layer, mode), ref)
    assert np.array_equal(run_conv_u8(sq, x, w, f, layer, mode, out_mode=mode), oracle.trim(ref, **mode.kwargs()))
    plain = oracle.requant(oracle.conv_gemm(x, w, layer.stride, layer.pad, **S.PLAIN8.kwargs())[0], f)
    assert np.array_equal(run_conv_u8(sq, x, w, f, layer, S.PLAIN8, out_mode=mode), oracle.trim(plain, **mode.kwargs()))


# The weights in registers: every number of steps held, steps past the layer's own, shares of the output channels (with idle wavefronts in
# the last), two wavefronts for the same channels, a stride, fewer pixels than a fragment and than workgroups, several tiles with an odd last one;
# then where the rule takes it, at the fewest pixels up to 512 channels.
COLS_SHAPES = [
    (1, S.ConvLayer("k_c132_n272", 1, 1031, 1, 132, 272)), (1, S.ConvLayer("k_c256_n48", 1, 31, 1, 256, 48)), (1, S.ConvLayer("k_c256_n528_s2", 3, 29, 31, 256, 528, 1, 1, (2, 2), (0, 0))),
    (1, S.ConvLayer("k_c200_n1040", 1, 7777, 1, 200, 1040)), (1, S.ConvLayer("k_c384_n272", 1, 9001, 1, 384, 272)), (1, S.ConvLayer("k_c330_n208", 1, 16421, 1, 330, 208)),
    (1, S.ConvLayer("k_c512_n560_s2", 2, 99, 101, 512, 560, 1, 1, (2, 2), (0, 0))), (1, S.ConvLayer("k_c448_n240", 1, 24611, 1, 448, 240)), (1, S.ConvLayer("k_c512_n33", 1, 65, 1, 512, 33)),
    (1, S.ConvLayer("k_c768_n288", 1, 8225, 1, 768, 288)), (1, S.ConvLayer("k_c580_n96", 1, 24577, 1, 580, 96)),
    (1, S.ConvLayer("k_c1024_n272", 1, 8225, 1, 1024, 272)), (1, S.ConvLayer("k_c780_n16", 1, 24577, 1, 780, 16)), (0, S.ConvLayer("k_c1024_n512", 1, 4099, 1, 1024, 512)),
    (0, S.ConvLayer("k_c256_n512", 1, 10656, 1, 256, 512)), (0, S.ConvLayer("k_c384_n512", 1, 32768, 1, 384, 512)), (0, S.ConvLayer("k_c512_n512", 1, 4096, 1, 512, 512)),
    (0, S.ConvLayer("k_c768_n144", 1, 12321, 1, 768, 144)),
]


@pytest.mark.parametrize("forced,layer", COLS_SHAPES, ids=lambda v: v.name if hasattr(v, "name") else str(v))
@pytest.mark.parametrize("mode", FORM_MODES, ids=lambda m: m.label)
def test_conv_weights_in_registers(sq, oracle, tuning, forced, layer, mode):
    if forced:
        tuning("form=cols")
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    assert "weights_in_registers" in sq.sparq_conv_plan(d, sq.mode(*mode.astuple()))
    x, w, sc = S.gen_layer(8, layer)
    ref_acc, ref_out = oracle.conv_gemm(x, w, layer.stride, layer.pad, scale=sc, **mode.kwargs())
    for want_acc, want_out in ((True, False), (False, True), (True, True)):
        acc, out = run_conv(sq, x, w, sc, layer, mode, want_acc, want_out)
        assert acc is None or np.array_equal(acc, ref_acc)
        assert out is None or np.all(np.abs(out.astype(np.float64) - ref_out) <= 1e-6 * np.abs(ref_out))
    f = S.gen_requant(layer, S.rng_for(8, 900 + layer.index))
    ref = oracle.requant(ref_acc, f)
    assert np.array_equal(run_conv_u8(sq, x, w, f, layer, mode), ref)
    assert np.array_equal(run_conv_u8(sq, x, w, f, layer, mode, out_mode=mode), oracle.trim(ref, **mode.kwargs()))


# Its kernel by name, for both results, and untrimmed input with the output trimmed for the next layer.
@pytest.mark.parametrize("forced,layer", COLS_SHAPES, ids=lambda v: v.name if hasattr(v, "name") else str(v))
def test_conv_weights_in_registers_by_name(sq, oracle, tuning, forced, layer):
    if forced:
        tuning("form=cols")
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    x, w, _ = S.gen_layer(8, layer)
    f = S.gen_requant(layer, S.rng_for(8, 900 + layer.index))
    plain = oracle.requant(oracle.conv_gemm(x, w, layer.stride, layer.pad, **S.PLAIN8.kwargs())[0], f)
    for mode in FORM_MODES:
        words = sq.sparq_conv_plan(d, sq.mode(*mode.astuple())).split()
        assert "kernel=conv_cols_kernel" in words and (layer.N % 16 or "u8_kernel=conv_cols_kernel" in words), words
        assert np.array_equal(run_conv_u8(sq, x, w, f, layer, S.PLAIN8, out_mode=mode), oracle.trim(plain, **mode.kwargs()))


# Shapes chosen for the input-patch kernel: tiles that span several image rows and several images,
# one-row tiles, every staging variant (64/128/256-channel units), several output-channel tiles.
PATCH_SHAPES = [
    S.ConvLayer("p_3x3_56_c64_n64", 2, 56, 56, 64, 64, 3, 3, (1, 1), (1, 1)),
    S.ConvLayer("p_3x3_8x8_c128_n300", 9, 8, 8, 128, 300, 3, 3, (1, 1), (1, 1)),
    S.ConvLayer("p_3x3_7x7_c64_n96", 11, 7, 7, 64, 96, 3, 3, (1, 1), (1, 1)),
    S.ConvLayer("p_3x3_wide_row", 1, 5, 300, 64, 40, 3, 3, (1, 1), (1, 1)),
    S.ConvLayer("p_5x5_c48", 3, 20, 20, 48, 70, 5, 5, (1, 1), (2, 2)),
    S.ConvLayer("p_1x3_c384", 5, 8, 8, 384, 130, 1, 3, (1, 1), (0, 1)),
    S.ConvLayer("p_3x1_c96", 5, 8, 8, 96, 64, 3, 1, (1, 1), (1, 0)),
    S.ConvLayer("p_1x1_c64", 1, 37, 41, 64, 256),
    S.ConvLayer("p_1x1_c128", 2, 30, 30, 128, 192),
    S.ConvLayer("p_1x1_c256", 1, 50, 27, 256, 72),
    S.ConvLayer("p_1x1_c768", 1, 33, 33, 768, 128),
    S.ConvLayer("p_1x1_c80", 1, 19, 23, 80, 50),
    S.ConvLayer("p_3x3_s2_small", 6, 9, 9, 64, 32, 3, 3, (2, 2), (1, 1)),
    S.ConvLayer("p_3x3_p2_dilated_pad", 2, 6, 6, 64, 16, 3, 3, (1, 1), (2, 2)),
    S.ConvLayer("p_2x2_even_taps", 2, 10, 10, 64, 16, 2, 2, (1, 1), (0, 0)),
    S.ConvLayer("p_1x1_s2_c64_n48", 3, 15, 13, 64, 48, 1, 1, (2, 2), (0, 0)),      # strided 1x1: pixel remap
    S.ConvLayer("p_1x1_s2_c128_n200", 5, 14, 14, 128, 200, 1, 1, (2, 2), (0, 0)),
    S.ConvLayer("p_1x1_s3x2_c256_n70", 2, 17, 19, 256, 70, 1, 1, (3, 2), (0, 0)),
]


@pytest.mark.parametrize("layer", PATCH_SHAPES, ids=lambda l: l.name)
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.Mode(3, S.OPT6_3B, 0, 1)], ids=lambda m: m.label)
def test_conv_patch_shapes(sq, oracle, layer, mode, path):
    check_layer(sq, oracle, layer, mode, seed_cfg=9)


@pytest.mark.parametrize("layer", SHAPES + PATCH_SHAPES, ids=lambda l: l.name)
def test_conv_u8_shapes(sq, oracle, layer, path):
    """The requantised-output entry point on every shape and through every kernel form."""
    check_layer_u8(sq, oracle, layer, S.Mode(4, S.OPT5, 1, 1), seed_cfg=9)


@pytest.mark.parametrize("layer", SHAPES + PATCH_SHAPES, ids=lambda l: l.name)
@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.Mode(3, S.OPT6_3B, 0, 1)], ids=lambda m: m.label)
def test_conv_u8_trimmed_for_the_next_layer(sq, oracle, layer, mode, path):
    """Output trimmed with the layer's own mode: inside the epilogue where N is a multiple of 4, by a pass of the
    standalone trim otherwise (odd N: the last channel of a pixel has no partner)."""
    check_layer_u8(sq, oracle, layer, mode, seed_cfg=9, out_mode=mode)


@pytest.mark.parametrize("layer", SHAPES + PATCH_SHAPES, ids=lambda l: l.name)
def test_conv_u8_untrimmed_input_trimmed_output(sq, oracle, layer, path):
    """The steady state of a chain: the input arrives trimmed (this layer runs at plain 8 bits) and the output is
    trimmed for the next one -- in the wave-specialised kernels' epilogue, by a trim pass in the other forms."""
    check_layer_u8(sq, oracle, layer, S.PLAIN8, seed_cfg=9, out_mode=S.Mode(4, S.OPT5, 1, 1))


@pytest.mark.parametrize("mode,out_mode", [(S.PLAIN8, S.Mode(4, S.OPT5, 1, 1)), (S.Mode(4, S.OPT5, 1, 1), S.Mode(4, S.OPT3, 0, 0)),
                                           (S.Mode(4, S.OPT2, 0, 1), S.PLAIN8)], ids=["plain-to-5opt", "5opt-to-3opt", "2opt-to-plain"])
def test_conv_u8_trimmed_with_another_mode(sq, oracle, mode, out_mode):
    """A first layer at plain 8 bits feeding a trimmed one, two different modes, and no output trim."""
    for layer in (S.ConvLayer("u8_tm_a", 2, 12, 12, 64, 96, 3, 3, (1, 1), (1, 1)), S.ConvLayer("u8_tm_b", 1, 9, 30, 3, 64, 7, 7, (2, 2), (3, 3))):
        check_layer_u8(sq, oracle, layer, mode, seed_cfg=9, out_mode=out_mode)


def test_conv_u8_trimmed_chain_runs_the_second_layer_untrimmed(sq, oracle):
    """Layer 1 trims its output for layer 2; layer 2 at plain 8 bits then equals layer 2 trimming on load."""
    l1 = S.ConvLayer("tchain1", 2, 12, 12, 64, 96, 3, 3, (1, 1), (1, 1))
    l2 = S.ConvLayer("tchain2", 2, 12, 12, 96, 40, 1, 1, index=1)
    mode = S.Mode(4, S.OPT5, 1, 1)
    x, w1, _ = S.gen_layer(9, l1)
    _, w2, _ = S.gen_layer(9, l2)
    f1, f2 = S.gen_requant(l1, S.rng_for(9, 950)), S.gen_requant(l2, S.rng_for(9, 951))
    y1t = run_conv_u8(sq, x, w1, f1, l1, mode, out_mode=mode)
    y2 = run_conv_u8(sq, y1t.reshape(l2.x_shape()), w2, f2, l2, S.PLAIN8)
    r1 = oracle.conv_gemm_u8(x, w1, f1, l1.stride, l1.pad, **mode.kwargs())            # untrimmed bytes
    r2 = oracle.conv_gemm_u8(r1.reshape(l2.x_shape()), w2, f2, l2.stride, l2.pad, **mode.kwargs())   # trimmed on load
    assert np.array_equal(y1t, oracle.trim(r1, **mode.kwargs())) and np.array_equal(y2, r2)


@pytest.mark.parametrize("tile", ["128x128", "128x256", "128x512"])
def test_conv_u8_gather_tiles(sq, oracle, tuning, tile):
    """Gather-kernel tiles with the byte output (the widest tile has none: the library picks the next one)."""
    tuning(f"path=gather,tile={tile}")
    check_layer_u8(sq, oracle, S.ConvLayer("u8_tiles", 1, 9, 31, 96, 520, 3, 3, (1, 1), (1, 1)), S.Mode(4, S.OPT3, 1, 1), seed_cfg=9)


def test_conv_u8_chain(sq, oracle):
    """Two layers chained on the device: the first layer's bytes are the second layer's NHWC input."""
    l1 = S.ConvLayer("chain1", 2, 12, 12, 64, 96, 3, 3, (1, 1), (1, 1))
    l2 = S.ConvLayer("chain2", 2, 12, 12, 96, 40, 1, 1, index=1)
    mode = S.Mode(4, S.OPT5, 1, 1)
    x, w1, _ = S.gen_layer(9, l1)
    _, w2, _ = S.gen_layer(9, l2)
    f1, f2 = S.gen_requant(l1, S.rng_for(9, 950)), S.gen_requant(l2, S.rng_for(9, 951))
    y1 = run_conv_u8(sq, x, w1, f1, l1, mode)
    y2 = run_conv_u8(sq, y1.reshape(l2.x_shape()), w2, f2, l2, mode)
    r1 = oracle.conv_gemm_u8(x, w1, f1, l1.stride, l1.pad, **mode.kwargs())
    r2 = oracle.conv_gemm_u8(r1.reshape(l2.x_shape()), w2, f2, l2.stride, l2.pad, **mode.kwargs())
    assert np.array_equal(y1, r1) and np.array_equal(y2, r2)


@pytest.mark.parametrize("tn", ["64", "128", "256"])
def test_conv_patch_channel_tiles(sq, oracle, tuning, tn):
    """Every output-channel tile width of the input-patch kernel on the same layer."""
    tuning(f"path=patch,patch_tn={tn}")
    check_layer(sq, oracle, S.ConvLayer("p_tn", 3, 14, 14, 128, 520, 3, 3, (1, 1), (1, 1)), S.Mode(4, S.OPT5, 1, 1), seed_cfg=9)


WIDE_TILE_LAYERS = [
    # reduction steps (64 indices each) per tile: 1, 2, 3, 4, 5 -- every remainder of the four-step unrolled loop
    S.ConvLayer("wide_1x1_c64", 1, 9, 31, 64, 300),
    S.ConvLayer("wide_1x1_c128", 1, 9, 31, 128, 300),
    S.ConvLayer("wide_1x1_c192", 2, 8, 9, 192, 512),
    S.ConvLayer("wide_1x1_c256", 1, 5, 27, 256, 260),
    S.ConvLayer("wide_1x1_c320", 1, 5, 27, 320, 900),          # two output-channel tiles, the second ragged
    # several taps with zero padding at the borders; 96 channels leave a tap's last chunks in its channel padding
    S.ConvLayer("wide_3x3_c64", 2, 12, 12, 64, 384, 3, 3, (1, 1), (1, 1)),
    S.ConvLayer("wide_3x3s2_c96", 1, 13, 17, 96, 300, 3, 3, (2, 2), (1, 1)),
    S.ConvLayer("wide_5x1_c80", 1, 11, 9, 80, 257, 5, 1, (1, 1), (2, 0)),
    S.ConvLayer("wide_1x1s2_c512", 1, 15, 15, 512, 300, 1, 1, (2, 2), (0, 0)),
]


@pytest.mark.parametrize("mode", [S.Mode(4, S.OPT5, 1, 1), S.Mode(4, S.OPT3, 0, 1), S.Mode(3, S.OPT6_3B, 1, 1), S.Mode(2, S.OPT7_2B, 0, 0), S.PLAIN8],
                         ids=lambda m: m.label + f"-{m.shift_mask:#x}")
@pytest.mark.parametrize("layer", WIDE_TILE_LAYERS, ids=lambda l: l.name)
def test_conv_widest_gather_tile(sq, oracle, tuning, layer, mode):
    """The 128 x 512 tile of the gather kernel (main loop pipelined by half steps, taps tracked in scalar
    registers) on every loop remainder, on multi-tap layers with padding, and on channel-padded taps."""
    tuning("path=gather,tile=128x512")
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    assert "tile=128x512" in sq.sparq_conv_plan(d, sq.mode(*mode.astuple()))
    check_layer(sq, oracle, layer, mode, seed_cfg=9)


def test_widest_gather_tile_needs_step_aligned_taps(sq, tuning):
    """With at most 32 channels a tap is shorter than a reduction step: the library takes the next tile."""
    tuning("path=gather,tile=128x512")
    d = sq.conv_desc(1, 9, 9, 32, 300, 3, 3, (1, 1), (1, 1))
    assert "tile=128x256" in sq.sparq_conv_plan(d, sq.mode(4, S.OPT5, 1, 1))


@pytest.mark.parametrize("mode", MODES_N4 + MODES_LOW + MODES_ODD, ids=lambda m: m.label + f"-{m.shift_mask:#x}")
def test_conv_all_modes(sq, oracle, mode, path):
    check_layer(sq, oracle, S.ConvLayer("3x3_modes", 1, 14, 14, 64, 48, 3, 3, (1, 1), (1, 1), index=3), mode)


def test_extreme_values(sq, oracle):
    """Saturation and accumulator extremes: all-255 / all-zero activations, all -127 / +127 weights, K = 4608."""
    layer = S.ConvLayer("extreme", 1, 70, 1, 4608, 8)
    sc = np.full(8, 0.005, dtype=np.float32)
    for xv in (255, 0, 128):
        for wv in (-127, 127):
            x = np.full(layer.x_shape(), xv, dtype=np.uint8)
            w = np.full(layer.w_shape(), wv, dtype=np.int8)
            for mode in (S.Mode(4, S.OPT5, 1, 1), S.PLAIN8):
                acc, _ = run_conv(sq, x, w, sc, layer, mode)
                ref, _ = oracle.conv_gemm(x, w, **mode.kwargs())
                assert np.array_equal(acc, ref)


def test_only_out_or_only_acc(sq, oracle):
    layer = S.ConvLayer("3x3_outs", 1, 9, 9, 32, 16, 3, 3, (1, 1), (1, 1))
    mode = S.Mode(4, S.OPT5, 1, 1)
    x, w, sc = S.gen_layer(8, layer)
    ref_acc, ref_out = oracle.conv_gemm(x, w, layer.stride, layer.pad, scale=sc, **mode.kwargs())
    acc, _ = run_conv(sq, x, w, sc, layer, mode, want_acc=True, want_out=False)
    assert np.array_equal(acc, ref_acc)
    _, out = run_conv(sq, x, w, sc, layer, mode, want_acc=False, want_out=True)
    assert np.all(np.abs(out.astype(np.float64) - ref_out) <= 1e-6 * np.abs(ref_out))


def test_fused_equals_trim_then_plain(sq):
    """GPU-internal cross-check: trimming with the standalone kernel and contracting at plain
    8 bits gives the same accumulators as the fused kernel."""
    layer = S.ConvLayer("3x3_x", 2, 12, 12, 64, 40, 3, 3, (1, 1), (1, 1))
    mode = S.Mode(4, S.OPT3, 1, 1)
    x, w, sc = S.gen_layer(8, layer)
    fused, _ = run_conv(sq, x, w, sc, layer, mode, want_out=False)
    xd = dev(x)
    y = torch.empty_like(xd)
    sq.sparq_trim(xd, y, sq.mode(*mode.astuple()))
    torch.cuda.synchronize()
    plain, _ = run_conv(sq, y.cpu().numpy(), w, sc, layer, S.PLAIN8, want_out=False)
    assert np.array_equal(fused, plain)
