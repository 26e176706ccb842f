"""GPU parity of the packed activation storage (Sections 3.1, 5.1, 6; Eq. 4): records bit-exact against the oracle's,
unpacked values against the oracle's, the round trip against the trim, and the convolution that reads packed input."""
import numpy as np
import pytest
import torch

import sparq_synth as S

pytestmark = pytest.mark.gpu

MODES = [(4, m, r, p) for m in (S.OPT5, S.OPT3, S.OPT2) for r in (0, 1) for p in (0, 1)] + \
        [(3, S.OPT6_3B, r, p) for r in (0, 1) for p in (0, 1)] + [(2, S.OPT7_2B, r, p) for r in (0, 1) for p in (0, 1)] + \
        [(4, 0x17, 1, 1), (3, 0x2B, 0, 0)]          # option sets of four placements: 2-bit ShiftCtrl with n = 4 and n = 3


@pytest.fixture(scope="module")
def sq():
    assert torch.cuda.is_available(), "GPU tests need a device"
    import paper_2105_11010_amd as sq_
    return sq_


def kw(mode):
    n, m, r, p = mode
    return dict(window_bits=n, shift_mask=m, round_nearest=r, pair=p)


def gpu_pack(sq, x, mode, group=1):
    m = sq.mode(*mode)
    xd = torch.from_numpy(x).cuda()
    nbytes = sq.sparq_packed_act_bytes(x.size // x.shape[-1], x.shape[-1], m, group)
    packed = torch.full((nbytes,), 0xAB, dtype=torch.uint8, device="cuda")
    sq.sparq_pack_act(xd, packed, m, group)
    y = torch.full(x.shape, 0xCD, dtype=torch.uint8, device="cuda")
    sq.sparq_unpack_act(packed, y, m, group)
    torch.cuda.synchronize()
    return packed.cpu().numpy(), y.cpu().numpy()


@pytest.mark.parametrize("mode", MODES, ids=str)
def test_every_pair_of_values(sq, oracle, mode):
    a, b = np.meshgrid(np.arange(256), np.arange(256), indexing="ij")
    x = np.stack([a.ravel(), b.ravel()], axis=1).astype(np.uint8).reshape(-1, 64)
    packed, y = gpu_pack(sq, x, mode)
    ref = oracle.pack_act(x, **kw(mode))
    assert np.array_equal(packed.reshape(ref.shape), ref), "records differ from the oracle's"
    assert np.array_equal(y, oracle.trim(x, **kw(mode))), "round trip is not the trim"


@pytest.mark.parametrize("C", [1, 2, 3, 31, 32, 33, 65, 96, 159, 256])
@pytest.mark.parametrize("mode", [(4, S.OPT5, 1, 1), (4, S.OPT3, 0, 1), (4, S.OPT2, 1, 0), (2, S.OPT7_2B, 1, 1)], ids=str)
def test_ragged_channel_counts_and_rows(sq, oracle, C, mode):
    x = S.gen_activations((3, 37, C), 0.5, S.rng_for(7, C))
    packed, y = gpu_pack(sq, x, mode)
    ref = oracle.pack_act(x, **kw(mode))
    assert np.array_equal(packed.reshape(ref.shape), ref)
    assert np.array_equal(y, oracle.unpack_act(ref, x.shape, **kw(mode)))
    assert np.array_equal(y, oracle.trim(x, **kw(mode)))


@pytest.mark.parametrize("group", [2, 4, 8, 16, 32])
@pytest.mark.parametrize("mode", [(4, S.OPT5, 0, 0), (4, S.OPT5, 1, 0), (4, S.OPT3, 1, 0), (4, S.OPT2, 0, 0), (3, S.OPT6_3B, 1, 0),
                                  (2, S.OPT7_2B, 0, 0)], ids=str)
def test_shared_shift_groups(sq, oracle, group, mode):
    x = S.gen_activations((1000, 96), 0.5, S.rng_for(7, 100 + group))
    x[0] = 0
    x[1] = 255
    x[2, ::group] = 255
    packed, y = gpu_pack(sq, x, mode, group)
    ref = oracle.pack_act(x, group, **kw(mode))
    assert np.array_equal(packed.reshape(ref.shape), ref)
    assert np.array_equal(y, oracle.unpack_act(ref, x.shape, group, **kw(mode)))


def test_sizes_and_rejections(sq, oracle):
    for mode in MODES:
        for group in (1, 2, 8, 32):
            want = oracle.packed_record_bytes(group, **kw(mode))
            assert sq.sparq_packed_act_bytes(5, 70, sq.mode(*mode), group) == 5 * 3 * want
    m = sq.mode(4, S.OPT5, 1, 1)
    x = torch.zeros((4, 64), dtype=torch.uint8, device="cuda")
    small = torch.zeros(10, dtype=torch.uint8, device="cuda")
    with pytest.raises(sq.SparqError) as e:
        sq.sparq_pack_act(x, small, m)
    assert e.value.status == 3
    with pytest.raises(sq.SparqError):
        sq.sparq_pack_act(x, torch.zeros(4096, dtype=torch.uint8, device="cuda"), sq.mode(8, 1, 0, 0))
    with pytest.raises(sq.SparqError):
        sq.sparq_pack_act(x, torch.zeros(4096, dtype=torch.uint8, device="cuda"), m, 4)       # shared shift needs vSPARQ off
    sq.sparq_pack_act(x[:0], small, m)                                                       # no rows: nothing to do


@pytest.mark.parametrize("layer,group", [
    (S.ConvLayer("p_1x1_256_64", 4, 28, 28, 256, 64, 1, 1, (1, 1), (0, 0), 0.5, S.Mode(4, S.OPT3, 0, 1)), 1),
    (S.ConvLayer("p_3x3_64_96", 2, 17, 17, 64, 96, 3, 3, (1, 1), (1, 1), 0.4, S.Mode(4, S.OPT5, 1, 1)), 1),
    (S.ConvLayer("p_3x3s2_65_48", 2, 19, 19, 65, 48, 3, 3, (2, 2), (1, 1), 0.5, S.Mode(4, S.OPT2, 1, 1)), 1),
    (S.ConvLayer("p_1x1_512_128_g8", 2, 14, 14, 512, 128, 1, 1, (1, 1), (0, 0), 0.5, S.Mode(4, S.OPT5, 1, 0)), 8),
    (S.ConvLayer("p_1x7_160_g4", 2, 17, 17, 160, 160, 1, 7, (1, 1), (0, 3), 0.5, S.Mode(3, S.OPT6_3B, 0, 0)), 4)], ids=lambda v: getattr(v, "name", v))
def test_convolution_on_packed_input(sq, oracle, layer, group):
    """Packed input -> the same int32 accumulators as the oracle's convolution over the values the oracle unpacks."""
    x, w, sc = S.gen_layer(8, layer)
    d = sq.conv_desc(layer.B, layer.H, layer.W, layer.C, layer.N, layer.KH, layer.KW, layer.stride, layer.pad)
    m = sq.mode(*layer.mode.astuple())
    dev = torch.device("cuda:0")
    xd, wd, sd = (torch.from_numpy(a).to(dev) for a in (x, w, sc))
    px = torch.empty(sq.sparq_packed_act_bytes(layer.B * layer.H * layer.W, layer.C, m, group), dtype=torch.uint8, device=dev)
    sq.sparq_pack_act(xd, px, m, group)
    pw = torch.empty(sq.sparq_packed_bytes(d), dtype=torch.uint8, device=dev)
    sq.sparq_pack_weights(wd, d, pw)
    ws = torch.empty(sq.sparq_conv_packed_workspace_bytes(d, m), dtype=torch.uint8, device=dev)
    acc = torch.empty((layer.M, layer.N), dtype=torch.int32, device=dev)
    out = torch.empty((layer.M, layer.N), dtype=torch.float32, device=dev)
    sq.sparq_conv_gemm_packed(px, group, pw, d, m, acc=acc, scale=sd, out=out, workspace=ws)
    torch.cuda.synchronize()
    values = oracle.unpack_act(oracle.pack_act(x, group, **layer.mode.kwargs()), x.shape, group, **layer.mode.kwargs())
    if group == 1:
        assert np.array_equal(values, oracle.trim(x, **layer.mode.kwargs()))
    ref_acc, ref_out = oracle.conv_gemm(values, w, layer.stride, layer.pad, scale=sc, **S.PLAIN8.kwargs())
    assert np.array_equal(acc.cpu().numpy(), ref_acc)
    assert np.all(np.abs(out.cpu().numpy().astype(np.float64) - ref_out) <= 1e-6 * np.abs(ref_out))
    if group == 1:      # and the per-value format gives what the fused convolution gives on the raw input
        acc2 = torch.empty_like(acc)
        wsb = sq.sparq_workspace_bytes(d, m)
        sq.sparq_conv_gemm(xd, pw, d, m, acc=acc2, workspace=torch.empty(wsb, dtype=torch.uint8, device=dev) if wsb else None)
        assert torch.equal(acc, acc2)


# Channel counts that are no multiple of four unpack into the channel-padded tensor: one and several records a row, a last record
# of one channel and of all but one, counts below a 16-channel word, every form of the contraction, and a folded first layer.
@pytest.mark.parametrize("layer,group", [
    (S.ConvLayer("p_1x1_315_224", 3, 19, 19, 315, 224, 1, 1, (1, 1), (0, 0), 0.5, S.Mode(4, S.OPT3, 0, 1)), 1),
    (S.ConvLayer("p_1x1s2_549_33", 1, 97, 33, 549, 33, 1, 1, (2, 2), (0, 0), 0.5, S.Mode(4, S.OPT5, 1, 0)), 8),
    (S.ConvLayer("p_3x3_33_40", 2, 11, 9, 33, 40, 3, 3, (1, 1), (1, 1), 0.5, S.Mode(2, S.OPT7_2B, 1, 1)), 1),
    (S.ConvLayer("p_3x3_63_96", 25, 35, 35, 63, 96, 3, 3, (1, 1), (1, 1), 0.5, S.Mode(4, S.OPT5, 1, 1)), 1),
    (S.ConvLayer("p_5x5_17_20", 2, 13, 12, 17, 20, 5, 5, (1, 1), (2, 2), 0.5, S.Mode(3, S.OPT6_3B, 0, 0)), 32),
    (S.ConvLayer("p_3x3_6_12", 2, 9, 7, 6, 12, 3, 3, (1, 1), (1, 1), 0.5, S.Mode(4, S.OPT3, 0, 1)), 1),
    (S.ConvLayer("p_1x1_3_8", 2, 9, 7, 3, 8, 1, 1, (1, 1), (0, 0), 0.5, S.Mode(4, S.OPT5, 1, 1)), 1),
    (S.ConvLayer("p_7x7s2_3_64", 1, 28, 28, 3, 64, 7, 7, (2, 2), (3, 3), 0.5, S.Mode(4, S.OPT5, 1, 1)), 1)], ids=lambda v: getattr(v, "name", v))
def test_convolution_on_packed_input_of_any_width(sq, oracle, layer, group):
    test_convolution_on_packed_input(sq, oracle, layer, group)


@pytest.mark.parametrize("mode,group", [((4, S.OPT5, 1, 1), 1), ((4, S.OPT3, 0, 1), 1), ((4, S.OPT5, 1, 0), 8)], ids=str)
def test_calls_larger_than_the_last_level_cache(sq, mode, group):
    """More than 256 MiB moved: unpacking goes through LDS; the last wavefront holds fewer than 64 records."""
    m = sq.mode(*mode)
    rows, C = 42037, 4064                                                    # 127 records a row
    x = torch.randint(0, 256, (rows, C), dtype=torch.uint8, device="cuda")
    x.mul_((torch.rand(rows, C, device="cuda") < 0.5).to(torch.uint8))
    packed = torch.empty(sq.sparq_packed_act_bytes(rows, C, m, group), dtype=torch.uint8, device="cuda")
    assert x.numel() + packed.numel() >= 256 << 20 and rows * (C // 32) % 64
    sq.sparq_pack_act(x, packed, m, group)
    y = torch.full_like(x, 0xCD)
    sq.sparq_unpack_act(packed, y, m, group)
    part = torch.empty_like(x)
    step = 5000                                                              # small calls take the other form
    for r in range(0, rows, step):
        n = min(step, rows - r)
        rec = packed.numel() // rows
        sq.sparq_unpack_act(packed[r * rec:(r + n) * rec], part[r:r + n], m, group)
    assert torch.equal(y, part)
    if group == 1:
        sq.sparq_trim(x, part, m)
        assert torch.equal(y, part)


@pytest.mark.parametrize("offset,C", [(1, 33), (3, 64), (4, 40), (2, 31)])
def test_activations_that_start_anywhere(sq, oracle, offset, C):
    """Activations at an odd address, ragged rows, and a last record that ends with the tensor."""
    mode = (4, S.OPT5, 1, 1)
    x = S.gen_activations((67, C), 0.5, S.rng_for(7, 300 + offset))
    m = sq.mode(*mode)
    buf = torch.zeros(x.size + 16, dtype=torch.uint8, device="cuda")
    xd = buf[offset:offset + x.size].view(x.shape)
    xd.copy_(torch.from_numpy(x))
    packed = torch.empty(sq.sparq_packed_act_bytes(67, C, m), dtype=torch.uint8, device="cuda")
    sq.sparq_pack_act(xd, packed, m)
    out = torch.full((x.size + 16,), 0xCD, dtype=torch.uint8, device="cuda")
    sq.sparq_unpack_act(packed, out[offset:offset + x.size].view(x.shape), m)
    ref = oracle.pack_act(x, **kw(mode))
    assert np.array_equal(packed.cpu().numpy().reshape(ref.shape), ref)
    o = out.cpu().numpy()
    assert np.array_equal(o[offset:offset + x.size].reshape(x.shape), oracle.trim(x, **kw(mode)))
    assert (o[:offset] == 0xCD).all() and (o[offset + x.size:] == 0xCD).all()
