"""Host-side planning of the convolution (no GPU): every layer of the workload tables gets a plan,
and the plan agrees with the workspace the library asks for."""
import ctypes
import os

import pytest

import sparq_synth as S

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2105_11010_amd", "libsparq.so")


class Mode(ctypes.Structure):
    _fields_ = [("window_bits", ctypes.c_int32), ("shift_mask", ctypes.c_uint32),
                ("round_nearest", ctypes.c_int32), ("pair", ctypes.c_int32)]


class Desc(ctypes.Structure):
    _fields_ = [(k, ctypes.c_int32) for k in
                ("B", "H", "W", "C", "N", "KH", "KW", "stride_h", "stride_w", "pad_h", "pad_w")]


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        pytest.skip("libsparq.so not built")
    L = ctypes.CDLL(LIB)
    L.sparq_workspace_bytes.restype = ctypes.c_size_t
    L.sparq_packed_bytes.restype = ctypes.c_size_t
    return L


def plan(lib, l, mode=None):
    d = Desc(l.B, l.H, l.W, l.C, l.N, l.KH, l.KW, l.stride[0], l.stride[1], l.pad[0], l.pad[1])
    m = Mode(*(mode or l.mode).astuple())
    buf = ctypes.create_string_buffer(256)
    assert lib.sparq_conv_plan(ctypes.byref(d), ctypes.byref(m), buf, len(buf)) == 0
    return buf.value.decode(), lib.sparq_workspace_bytes(ctypes.byref(d), ctypes.byref(m)), lib.sparq_packed_bytes(ctypes.byref(d))


ALL = [(c, l) for c, ls in ((0, S.config0()), (1, S.config1()), (2, S.config2()), (4, S.config4())) for l in ls]


@pytest.mark.parametrize("cfg,layer", ALL, ids=lambda v: v.name if hasattr(v, "name") else f"cfg{v}")
def test_every_workload_layer_has_a_consistent_plan(lib, cfg, layer):
    text, ws, packed = plan(lib, layer)
    assert text.startswith(("conv_patch_kernel", "conv_gemm_kernel"))
    pixels = layer.B * layer.H * layer.W
    if layer.C <= 4:
        assert "pixel_folded" in text and ws >= pixels * 4           # 4-channel padded copy
    elif layer.C % 16:
        assert "padded_copy" in text and ws >= pixels * ((layer.C + 15) // 16 * 16)
    else:
        assert "padded_copy" not in text
    if layer.C % 16 == 0:
        assert ws == 0                                                # nothing to stage
    assert packed >= layer.K * layer.N


def test_plan_of_the_headline_shapes(lib):
    conv = S.ConvLayer("conv3x3", 64, 32, 32, 512, 512, 3, 3, (1, 1), (1, 1), 0.5, S.Mode(4, S.OPT5, 1, 1))
    text, ws, _ = plan(lib, conv)
    assert text.startswith("conv_patch_kernel tile=128x256") and "wave_specialised" in text and ws == 0
    text, ws, _ = plan(lib, S.config3_layer())
    assert text.startswith("conv_gemm_kernel tile=128x512") and ws == 0


def words(text, key):
    return [w[len(key):] for w in text.split() if w.startswith(key)]


@pytest.mark.parametrize("shape,kernel,u8_kernel", [
    ((64, 32, 32, 512, 512, 3, 1), "conv_patch_kernel", "conv_patch_kernel"),
    ((1, 65536, 1, 4608, 512, 1, 0), "conv_wide_kernel", "conv_wide_kernel:128x512"),
    ((256, 56, 56, 64, 256, 1, 0), "conv_patch_kernel", "conv_rows_kernel"),            # large four-byte rows / byte rows
    ((256, 14, 14, 256, 1024, 1, 0), "conv_cols_kernel", "conv_cols_kernel"),             # weights in registers
    ((256, 56, 56, 64, 64, 3, 1), "conv_block_kernel", "conv_block_kernel"),
    ((256, 28, 28, 128, 128, 3, 1), "conv_patch_kernel", "conv_block_kernel"),          # 113 to 128 channels: bytes only
    ((128, 35, 35, 96, 96, 3, 1), "conv_patch_kernel", "conv_patch_kernel"),
    ((1, 56, 56, 64, 64, 3, 1), "conv_split_kernel", "conv_split_kernel:32x32"),
    ((1, 7, 7, 512, 514, 3, 1), "conv_split_kernel", "conv_split_kernel:32x32"),        # this form takes any N for bytes
    ((64, 28, 28, 64, 250, 1, 0), "conv_patch_kernel", "conv_patch_kernel"),            # rows off a 64-byte border, bytes not 16
    ((2, 9, 9, 32, 300, 3, 1), "conv_gemm_kernel", "conv_gemm_kernel:128x256"),
    ((64, 32, 32, 512, 514, 1, 0), "conv_patch_kernel", "conv_patch_kernel"),
    ((1, 65536, 1, 4608, 508, 1, 0), "conv_wide_kernel", "conv_gemm_kernel:128x256"),   # bytes: N off 16
    ((1, 4000, 1, 64, 6000, 1, 0), "conv_rows_kernel", "conv_patch_kernel"),            # bytes: more channels than its LDS constants hold
], ids=str)
def test_plan_names_the_kernel_of_either_result(lib, shape, kernel, u8_kernel):
    """kernel=: what sparq_conv_gemm launches; u8_kernel=: what sparq_conv_gemm_u8 does (with the gather kernel's, the split and
    the eight-wavefront form's tile)."""
    B, H, W, C, N, k, pad = shape
    text = plan(lib, S.ConvLayer("p", B, H, W, C, N, k, k, (1, 1), (pad, pad)), S.Mode(4, S.OPT5, 1, 1))[0]
    assert words(text, "kernel=") == [kernel] and words(text, "u8_kernel=") == [u8_kernel], text


M45, PLAIN = S.Mode(4, S.OPT5, 1, 1), S.PLAIN8
FLOOR = S.Mode(4, S.OPT3, 0, 0)


@pytest.mark.parametrize("form,shape,mode,takes", [
    # eight wavefronts: tiles for less than half the CUs, untrimmed layers of few outputs or half-empty rounds, mostly padding
    ("wide", (1, 867, 1, 4336, 960, 1, 0), PLAIN, (False, False)), ("wide", (1, 12544, 1, 4432, 128, 1, 0), PLAIN, (False, False)),
    ("wide", (1, 2000, 1, 832, 816, 1, 0), M45, (False, False)), ("wide", (1, 1500, 1, 1040, 816, 1, 0), M45, (True, False)),
    ("wide", (1, 2500, 1, 1040, 816, 1, 0), M45, (True, True)), ("wide", (1, 9408, 1, 2688, 288, 1, 0), PLAIN, (False, False)),
    ("wide", (1, 9408, 1, 2688, 288, 1, 0), M45, (True, True)), ("wide", (1, 9218, 1, 576, 272, 1, 0), M45, (False, False)),
    ("wide", (1, 65536, 1, 4608, 512, 1, 0), PLAIN, (True, True)), ("wide", (2, 33, 33, 4336, 960, 1, 0), M45, (True, True)),
    ("wide", (2, 33, 33, 4337, 960, 1, 0), M45, (False, False)),                     # an odd channel count: the padded copy is trimmed already
    # small workgroups: rows off a 64-byte border, few taps, narrow images, more than 64 outputs at 113 to 128 channels
    ("block", (56, 56, 56, 48, 86, 3, 1), M45, (False, False)), ("block", (56, 56, 56, 48, 96, 3, 1), M45, (True, True)),
    ("block", (72, 40, 40, 48, 80, (1, 3), (0, 1)), M45, (False, True)), ("block", (72, 40, 40, 48, 48, (1, 3), (0, 1)), M45, (False, True)),
    ("block", (72, 40, 40, 48, 48, (1, 7), (0, 3)), M45, (True, True)), ("block", (409, 8, 8, 64, 160, 3, 1), M45, (False, False)),
    ("block", (409, 8, 8, 64, 160, 3, 1), PLAIN, (True, True)), ("block", (400, 12, 12, 48, 192, 3, 1), M45, (True, False)),
    ("block", (128, 35, 35, 128, 256, 3, 1), M45, (False, False)), ("block", (128, 35, 35, 128, 256, 3, 1), PLAIN, (False, True)),
    ("block", (256, 14, 14, 128, 96, 3, 1), M45, (False, False)), ("block", (256, 28, 28, 128, 128, 3, 1), M45, (False, True)),
    # small workgroups on layers whose patch the tile kernel cannot stage: one 128-wide column tile of the gather kernel, filters one column wide
    ("block", (51, 56, 56, 64, 112, (3, 1), (1, 0)), PLAIN, (False, True)), ("block", (51, 56, 56, 64, 144, (3, 1), (1, 0)), PLAIN, (True, True)),
    ("block", (51, 56, 56, 64, 64, (3, 1), (1, 0)), PLAIN, (True, True)), ("block", (51, 56, 56, 64, 112, (3, 1), (1, 0)), M45, (True, True)),
    ("block", (33, 56, 56, 64, 112, (3, 1), (1, 0)), M45, (False, True)), ("block", (202, 40, 40, 64, 112, (7, 1), (3, 0)), PLAIN, (False, False)),
    ("block", (202, 40, 40, 64, 112, (7, 1), (3, 0)), M45, (True, True)), ("block", (51, 56, 56, 64, 112, 4, 2), PLAIN, (True, True)),
    ("block", (206, 32, 32, 64, 72, 2, 1), PLAIN, (False, False)), ("block", (206, 32, 32, 64, 80, 2, 1), PLAIN, (True, True)),
    ("block", (51, 56, 56, 64, 100, (3, 1), (1, 0)), PLAIN, (True, False)), ("block", (33, 56, 56, 64, 100, (3, 1), (1, 0)), M45, (True, False)),
    # activations in registers: four-byte results of half the last-level cache and more beside little arithmetic
    # (from 129 channels on wide ones hold the weights there instead)
    ("rows", (1, 144611, 1, 128, 448, 1, 0), M45, (False, True)), ("cols", (1, 144611, 1, 256, 448, 1, 0), M45, (True, True)),
    ("cols", (1, 144611, 1, 256, 448, 1, 0), PLAIN, (False, True)), ("rows", (1, 70000, 1, 128, 448, 1, 0), M45, (True, True)),
    ("rows", (1, 802816, 1, 256, 64, 1, 0), M45, (True, True)), ("rows", (1, 802816, 1, 256, 128, 1, 0), M45, (False, True)),
], ids=str)
def test_rules_leave_layers_to_the_tile_kernels(lib, form, shape, mode, takes):
    """Both sides of the lines at which a form stops being ahead of the tile kernels; takes: (four-byte results, bytes)."""
    B, H, W, C, N, k, pad = shape
    kh, kw = k if isinstance(k, tuple) else (k, k)
    text = plan(lib, S.ConvLayer("p", B, H, W, C, N, kh, kw, (1, 1), pad if isinstance(pad, tuple) else (pad, pad)), mode)[0]
    tiles = ("conv_patch_kernel", "conv_gemm_kernel")
    for got, want in ((words(text, "kernel=")[0], takes[0]), (words(text, "u8_kernel=")[0].split(":")[0], takes[1])):
        assert got == f"conv_{form}_kernel" if want else got in tiles, text


@pytest.mark.parametrize("m,c,n,takes", [
    (46644, 284, 1625, False), (46644, 320, 1632, True), (13900, 256, 450, True), (14100, 256, 450, False), (163072, 432, 493, False),
    (726180, 352, 190, False), (4100, 512, 500, False), (4200, 512, 512, True), (101300, 768, 362, True), (101400, 768, 362, False),
    (267600, 768, 376, True), (267800, 768, 376, False), (33600, 1024, 1001, True)])
def test_weights_in_registers_leave_rows_off_a_line(lib, m, c, n, takes):
    """Four-byte rows off a 64-byte border leave that kernel as pieces of lines: up to the results that the caches put together."""
    text = plan(lib, S.ConvLayer("rows", 1, m, 1, c, n), S.Mode(4, S.OPT5, 1, 1))[0]
    assert (words(text, "kernel=") == ["conv_cols_kernel"]) == takes, text


@pytest.mark.parametrize("m,c,n,takes", [
    # (four-byte results, bytes), for 256 CUs.  Up to 256 outputs: 32 pixels for each of two wavefronts per SIMD are 65536
    (49152, 512, 128, (False, True)), (49153, 512, 128, (False, False)), (65536, 512, 128, (False, False)), (65537, 512, 128, (False, True)),
    (60000, 512, 256, (False, True)), (60000, 384, 192, (False, False)), (48000, 384, 192, (True, True)),
    # four-byte results of 384 channels, the outputs of one, two and three shares
    (49152, 384, 512, (True, True)), (49153, 384, 512, (False, True)), (24577, 384, 1024, (False, True)), (32769, 384, 1024, (True, True)),
    (16384, 384, 1536, (False, True)), (16385, 384, 1536, (True, True)),
    # bytes, 64 pixels per wavefront: three quarters of 131072 pixels and seven eighths, all wavefronts at work and not; half a round
    (98304, 256, 1280, (True, True)), (98305, 256, 1280, (True, False)), (114688, 256, 1024, (True, True)), (114689, 256, 1024, (True, False)),
    (131072, 256, 1024, (True, False)), (131073, 256, 1024, (True, True)), (100000, 256, 896, (True, True)), (100000, 384, 896, (True, False)),
    (100000, 320, 1024, (True, False)), (100000, 512, 1024, (True, True)), (60000, 320, 1024, (True, False)), (66000, 320, 1024, (True, True)),
    (60000, 256, 1280, (True, False)), (60000, 512, 1280, (True, True))])
def test_weights_in_registers_leave_full_rounds_of_the_other_form(lib, m, c, n, takes):
    """Where the form with the activations in registers fills its last round, it keeps the layers it is ahead on."""
    text = plan(lib, S.ConvLayer("rounds", 1, m, 1, c, n), S.Mode(4, S.OPT5, 1, 1))[0]
    assert (words(text, "kernel=") == ["conv_cols_kernel"], words(text, "u8_kernel=") == ["conv_cols_kernel"]) == takes, text


@pytest.mark.parametrize("m,c,n,mode,takes", [
    # 448 and 512 channels, four-byte results: untrimmed below one round but where all wavefronts are at work, and up to 2.5 beside the eight-wavefront form
    (2500, 448, 1088, PLAIN, False), (2600, 448, 1088, PLAIN, True), (4000, 448, 720, PLAIN, False), (4200, 512, 512, PLAIN, True), (8487, 464, 512, PLAIN, False),
    (5156, 512, 1248, PLAIN, False), (2600, 448, 1088, M45, True),
    # windows that round down, between 1.0 and 1.3 rounds
    (2600, 448, 1088, FLOOR, False), (2300, 448, 1088, FLOOR, True), (3600, 448, 1088, FLOOR, True), (4352, 448, 1024, FLOOR, True),
    # 193 to 256 channels: from 1.6 to 2.2 rounds with a tenth of the wavefronts idle
    (14060, 256, 432, FLOOR, False), (14060, 256, 512, FLOOR, True), (14060, 256, 432, PLAIN, False), (12800, 256, 432, PLAIN, True), (18100, 256, 432, PLAIN, True), (14060, 256, 432, M45, True)])
def test_weights_in_registers_leave_trims_with_little_arithmetic(lib, m, c, n, mode, takes):
    """The first rounds of four-byte results, where the trim does not fill them: the forms above and below keep these."""
    text = plan(lib, S.ConvLayer("light", 1, m, 1, c, n), mode)[0]
    assert (words(text, "kernel=") == ["conv_cols_kernel"]) == takes and words(text, "u8_kernel=") == ["conv_cols_kernel"], text


@pytest.mark.parametrize("m,c,n,takes", [
    # an even number of 256-output shares: up to 768 channels and up to 1024; then an odd one, and more
    (24500, 768, 512, True), (24600, 768, 512, False), (32700, 768, 512, False), (32800, 768, 512, True), (81800, 768, 512, True), (81950, 768, 512, False),
    (80384, 768, 1024, False), (16400, 1024, 512, False), (32700, 1024, 512, False), (32800, 1024, 512, True), (41000, 1024, 512, False),
    (20400, 1024, 768, True), (60000, 768, 768, True), (3500, 1024, 1024, True)])
def test_weights_in_registers_leave_trims_that_cost_more_twice(lib, m, c, n, takes):
    """Windows of two and three bits with rounding and pairs, four-byte results: trimmed once per 256 outputs, where the eight-wavefront form
    trims once per 512.  Other trims stay."""
    layer = S.ConvLayer("heavy", 1, m, 1, c, n)
    for mode in (S.Mode(2, S.OPT7_2B, 1, 1), S.Mode(3, S.OPT6_3B, 1, 1)):
        assert words(plan(lib, layer, mode)[0], "kernel=") == ["conv_cols_kernel" if takes else "conv_wide_kernel"]
    assert words(plan(lib, layer, S.Mode(2, S.OPT7_2B, 0, 1))[0], "kernel=") == ["conv_cols_kernel"]
    # (rows off a 64-byte border)
    assert words(plan(lib, S.ConvLayer("heavy", 1, 17000, 1, 1024, 501), S.Mode(2, S.OPT7_2B, 1, 1))[0], "kernel=") == ["conv_cols_kernel"]


@pytest.mark.parametrize("m,c,n,held,run", [
    # pixels for every wavefront slot: bytes 16 a CU (up to 64 channels) and 12; four-byte results 1.1, 1.4, 1.5 and 2 times that
    (131072, 64, 64, False, 128), (131040, 64, 64, False, 0), (98304, 128, 64, False, 128), (98272, 128, 64, False, 0),
    (144192, 256, 64, True, 128), (144160, 256, 64, False, 128), (137632, 320, 64, True, 128), (137600, 320, 64, False, 128),
    (147456, 512, 80, True, 128), (147424, 512, 80, False, 128), (262144, 128, 112, True, 128), (262112, 128, 112, False, 128),
    # more weights than fit beside 128 bytes of result rows, and beside 64
    (196577, 384, 288, False, 64), (196576, 384, 288, False, 0), (196609, 512, 224, False, 64), (196609, 256, 400, False, 0)])
def test_plan_names_the_weights_in_lds(lib, m, c, n, held, run):
    """The plan says where the activations-in-registers form holds its weights in LDS, for four-byte results and for bytes."""
    text = plan(lib, S.ConvLayer("held", 1, m, 1, c, n), S.Mode(4, S.OPT5, 1, 1))[0]
    assert ("weights_in_lds" in text.split()) == held and words(text, "u8_weights_in_lds=") == [str(run)] * (run != 0), text


def test_tuning_hook_forces_and_clears_the_choice(lib):
    """sparq_set_tuning: the documented keys change the plan, NULL restores the rules, junk is refused and changes nothing."""
    conv = S.ConvLayer("conv3x3", 64, 32, 32, 512, 512, 3, 3, (1, 1), (1, 1), 0.5, S.Mode(4, S.OPT5, 1, 1))
    lib.sparq_set_tuning.argtypes = [ctypes.c_char_p]
    base = plan(lib, conv)[0]
    try:
        assert lib.sparq_set_tuning(b"path=gather,tile=128x256") == 0
        assert plan(lib, conv)[0].startswith("conv_gemm_kernel tile=128x256")
        assert lib.sparq_set_tuning(b"path=patch,patch_tn=64,patch_ws=0") == 0
        text = plan(lib, conv)[0]
        assert text.startswith("conv_patch_kernel tile=128x64") and "wave_specialised" not in text
        for junk in (b"path=fast", b"tile=64x64", b"patch_tn=100", b"patch_ws=2", b"colour=red", b"path", b","):
            assert lib.sparq_set_tuning(junk) == 1
        assert plan(lib, conv)[0] == text                            # a refused spec leaves the override as it was
    finally:
        assert lib.sparq_set_tuning(None) == 0
    assert plan(lib, conv)[0] == base


def test_tuning_hook_forces_the_other_forms(lib):
    """form=: wherever the layer fits the form, for four-byte and byte results; the tile kernels where it does not."""
    lib.sparq_set_tuning.argtypes = [ctypes.c_char_p]
    mode = S.Mode(4, S.OPT5, 1, 1)
    big = S.ConvLayer("conv3x3", 64, 32, 32, 512, 512, 3, 3, (1, 1), (1, 1))
    taps = S.ConvLayer("t", 2, 13, 11, 72, 80, 3, 3, (1, 1), (1, 1))
    one = S.ConvLayer("o", 1, 100, 1, 330, 48)
    odd = S.ConvLayer("n", 1, 100, 1, 330, 50)
    few = S.ConvLayer("c32", 2, 13, 11, 32, 80, 3, 3, (1, 1), (1, 1))
    tiles = ("conv_patch_kernel", "conv_gemm_kernel")
    cases = {"split": ((taps, True, True), (one, True, True), (odd, True, True), (few, False, False)),
             "rows": ((one, True, True), (odd, True, False), (taps, False, False), (big, False, False)),
             "cols": ((one, True, True), (odd, True, False), (taps, False, False), (S.ConvLayer("k", 1, 100, 1, 1030, 48), False, False)),
             "wide": ((one, True, True), (odd, True, False), (taps, False, False), (S.ConvLayer("k", 1, 100, 1, 256, 48), False, False)),
             "block": ((taps, True, True), (big, True, True), (one, False, False), (few, False, False))}
    base = [plan(lib, l, mode)[0] for l in (big, taps, one, odd, few)]
    try:
        for form, layers in cases.items():
            assert lib.sparq_set_tuning(f"form={form}".encode()) == 0
            for layer, acc, u8 in layers:
                text = plan(lib, layer, mode)[0]
                k, k8 = words(text, "kernel=")[0], words(text, "u8_kernel=")[0].split(":")[0]
                assert (k == f"conv_{form}_kernel") == acc and (acc or k in tiles), text
                assert (k8 == f"conv_{form}_kernel") == u8 and (u8 or k8 in tiles), text
        assert lib.sparq_set_tuning(b"form=fast") == 1
    finally:
        assert lib.sparq_set_tuning(None) == 0
    assert [plan(lib, l, mode)[0] for l in (big, taps, one, odd, few)] == base


def test_widest_gather_tile_only_with_step_aligned_taps(lib):
    """The 128 x 512 tile tracks a step's filter tap in scalar registers, so every 64-byte reduction step must lie
    inside one tap (more than 32 channels); otherwise, and when 512 columns would read past the padded weights, the
    library takes the next tile, also when the hook asks for the widest one."""
    lib.sparq_set_tuning.argtypes = [ctypes.c_char_p]
    mode = S.Mode(4, S.OPT5, 1, 1)
    try:
        assert lib.sparq_set_tuning(b"path=gather,tile=128x512") == 0
        assert plan(lib, S.ConvLayer("c64", 1, 9, 9, 64, 300, 3, 3, (1, 1), (1, 1)), mode)[0].startswith("conv_gemm_kernel tile=128x512")
        assert plan(lib, S.ConvLayer("c32", 1, 9, 9, 32, 300, 3, 3, (1, 1), (1, 1)), mode)[0].startswith("conv_gemm_kernel tile=128x256")
        assert plan(lib, S.ConvLayer("n520", 1, 9, 9, 64, 520, 3, 3, (1, 1), (1, 1)), mode)[0].startswith("conv_gemm_kernel tile=128x256")
    finally:
        assert lib.sparq_set_tuning(None) == 0


def test_small_workgroups_only_where_they_can_be_launched(lib):
    """A tile of 256 rows of results is addressed in 32 bits: from 2^21 output channels on a few-channel layer is planned
    for the kernels that still take it (the call would otherwise return "unsupported")."""
    mode = S.Mode(4, S.OPT5, 1, 1)
    for n, small in (((1 << 21) - 64, True), (1 << 21, False)):
        for layer in (S.ConvLayer("n_3x3", 1, 16, 16, 64, n, 3, 3, (1, 1), (1, 1)), S.ConvLayer("n_1x9", 1, 1, 16, 64, n, 1, 9, (1, 1), (0, 4))):
            text = plan(lib, layer, mode)[0]
            assert ("small_workgroups" in text) == small, text


def test_few_channel_tiles_stay_inside_32_bit_offsets(lib):
    """Layers of at most four channels: a tile's four-byte results are addressed in 32 bits, with 2^31 as the offset of what is to be
    dropped, so wider layers get lower tiles.  So are the packed weights: 2 GiB of them are for the gather kernel."""
    for n, height in ((262144, 1024), (524272, 1024), (524288, 512), (524304, 512), (600016, 512), (1048560, 512), (1 << 20, 256)):
        text, _, packed = plan(lib, S.ConvLayer("few", 1, 32, 32, 3, n, 5, 5, (1, 1), (2, 2)), S.Mode(4, S.OPT5, 1, 1))
        assert f"few_channels tile={height}x64" in text and packed - 16 * n < 1 << 31, text
    for n, few in (((1 << 20) - 64, True), (1 << 20, False)):        # 15 rows of two taps of 16 bytes for each of 4 n columns
        text, _, packed = plan(lib, S.ConvLayer("tall", 1, 32, 32, 4, n, 15, 1, (1, 1), (7, 2)), S.Mode(4, S.OPT5, 1, 1))
        assert (packed - 16 * n < 1 << 31) == few and words(text, "kernel=") == ["conv_few_kernel" if few else "conv_gemm_kernel"], text


@pytest.mark.parametrize("b,h,w,c,n,k,stride,pad,takes", [
    # few outputs of many pixels: the gather kernel works out four pixels' side by side
    (14, 230, 196, 4, 5, (1, 7), 1, (0, 3), False), (2, 230, 196, 4, 5, (1, 7), 1, (0, 3), True), (9, 150, 148, 2, 14, (3, 3), 1, (1, 1), False),
    (9, 150, 148, 2, 16, (3, 3), 1, (1, 1), False), (9, 150, 148, 2, 17, (3, 3), 1, (1, 1), True), (9, 150, 148, 2, 32, (3, 3), 1, (1, 1), False),
    (9, 150, 148, 2, 36, (3, 3), 1, (1, 1), True), (36, 150, 148, 2, 5, (3, 1), 2, (1, 0), True),
    # rows off a 64-byte border: stored by whole lines as the folded rows of the gather kernel
    (16, 128, 128, 1, 300, (3, 3), 1, (1, 1), False), (2, 128, 128, 1, 300, (7, 7), 1, (3, 3), False), (1, 128, 128, 1, 300, (7, 7), 1, (3, 3), True),
    (16, 128, 128, 1, 304, (7, 7), 1, (3, 3), True), (16, 128, 128, 1, 60, (3, 3), 1, (1, 1), True), (40, 128, 128, 1, 60, (3, 3), 1, (1, 1), False),
    (16, 256, 256, 3, 120, (7, 7), 2, (3, 3), False), (4, 256, 256, 3, 120, (7, 7), 2, (3, 3), True), (32, 128, 128, 1, 65, (3, 3), 1, (1, 1), False),
    (16, 128, 128, 1, 65, (3, 3), 1, (1, 1), True), (40, 128, 128, 1, 61, (3, 3), 1, (1, 1), True), (16, 256, 256, 3, 200, (4, 4), 4, (0, 0), True)], ids=str)
def test_few_channel_layers_the_gather_kernel_is_ahead_on(lib, b, h, w, c, n, k, stride, pad, takes):
    """Both sides of the lines at which four-byte results go to the folded gather kernel; bytes stay."""
    text = plan(lib, S.ConvLayer("few", b, h, w, c, n, *k, (stride, stride), pad), S.Mode(4, S.OPT5, 1, 1))[0]
    assert words(text, "kernel=") == ["conv_few_kernel" if takes else "conv_gemm_kernel"], text
    assert n % 16 or words(text, "u8_kernel=") == ["conv_few_kernel"], text


@pytest.mark.parametrize("shape,k,stride,pad,mode,copy", [
    # few tiles, each with a patch of its own beside few taps' products: the trim of many channels would be left to a few CUs
    ((7, 15, 15, 1396, 96), (1, 7), 2, (0, 3), S.Mode(3, S.OPT6_3B, 1, 1), True), ((16, 7, 7, 2148, 349), (1, 7), 2, (0, 3), S.Mode(4, S.OPT5, 1, 1), True),
    ((10, 5, 63, 836, 320), (1, 7), 2, (0, 0), S.Mode(4, S.OPT5, 1, 1), True), ((6, 7, 17, 980, 32), (7, 1), 3, (0, 0), S.Mode(4, S.OPT3, 0, 1), True),
    ((6, 8, 8, 892, 320), (7, 1), 3, (3, 0), S.Mode(4, S.OPT5, 0, 0), True), ((5, 31, 5, 1016, 18), (3, 3), 2, (0, 0), S.Mode(2, S.OPT7_2B, 1, 1), True),
    # ... against short reductions, patches that the taps reuse, tiles for every CU, nothing to trim
    ((128, 15, 15, 60, 96), (1, 7), 2, (0, 3), S.Mode(4, S.OPT5, 1, 1), False), ((16, 14, 14, 1396, 96), (3, 3), 1, (1, 1), S.Mode(4, S.OPT5, 1, 1), False),
    ((64, 28, 28, 244, 256), (3, 3), 1, (1, 1), S.Mode(4, S.OPT5, 1, 1), False), ((16, 7, 7, 2148, 349), (1, 7), 2, (0, 3), S.PLAIN8, False),
    ((64, 12, 12, 1000, 96), (3, 3), 1, (1, 1), S.Mode(4, S.OPT5, 0, 0), False)], ids=str)
def test_tile_kernels_that_would_trim_longer_than_a_copy_takes(lib, shape, k, stride, pad, mode, copy):
    """Channel counts in whole words are read where they are, except by a tile kernel whose staging is the longer side then."""
    text = plan(lib, S.ConvLayer("words", *shape, *k, (stride, stride), pad), mode)[0]
    assert words(text, "kernel=") == ["conv_patch_kernel"] and ("padded_copy" in text) == copy, text


@pytest.mark.parametrize("b,hw,c,n,square", [(12, 93, 112, 320, False), (52, 69, 128, 160, False), (64, 65, 112, 80, False), (57, 45, 96, 160, True), (52, 69, 64, 160, True)])
def test_square_tile_while_three_workgroups_share_a_cu(lib, b, hw, c, n, square):
    """Strided layers of 65 to 128 channels that the 256 x 64 tile leaves to the gather kernel: the 128 x 128 tile up to 803 patch pixels."""
    text = plan(lib, S.ConvLayer("strided", b, hw, hw, c, n, 3, 3, (2, 2), (1, 1)), S.Mode(4, S.OPT5, 1, 1))[0]
    assert ("small_workgroups tile=128x128" in text) == square and words(text, "u8_kernel=") == ["conv_block_kernel" if square else "conv_gemm_kernel:128x%d" % (256 if n > 128 else 128)], text


@pytest.mark.parametrize("n,mode,copy", [
    (566, S.Mode(3, S.OPT6_3B, 1, 1), True), (512, S.Mode(3, S.OPT6_3B, 1, 1), False), (566, S.Mode(4, S.OPT5, 1, 1), False), (1100, S.Mode(4, S.OPT5, 1, 1), True),
    (1100, S.Mode(4, S.OPT5, 1, 0), False), (1700, S.Mode(4, S.OPT5, 1, 0), False), (1700, S.Mode(4, S.OPT3, 0, 1), False), (1700, S.PLAIN8, False)], ids=str)
def test_1x1_layers_that_would_trim_once_per_column_tile(lib, n, mode, copy):
    """Read where they are while the columns of tiles and the trim's instructions are few enough for the products to cover."""
    text = plan(lib, S.ConvLayer("columns", 1, 11669, 1, 3444, n), mode)[0]
    assert (copy or words(text, "kernel=") == ["conv_wide_kernel"]) and ("padded_copy" in text) == copy, text


@pytest.mark.parametrize("shape,k,stride,mode,copy", [
    # trims of two and three bits with rounding: patches that tiles stage more than five times over, and those that outlast the copy
    ((2, 54, 54, 116, 131), (3, 3), 1, S.Mode(2, S.OPT7_2B, 1, 1), False), ((3, 21, 21, 60, 274), (3, 1), 1, S.Mode(3, S.OPT6_3B, 1, 0), False),
    ((35, 35, 35, 908, 736), (3, 3), 2, S.Mode(3, S.OPT6_3B, 1, 1), True), ((9, 31, 31, 2724, 375), (1, 3), 1, S.Mode(2, S.OPT7_2B, 1, 1), True)], ids=str)
def test_costly_trims_in_tile_kernels_copy_where_staging_outlasts_it(lib, shape, k, stride, mode, copy):
    """The trims with the most arithmetic are decided on as the others are, by the present instruction counts."""
    text = plan(lib, S.ConvLayer("words", *shape, *k, (stride, stride), (k[0] // 2, k[1] // 2)), mode)[0]
    assert words(text, "kernel=") == ["conv_patch_kernel"] and ("padded_copy" in text) == copy, text


@pytest.mark.parametrize("n,mode,copy", [
    (1100, S.Mode(3, S.OPT6_3B, 1, 0), True), (1000, S.Mode(3, S.OPT6_3B, 1, 0), False), (1000, S.Mode(4, S.OPT5, 1, 1), False),
    (500, S.Mode(2, S.OPT7_2B, 1, 1), False), (600, S.Mode(2, S.OPT7_2B, 1, 1), True),
    (3500, S.Mode(2, S.OPT7_2B, 0, 1), False)], ids=str)
def test_1x1_columns_by_the_present_instruction_counts(lib, n, mode, copy):
    """Either side of the column tiles from which a 1x1 layer's trims outlast the copy: four and five, two and three; windows that
    round down with pairs as before, at seven."""
    text = plan(lib, S.ConvLayer("columns", 1, 11669, 1, 3444, n), mode)[0]
    assert ("padded_copy" in text) == copy, text


@pytest.mark.parametrize("m,c,n,mode,copy", [
    (3119, 776, 640, S.Mode(4, S.OPT5, 1, 1), False), (3119, 776, 640, S.Mode(2, S.OPT7_2B, 1, 1), False), (36864, 780, 640, S.Mode(3, S.OPT6_3B, 1, 0), False),
    (1110, 760, 1392, S.Mode(4, S.OPT5, 1, 1), False), (46644, 300, 1632, S.Mode(4, S.OPT5, 1, 1), False), (40000, 660, 1280, S.Mode(4, S.OPT5, 1, 1), False),
    # two- and three-bit windows with rounding and pairs, trimmed by several shares in many rounds: up to 768 channels, up to 1024
    (59800, 580, 640, S.Mode(2, S.OPT7_2B, 1, 1), False), (59900, 580, 640, S.Mode(2, S.OPT7_2B, 1, 1), True), (59900, 580, 640, S.Mode(4, S.OPT5, 1, 1), False),
    (34000, 900, 640, S.Mode(3, S.OPT6_3B, 1, 1), False), (34400, 900, 640, S.Mode(3, S.OPT6_3B, 1, 1), True)])
def test_weights_in_registers_decide_on_the_copy_themselves(lib, m, c, n, mode, copy):
    """Channel counts in whole words that the weights-in-registers form takes are read where they are, by what that form trims and not by what the
    forms behind it would."""
    text = plan(lib, S.ConvLayer("words", 1, m, 1, c, n), mode)[0]
    assert words(text, "kernel=") == ["conv_cols_kernel"] and ("padded_copy" in text) == copy, text


def test_layers_in_turn_do_not_walk_their_tiles_again(lib):
    """The largest patch of a layer comes from a walk over its tile positions (193 us for 147 x 147 pixels) and is kept per
    geometry.  These two geometries share the low nine bits of the cache's hash: called in turn, neither pushes the other out."""
    import time
    mode = S.Mode(4, S.OPT5, 1, 1)
    layers = [S.ConvLayer(f"b{b}", b, 147, 147, 256, 256, 3, 3, (1, 1), (1, 1)) for b in (136, 140)]

    def us(l):
        t = time.perf_counter()
        plan(lib, l, mode)
        return (time.perf_counter() - t) * 1e6

    first = min(us(l) for l in layers)
    again = sorted(us(l) for _ in range(50) for l in layers)[50]
    assert again < first / 3, (first, again)


def test_plan_rejects_bad_arguments(lib):
    buf = ctypes.create_string_buffer(64)
    m = Mode(4, 0x1F, 1, 1)
    bad = Desc(1, 2, 2, 64, 64, 3, 3, 1, 1, 0, 0)
    assert lib.sparq_conv_plan(ctypes.byref(bad), ctypes.byref(m), buf, len(buf)) == 1
    ok = Desc(1, 8, 8, 64, 64, 3, 3, 1, 1, 1, 1)
    assert lib.sparq_conv_plan(ctypes.byref(ok), ctypes.byref(m), None, 0) == 1
    assert lib.sparq_conv_plan(ctypes.byref(ok), ctypes.byref(Mode(5, 1, 0, 0)), buf, len(buf)) == 1


def sparse_plan(lib, d, m):
    buf = ctypes.create_string_buffer(256)
    assert lib.sparq_sparse24_plan(ctypes.byref(d), ctypes.byref(m), buf, len(buf)) == 0
    return buf.value.decode()


def test_sparse24_layers_of_one_step_keep_the_sparse_instruction(lib):
    """1x1 layers of at most 64 channels, vSPARQ off, whose results are too many for the activations-in-registers form."""
    for c, n in ((48, 60), (36, 61), (64, 250)):
        for m in (Mode(4, 0x15, 0, 0), Mode(8, 1, 0, 0)):
            text = sparse_plan(lib, Desc(171, 62, 62, c, n, 1, 1, 1, 1, 0, 0), m)
            assert " kernel=conv_patch_kernel" in text and text.endswith("sparse_mfma"), text


def test_sparse24_plan_names_the_matrix_instruction(lib):
    """2:4 pruned weights: the sparse matrix instruction wherever the (expanded) layer takes the wave-specialised
    input-patch kernel, for every mode; the dense kernels where it does not; and the packed buffer holds both forms."""
    lib.sparq_sparse24_packed_bytes.restype = ctypes.c_size_t
    conv = Desc(64, 32, 32, 512, 512, 3, 3, 1, 1, 1, 1)
    for m in (Mode(4, 0x1F, 1, 1), Mode(4, 0x1F, 1, 0), Mode(4, 0x15, 0, 0), Mode(3, 0x3F, 1, 0), Mode(8, 1, 0, 0)):
        text = sparse_plan(lib, conv, m)
        assert text.startswith("conv_patch_kernel tile=128x256") and text.endswith("sparse_mfma"), text
        assert ("expanded_x4" in text) == bool(m.pair and m.window_bits != 8), text
    thin = Desc(2, 8, 8, 4, 8, 1, 1, 1, 1, 0, 0)                      # expands to 16 channels: taps are not step-aligned
    assert sparse_plan(lib, thin, Mode(4, 0x1F, 1, 1)).endswith("dense_mfma")
    assert lib.sparq_set_tuning(b"path=gather") == 0
    try:
        assert sparse_plan(lib, conv, Mode(4, 0x1F, 1, 1)).endswith("dense_mfma")
    finally:
        assert lib.sparq_set_tuning(None) == 0
    m = Mode(4, 0x1F, 1, 1)
    lib.sparq_packed_bytes.restype = ctypes.c_size_t
    eff = Desc(64, 32, 32, 2048, 512, 3, 3, 1, 1, 1, 1)
    dense_tiles = lib.sparq_packed_bytes(ctypes.byref(eff))
    kp_np = 9 * 2048 * 512
    assert lib.sparq_sparse24_packed_bytes(ctypes.byref(conv), ctypes.byref(m)) >= dense_tiles + kp_np + kp_np // 2 + kp_np // 8
    buf = ctypes.create_string_buffer(64)
    assert lib.sparq_sparse24_plan(ctypes.byref(Desc(1, 4, 4, 6, 8, 1, 1, 1, 1, 0, 0)), ctypes.byref(m), buf, len(buf)) == 1   # C % 4


def test_sparse24_plan_says_where_the_expansion_happens(lib):
    """While staging: blocked channel counts, vSPARQ on, the sparse instruction, at most 32 patch pixels per tap."""
    m = Mode(4, 0x1F, 0, 1)
    for d, staging in (((2, 13, 11, 176, 100, 3, 3, 1, 1, 1, 1), True), ((2, 4, 4, 256, 136, 1, 1, 1, 1, 0, 0), True),
                       ((1, 3, 11, 256, 136, 1, 1, 1, 1, 0, 0), False), ((2, 15, 15, 256, 70, 1, 1, 1, 1, 0, 0), False),
                       ((2, 13, 11, 96, 100, 3, 3, 1, 1, 1, 1), False)):          # 96 channels: a third of padding
        text = sparse_plan(lib, Desc(*d), m)
        assert ("expanded_while_staging" in text) == staging and text.endswith("sparse_mfma"), text
    for m in (Mode(4, 0x1F, 0, 0), Mode(8, 1, 0, 0)):
        assert "expanded" not in sparse_plan(lib, Desc(2, 13, 11, 176, 100, 3, 3, 1, 1, 1, 1), m)


def test_one_tap_sparse24_layers_take_whole_units(lib):
    """Expanded 1x1 layers are filled up with zero channels to units of four or two 64-channel blocks where that adds little: their
    number of blocks is a multiple of three, and a unit of one costs a barrier per block."""
    lib.sparq_sparse24_packed_bytes.restype = ctypes.c_size_t
    for c, unit in ((64, 64), (96, 64), (128, 128), (192, 64), (256, 256), (320, 256), (448, 128), (640, 128), (576, 256), (832, 256), (1216, 256)):
        text = sparse_plan(lib, Desc(1, 14, 14, c, 256, 1, 1, 1, 1, 0, 0), Mode(4, 0x1F, 1, 1))
        assert f"unit_channels={unit} " in text and text.endswith("sparse_mfma"), (c, text)
    for m, c, n, unit in ((32768, 576, 300, 256), (33000, 576, 300, 64), (32768, 72, 16, 256), (33000, 72, 16, 128), (33000, 72, 80, 256)):
        text = sparse_plan(lib, Desc(1, m, 1, c, n, 1, 1, 1, 1, 0, 0), Mode(4, 0x1F, 1, 1))
        assert f"unit_channels={unit} " in text, (m, c, n, text)
