"""Timed cases of the library: what its users have it do, through the public entry points.

A case is a dict of plain values; ``listed()`` names the fixed ones, ``draw(rng)`` makes another one of the same
ranges.  ``prepare`` makes what a program holds before the call (device tensors, packed weights, scratch), ``run``
is one pass through the entry points, ``work`` the bytes and operations the pass cannot do without and
``tolerance`` how far a correct result may be off.

Kinds of cases:
  stack    every convolution of a network's table in order, one library call each, on its own input (what pooling,
           residual additions and concatenations would hand over), each layer with weights of its own
  conv     one convolution layer (an explicit matrix product is the 1x1 case with H = M, W = 1)
  sparse24 one convolution with 2:4 pruned weights
  packed   one convolution whose input is held in packed storage
  codec    activations packed and unpacked again
  trim     the standalone trim of a tensor
  post     int32 accumulators dequantised to fp32 and requantised to uint8

Every entry point is defined to the bit (int32 sums; one int32 -> fp32 conversion and one fp32 product per
result; bytes), so every case is compared exactly.
"""
import math

import torch

import paper_2105_11010_amd as sq

# ------------------------------------------------------------------------------------------------------------
# trim modes: (window bits, allowed shifts, round to nearest, vSPARQ pairs)
# ------------------------------------------------------------------------------------------------------------
MODES = {
    "4b-5opt-round-pair": (4, 0x1F, 1, 1),
    "4b-5opt-floor": (4, 0x1F, 0, 0),
    "4b-5opt-round": (4, 0x1F, 1, 0),
    "4b-3opt-floor-pair": (4, 0x15, 0, 1),
    "4b-3opt-floor": (4, 0x15, 0, 0),
    "4b-2opt-round-pair": (4, 0x11, 1, 1),
    "3b-6opt-round-pair": (3, 0x3F, 1, 1),
    "2b-7opt-round-pair": (2, 0x7F, 1, 1),
    "plain8": (8, 0x01, 0, 0),
}
MAIN_MODE = "4b-5opt-round-pair"


def _mode(name):
    return sq.mode(*MODES[name])


# ------------------------------------------------------------------------------------------------------------
# layer tables: (H, W, C, N, KH, KW, stride, pad_h, pad_w, plain 8 bits)
# ------------------------------------------------------------------------------------------------------------
def _resnet18():
    L = [(224, 224, 3, 64, 7, 7, 2, 3, 3, True)]
    L += [(56, 56, 64, 64, 3, 3, 1, 1, 1, False)] * 4
    hw, c = 56, 64
    for n in (128, 256, 512):
        L.append((hw, hw, c, n, 3, 3, 2, 1, 1, False))
        L.append((hw, hw, c, n, 1, 1, 2, 0, 0, False))
        hw //= 2
        L += [(hw, hw, n, n, 3, 3, 1, 1, 1, False)] * 3
        c = n
    return L


def _resnet50():
    L = [(224, 224, 3, 64, 7, 7, 2, 3, 3, True)]
    hw, c = 56, 64
    for mid, n, blocks, s in ((64, 256, 3, 1), (128, 512, 4, 2), (256, 1024, 6, 2), (512, 2048, 3, 2)):
        for b in range(blocks):
            st = s if b == 0 else 1
            L.append((hw, hw, c, mid, 1, 1, 1, 0, 0, False))
            L.append((hw, hw, mid, mid, 3, 3, st, 1, 1, False))
            L.append((hw // st, hw // st, mid, n, 1, 1, 1, 0, 0, False))
            if b == 0:
                L.append((hw, hw, c, n, 1, 1, st, 0, 0, False))
            hw, c = hw // st, n
    return L


def _inception():
    L = []
    for c in (192, 256, 288):
        L += [(35, 35, c, 64, 1, 1, 1, 0, 0, False), (35, 35, c, 48, 1, 1, 1, 0, 0, False)]
    L += [(35, 35, 288, 96, 1, 1, 1, 0, 0, False), (35, 35, 48, 64, 5, 5, 1, 2, 2, False),
          (35, 35, 64, 96, 3, 3, 1, 1, 1, False), (35, 35, 96, 96, 3, 3, 1, 1, 1, False),
          (35, 35, 288, 384, 3, 3, 2, 0, 0, False), (35, 35, 96, 96, 3, 3, 2, 0, 0, False)]
    for c in (128, 160, 192):
        L += [(17, 17, 768, c, 1, 1, 1, 0, 0, False), (17, 17, c, c, 1, 7, 1, 0, 3, False),
              (17, 17, c, c, 7, 1, 1, 3, 0, False)]
    L += [(17, 17, 192, 192, 7, 1, 1, 3, 0, False), (17, 17, 192, 320, 3, 3, 2, 0, 0, False),
          (17, 17, 192, 192, 3, 3, 2, 0, 0, False), (8, 8, 768, 320, 1, 1, 1, 0, 0, False),
          (8, 8, 768, 384, 1, 1, 1, 0, 0, False), (8, 8, 384, 384, 1, 3, 1, 0, 1, False),
          (8, 8, 384, 384, 3, 1, 1, 1, 0, False), (8, 8, 448, 384, 3, 3, 1, 1, 1, False)]
    # odd channel counts: an unpaired last channel, ragged reductions and outputs
    L += [(35, 35, 65, 96, 3, 3, 1, 1, 1, False), (17, 17, 159, 161, 1, 7, 1, 0, 3, False)]
    return L


TABLES = {"resnet18": (_resnet18(), "4b-3opt-floor-pair"), "resnet50": (_resnet50(), MAIN_MODE),
          "inception": (_inception(), MAIN_MODE)}


def _conv_case(name, B, H, W, C, N, KH, KW, stride, ph, pw, output, mode=MAIN_MODE, zf=0.5, kind="conv", **more):
    case = {"kind": kind, "B": B, "H": H, "W": W, "C": C, "N": N, "KH": KH, "KW": KW, "stride": stride,
            "pad_h": ph, "pad_w": pw, "output": output, "mode": mode, "zf": zf, **more}
    return {"name": name, **case} if name else case


def listed():
    return [
        # one image, one 3x3 layer of a network's first stage: the smallest call, bound by latency
        _conv_case("conv3x3_64_b1", 1, 56, 56, 64, 64, 3, 3, 1, 1, 1, "fp32"),
        # a network serving one request at a time: twenty short launches
        {"name": "resnet18_b1_u8", "kind": "stack", "table": "resnet18", "batch": 1, "output": "u8"},
        # the same network evaluated in batches, results dequantised (calibration, accuracy runs)
        {"name": "resnet18_b32_fp32", "kind": "stack", "table": "resnet18", "batch": 32, "output": "fp32"},
        # a large network at serving throughput: the largest case
        {"name": "resnet50_b256_u8", "kind": "stack", "table": "resnet50", "batch": 256, "output": "u8"},
        # mixed filter shapes, channel counts that fit no tile, odd channels
        {"name": "inception_b128_fp32", "kind": "stack", "table": "inception", "batch": 128, "output": "fp32"},
        # one wide 3x3 layer at full occupancy: the matrix-bound end
        _conv_case("conv3x3_512_b64", 64, 32, 32, 512, 512, 3, 3, 1, 1, 1, "fp32"),
        # the same contraction on a materialised A: a plain trimmed matrix product with exact int32 results
        _conv_case("gemm_65536x4608x512", 1, 65536, 1, 4608, 512, 1, 1, 1, 0, 0, "int32"),
        # the layer with 2:4 pruned weights, pairs formed by the weights' coordinates
        _conv_case("sparse24_512_b64", 64, 32, 32, 512, 512, 3, 3, 1, 1, 1, "fp32", kind="sparse24"),
        # the layer reading an input kept in packed storage (7 bits per activation)
        _conv_case("packed_512_b64", 64, 32, 32, 512, 512, 3, 3, 1, 1, 1, "fp32", mode="4b-3opt-floor-pair",
                   kind="packed", group=1),
        # activations written to packed storage and read back
        {"name": "codec_65536x4608", "kind": "codec", "rows": 65536, "C": 4608, "mode": MAIN_MODE, "group": 1, "zf": 0.5},
        # the trim on its own, on a tensor with an odd channel count
        {"name": "trim_156800x289", "kind": "trim", "rows": 156800, "C": 289, "mode": MAIN_MODE, "zf": 0.5},
        # accumulators of a ragged layer turned into fp32 results and into the next layer's bytes
        {"name": "post_36992x161", "kind": "post", "rows": 36992, "N": 161},
    ]


# ------------------------------------------------------------------------------------------------------------
# drawn cases
# ------------------------------------------------------------------------------------------------------------
def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """A channel count: mostly multiples of 16, some of 4, some odd."""
    c = _log_int(rng, lo, hi)
    r = rng.random()
    if r < 0.6:
        return max(16, c // 16 * 16)
    if r < 0.8:
        return max(4, c // 4 * 4)
    return c | 1


def _layer_ok(case):
    M = _out_rows(case)
    return 2 * M * _k(case) * case["N"] <= 3.2e11 and case["B"] * case["H"] * case["W"] * case["C"] <= 4e8 and \
        M * case["N"] <= 2e8


def _draw_layer(rng):
    while True:
        kh, kw, ph, pw = rng.choice([(1, 1, 0, 0), (3, 3, 1, 1), (3, 3, 1, 1), (3, 3, 0, 0), (5, 5, 2, 2), (1, 7, 0, 3), (7, 1, 3, 0)])
        hw = _log_int(rng, 7, 112)
        case = _conv_case(None, _log_int(rng, 1, 256), hw, hw, _channels(rng, 32, 1024), _channels(rng, 32, 1024), kh, kw,
                          rng.choice([1, 1, 1, 2]), ph, pw, rng.choice(["fp32", "int32", "u8", "u8", "u8trim"]),
                          mode=rng.choice(list(MODES)), zf=round(rng.uniform(0.2, 0.8), 2))
        if _layer_ok(case):
            return case


def draw(rng):
    kind = rng.choice(["stack", "conv", "conv", "conv", "gemm", "gemm", "sparse24", "packed", "codec", "trim", "post"])
    if kind == "stack":
        table = rng.choice(list(TABLES))
        return {"kind": "stack", "table": table, "batch": _log_int(rng, 1, 128 if table == "inception" else 224),
                "output": rng.choice(["fp32", "u8"]) if table != "resnet50" else "u8"}
    if kind == "conv":
        return _draw_layer(rng)
    if kind == "gemm":
        while True:
            case = _conv_case(None, 1, _log_int(rng, 64, 65536), 1, _channels(rng, 128, 4608), _channels(rng, 32, 2048), 1, 1, 1, 0, 0,
                              rng.choice(["fp32", "int32", "u8"]), mode=rng.choice(list(MODES)), zf=round(rng.uniform(0.2, 0.8), 2))
            if _layer_ok(case):
                return case
    if kind in ("sparse24", "packed"):
        while True:
            case = _draw_layer(rng)
            case["kind"] = kind
            case["output"] = rng.choice(["fp32", "int32"])
            if kind == "sparse24":
                case["C"] = max(32, case["C"] // 16 * 16) if rng.random() < 0.8 else max(32, case["C"] // 4 * 4)
                case["C"] = min(case["C"], 512)
            else:
                case["group"] = 1
                if case["mode"] == "plain8":
                    case["mode"] = MAIN_MODE
                if not MODES[case["mode"]][3]:
                    case["group"] = rng.choice([1, 2, 8, 32])
            if _layer_ok(case):
                return case
    if kind == "post":
        return {"kind": "post", "rows": _log_int(rng, 49, 802816 // 4), "N": _channels(rng, 32, 512)}
    rows, C = _log_int(rng, 49, 156800), _channels(rng, 16, 4608)
    rows = min(rows, 302000000 // C)
    mode = rng.choice([m for m in MODES if m != "plain8"])
    case = {"kind": kind, "rows": rows, "C": C, "mode": mode, "zf": round(rng.uniform(0.2, 0.8), 2)}
    if kind == "codec":
        case["group"] = 1 if MODES[mode][3] else rng.choice([1, 2, 8, 32])
    return case


# ------------------------------------------------------------------------------------------------------------
# sizes
# ------------------------------------------------------------------------------------------------------------
def _out_rows(c):
    ho = (c["H"] + 2 * c["pad_h"] - c["KH"]) // c["stride"] + 1
    wo = (c["W"] + 2 * c["pad_w"] - c["KW"]) // c["stride"] + 1
    return c["B"] * ho * wo


def _k(c):
    return c["KH"] * c["KW"] * c["C"]


def _layers(case):
    """The convolution cases of a stack, in order."""
    table, mode = TABLES[case["table"]]
    return [_conv_case(None, case["batch"], h, w, c, n, kh, kw, s, ph, pw, case["output"],
                       mode="plain8" if plain else mode, zf=0.0 if plain else 0.5)
            for h, w, c, n, kh, kw, s, ph, pw, plain in table]


def _packed_bytes(rows, C, mode, group):
    n, mask, _, pair = MODES[mode]
    bits = max(1, (bin(mask).count("1") - 1).bit_length())
    words = n + (32 // group * bits + 31) // 32 + (1 if pair else 0)
    return rows * ((C + 31) // 32) * words * 4


def work(case):
    kind = case["kind"]
    if kind == "stack":
        parts = [work(c) for c in _layers(case)]
        return {"bytes": sum(p["bytes"] for p in parts), "flops": sum(p["flops"] for p in parts)}
    if kind in ("conv", "sparse24", "packed"):
        M, K, N = _out_rows(case), _k(case), case["N"]
        # 1x1 layers with a stride do not read the pixels in between
        pixels = M if case["KH"] == case["KW"] == 1 else case["B"] * case["H"] * case["W"]
        read = pixels * case["C"]
        if kind == "packed":
            read = _packed_bytes(pixels, case["C"], case["mode"], case["group"])
        kept = 2 if kind == "sparse24" else 1                      # pruned weights are not multiplied; 10 bits per kept one
        weights = K * N if kept == 1 else K * N * 5 // 8
        return {"bytes": read + weights + M * N * (1 if case["output"].startswith("u8") else 4) + 4 * N,
                "flops": 2 * M * K * N // kept}
    if kind == "codec":
        n = case["rows"] * case["C"]
        return {"bytes": 2 * (n + _packed_bytes(case["rows"], case["C"], case["mode"], case["group"])), "flops": 0}
    if kind == "trim":
        return {"bytes": 2 * case["rows"] * case["C"], "flops": 0}
    n = case["rows"] * case["N"]
    return {"bytes": 2 * 4 * n + 5 * n, "flops": 2 * n}             # each of the two calls reads the accumulators


def tolerance(case):
    return "exact"


# ------------------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------------------
def _activations(shape, zf, gen):
    """ReLU-sparse half-normal bytes: exact zeros at fraction zf, the rest clip(rint(|N(0,1)| * 40), 1, 255)."""
    n = math.prod(shape)
    out = torch.empty(n, dtype=torch.uint8, device="cuda")
    for lo in range(0, n, 1 << 27):
        hi = min(n, lo + (1 << 27))
        v = torch.randn(hi - lo, device="cuda", generator=gen).abs_().mul_(40.0).round_().clamp_(1, 255)
        v.mul_(torch.rand(hi - lo, device="cuda", generator=gen) >= zf)
        out[lo:hi] = v.to(torch.uint8)
    return out.view(shape)


def _weights(shape, gen):
    return torch.randint(-127, 128, shape, dtype=torch.int8, device="cuda", generator=gen)


def _uniform(n, lo, hi, gen):
    return torch.rand(n, device="cuda", generator=gen) * (hi - lo) + lo


def _pruned_weights(N, KH, KW, C, gen):
    """2:4 compressed weights: two kept positions of every four channels (ascending), about 3 % zeros among them."""
    pairs = torch.tensor([[0, 1], [0, 2], [0, 3], [1, 2], [1, 3], [2, 3]], dtype=torch.uint8, device="cuda")
    groups = N * KH * KW * (C // 4)
    idx = pairs[torch.randint(0, 6, (groups,), device="cuda", generator=gen)].reshape(N, KH, KW, C // 2)
    vals = _weights((groups, 2), gen)
    vals.mul_((torch.rand((groups, 2), device="cuda", generator=gen) >= 0.03).to(torch.int8))
    return vals.reshape(N, KH, KW, C // 2).contiguous(), idx.contiguous()


def _buffer(n):
    return torch.empty(n, dtype=torch.uint8, device="cuda") if n else None


def _prepare_conv(case, gen):
    m = _mode(case["mode"])
    s = case["stride"]
    d = sq.conv_desc(case["B"], case["H"], case["W"], case["C"], case["N"], case["KH"], case["KW"], (s, s),
                     (case["pad_h"], case["pad_w"]))
    x = _activations((case["B"], case["H"], case["W"], case["C"]), case["zf"], gen)
    st = {"kind": case["kind"], "d": d, "m": m, "x": x, "output": case["output"]}
    if case["kind"] == "sparse24":
        vals, idx = _pruned_weights(case["N"], case["KH"], case["KW"], case["C"], gen)
        st["w"] = _buffer(sq.sparq_sparse24_packed_bytes(d, m))
        sq.sparq_pack_weights_sparse24(vals, idx, d, m, st["w"])
        st["ws"] = _buffer(sq.sparq_sparse24_workspace_bytes(d, m))
    else:
        st["w"] = _buffer(sq.sparq_packed_bytes(d))
        sq.sparq_pack_weights(_weights((case["N"], case["KH"], case["KW"], case["C"]), gen), d, st["w"])
        if case["kind"] == "packed":
            st["group"] = case["group"]
            st["x"] = _buffer(sq.sparq_packed_act_bytes(x.numel() // case["C"], case["C"], m, case["group"]))
            sq.sparq_pack_act(x, st["x"], m, case["group"])
            st["ws"] = _buffer(sq.sparq_conv_packed_workspace_bytes(d, m))
        else:
            st["ws"] = _buffer(sq.sparq_workspace_bytes(d, m))
    M, N = sq.out_rows(d), case["N"]
    if case["output"].startswith("u8"):
        # factors that spread the results over the byte range: about half clamp at 0, under 1 % at 255
        st["scale"] = _uniform(N, 0.7, 1.3, gen) * (0.044 / math.sqrt(_k(case)))
        st["out_mode"] = m if case["output"] == "u8trim" else None
        st["y"] = torch.empty((M, N), dtype=torch.uint8, device="cuda")
    elif case["output"] == "fp32":
        st["scale"] = _uniform(N, 1e-3, 1e-2, gen)
        st["y"] = torch.empty((M, N), dtype=torch.float32, device="cuda")
    else:
        st["y"] = torch.empty((M, N), dtype=torch.int32, device="cuda")
    return st


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind = case["kind"]
    if kind == "stack":
        return {"kind": kind, "layers": [_prepare_conv(c, gen) for c in _layers(case)]}
    if kind in ("conv", "sparse24", "packed"):
        return _prepare_conv(case, gen)
    if kind == "post":
        shape = (case["rows"], case["N"])
        acc = (torch.randn(shape, device="cuda", generator=gen) * 60000.0).to(torch.int32)
        return {"kind": kind, "acc": acc, "scale": _uniform(case["N"], 1e-3, 1e-2, gen),
                "factor": _uniform(case["N"], 0.7, 1.3, gen) * (0.044 / 30.0),
                "out": torch.empty(shape, dtype=torch.float32, device="cuda"),
                "y": torch.empty(shape, dtype=torch.uint8, device="cuda")}
    x = _activations((case["rows"], case["C"]), case["zf"], gen)
    st = {"kind": kind, "m": _mode(case["mode"]), "x": x, "y": torch.empty_like(x)}
    if kind == "codec":
        st["group"] = case["group"]
        st["packed"] = _buffer(sq.sparq_packed_act_bytes(case["rows"], case["C"], st["m"], case["group"]))
    return st


# ------------------------------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------------------------------
def _run_conv(st):
    y = st["y"]
    if st["output"].startswith("u8"):
        sq.sparq_conv_gemm_u8(st["x"], st["w"], st["d"], st["m"], st["scale"], y, workspace=st["ws"], out_mode=st["out_mode"])
        return y
    kw = {"workspace": st["ws"]}
    if st["output"] == "fp32":
        kw.update(scale=st["scale"], out=y)
    else:
        kw.update(acc=y)
    if st["kind"] == "packed":
        sq.sparq_conv_gemm_packed(st["x"], st["group"], st["w"], st["d"], st["m"], **kw)
    elif st["kind"] == "sparse24":
        sq.sparq_conv_gemm_sparse24(st["x"], st["w"], st["d"], st["m"], **kw)
    else:
        sq.sparq_conv_gemm(st["x"], st["w"], st["d"], st["m"], **kw)
    return y


def run(state):
    kind = state["kind"]
    if kind == "stack":
        return [_run_conv(st) for st in state["layers"]]
    if kind in ("conv", "sparse24", "packed"):
        return _run_conv(state)
    if kind == "codec":
        sq.sparq_pack_act(state["x"], state["packed"], state["m"], state["group"])
        sq.sparq_unpack_act(state["packed"], state["y"], state["m"], state["group"])
        return [state["packed"], state["y"]]
    if kind == "trim":
        sq.sparq_trim(state["x"], state["y"], state["m"])
        return state["y"]
    sq.sparq_dequant(state["acc"], state["scale"], state["out"])
    sq.sparq_requant(state["acc"], state["factor"], state["y"])
    return [state["out"], state["y"]]
