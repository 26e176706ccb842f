"""The packed-storage codec's record arithmetic, built for the host, against the oracle (CPU only)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import sparq_synth as S

HERE = os.path.dirname(os.path.abspath(__file__))

# every ShiftCtrl width for every window width, full and thinned option sets
MODES = [(4, 0x1F), (4, 0x15), (4, 0x11), (4, 0x17), (3, 0x3F), (3, 0x29), (3, 0x2D), (3, 0x21), (2, 0x7F), (2, 0x55), (2, 0x41), (2, 0x5F)]


@pytest.fixture(scope="module")
def codec(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("codec") / "libcodec_host.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so,
                    os.path.join(HERE, "packed_swar_host_check.cpp")], check=True)
    lib = ctypes.CDLL(so)
    lib.codec_records.argtypes = [ctypes.c_int, ctypes.c_uint] + [ctypes.c_int] * 4 + [ctypes.c_void_p, ctypes.c_long] + [ctypes.c_void_p] * 2

    def run(x, n, mask, rnd, pair, group, rec_bytes):
        sb = max(1, (bin(mask).count("1") - 1).bit_length())
        x = np.ascontiguousarray(x, dtype=np.uint8).reshape(-1, 32)
        packed = np.empty((len(x), rec_bytes), dtype=np.uint8)
        y = np.empty_like(x)
        p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
        assert lib.codec_records(n, mask, rnd, pair, group, sb, p(x), len(x), p(packed), p(y)) == 0
        return packed, y
    return run


@pytest.mark.parametrize("n,mask", MODES)
@pytest.mark.parametrize("rnd", [0, 1])
@pytest.mark.parametrize("pairing", [0, 1])
def test_records_of_all_pairs(oracle, codec, n, mask, rnd, pairing):
    if oracle.mode_check(n, mask, rnd, pairing):
        pytest.skip("mode not valid with pairing")
    kw = dict(window_bits=n, shift_mask=mask, round_nearest=rnd, pair=pairing)
    a, b = np.meshgrid(np.arange(256, dtype=np.uint8), np.arange(256, dtype=np.uint8), indexing="ij")
    x = np.stack([a, b], axis=-1).reshape(-1, 32)
    packed, y = codec(x, n, mask, rnd, pairing, 1, oracle.packed_record_bytes(1, **kw))
    assert np.array_equal(packed, oracle.pack_act(x, **kw))
    assert np.array_equal(y, oracle.trim(x, **kw))


@pytest.mark.parametrize("n,mask", MODES)
@pytest.mark.parametrize("rnd", [0, 1])
@pytest.mark.parametrize("group", [2, 4, 8, 16, 32])
def test_records_with_shared_shifts(oracle, codec, n, mask, rnd, group):
    kw = dict(window_bits=n, shift_mask=mask, round_nearest=rnd, pair=0)
    x = S.gen_activations((4096, 32), 0.6, S.rng_for(7, 40 + group))
    x[0], x[1] = 0, 255
    packed, y = codec(x, n, mask, rnd, 0, group, oracle.packed_record_bytes(group, **kw))
    ref = oracle.pack_act(x, group, **kw)
    assert np.array_equal(packed, ref)
    assert np.array_equal(y, oracle.unpack_act(ref, x.shape, group, **kw))
