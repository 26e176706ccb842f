"""Kernels that turn results through a wavefront's own piece of LDS, where lanes read what other lanes wrote without a
barrier: the compiler's output must hold a wavefront fence on either side of the reads (hardware order alone would not keep
the compiler from moving them)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2105_11010_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

KERNELS = {
    "rows": ("sparq_conv_rows_kernel.h", "conv_rows_kernel<RowsCfg<2, 1, true, 4>, kTrimNone, true>(const RowsParams)"),
    "cols": ("sparq_conv_cols_kernel.h", "conv_cols_kernel<ColsCfg<8, 2, 1, 2>, kTrimNone, true>(const ColsParams)"),
    "wide": ("sparq_conv_wide_kernel.h", "conv_wide_kernel<Wide256, kTrimNone, true>(const WideParams)"),
    "sparse": ("sparq_conv_patch_kernel.h", "conv_patch_kernel<PatchCfg<64, 4, 1, 2, 1, 2, true, true>, kTrimNone>(const PatchParams)"),
    "codec": ("sparq_packed_act_kernel.h", "unpack_act_kernel<4, 3, 1, true, true>(const CodecParams)"),
}


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs hipcc")
@pytest.mark.parametrize("name", KERNELS)
def test_lds_turn_is_fenced(tmp_path, name):
    header, kernel = KERNELS[name]
    src = tmp_path / "one.hip"
    src.write_text(f'#include "{header}"\nnamespace sparq {{\ntemplate __global__ void {kernel};\n}}\n')
    out = tmp_path / "one.ll"
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", CSRC, "--cuda-device-only", "-S", "-emit-llvm",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", str(src), "-o", str(out)], check=True, capture_output=True)
    assert out.read_text().count('fence syncscope("wavefront") acq_rel') >= 2
