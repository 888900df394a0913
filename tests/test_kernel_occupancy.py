"""What the compiler makes of kernels whose speed hangs on how many of their waves a compute unit holds (host only)."""
import os
import re
import subprocess

from paper_2411_02820_amd import build


def _occupancy(src):
    """{mangled kernel name: waves per SIMD by registers and LDS}"""
    cmd = [build.HIPCC, *build.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c", os.path.join(build.CSRC, src),
           "-o", os.devnull]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return {m[0]: int(m[1]) for m in re.findall(r"Function Name: (\S+).*?Occupancy \[waves/SIMD\]: (\d+)", r.stderr, re.S)}


def test_fp32_qkv_on_medium_tiles_is_no_heavier_than_the_plain_projection():
    occ = {tuple(int(v) for v in re.findall(r"L[ib](\d+)E", name.split("gemm_fp32_kernelI")[1])): n
           for name, n in _occupancy("fp32_mfma.hip").items() if "gemm_fp32_kernelI" in name}
    medium = {t[7]: n for t, n in occ.items() if t[:6] == (2, 2, 1, 1, 4, 2)}   # by epilogue: plain, SwiGLU, RoPE
    assert set(medium) == {0, 1, 2} and medium[2] >= medium[1] >= medium[0] > 1, medium
