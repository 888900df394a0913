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


def test_lower_tiles_do_not_wait_for_w_that_is_not_due(tmp_path):
    # GEMM tiles of 128 and 192 rows, W through LDS with stages ahead (four and three; none, i.e. two, up to 128 rows).  Loads return in order, so a wait names how many
    # may be outstanding.  In the middle of a k-tile half of the loads of A (a k-tile is a loads of A and w of W to a wave) have gone
    # out behind A of the next one, and, until W has ended for a whole k-tile, w loads of W that are not due yet.  In front of the loop
    # only the first k-tile is due, with fewer k-tiles than stages too.
    asm = tmp_path / "gemm.s"
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "gemm_mfma.hip"), "-o", str(asm)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    seen = []
    for name, body in re.findall(r"^(\S*gemm16_bf16_kernelI\S+):(.*?)^\.Lfunc_end", asm.read_text(), re.S | re.M):
        bm, bn, wm, wn, stages = (int(v) for v in re.findall(r"Li(\d+)E", name))
        if bm == 256:
            continue
        waits = [int(v) for v in re.findall(r"ASMSTART\s+s_waitcnt vmcnt\((\d+)\)", body)]
        a, w, ahead = bm // (8 * wm * wn), bn // (8 * wm * wn), stages - 2
        loop = [set(), {a // 2 + w}, {a // 2 + w, a // 2}][ahead]              # the k-tiles that bring A alone
        front = {a + w + u * w for u in range(ahead + 1)}
        assert loop | front | {(a + w) // 2 + (w if ahead else 0), 0} == set(waits), (name, waits)
        seen.append((bm, stages))
    assert set(seen) == {(128, 2), (128, 4), (192, 3)} and len(seen) >= 8
