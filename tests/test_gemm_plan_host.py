"""How the bf16 GEMM splits its work, over random sizes (host code): what the launches and their scratch rely on."""
import random

from paper_2411_02820_amd import binding as B


def test_plans_keep_their_bounds():
    rng = random.Random(3)
    seen = set()
    for _ in range(20000):
        M, N, K = (round(2 ** rng.uniform(lo, hi)) for lo, hi in ((6.03, 16), (6, 16), (0, 9)))
        M, N, K = max(M, 65), N // 4 * 4, K * 64
        bm, splits, head, rest = B.dsk_gemm_plan(M, N, K)
        tiles = -(-M // bm) * -(-N // 256)
        assert bm in (128, 192, 256)
        if splits > 1:   # 256 workgroups, so 64 MiB of partial sums; four k-tiles each, none without any
            assert head == 0 and tiles * splits <= 256 and splits * M * N * 4 <= 64 << 20
            per = -(-(K // 64) // splits)
            assert K // 64 >= 4 * splits and per * (splits - 1) < K // 64
        if head:
            assert bm == 256 and head % 256 == 0 and 64 < M - head and rest in (128, 192, 256)
        unsplit = B.dsk_gemm_plan(M, N, K, False)
        assert unsplit[1] == 1
        seen.add((bm, splits > 1, rest))
    assert len(seen) >= 8, seen   # every height with and without a split, and a rest of either lower height


def test_sizes_that_have_no_plan():
    import ctypes as C
    plan = (C.c_int32 * 4)()
    for M, N, K in ((64, 256, 256), (100, 0, 256), (100, 256, 0), (100, 256, 100), (2 ** 31 - 1, 256, 256), (100, 2 ** 31 - 1, 256)):
        assert B.lib.dsk_gemm_plan(M, N, K, 1, plan) == B.DSK_EINVAL
    assert B.lib.dsk_gemm_plan(100, 256, 256, 1, None) == B.DSK_EINVAL
