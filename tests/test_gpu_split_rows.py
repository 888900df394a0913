"""Projections over 65 to a few thousand rows: every tile height, a contraction split over workgroups with RoPE, residual and
RMSNorm in its reduction, ragged tiles, against float64 and against the kernels that do not split."""
import numpy as np
import pytest
import torch

from oracle import dsk_oracle as O
from paper_2411_02820_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2411_02820_amd import binding
    return binding


# row-major weights through the component call: rows around multiples of 128, 192 and 256, columns that end inside a tile; on
# every form a projection can take: each tile height unsplit and split (an uneven last share), and two launches, whole
# rounds of 256-row tiles and a rest in either lower height, with the residual's and the result's rows of the second
@pytest.mark.parametrize("M,N,K,residual,plan", [
    (65, 64, 64, False, (128, 1, 0, 0)), (129, 516, 320, True, (128, 1, 0, 0)), (2000, 2560, 256, False, (128, 1, 0, 0)),
    (4200, 4612, 128, True, (192, 1, 0, 0)), (3000, 5000, 192, True, (256, 1, 0, 0)),
    (191, 1028, 1984, False, (128, 7, 0, 0)), (193, 256, 4096, True, (128, 16, 0, 0)), (257, 2052, 1024, True, (128, 4, 0, 0)),
    (385, 512, 8192, False, (128, 16, 0, 0)), (1025, 1024, 2048, True, (128, 4, 0, 0)),
    (129, 4100, 4096, True, (192, 8, 0, 0)), (129, 3076, 8192, False, (192, 13, 0, 0)), (700, 2052, 8192, True, (192, 7, 0, 0)),
    (385, 4100, 8192, True, (256, 7, 0, 0)), (769, 3076, 4096, False, (256, 4, 0, 0)),
    (5000, 4612, 4096, True, (256, 1, 3328, 192)), (7700, 4612, 2048, True, (256, 1, 6656, 128))])
def test_linear_bf16_medium_rows(B, M, N, K, residual, plan):
    assert B.dsk_gemm_plan(M, N, K, M <= 4096) == plan
    bf = lambda a: synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(a))
    x = bf(synth.normal(M * K, 51, 0, 1.0).reshape(M, K))
    w = bf(synth.normal(N * K, 51, 1, 0.05).reshape(N, K))
    r = bf(synth.normal(M * N, 51, 2, 1.0).reshape(M, N)) if residual else None
    ref = x.astype(np.float64) @ w.astype(np.float64).T + (0 if r is None else r.astype(np.float64))
    dev = lambda a: torch.from_numpy(a).to(torch.bfloat16).cuda()
    xd, wd, rd = dev(x), dev(w), None if r is None else dev(r)
    y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.dsk_linear(B.DSK_BF16, xd, wd, y, rd, M, N, K)
    torch.cuda.synchronize()
    # one bf16 rounding of the result
    assert O.max_rel_err(y.float().cpu().numpy(), ref) <= 2 ** -8
    if plan[1] == 1:   # unsplit, every tile height adds in one order
        y256 = torch.full_like(y, float("nan"))
        B.dsk_set_option("gemm_tiling", 1)
        try:
            B.dsk_linear(B.DSK_BF16, xd, wd, y256, rd, M, N, K)
            torch.cuda.synchronize()
        finally:
            B.dsk_set_option("gemm_tiling", 0)
        assert torch.equal(y, y256)


# contractions of one k-tile up to more than the stages of W that a lower tile has (four and three): the bits of the 256-row tiles,
# whose sums have the same order
@pytest.mark.parametrize("K", [64, 128, 192, 256, 320, 384, 448, 512, 576])
@pytest.mark.parametrize("M,N,bm", [(65, 64, 128), (200, 516, 128), (4200, 4612, 192)])
def test_lower_tiles_run_ahead_on_w(B, M, N, bm, K):
    assert B.dsk_gemm_plan(M, N, K, False) == (bm, 1, 0, 0)
    x, w = torch.randn(M, K, device="cuda").bfloat16(), torch.randn(N, K, device="cuda").bfloat16()
    y, y256 = (torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    for tiling, out in ((0, y), (1, y256)):
        B.dsk_set_option("gemm_tiling", tiling)
        try:
            B.dsk_linear(B.DSK_BF16, x, w, out, None, M, N, K)
            torch.cuda.synchronize()
        finally:
            B.dsk_set_option("gemm_tiling", 0)
    # one bf16 rounding of the result
    assert O.max_rel_err(y.float().cpu().numpy(), x.double().cpu().numpy() @ w.double().cpu().numpy().T) <= 2 ** -8
    assert torch.equal(y, y256)


# two layers, so that the split down projection also leaves the next layer's norm input; against the same model with the
# tiling forced (which neither splits nor fuses).  plans: (tile rows, splits) of QKV, O and down: RoPE + KV write with heads
# of 64 and 128 and RMSNorm at widths up to 4096 and beyond in the reduction, every tile height, QKV unsplit
@pytest.mark.parametrize("d,Hq,Hkv,dh,F,rows,plans", [
    (512, 4, 2, 128, 2048, 65, ((128, 1), (128, 1), (128, 8))), (512, 4, 2, 128, 2048, 130, ((128, 1), (128, 1), (128, 8))),
    (512, 4, 2, 128, 2048, 200, ((128, 1), (128, 1), (128, 8))), (512, 4, 2, 128, 2048, 390, ((128, 1), (128, 1), (128, 8))),
    (1088, 17, 1, 64, 1472, 65, ((128, 4), (128, 4), (128, 5))), (1088, 17, 1, 64, 1472, 130, ((128, 4), (128, 4), (128, 5))),
    (1088, 17, 1, 64, 1472, 200, ((128, 4), (128, 4), (128, 5))), (1088, 17, 1, 64, 1472, 390, ((128, 3), (128, 3), (128, 4))),
    (1024, 8, 2, 128, 4096, 65, ((128, 4), (128, 4), (128, 16))), (1024, 8, 2, 128, 4096, 257, ((128, 4), (128, 4), (128, 11))),
    (4096, 32, 8, 128, 14336, 257, ((192, 4), (128, 5), (192, 8))), (4096, 32, 8, 128, 14336, 333, ((128, 3), (128, 5), (192, 8))),
    (4096, 32, 8, 128, 14336, 700, ((256, 3), (192, 4), (256, 5))), (8192, 64, 8, 128, 14336, 130, ((192, 6), (192, 8), (192, 8))),
    (8192, 64, 8, 128, 14336, 400, ((256, 3), (256, 4), (256, 4)))])
def test_layers_with_split_projections(B, d, Hq, Hkv, dh, F, rows, plans):
    from tests import gpu_util as G
    assert tuple(B.dsk_gemm_plan(rows, n, k)[:2] for n, k in (((Hq + 2 * Hkv) * dh, d), (d, Hq * dh), (d, F))) == plans
    shape = synth.ModelShape(2, d, Hq, Hkv, dh, F, 10000.0, 1e-5, "bf16")
    x = G.to_dev(synth.hidden_states(shape, rows), shape)
    with G.GpuModel(shape, rows) as m:
        m.init_random(7)
        kv, h = m.partial(x, 0, 2, None, [rows - 9, 9])
        B.dsk_set_option("gemm_tiling", 2)
        try:
            kv_ref, h_ref = m.partial(x, 0, 2, None, [rows - 9, 9])
            torch.cuda.synchronize()
        finally:
            B.dsk_set_option("gemm_tiling", 0)
    # both are bf16 evaluations of the same layers, each within 1e-2 of the exact ones at this weight scale
    for a, b in ((kv, kv_ref), (h, h_ref)):
        assert O.max_rel_err(G.to_np(a), G.to_np(b).astype(np.float64)) <= 2e-2


# O and down in two launches (residual bf16 and fp32, result fp32 and bf16, two layers): the rows of a call are those of a call
# over fewer of the sequences, which has no second launch, bit for bit
def test_layers_with_projections_in_two_launches(B):
    from tests import gpu_util as G
    shape = synth.ModelShape(2, 2048, 32, 4, 128, 4096, 10000.0, 1e-5, "bf16")
    n, few = 12400, 6000
    assert B.dsk_gemm_plan(n, 2048, 4096)[2:] == (8192, 192) and B.dsk_gemm_plan(few, 2048, 4096)[1:3] == (1, 0)
    assert B.dsk_gemm_plan(few, 5120, 2048)[1] == 1   # and QKV is not split either
    x = G.to_dev(synth.hidden_states(shape, n), shape)
    with G.GpuModel(shape, n) as m:
        m.init_random(17)
        kv, h = m.partial(x, 0, 2, None, [100] * (n // 100))
        for r0 in (0, n - few):   # rows of the first launch, and of both
            kv_few, h_few = m.partial(x[r0:r0 + few].contiguous(), 0, 2, None, [100] * (few // 100))
            torch.cuda.synchronize()
            assert torch.equal(h[r0:r0 + few], h_few) and torch.equal(kv[:, :, r0:r0 + few], kv_few)


# how a contraction is split, and with it the order of its sums, is a matter of the call's sizes alone: the same rows on a
# model that takes no more than them and on one that takes more
@pytest.mark.parametrize("d,F,rows", [(2048, 8192, 500), (4096, 14336, 333), (4096, 14336, 700), (4096, 14336, 1024)])
def test_split_does_not_depend_on_the_models_capacity(B, d, F, rows):
    from tests import gpu_util as G
    shape = synth.ModelShape(1, d, d // 128, d // 512, 128, F, 10000.0, 1e-5, "bf16")
    x = G.to_dev(synth.hidden_states(shape, rows), shape)
    got = []
    for max_tokens in (rows, 4096):
        with G.GpuModel(shape, max_tokens) as m:
            m.init_random(13)
            kv, h = m.partial(x, 0, 1, None, [rows])
            torch.cuda.synchronize()
            got.append((kv, h))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


def test_linear_does_not_depend_on_earlier_calls(B):
    # the first wide call of the process makes the shared scratch grow
    M, N, K = 400, 4096, 14336
    x, w, wide = (torch.randn(n, k, device="cuda").to(torch.bfloat16) for n, k in ((M, K), (N, K), (60000, 64)))
    y = [torch.empty((M, N), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    B.dsk_linear(B.DSK_BF16, x, w, y[0], None, M, N, K)
    B.dsk_linear(B.DSK_BF16, x[:, :64].contiguous(), wide, torch.empty((M, 60000), dtype=torch.bfloat16, device="cuda"), None, M, 60000, 64)
    B.dsk_linear(B.DSK_BF16, x, w, y[1], None, M, N, K)
    torch.cuda.synchronize()
    assert torch.equal(y[0], y[1])


# the router on the matrix cores: token counts around multiples of 16, one to four blocks of experts, contractions shorter
# and longer than the steps in flight, a row of NaN; the choice must be one of the best by more than fp32 sums can differ
@pytest.mark.parametrize("n,d,E,k", [(65, 32, 2, 1), (80, 320, 16, 2), (100, 4096, 17, 8), (129, 1056, 33, 3), (70, 2080, 64, 8)])
def test_router_on_the_matrix_cores(B, n, d, E, k):
    bf = lambda a: synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(a))
    x, w = bf(synth.normal(n * d, 61, 0, 1.0).reshape(n, d)), bf(synth.normal(E * d, 61, 1, 0.05).reshape(E, d))
    x[3] = np.nan
    w[E - 1] = w[0]   # equal logits: the lower index goes first
    dev = lambda a: torch.from_numpy(a).to(torch.bfloat16).cuda()
    experts = torch.full((n, k), -7, dtype=torch.int32, device="cuda")
    gates = torch.full((n, k), float("nan"), device="cuda")
    B.dsk_moe_route(B.DSK_BF16, dev(x), dev(w), n, d, E, k, experts, gates)
    torch.cuda.synchronize()
    experts, gates = experts.cpu().numpy(), gates.cpu().numpy()
    logits = x.astype(np.float64) @ w.astype(np.float64).T
    assert np.all(np.sort(experts, axis=1)[:, 1:] != np.sort(experts, axis=1)[:, :-1]) and experts.min() >= 0 and experts.max() < E
    for t in range(n):
        if t == 3:
            continue
        got, best = logits[t, experts[t]], np.sort(logits[t])[::-1][:k]
        # fp32 sums of d products: 2^-24 sqrt(d) of their scale, far below 1e-4
        assert np.abs(got - best).max() <= 1e-4
        assert np.abs(gates[t] - np.exp(got - got[0]) / np.exp(got - got[0]).sum()).max() <= 1e-4
        if 0 in experts[t] and E - 1 in experts[t]:
            assert list(experts[t]).index(0) < list(experts[t]).index(E - 1)
        assert not (E - 1 in experts[t] and 0 not in experts[t])


# RoPE + KV write in the epilogue of an unsplit QKV projection (heads of 128): every tile height, a last column tile that is
# half full, rows that end inside a tile, whole rounds and a rest in two launches; against the same model with
# the tiling forced, where the rotation is a pass of its own over the rounded projection
@pytest.mark.parametrize("d,Hq,lens,plan", [
    (128, 3, [65], (128, 1, 0, 0)), (128, 3, [150, 1], (128, 1, 0, 0)), (128, 3, [500, 140], (128, 1, 0, 0)),
    (128, 3, [1000] * 11, (192, 1, 0, 0)), (128, 3, [1000] * 17 + [30], (256, 1, 0, 0)),
    (2048, 25, [200] * 55 + [30], (256, 1, 9216, 128)), (4096, 25, [200] * 35 + [30], (256, 1, 4608, 192))])
def test_rope_in_the_projection(B, d, Hq, lens, plan):
    assert B.dsk_gemm_plan(sum(lens), (Hq + 2) * 128, d) == plan
    from tests import gpu_util as G
    shape = synth.ModelShape(1, d, Hq, 1, 128, 128, 10000.0, 1e-5, "bf16")
    x = G.to_dev(synth.hidden_states(shape, sum(lens)), shape)
    with G.GpuModel(shape, sum(lens)) as m:
        m.init_random(9)
        kv, h = m.partial(x, 0, 1, None, lens)
        B.dsk_set_option("gemm_tiling", 2)
        try:
            kv_ref, h_ref = m.partial(x, 0, 1, None, lens)
            torch.cuda.synchronize()
        finally:
            B.dsk_set_option("gemm_tiling", 0)
    # k: one rounding here, up to two of each of the pair's elements there (2^-9 each); v and the state: one each
    for a, b in ((kv, kv_ref), (h, h_ref)):
        assert O.max_rel_err(G.to_np(a), G.to_np(b).astype(np.float64)) <= 2 ** -7


# unsplit 256-row tiles of short contractions: one to five and 17 k-tiles, last column tiles that end early, rows that end inside a
# tile; QKV with the rotation, O with residual, gate/up with SwiGLU, down, with weights with which a k-tile left out of any
# of them shows in the state (a tenth of it and more).  Against the 128-row tiles of the other kernel.
@pytest.mark.parametrize("d,Hq,F,n", [(64, 3, 128, 18030), (128, 3, 320, 18030), (192, 5, 192, 13001), (320, 3, 1088, 18030)])
def test_unsplit_256_row_tiles(B, d, Hq, F, n):
    from tests import gpu_util as G
    assert B.dsk_gemm_plan(n, (Hq + 2) * 128, d)[:2] == (256, 1)
    shape = synth.ModelShape(1, d, Hq, 1, 128, F, 10000.0, 1e-5, "bf16")
    lens = [250] * (n // 250) + [n % 250]
    x = G.to_dev(synth.hidden_states(shape, n), shape)
    with G.GpuModel(shape, n) as m:
        m.init_random(19, std=0.1)
        for t, rows in ((B.DSK_WQ, Hq * 128), (B.DSK_WK, 128)):
            w = synth.normal(rows * d, 19, t, 0.02).reshape(rows, d)
            B.dsk_model_set_tensor(m.handle, 0, t, G.to_dev(w, shape))
        B.dsk_set_option("gemm_tiling", 1)   # 256-row tiles for every projection; the rotation is a pass of its own
        try:
            forced = m.partial(x, 0, 1, None, lens)
            B.dsk_set_option("gemm_tiling", 2)
            ref = m.partial(x, 0, 1, None, lens)
            torch.cuda.synchronize()
        finally:
            B.dsk_set_option("gemm_tiling", 0)
        planned = m.partial(x, 0, 1, None, lens)
        torch.cuda.synchronize()
    # as above: up to two roundings of 2^-9 for each of a pair's elements, one for v and the state.  The roundings of q and k reach the
    # state as changes of a score: with wq and wk at 0.02 a score is the mean of 128 products of at most 0.36 x 0.36 in the mean
    # square, times sqrt(128), so 1.5 in the mean square at most and its error 1.5 * 2^-8 / sqrt(128), a tenth of a rounding (at 0.1
    # scores are 25 times that); those in front of down as a mean over F columns.
    for got in (forced, planned):
        for a, b in zip(got, ref):
            assert O.max_rel_err(G.to_np(a), G.to_np(b).astype(np.float64)) <= 2 ** -7


def _count_direct(B, m, x, lens):
    B.dsk_set_option("reset_stats", 0)
    out = m.partial(x[:sum(lens)].contiguous(), 0, 1, None, lens)
    torch.cuda.synchronize()
    return (*out, B.dsk_get_stat("gemm_direct_launches"))


# Unsplit 256-row tiles with W straight to registers add in the order of every other tile of that kernel: the rows of a call that
# takes them are those of a call over fewer sequences that does not, bit for bit, with weights that make the MLP the larger part
# of the state.  On both sides of the rule's lines: QKV, O and down past 256 rows (contractions of 57, 58 and 59 k-tiles, of 64,
# 56 and 56), gate/up from 1536 rows on at 8192 and from 2^25 elements on below (128, 129, 65 k-tiles, a last column tile that
# ends early); no launch at a contraction of 3520, nor for gate/up over the 512 rows of an 8B layer.
@pytest.mark.parametrize("d,Hq,F,n,few,unit,launches", [
    (3648, 29, 3776, 300, 256, 64, (3, 0)), (4096, 28, 3584, 300, 256, 64, (3, 0)), (3520, 5, 64, 300, 256, 64, (0, 0)),
    (8192, 3, 192, 1536, 1500, 100, (2, 1)), (8256, 3, 320, 1536, 1500, 100, (2, 1)), (4160, 3, 192, 8100, 8000, 100, (2, 1)),
    (4096, 3, 64, 512, 500, 100, (1, 1))])
def test_weights_straight_to_registers(B, d, Hq, F, n, few, unit, launches):
    from tests import gpu_util as G
    shape = synth.ModelShape(1, d, Hq, 1, 128, F, 10000.0, 1e-5, "bf16")
    lens = [unit] * (n // unit) + [n % unit] * (n % unit > 0)
    assert few % unit == 0
    x = torch.randn((n, d), generator=torch.Generator(device="cuda").manual_seed(19), device="cuda").to(torch.bfloat16)
    with G.GpuModel(shape, n) as m:
        m.init_random(19, std=0.1)
        B.dsk_set_option("gemm_tiling", 1)   # 256-row tiles for every projection; the rotation is a pass of its own
        try:
            kv, h, got = _count_direct(B, m, x, lens)
            kv_few, h_few, got_few = _count_direct(B, m, x, [unit] * (few // unit))
        finally:
            B.dsk_set_option("gemm_tiling", 0)
    assert (got, got_few) == launches and torch.isfinite(h).all()
    assert torch.equal(h[:few], h_few) and torch.equal(kv[:, :, :few], kv_few)


# ... and QKV with the rotation, as planned: 57 and 64 k-tiles of 256-row tiles, against 192-row tiles of the other form
@pytest.mark.parametrize("d,n,few,launches", [(3648, 4000, 2500, (2, 0)), (4096, 4000, 2500, (2, 0))])
def test_rotation_with_weights_straight_to_registers(B, d, n, few, launches):
    from tests import gpu_util as G
    Hq, F = 28, 128
    assert B.dsk_gemm_plan(n, (Hq + 2) * 128, d, False) == (256, 1, 0, 0) and B.dsk_gemm_plan(few, (Hq + 2) * 128, d, False)[0] == 192
    assert B.dsk_gemm_plan(n, d, Hq * 128)[1] == B.dsk_gemm_plan(few, d, Hq * 128)[1] == 1   # nor is O split
    shape = synth.ModelShape(1, d, Hq, 1, 128, F, 10000.0, 1e-5, "bf16")
    x = torch.randn((n, d), generator=torch.Generator(device="cuda").manual_seed(20), device="cuda").to(torch.bfloat16)
    with G.GpuModel(shape, n) as m:
        m.init_random(20, std=0.1)
        kv, h, got = _count_direct(B, m, x, [100] * (n // 100))
        kv_few, h_few, got_few = _count_direct(B, m, x, [100] * (few // 100))
    assert (got, got_few) == launches and torch.isfinite(h).all()
    assert torch.equal(h[:few], h_few) and torch.equal(kv[:, :, :few], kv_few)


# ... and over experts (every token chooses both) of more than 256 rows in the mean: gate/up of 56 and 65 k-tiles, down of 65 and
# 56, rows of another expert behind the last tile of the first, one scheduling group an expert and three
@pytest.mark.parametrize("d,F,n", [(3584, 4160, 300), (4160, 3584, 300), (3584, 3584, 7040)])
def test_expert_weights_straight_to_registers(B, d, F, n):
    from tests import gpu_util as G
    few = 256
    shape = synth.ModelShape(1, d, 2, 1, 64, F, 10000.0, 1e-5, "bf16", 2, 2)
    lens = [64] * (n // 64) + [n % 64] * (n % 64 > 0)
    x = torch.randn((n, d), generator=torch.Generator(device="cuda").manual_seed(23), device="cuda").to(torch.bfloat16)
    with G.GpuModel(shape, n) as m:
        m.init_random(23, std=0.1)
        B.dsk_set_option("gemm_tiling", 1)   # (of the other projections)
        try:
            kv, h, got = _count_direct(B, m, x, lens)
            kv_few, h_few, got_few = _count_direct(B, m, x, [64] * (few // 64))
        finally:
            B.dsk_set_option("gemm_tiling", 0)
    assert (got, got_few) == (3, 0) and torch.isfinite(h).all()
    assert torch.equal(h[:few], h_few) and torch.equal(kv[:, :, :few], kv_few)


# experts in tiles of 256 rows with W through LDS: one, three and five k-tiles, an expert's tiles in one scheduling group and in
# three, against the plain kernels
@pytest.mark.parametrize("d,F,n", [(64, 192, 601), (320, 128, 601), (192, 320, 601), (128, 128, 7001)])
def test_expert_tiles_of_256_rows(B, d, F, n):
    from tests import gpu_util as G
    shape = synth.ModelShape(1, d, 2, 1, 64, F, 10000.0, 1e-5, "bf16", 2, 2)
    x = G.to_dev(synth.hidden_states(shape, n), shape)
    with G.GpuModel(shape, n) as m:
        m.init_random(23, 0.05)
        kv, h = m.partial(x, 0, 1, None, [n])
        B.dsk_set_option("force_generic", 1)
        try:
            kv_ref, h_ref = m.partial(x, 0, 1, None, [n])
            torch.cuda.synchronize()
        finally:
            B.dsk_set_option("force_generic", 0)
    # two bf16 evaluations of one layer
    for a, b in ((kv, kv_ref), (h, h_ref)):
        assert O.max_rel_err(G.to_np(a), G.to_np(b).astype(np.float64)) <= 1e-2
