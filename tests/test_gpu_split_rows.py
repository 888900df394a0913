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


# row-major weights through the component call: rows around multiples of 128, 192 and 256, columns that end inside a tile,
# contractions of a few k-tiles (unsplit) and many (split with an uneven last share), and more than one round of tiles
@pytest.mark.parametrize("M,N,K,residual", [(65, 64, 64, False), (129, 516, 320, True), (191, 1028, 1984, False),
                                            (193, 256, 4096, True), (257, 2052, 1024, True), (385, 512, 8192, False),
                                            (1025, 1024, 2048, True), (2000, 2560, 256, False), (3000, 5000, 192, True),
                                            (4200, 4612, 128, True)])   # whole rounds and a rest, in two launches
def test_linear_bf16_medium_rows(B, M, N, K, residual):
    bf = lambda a: synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(a))
    x = bf(synth.normal(M * K, 51, 0, 1.0).reshape(M, K))
    w = bf(synth.normal(N * K, 51, 1, 0.05).reshape(N, K))
    r = bf(synth.normal(M * N, 51, 2, 1.0).reshape(M, N)) if residual else None
    ref = x.astype(np.float64) @ w.astype(np.float64).T + (0 if r is None else r.astype(np.float64))
    dev = lambda a: torch.from_numpy(a).to(torch.bfloat16).cuda()
    y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.dsk_linear(B.DSK_BF16, dev(x), dev(w), y, None if r is None else dev(r), M, N, K)
    torch.cuda.synchronize()
    # one bf16 rounding of the result
    assert O.max_rel_err(y.float().cpu().numpy(), ref) <= 2 ** -8


# two layers, so that the split down projection also leaves the next layer's norm input; dh 64 and 128; against the same
# model with the tiling forced (which neither splits nor fuses)
@pytest.mark.parametrize("rows", [65, 130, 200, 390])
@pytest.mark.parametrize("d,Hq,Hkv,dh,F", [(512, 4, 2, 128, 2048), (1088, 17, 1, 64, 1472)])
def test_layers_with_split_projections(B, rows, d, Hq, Hkv, dh, F):
    from tests import gpu_util as G
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
# half full, rows that end inside a tile, whole rounds and a rest in two launches (22000 rows); against the same model with
# the tiling forced, where the rotation is a pass of its own over the rounded projection
@pytest.mark.parametrize("lens", [[65], [150, 1], [300], [500, 140], [1000] * 22])
def test_rope_in_the_projection(B, lens):
    from tests import gpu_util as G
    shape = synth.ModelShape(1, 128, 3, 1, 128, 128, 10000.0, 1e-5, "bf16")
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
