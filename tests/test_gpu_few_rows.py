"""The few-row projections (activations and weights in blocks) at the edges of their tilings: row counts around multiples of
16, every row tiling, narrow and odd widths, a contraction split over workgroups, against the plain kernels and the oracle."""
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


# d = 64 (four sums of squares a row), widths that are odd multiples of 64, dh 64 and 128
@pytest.mark.parametrize("rows", [1, 15, 16, 17, 33, 48, 49, 64])
@pytest.mark.parametrize("d,Hq,Hkv,dh,F", [(64, 1, 1, 64, 64), (448, 7, 1, 64, 832), (512, 6, 2, 128, 320)])
def test_layers_over_few_rows_match_the_oracle(B, rows, d, Hq, Hkv, dh, F):
    from tests import gpu_util as G
    from tests.helpers import kv_list, oracle_config, weights_fn
    shape = synth.ModelShape(2, d, Hq, Hkv, dh, F, 10000.0, 1e-5, "bf16")
    lens = [rows] if rows < 3 else [rows - 2, 2]
    x = synth.hidden_states(shape, rows)
    with G.GpuModel(shape, rows) as m:   # the workspace is sized for exactly these rows
        m.load_from_generator(3)
        B.dsk_set_option("reset_stats", 0)
        kv, h = m.partial(G.to_dev(x, shape), 0, 2, None, lens)
        torch.cuda.synchronize()
        assert B.dsk_get_stat("gemm_mfma_launches") == 8 and B.dsk_get_stat("gemm_generic_launches") == 0
        w = m.get_tensor(1, synth.WU)    # blocks and back
        assert np.array_equal(G.to_np(w), synth.layer_tensor(shape, 3, 1, synth.WU))
    kv_ref, h_ref = O.partial_prefill(oracle_config(shape), weights_fn(shape, 3), x.astype(np.float64), 0, 2,
                                      [(None, None)] * 2, synth.packed_positions(lens), synth.cu_seqlens(lens))
    # the bound of the bf16 path at this weight scale
    assert O.max_rel_err(G.to_np(h), h_ref) <= 2e-2
    for l in range(2):
        assert O.max_rel_err(G.to_np(kv[l, 0]), kv_ref[l][0]) <= 2e-2 and O.max_rel_err(G.to_np(kv[l, 1]), kv_ref[l][1]) <= 2e-2


@pytest.mark.parametrize("rows", [40, 64])
def test_split_contraction_matches_the_unsplit_one(B, rows):
    # the down projection's 256 column tiles would read 48 or 64 rows of 28672 each, more than 256 MB, so it is split over
    # workgroups; the same rows one at a time take the unsplit kernel.  The order of fp32 sums differs, and with it now and
    # then a bf16 rounding (2^-9) of an intermediate: a few of those on the way to a result.
    from tests import gpu_util as G
    shape = synth.ModelShape(1, 4096, 32, 8, 128, 28672, 500000.0, 1e-5, "bf16")
    x = G.to_dev(synth.hidden_states(shape, rows), shape)
    with G.GpuModel(shape, rows) as m:
        m.init_random(0)
        _, h = m.partial(x, 0, 1, None, [1] * rows)
        singles = [m.partial(x[i:i + 1].contiguous(), 0, 1, None, [1], positions=np.zeros(1, np.int32))[1].clone() for i in (0, 17, rows - 1)]
        torch.cuda.synchronize()
    for i, one in zip((0, 17, rows - 1), singles):
        assert O.max_rel_err(G.to_np(h[i:i + 1]), G.to_np(one).astype(np.float64)) <= 2 ** -6


# experts without a token (9 choices over 64 experts, a single token), one choice, several tokens, row tilings 1 to 4; an
# expert count that is no multiple of the router's eight; and beyond 64 rows the grouped projections on each tile height
# (about 17, 120, 140 and 300 rows an expert) with the matrix-core router over one, two and four blocks of experts
@pytest.mark.parametrize("rows,E,k", [(1, 8, 2), (3, 64, 3), (17, 5, 1), (40, 9, 4), (64, 8, 2),
                                      (70, 17, 4), (300, 5, 2), (350, 5, 2), (600, 4, 2), (900, 40, 3)])
def test_expert_layers_match_the_plain_kernels(B, rows, E, k):
    from tests import gpu_util as G
    shape = synth.ModelShape(1, 320, 5, 1, 64, 192, 10000.0, 1e-5, "bf16", E, k)
    with G.GpuModel(shape, rows) as m:
        m.init_random(5, std=0.05)
        # a part along one router row per token, so that the choice of experts does not hang on rounding
        wr = G.to_np(m.get_tensor(0, synth.WR))
        x = synth.hidden_states(shape, rows)
        for j in range(k):
            x += (9.0 - 1.5 * j) * wr[(np.arange(rows) * 3 + 5 * j) % E] / np.linalg.norm(wr, axis=1).mean()
        x = G.to_dev(x, shape)
        kv, h = m.partial(x, 0, 1, None, [rows])
        B.dsk_set_option("force_generic", 1)
        try:
            kv_ref, h_ref = m.partial(x, 0, 1, None, [rows])
            torch.cuda.synchronize()
        finally:
            B.dsk_set_option("force_generic", 0)
    # two bf16 evaluations of one layer: each within 1e-2 of the exact one at this weight scale
    assert O.max_rel_err(G.to_np(h), G.to_np(h_ref).astype(np.float64)) <= 2e-2
    assert O.max_rel_err(G.to_np(kv[0]), G.to_np(kv_ref[0]).astype(np.float64)) <= 2e-2


# activations of up to eight rows stand in rows, of more in blocks: the same sums in the same order, bit for bit; a single
# row, the most rows, dense and expert layers, an odd number of 64-column steps
@pytest.mark.parametrize("d,Hq,Hkv,dh,F,E", [(448, 7, 1, 64, 832, 0), (512, 6, 2, 128, 320, 0), (320, 5, 1, 64, 192, 5)])
def test_activations_in_rows_and_in_blocks_agree(B, d, Hq, Hkv, dh, F, E):
    from tests import gpu_util as G
    shape = synth.ModelShape(2, d, Hq, Hkv, dh, F, 10000.0, 1e-5, "bf16", E, 2 if E else 0)
    x = G.to_dev(synth.hidden_states(shape, 9), shape)
    with G.GpuModel(shape, 9) as m:
        m.init_random(5, std=0.05)
        kv, h = m.partial(x, 0, 2, None, [1] * 9)
        for r0, n in ((0, 8), (8, 1), (3, 5)):
            kv_n, h_n = m.partial(x[r0:r0 + n].contiguous(), 0, 2, None, [1] * n)
            torch.cuda.synchronize()
            assert torch.equal(h[r0:r0 + n], h_n) and torch.equal(kv[:, :, r0:r0 + n], kv_n)


# three to seven steps a wave, waves that differ by one: the loop and the steps behind it, one to four row tiles, against the
# plain kernels
@pytest.mark.parametrize("rows", [1, 9, 30, 46, 64])
@pytest.mark.parametrize("d,F", [(1536, 1984), (2048, 2112), (2624, 3136)])
def test_steps_behind_the_loop(B, rows, d, F):
    from tests import gpu_util as G
    shape = synth.ModelShape(1, d, d // 64, 1, 64, F, 10000.0, 1e-5, "bf16")
    x = G.to_dev(synth.hidden_states(shape, rows), shape)
    with G.GpuModel(shape, rows) as m:
        m.init_random(11)
        kv, h = m.partial(x, 0, 1, None, [rows])
        B.dsk_set_option("force_generic", 1)
        try:
            kv_ref, h_ref = m.partial(x, 0, 1, None, [rows])
            torch.cuda.synchronize()
        finally:
            B.dsk_set_option("force_generic", 0)
    # two bf16 evaluations of one layer, each within 1e-2 of the exact one at this weight scale
    assert O.max_rel_err(G.to_np(h), G.to_np(h_ref).astype(np.float64)) <= 2e-2
    assert O.max_rel_err(G.to_np(kv[0]), G.to_np(kv_ref[0]).astype(np.float64)) <= 2e-2


# the wider tiles of 9 to 64 rows: experts enough for 256 workgroups of 64 and 128 columns (one to four row tiles), a dense gate/up of
# 192 tiles and down split over workgroups at 17 to 32 rows, O split from 17 rows on (8192 wide) and from 49 on (5120); against the plain
# kernels
@pytest.mark.parametrize("rows", [9, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("d,F,E", [(2048, 1600, 16), (256, 12352, 0), (2048, 28736, 0), (8192, 64, 0), (5120, 64, 0)])
def test_wide_tiles_of_few_rows(B, rows, d, F, E):
    from tests import gpu_util as G
    shape = synth.ModelShape(1, d, d // 128, 1, 128, F, 10000.0, 1e-5, "bf16", E, 1 if E else 0)
    with G.GpuModel(shape, rows) as m:
        m.init_random(11)
        x = synth.hidden_states(shape, rows)
        if E:  # a part along one router row per token, so that the choice of experts does not hang on rounding
            wr = G.to_np(m.get_tensor(0, synth.WR))
            x += 9.0 * wr[np.arange(rows) * 3 % E] / np.linalg.norm(wr, axis=1).mean()
        x = G.to_dev(x, shape)
        kv, h = m.partial(x, 0, 1, None, [rows])
        B.dsk_set_option("force_generic", 1)
        try:
            kv_ref, h_ref = m.partial(x, 0, 1, None, [rows])
            torch.cuda.synchronize()
        finally:
            B.dsk_set_option("force_generic", 0)
    # two bf16 evaluations of one layer, each within 1e-2 of the exact one at this weight scale
    assert O.max_rel_err(G.to_np(h), G.to_np(h_ref).astype(np.float64)) <= 2e-2
    assert O.max_rel_err(G.to_np(kv[0]), G.to_np(kv_ref[0]).astype(np.float64)) <= 2e-2
