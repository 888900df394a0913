"""The fp32 matrix-instruction kernels at the edges of their tilings, against float64."""
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


# 16 x 32 tiles with the contraction over eight waves (first five: one chunk, a ragged chunk, fewer chunks than waves),
# 32 x 64 tiles (600 x 1400), 128 x 128 tiles (2100 x 2052); rows of 4-element granularity, and the plain kernel
# beyond it (K = 42, N = 37).  A sum of K products of N(0,1) x N(0,0.05) has max-abs error <= about
# 5 sqrt(K) 2^-24 of its scale: below 1e-5 for K <= 700.
@pytest.mark.parametrize("M,N,K", [(1, 4, 4), (17, 36, 20), (16, 32, 128), (130, 260, 700), (45, 1376, 256), (600, 1400, 100),
                                   (2100, 2052, 36), (33, 40, 42), (33, 37, 40)])
@pytest.mark.parametrize("residual", [False, True])
def test_linear_fp32_tilings(B, M, N, K, residual):
    x = synth.normal(M * K, 31, 0, 1.0).reshape(M, K)
    w = synth.normal(N * K, 31, 1, 0.05).reshape(N, K)
    r = synth.normal(M * N, 31, 2, 1.0).reshape(M, N) if residual else None
    ref = x.astype(np.float64) @ w.astype(np.float64).T + (0 if r is None else r)
    y = torch.full((M, N), float("nan"), device="cuda")
    B.dsk_linear(B.DSK_F32, torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), y,
                 None if r is None else torch.from_numpy(r).cuda(), M, N, K)
    torch.cuda.synchronize()
    assert O.max_rel_err(y.cpu().numpy(), ref) <= 1e-5


def _attention(B, q, k, v, lens, plens, own_row0, Hq, Hkv, dh):
    qb, pb = B.Batch(synth.cu_seqlens(lens)), B.Batch(synth.cu_seqlens(plens)) if plens else None
    out = torch.full((sum(lens), Hq * dh), float("nan"), device="cuda")
    B.dsk_attention(B.DSK_F32, *[torch.from_numpy(t).cuda() for t in (q, k, v)], out, qb.desc, None if pb is None else pb.desc,
                    own_row0, Hq, Hkv, dh)
    torch.cuda.synchronize()
    return out.cpu().numpy().reshape(-1, Hq, dh)


# ragged query tiles (16), key chunks (32) and waves without a chunk; head_dim 96 stays on the plain kernel
@pytest.mark.parametrize("dh", [64, 128, 96])
@pytest.mark.parametrize("lens,plens", [([1], None), ([17, 1, 40], None), ([200], None), ([5, 18], [33, 150])])
def test_attention_fp32(B, lens, plens, dh):
    _attention_against_float64(B, lens, plens, dh)


# on both sides of the lines between four and eight waves: 128 keys; 256 workgroups (heads of 64), 4 heads a tile of 16 queries
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("lens,plens", [([128], None), ([129], None), ([16] * 64, [113] * 64), ([16] * 64 + [1], [113] * 65),
                                        ([3, 20], [300, 1])])
def test_attention_fp32_four_and_eight_waves(B, lens, plens, dh):
    _attention_against_float64(B, lens, plens, dh)


def _attention_against_float64(B, lens, plens, dh):
    Hq, Hkv = 4, 2
    n, n_pre = sum(lens), sum(plens or [])
    own0 = n_pre + 3 if plens else 0
    q = synth.normal(n * Hq * dh, 32, 0, 1.0).reshape(n, Hq, dh)
    k, v = (synth.normal((own0 + n) * Hkv * dh, 32, j, 1.0).reshape(-1, Hkv, dh) for j in (1, 2))
    ref = np.empty((n, Hq, dh))
    cu, pcu = synth.cu_seqlens(lens), synth.cu_seqlens(plens) if plens else None
    for b in range(len(lens)):
        for i in range(cu[b], cu[b + 1]):
            vis = (list(range(pcu[b], pcu[b + 1])) if plens else []) + list(range(own0 + cu[b], own0 + i + 1))
            ref[i] = O.attend_row(*(t.astype(np.float64) for t in (q[i], k[vis], v[vis])))
    assert O.max_rel_err(_attention(B, q, k, v, lens, plens, own0, Hq, Hkv, dh), ref) <= 1e-5


def test_attention_fp32_rows_that_are_not_finite_reach_later_queries_only(B):
    _rows_that_are_not_finite(B, 50, 37)


def test_attention_fp32_rows_that_are_not_finite_eight_waves(B):
    _rows_that_are_not_finite(B, 150, 133)


def _rows_that_are_not_finite(B, n, bad):
    Hq, Hkv, dh = 4, 2, 64
    q = synth.normal(n * Hq * dh, 33, 0, 1.0).reshape(n, Hq, dh)
    k, v = (synth.normal(n * Hkv * dh, 33, j, 1.0).reshape(n, Hkv, dh) for j in (1, 2))
    clean = _attention(B, q, k, v, [n], None, 0, Hq, Hkv, dh)
    k[bad], v[bad] = np.inf, np.nan
    got = _attention(B, q, k, v, [n], None, 0, Hq, Hkv, dh)
    # the sums of the queries that see only finite rows are the same up to their order
    assert np.abs(got[:bad] - clean[:bad]).max() <= 1e-5 * np.abs(clean).max() and np.isnan(got[bad:]).all()


# RMSNorm, RoPE + KV write and SwiGLU on the projections: widths with ragged chunks, gate/up blocks of 16 and 32, and
# blocks of 8 (F = 40) and a head_dim of 48, which take the separate steps; enough rows for each tiling
@pytest.mark.parametrize("rows,d,Hq,Hkv,dh,F", [(21, 68, 2, 1, 64, 80), (9, 72, 2, 2, 32, 96), (9, 72, 2, 1, 48, 40),
                                                (300, 512, 8, 2, 64, 1376), (1100, 512, 16, 8, 128, 2048)])
def test_layer_fp32_fused_steps_match_the_plain_kernels(B, rows, d, Hq, Hkv, dh, F):
    from tests import gpu_util as G
    shape = synth.ModelShape(2, d, Hq, Hkv, dh, F, 10000.0, 1e-5, "f32")
    x = G.to_dev(synth.hidden_states(shape, rows), shape)
    with G.GpuModel(shape, rows) as m:
        m.init_random(3, std=0.05)
        kv, h = m.partial(x, 0, 2, None, [rows - 4, 4])
        B.dsk_set_option("force_generic", 1)
        try:
            kv_ref, h_ref = m.partial(x, 0, 2, None, [rows - 4, 4])
            torch.cuda.synchronize()
        finally:
            B.dsk_set_option("force_generic", 0)
    # two evaluations in fp32 of the same layers: a few sums of at most 2048 terms each
    for a, b in ((kv, kv_ref), (h, h_ref)):
        assert O.max_rel_err(G.to_np(a), G.to_np(b).astype(np.float64)) <= 2e-5


# where the tile narrows to eight columns of either side (256 workgroups; QKV, then gate/up, on both sides of it), and 32-row
# tiles, each with the rotary table filled by the first layer's projection and read by the second's
@pytest.mark.parametrize("rows,d,Hq,Hkv,dh,F", [(128, 64, 4, 2, 64, 688), (129, 64, 4, 2, 64, 96), (256, 64, 1, 1, 32, 128),
                                                (257, 64, 1, 1, 32, 128), (600, 128, 16, 8, 128, 128)])
def test_layer_fp32_narrow_tiles(B, rows, d, Hq, Hkv, dh, F):
    from tests import gpu_util as G
    shape = synth.ModelShape(2, d, Hq, Hkv, dh, F, 10000.0, 1e-5, "f32")
    x = G.to_dev(synth.hidden_states(shape, rows), shape)
    with G.GpuModel(shape, rows) as m:
        m.init_random(3, std=0.05)
        kv, h = m.partial(x, 0, 2, None, [rows - 4, 4])
        B.dsk_set_option("force_generic", 1)
        try:
            kv_ref, h_ref = m.partial(x, 0, 2, None, [rows - 4, 4])
            torch.cuda.synchronize()
        finally:
            B.dsk_set_option("force_generic", 0)
    # two evaluations in fp32 of the same layers: a few sums of at most 688 terms each
    for a, b in ((kv, kv_ref), (h, h_ref)):
        assert O.max_rel_err(G.to_np(a), G.to_np(b).astype(np.float64)) <= 2e-5
