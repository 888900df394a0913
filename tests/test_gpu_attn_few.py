"""Attention of few queries against a long cache at the edges of its tilings, against the oracle."""
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


# columns (queries x heads of a group) on both sides of 16, 64 and 128; one, three (no power of two) and eight heads per
# group; keys on both sides of a 32-key step and of a stage, key ranges cut through prefix and own rows; ragged
# sequences; through a model, so that the key split has its workspace and the result goes out in blocks or rows
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("Hq,Hkv", [(4, 1), (2, 2), (6, 2), (16, 2)])
@pytest.mark.parametrize("lens,plens", [([1], [31]), ([4], [4000]), ([5], [700]), ([16], [95]), ([17, 1], [300, 1500]),
                                        ([33], [1000]), ([64, 64], [129, 640]), ([128, 100, 7], [900, 2300, 130])])
def test_attention_few_queries(B, Hq, Hkv, dh, lens, plens):
    from tests import gpu_util as G
    from tests.helpers import kv_list, oracle_config, weights_fn
    shape = synth.ModelShape(1, 128, Hq, Hkv, dh, 128, 10000.0, 1e-5, "bf16")
    T, S = sum(plens), sum(lens)
    kv = synth.kv_cache(shape, T)
    xs = synth.hidden_states(shape, S, seed=synth.SEED_SUFFIX)
    cache = torch.full((1, 2, T + 2 + S, Hkv, dh), float("nan"), dtype=torch.bfloat16, device="cuda")
    cache[:, :, :T] = G.to_dev(kv, shape)   # two rows between the prefix and the own rows stay NaN
    with G.GpuModel(shape, S, T + 2 + S) as m:
        m.load_from_generator(0, scale=8.0)
        B.dsk_set_option("reset_stats", 0)
        h = m.suffix(G.to_dev(xs, shape), cache, plens, lens, suffix_row0=T + 2)
        torch.cuda.synchronize()
        assert B.dsk_get_stat("attn_mfma_launches") == 1
    base = weights_fn(shape, 0)
    scaled = lambda l: {k: (v if k in ("g1", "g2") else (v.astype(np.float32) * np.float32(8.0)).astype(np.float64))
                        for k, v in base(l).items()}
    _, ref = O.suffix_prefill(oracle_config(shape), scaled, xs.astype(np.float64), kv_list(kv),
                              synth.packed_positions(lens, start=plens), synth.cu_seqlens(plens), synth.cu_seqlens(lens))
    # one layer, attention output a fair part of it at this weight scale; the bound of the bf16 path
    assert O.max_rel_err(G.to_np(h), ref) <= 2e-2


def test_attention_few_queries_component_call(B):
    # rows out, no workspace (one key range per workgroup), peaked scores
    Hq, Hkv, dh, n, pre = 8, 2, 128, 40, 500
    bf = lambda a: synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(a))
    q = bf(synth.normal(n * Hq * dh, 41, 0, 3.0).reshape(n, Hq, dh))
    k = bf(synth.normal((pre + n) * Hkv * dh, 41, 1, 2.0).reshape(-1, Hkv, dh))
    v = bf(synth.normal((pre + n) * Hkv * dh, 41, 2, 1.0).reshape(-1, Hkv, dh))
    ref = np.stack([O.attend_row(*(t.astype(np.float64) for t in (q[i], k[:pre + i + 1], v[:pre + i + 1]))) for i in range(n)])
    dev = lambda a: torch.from_numpy(a).to(torch.bfloat16).cuda()
    out = torch.empty((n, Hq * dh), dtype=torch.bfloat16, device="cuda")
    scratch = torch.empty(Hkv * dh * ((pre + n + 63) // 64 * 64), dtype=torch.bfloat16, device="cuda")
    qb, pb = B.Batch(synth.cu_seqlens([n])), B.Batch(synth.cu_seqlens([pre]))
    B.dsk_attention(B.DSK_BF16, dev(q), dev(k), dev(v), out, qb.desc, pb.desc, pre, Hq, Hkv, dh, scratch)
    torch.cuda.synchronize()
    # rounding of the probabilities and of the result: 2^-9 each
    assert O.max_rel_err(out.float().cpu().numpy().reshape(n, Hq, dh), ref) <= 1e-2


# prefixes that end on both sides of a stage of 128 keys, from one stage to more than the ring holds: stages wholly inside the prefix
# are loaded another way than those that reach past it; every column form, a second sequence whose rows start elsewhere
@pytest.mark.parametrize("pre", [1, 127, 128, 129, 255, 256, 257, 511, 512, 640])
@pytest.mark.parametrize("n", [2, 9, 40])
@pytest.mark.parametrize("Hkv,dh", [(1, 128), (3, 64)])
def test_attention_prefix_ends_at_a_stage(B, pre, n, Hkv, dh):
    Hq, lens, plens = 4 * Hkv, [n, n], [pre, pre + 128]
    torch.manual_seed(pre)
    q, k, v = (torch.randn(r, h, dh, device="cuda").bfloat16() for r, h in ((2 * n, Hq), (sum(plens) + 2 * n, Hkv), (sum(plens) + 2 * n, Hkv)))
    out = torch.empty((2 * n, Hq * dh), dtype=torch.bfloat16, device="cuda")
    scratch = torch.empty(Hkv * dh * ((k.shape[0] + 63) // 64 * 64), dtype=torch.bfloat16, device="cuda")
    qb, pb = B.Batch(synth.cu_seqlens(lens)), B.Batch(synth.cu_seqlens(plens))
    B.dsk_attention(B.DSK_BF16, q, k, v, out, qb.desc, pb.desc, sum(plens), Hq, Hkv, dh, scratch)
    torch.cuda.synchronize()
    qd, kd, vd = (t.double().cpu().numpy() for t in (q, k, v))
    got = out.float().cpu().numpy().reshape(2 * n, Hq, dh)
    for b, p0 in ((0, 0), (1, plens[0])):
        for i in range(n):
            rows = np.r_[p0:p0 + plens[b], sum(plens) + b * n:sum(plens) + b * n + i + 1]
            # rounding of the probabilities and of the result: 2^-9 each
            assert O.max_rel_err(got[b * n + i], O.attend_row(qd[b * n + i], kd[rows], vd[rows])) <= 1e-2


# more than 128 queries over short key ranges: the first and the last sizes of the rule and one past it, without and with
# keys in front, ragged
@pytest.mark.parametrize("lens,plens", [([129], None), ([333, 130, 1], None), ([500, 161], [524, 17]), ([1024], None),
                                        ([1025], None)])
@pytest.mark.parametrize("Hq,Hkv,dh", [(8, 2, 128), (6, 2, 64)])
def test_attention_short_prompts(B, Hq, Hkv, dh, lens, plens):
    n, pre = sum(lens), sum(plens or [0])
    bf = lambda a: synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(a))
    q = bf(synth.normal(n * Hq * dh, 43, 0, 3.0).reshape(n, Hq, dh))
    k = bf(synth.normal((pre + n) * Hkv * dh, 43, 1, 2.0).reshape(-1, Hkv, dh))
    v = bf(synth.normal((pre + n) * Hkv * dh, 43, 2, 1.0).reshape(-1, Hkv, dh))
    qc, pc = synth.cu_seqlens(lens), synth.cu_seqlens(plens or [0] * len(lens))
    ref = np.empty((n, Hq, dh))
    for b in range(len(lens)):
        rows = np.r_[pc[b]:pc[b + 1], pre + qc[b]:pre + qc[b + 1]]
        n_pre = pc[b + 1] - pc[b]
        for h in range(Hq):
            kk, vv = (t[rows, h * Hkv // Hq].astype(np.float64) for t in (k, v))
            s = q[qc[b]:qc[b + 1], h].astype(np.float64) @ kk.T / np.sqrt(dh)
            s[np.arange(len(rows))[None] > n_pre + np.arange(lens[b])[:, None]] = -np.inf
            p = np.exp(s - s.max(axis=1, keepdims=True))
            ref[qc[b]:qc[b + 1], h] = p @ vv / p.sum(axis=1, keepdims=True)
    dev = lambda a: torch.from_numpy(a).to(torch.bfloat16).cuda()
    out = torch.empty((n, Hq * dh), dtype=torch.bfloat16, device="cuda")
    scratch = torch.empty(Hkv * dh * ((pre + n + 63) // 64 * 64), dtype=torch.bfloat16, device="cuda")
    qb, pb = B.Batch(qc), B.Batch(pc) if plens else None
    B.dsk_attention(B.DSK_BF16, dev(q), dev(k), dev(v), out, qb.desc, pb.desc if plens else None, pre, Hq, Hkv, dh, scratch)
    torch.cuda.synchronize()
    # rounding of the probabilities and of the result: 2^-9 each
    assert O.max_rel_err(out.float().cpu().numpy().reshape(n, Hq, dh), ref) <= 1e-2


# V rows that are not finite reach the queries that see them and no others (a probability of 0 does not take them out of a
# product): every column form, one and four heads per group, the bad row in front of, inside and behind a wave's own columns,
# in the last key too (its row is repeated up to the end of a stage)
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,n,pre,bad", [(4, 4, 10, 250, 7), (4, 4, 50, 100, 49), (4, 4, 128, 0, 100), (4, 4, 128, 300, 3),
                                              (8, 2, 4, 127, 3), (8, 2, 16, 130, 9), (8, 2, 100, 64, 70), (4, 1, 300, 0, 120)])
def test_attention_rows_that_are_not_finite_reach_later_queries_only(B, Hq, Hkv, n, pre, bad, dh):
    bf = lambda a: torch.from_numpy(a).to(torch.bfloat16).cuda()
    q = bf(synth.normal(n * Hq * dh, 45, 0, 1.0).reshape(n, Hq, dh))
    k, v = (bf(synth.normal((pre + n) * Hkv * dh, 45, j, 1.0).reshape(-1, Hkv, dh)) for j in (1, 2))
    scratch = torch.empty(Hkv * dh * ((pre + n + 63) // 64 * 64), dtype=torch.bfloat16, device="cuda")
    qb, pb = B.Batch(synth.cu_seqlens([n])), B.Batch(synth.cu_seqlens([pre])) if pre else None

    def run():
        out = torch.empty((n, Hq, dh), dtype=torch.bfloat16, device="cuda")
        B.dsk_attention(B.DSK_BF16, q, k, v, out, qb.desc, pb.desc if pre else None, pre, Hq, Hkv, dh, scratch)
        torch.cuda.synchronize()
        return out.float().cpu().numpy()

    clean = run()
    v[pre + bad, :, 0] = float("inf")
    v[pre + bad, :, 1:dh // 2] = float("nan")
    got = run()
    # what does not take part in a sum does not change it
    assert np.array_equal(got[:bad], clean[:bad]) and np.array_equal(got[bad:, :, dh // 2:], clean[bad:, :, dh // 2:])
    assert np.isposinf(got[bad:, :, 0]).all() and np.isnan(got[bad:, :, 1:dh // 2]).all()


@pytest.mark.parametrize("n,pre,bad", [(40, 4000, 21), (100, 2000, 60)])
def test_suffix_token_that_is_not_finite_reaches_later_tokens_only(B, n, pre, bad):
    # through a model: the keys split over workgroups, the partial results merged
    from tests import gpu_util as G
    shape = synth.ModelShape(2, 256, 4, 4, 64, 256, 10000.0, 1e-5, "bf16")
    cache = torch.full((2, 2, pre + n, 4, 64), float("nan"), dtype=torch.bfloat16, device="cuda")
    cache[:, :, :pre] = G.to_dev(synth.kv_cache(shape, pre), shape)
    xs = G.to_dev(synth.hidden_states(shape, n, seed=synth.SEED_SUFFIX), shape)
    with G.GpuModel(shape, n, pre + n) as m:
        m.init_random(11)
        B.dsk_set_option("reset_stats", 0)
        clean = G.to_np(m.suffix(xs, cache, [pre], [n]))
        assert B.dsk_get_stat("attn_key_split_launches") == 2
        xs[bad] = float("nan")
        got = G.to_np(m.suffix(xs, cache, [pre], [n]))
    assert np.array_equal(got[:bad], clean[:bad]) and np.isnan(got[bad:]).all()


# the timing hook takes every attention launch of a prefix pass of 1024 rows and more, on whichever kernel
@pytest.mark.parametrize("lens,timed", [([1024], 2), ([100] * 11, 2), ([1200], 2), ([1023], 0)])
def test_prefix_attention_is_timed(B, lens, timed):
    from tests import gpu_util as G
    shape = synth.ModelShape(2, 256, 4, 2, 64, 256, 10000.0, 1e-5, "bf16")
    x = G.to_dev(synth.hidden_states(shape, sum(lens)), shape)
    with G.GpuModel(shape, sum(lens)) as m:
        m.init_random(1)
        B.dsk_set_option("reset_stats", 0)
        B.dsk_set_option("time_gemm", 1)
        try:
            m.partial(x, 0, 2, None, lens)
            torch.cuda.synchronize()
        finally:
            B.dsk_set_option("time_gemm", 0)
        assert B.dsk_get_stat("attn_mfma_launches") == 2 and B.dsk_get_stat("timed_attn_launches") == timed
        assert (B.dsk_get_stat("timed_attn_ms") > 0) == (timed > 0)
        assert B.dsk_get_stat("timed_attn_flops") == (2 * 4.0 * 4 * 64 * sum(n * (n + 1) / 2 for n in lens) if timed else 0)
