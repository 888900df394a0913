"""The work that users of this library have it do, as measurable cases.

Every case goes through the two calls a serving engine makes, dsk_partial_prefill (selective prefill of a context) and
dsk_suffix_prefill (the new tokens against the mixed cache), on the model shapes of the workloads in bench.py.  Four kinds:

  "layer"      the recomputation of one decoder layer over a packed batch of contexts (attention block and MLP)
  "suffix"     the new tokens through a few layers against caches that are already there
  "selective"  the whole flow on a model: recompute [lo, hi), splice the rest, then the suffix pass

Weights, hidden states and caches are drawn with torch on the device from the seed alone: weights N(0, 0.02), gains
1 + N(0, 0.02), hidden states and caches N(0, 1), as in the repository's synthetic workloads.
"""
import dataclasses
import math
import random

import torch

from paper_2411_02820_amd import binding as B
from paper_2411_02820_amd import synth

SHAPES = {"tiny": synth.TINY, "8b": synth.LLAMA_8B, "70b": synth.LLAMA_70B, "mixtral": synth.MIXTRAL_8X7B}


def listed():
    return [
        # The smallest call: the fp32 model of the first workload, whole; launches and latency are what counts.
        dict(name="tiny-f32", kind="selective", shape="tiny", layers=4, lo=1, hi=3, seqs=1, len_min=128, len_max=128,
             len_seed=0, suffix=16, host=False),
        # A short prompt: too few rows to fill the chip with large tiles, weights and products weigh alike.
        dict(name="layer-8b-333", kind="layer", shape="8b", seqs=1, len_min=333, len_max=333, len_seed=0),
        # An ordinary context at the 8B width.
        dict(name="layer-8b-4k", kind="layer", shape="8b", seqs=1, len_min=4096, len_max=4096, len_seed=0),
        # Eight contexts of uneven length packed into one call (about 40k rows), the batch a loaded engine prefills.
        dict(name="layer-8b-ragged", kind="layer", shape="8b", seqs=8, len_min=1024, len_max=8192, len_seed=5),
        # The widest model.
        dict(name="layer-70b-8k", kind="layer", shape="70b", seqs=1, len_min=8192, len_max=8192, len_seed=0),
        # The mixture-of-experts receiver.
        dict(name="layer-mixtral-8k", kind="layer", shape="mixtral", seqs=1, len_min=8192, len_max=8192, len_seed=0),
        # The question after a reused context: 64 new tokens, a pass over the weights.
        dict(name="suffix-8b-64", kind="suffix", shape="8b", layers=4, seqs=1, len_min=8192, len_max=8192, len_seed=0, suffix=64),
        # One new token: a generation step.
        dict(name="suffix-8b-1", kind="suffix", shape="8b", layers=4, seqs=1, len_min=4096, len_max=4096, len_seed=0, suffix=1),
        # 128 new tokens for each of eight contexts of uneven length.
        dict(name="suffix-8b-ragged", kind="suffix", shape="8b", layers=2, seqs=8, len_min=1024, len_max=8192, len_seed=5,
             suffix=128),
        # The new tokens through expert layers: every expert's weights are streamed.
        dict(name="suffix-mixtral-64", kind="suffix", shape="mixtral", layers=1, seqs=1, len_min=8192, len_max=8192, len_seed=0,
             suffix=64),
        # The sender's caches wait in pinned host memory and are loaded under the recomputation (fewer layers than the
        # whole model, so that the pinned buffers stay small; the share that is recomputed is the workload's).
        dict(name="8b-16k-hostkv", kind="selective", shape="8b", layers=8, lo=2, hi=4, seqs=1, len_min=16384, len_max=16384,
             len_seed=0, suffix=64, host=True),
        # The point the headline figure is quoted on, whole.
        dict(name="8b-8k", kind="selective", shape="8b", layers=32, lo=8, hi=16, seqs=1, len_min=8192, len_max=8192,
             len_seed=0, suffix=64, host=False),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """Another case of the same ranges: contexts of 64 tokens to 16k, 1 to 8 of them, 1 to 1024 new tokens."""
    kind = rng.choice(["tiny", "layer", "layer", "layer", "suffix", "suffix", "suffix", "selective"])
    if kind == "tiny":
        lo = rng.randint(0, 3)
        seqs = rng.choice([1, 1, 2])
        n = _log_int(rng, 16, 512)
        return dict(kind="selective", shape="tiny", layers=4, lo=lo, hi=rng.randint(lo + 1, 4), seqs=seqs, len_min=max(1, n // seqs),
                    len_max=n, len_seed=rng.randint(0, 999), suffix=rng.randint(1, 32), host=False)
    if kind == "layer":
        shape = rng.choice(["8b", "8b", "70b", "mixtral"])
        seqs = rng.choice([1, 1, 2, 4, 8])
        most = {"8b": 16384, "70b": 8192, "mixtral": 8192}[shape]
        n = _log_int(rng, 96, most) if seqs == 1 else _log_int(rng, 32, min(4096, most // seqs))
        return dict(kind="layer", shape=shape, seqs=seqs, len_min=n if seqs == 1 else max(1, n // 4), len_max=n,
                    len_seed=rng.randint(0, 999))
    if kind == "suffix":
        shape = rng.choice(["8b", "8b", "8b", "mixtral"])
        seqs = rng.choice([1, 1, 1, 2, 4, 8])
        suffix = _log_int(rng, 1, 64 if shape == "mixtral" else 128)
        n = _log_int(rng, 512, 16384 // (1 if seqs == 1 else 2))
        return dict(kind="suffix", shape=shape, layers=1 if shape == "mixtral" else rng.randint(2, 4), seqs=seqs,
                    len_min=n if seqs == 1 else max(1, n // 4), len_max=n, len_seed=rng.randint(0, 999),
                    suffix=max(1, suffix // (seqs if shape == "mixtral" else 1)))
    lo = rng.randint(0, 3)
    n = _log_int(rng, 512, 16384)
    return dict(kind="selective", shape="8b", layers=6, lo=lo, hi=lo + rng.randint(1, 2), seqs=1, len_min=n, len_max=n, len_seed=0,
                suffix=rng.randint(1, 64), host=rng.random() < 0.5)


# ---- inputs ----

def _shape(case):
    return dataclasses.replace(SHAPES[case["shape"]], n_layers=case.get("layers", 1))


def _lens(case):
    rng = random.Random(case["len_seed"])
    return [rng.randint(case["len_min"], case["len_max"]) for _ in range(case["seqs"])]


def _dtype(shape):
    return torch.float32 if shape.dtype == "f32" else torch.bfloat16


def _normal(shape, size, seed, stream, std=1.0, mean=0.0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1_000_003 + stream)
    return torch.randn(size, generator=g, device="cuda", dtype=torch.float32).mul_(std).add_(mean).to(_dtype(shape))


def _weights(shape, seed, layer):
    """The tensors of one layer as (binding's tensor id, tensor), one at a time."""
    kinds = [B.DSK_G1, B.DSK_WQ, B.DSK_WK, B.DSK_WV, B.DSK_WO, B.DSK_G2]
    kinds += [synth.WR] if shape.n_experts else [B.DSK_WG, B.DSK_WU, B.DSK_WD]
    for k in kinds:
        yield k, _normal(shape, shape.tensor_shape(k), seed, 100_000 + layer * 1000 + k, 0.02, 1.0 if k in (B.DSK_G1, B.DSK_G2) else 0.0)
    for e in range(shape.n_experts):
        for k in (B.DSK_WG, B.DSK_WU, B.DSK_WD):
            yield B.DSK_EXPERT(e, k), _normal(shape, shape.tensor_shape(k), seed, 100_000 + layer * 1000 + 16 + e * 16 + k, 0.02)


def _hidden(shape, rows, seed, stream):
    """Hidden states N(0, 1).  For an expert model every token carries a part along the router rows of two experts of
    its own: a trained router is decisive, and the choice of experts does not hang on the last bit of a sum."""
    x = _normal(shape, (rows, shape.hidden), seed, stream)
    if shape.n_experts:
        r = _normal(shape, shape.tensor_shape(synth.WR), seed, 100_000 + synth.WR, 0.02).float()
        r = r / r.norm(dim=1, keepdim=True)
        pick = _normal(dataclasses.replace(shape, dtype="f32"), (rows, shape.n_experts), seed, stream + 1).topk(2, dim=1).indices
        x = (x.float() + 8.0 * r[pick[:, 0]] + 6.0 * r[pick[:, 1]]).to(x.dtype)
    return x


def _cache(shape, rows, seed, stream, new_rows=0):
    """[L, 2, rows + new_rows, Hkv, dh], N(0, 1) in the first `rows` rows and 0 in the others."""
    t = torch.zeros((shape.n_layers, 2, rows + new_rows, shape.n_kv_heads, shape.head_dim), device="cuda", dtype=_dtype(shape))
    for l in range(shape.n_layers):
        t[l, :, :rows] = _normal(shape, (2, rows, shape.n_kv_heads, shape.head_dim), seed, stream + l)
    return t


class _Model:
    """A receiver with its weights, released with the state that holds it."""

    def __init__(self, shape, seed, max_tokens, max_rows):
        self.handle = B.dsk_model_create(B.config_from_shape(shape), max_tokens, max_rows)
        for l in range(shape.n_layers):
            for k, w in _weights(shape, seed, l):
                B.dsk_model_set_tensor(self.handle, l, k, w)
        torch.cuda.synchronize()

    def __del__(self):
        if getattr(self, "handle", None):
            B.dsk_model_destroy(self.handle)


def _pinned(t):
    p = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
    p.copy_(t)
    return p


def prepare(case, seed):
    shape, lens = _shape(case), _lens(case)
    T = sum(lens)
    s = {"case": case, "T": T}
    if case["kind"] == "layer":
        s["model"] = _Model(shape, seed, T, T)
        s["prefix"] = B.Batch(synth.cu_seqlens(lens), synth.packed_positions(lens))
        s["x"] = _hidden(shape, T, seed, 1)
        s["kv"] = torch.empty((1, 2, T, shape.n_kv_heads, shape.head_dim), device="cuda", dtype=_dtype(shape))
        s["out"] = torch.empty_like(s["x"])
        s["kv_desc"] = B.kv_desc(s["kv"])
        return s
    slens = [case["suffix"]] * len(lens)
    S = sum(slens)
    s["model"] = _Model(shape, seed, max(S, T if case["kind"] == "selective" else 1), T + S)
    s["prefix"] = B.Batch(synth.cu_seqlens(lens), synth.packed_positions(lens))
    s["suffix"] = B.Batch(synth.cu_seqlens(slens), synth.packed_positions(slens, start=lens))
    s["xs"] = _hidden(shape, S, seed, 3)
    s["out"] = torch.empty_like(s["xs"])
    if case["kind"] == "suffix":
        s["kv"] = _cache(shape, T, seed, 1000, S)
        s["kv_desc"] = B.kv_desc(s["kv"])
        return s
    reused, x = _cache(shape, T, seed, 1000), _hidden(shape, T, seed, 1)
    s["reused"], s["x"] = (_pinned(reused), _pinned(x)) if case["host"] else (reused, x)
    s["kv"] = torch.zeros((shape.n_layers, 2, T + S, shape.n_kv_heads, shape.head_dim), device="cuda", dtype=_dtype(shape))
    s["reused_desc"], s["kv_desc"] = B.kv_desc(s["reused"]), B.kv_desc(s["kv"])
    return s


def run(s):
    case, T = s["case"], s["T"]
    m = s["model"].handle
    if case["kind"] == "layer":
        B.dsk_partial_prefill(m, s["x"], 0, 1, None, s["kv_desc"], s["prefix"].desc, s["out"])
        return {"hidden": s["out"], "kv": s["kv"]}
    if case["kind"] == "suffix":
        B.dsk_suffix_prefill(m, s["xs"], s["kv_desc"], s["prefix"].desc, s["suffix"].desc, T, s["out"])
        return {"hidden": s["out"], "kv_new": s["kv"][:, :, T:]}
    lo, hi = case["lo"], case["hi"]
    B.dsk_partial_prefill(m, s["x"], lo, hi, s["reused_desc"], s["kv_desc"], s["prefix"].desc, None, B.DSK_DEFER_JOIN)
    B.dsk_suffix_prefill(m, s["xs"], s["kv_desc"], s["prefix"].desc, s["suffix"].desc, T, s["out"])
    return {"hidden": s["out"], "kv_recomputed": s["kv"][lo:hi], "kv_spliced_below": s["kv"][:lo], "kv_spliced_above": s["kv"][hi:]}


# ---- what a pass cannot do without ----

def _layer_params(shape, rows):
    d, hq, hkv, dh, f = shape.hidden, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, shape.ffn
    attn = d * (hq + 2 * hkv) * dh + hq * dh * d
    if not shape.n_experts:
        return attn + 3 * d * f, attn + 3 * d * f
    touched = min(shape.n_experts, rows * shape.top_k)  # experts whose weights are read, at most
    return attn + touched * 3 * d * f + shape.n_experts * d, attn + shape.top_k * 3 * d * f + shape.n_experts * d


def _attn_flops(shape, lens, pre):
    return sum(4.0 * shape.n_q_heads * shape.head_dim * (n * (n + 1) / 2.0 + n * p) for n, p in zip(lens, pre))


def work(case):
    shape, lens = _shape(case), _lens(case)
    T, b, kvw = sum(lens), shape.elem_bytes, shape.n_kv_heads * shape.head_dim
    total_bytes = total_flops = 0.0
    if case["kind"] in ("layer", "selective"):
        n = 1 if case["kind"] == "layer" else case["hi"] - case["lo"]
        stored, used = _layer_params(shape, T)
        total_bytes += n * (stored * b + 2 * T * kvw * b) + T * shape.hidden * b * (2 if case["kind"] == "layer" else 1)
        total_flops += n * (2.0 * T * used + _attn_flops(shape, lens, [0] * len(lens)))
        total_bytes += 2.0 * (shape.n_layers - n) * 2 * T * kvw * b  # spliced rows: read and written
    if case["kind"] in ("suffix", "selective"):
        slens = [case["suffix"]] * len(lens)
        S = sum(slens)
        stored, used = _layer_params(shape, S)
        total_bytes += shape.n_layers * (stored * b + 2 * T * kvw * b + 2 * S * kvw * b) + 2 * S * shape.hidden * b
        total_flops += shape.n_layers * (2.0 * S * used + _attn_flops(shape, slens, lens))
    return {"bytes": total_bytes, "flops": total_flops}


def tolerance(case):
    # Four times what the kernels are off by against `exact` over the listed and some drawn cases (2-norm; largest
    # difference over the root mean square): fp32 3e-7 / 1.8e-6; one bf16 layer 4.6e-3 / 0.03 at the 8B width and
    # 1.1e-2 / 0.07 at the 70B one; the suffix pass 5.9e-3 / 0.025 (the bf16 rounding of the operands in each layer, and
    # more with every layer it travels through); the whole flow 1.7e-2 / 0.09.
    if SHAPES[case["shape"]].dtype == "f32":
        return {"rel": 2e-6, "max": 1e-5}
    if case["kind"] == "layer":
        return {"rel": 0.03, "max": 0.28} if case["shape"] == "70b" else {"rel": 0.018, "max": 0.12}
    if case["kind"] == "suffix":
        return {"rel": 0.024, "max": 0.1}
    return {"rel": 0.03, "max": 0.36}


# ---- the same in 64 bits, with plain torch ----

def _rope(x, pos, base):
    half = x.shape[-1] // 2
    theta = base ** (-2.0 * torch.arange(half, device=x.device, dtype=torch.float64) / (2 * half))
    a = pos.to(torch.float64)[:, None, None] * theta
    c, s = a.cos(), a.sin()
    x1, x2 = x[..., :half], x[..., half:]
    return torch.cat([x1 * c - x2 * s, x2 * c + x1 * s], dim=-1)


def _norm(x, g, eps):
    return x * torch.rsqrt(x.square().mean(dim=-1, keepdim=True) + eps) * g


def _attend(q, k, v, n_pre):
    """q [n, Hq, dh] against k, v [n_pre + n, Hkv, dh]; query i sees the first n_pre + i + 1 keys."""
    n, hq, dh = q.shape
    hkv = k.shape[1]
    q = q.view(n, hkv, hq // hkv, dh).permute(1, 2, 0, 3)
    k, v = k.permute(1, 2, 0).contiguous(), v.permute(1, 0, 2).contiguous()
    out = torch.empty((n, hkv, hq // hkv, dh), device=q.device, dtype=torch.float64)
    for h in range(hkv):
        for r in range(0, n, 1024):
            e = min(n, r + 1024)
            m = n_pre + e
            s = q[h, :, r:e].reshape(-1, dh) @ k[h, :, :m].contiguous() / math.sqrt(dh)
            s = s.view(-1, e - r, m)
            keys = torch.arange(m, device=q.device)
            s.masked_fill_(keys[None, :] > n_pre + torch.arange(r, e, device=q.device)[:, None], -math.inf)
            o = torch.softmax(s, dim=-1).view(-1, m) @ v[h, :m]
            out[r:e, h] = o.view(-1, e - r, dh).permute(1, 0, 2)
    return out.view(n, hq * dh)


def _exact_layer(shape, seed, layer, x, pos, lens, pre_kv=None, pre_lens=None):
    """State leaving the layer, and the new K and V rows; pre_kv: [2, rows, Hkv, dh] of the contexts."""
    w = {k: t.to(torch.float64) for k, t in _weights(shape, seed, layer) if k < 16 and k != synth.WR}
    hq, hkv, dh = shape.n_q_heads, shape.n_kv_heads, shape.head_dim
    xn = _norm(x, w[B.DSK_G1], shape.rms_eps)
    q = _rope((xn @ w[B.DSK_WQ].T).view(-1, hq, dh), pos, shape.rope_base)
    k = _rope((xn @ w[B.DSK_WK].T).view(-1, hkv, dh), pos, shape.rope_base)
    v = (xn @ w[B.DSK_WV].T).view(-1, hkv, dh)
    att = torch.empty((x.shape[0], hq * dh), device=x.device, dtype=torch.float64)
    a = p = 0
    for i, n in enumerate(lens):
        kk, vv, m = k[a:a + n], v[a:a + n], 0
        if pre_kv is not None:
            m = pre_lens[i]
            kk = torch.cat([pre_kv[0, p:p + m].to(torch.float64), kk])
            vv = torch.cat([pre_kv[1, p:p + m].to(torch.float64), vv])
        att[a:a + n] = _attend(q[a:a + n], kk, vv, m)
        a, p = a + n, p + m
    h = x + att @ w[B.DSK_WO].T
    y = _norm(h, w[B.DSK_G2], shape.rms_eps)
    silu = torch.nn.functional.silu
    if not shape.n_experts:
        return h + (silu(y @ w[B.DSK_WG].T) * (y @ w[B.DSK_WU].T)) @ w[B.DSK_WD].T, k, v
    ids, out = None, h.clone()
    expert = {}
    for key, t in _weights(shape, seed, layer):
        if key == synth.WR:
            val, ids = (y @ t.to(torch.float64).T).topk(shape.top_k, dim=1)
            gate = torch.softmax(val, dim=1)
        elif key >= 16:
            expert[key % 16] = t.to(torch.float64)
            if key % 16 == B.DSK_WD:
                rows, choice = (ids == (key - 16) // 16).nonzero(as_tuple=True)
                z = y[rows]
                z = (silu(z @ expert[B.DSK_WG].T) * (z @ expert[B.DSK_WU].T)) @ expert[B.DSK_WD].T
                out.index_add_(0, rows, z * gate[rows, choice][:, None])
    return out, k, v


def exact(case, seed):
    shape, lens = _shape(case), _lens(case)
    T = sum(lens)
    pos = torch.from_numpy(synth.packed_positions(lens)).cuda()
    if case["kind"] == "layer":
        h, k, v = _exact_layer(shape, seed, 0, _hidden(shape, T, seed, 1).to(torch.float64), pos, lens)
        return {"hidden": h, "kv": torch.stack([k, v])[None]}
    slens = [case["suffix"]] * len(lens)
    S = sum(slens)
    spos = torch.from_numpy(synth.packed_positions(slens, start=lens)).cuda()
    prefix = _cache(shape, T, seed, 1000)
    if case["kind"] == "selective":
        lo, hi = case["lo"], case["hi"]
        mixed = prefix.to(torch.float64)
        h = _hidden(shape, T, seed, 1).to(torch.float64)
        for l in range(lo, hi):
            h, mixed[l, 0], mixed[l, 1] = _exact_layer(shape, seed, l, h, pos, lens)
        prefix = mixed
    new = torch.empty((shape.n_layers, 2, S, shape.n_kv_heads, shape.head_dim), device="cuda", dtype=torch.float64)
    h = _hidden(shape, S, seed, 3).to(torch.float64)
    for l in range(shape.n_layers):
        h, new[l, 0], new[l, 1] = _exact_layer(shape, seed, l, h, spos, slens, prefix[l], lens)
    if case["kind"] == "suffix":
        return {"hidden": h, "kv_new": new}
    kv = torch.cat([prefix, new], dim=2)
    return {"hidden": h, "kv_recomputed": kv[lo:hi], "kv_spliced_below": kv[:lo], "kv_spliced_above": kv[hi:]}
