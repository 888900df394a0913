"""The three KV-loading strategies (Sec. 4.3, Fig. 13) on the GPU, over an emulated slow link: results stay
bit-identical, the strategies finish in the figure's order, and the delay of each strategy RELATIVE to "load
everything, then compute" follows the unit-cost schedule model that reproduces the figure's totals, fed with the
per-layer transfer and recompute times measured on the same box.  Ratios of minima over several repetitions are
compared, not wall-clock values, so that a busy box shifts both sides alike."""
import numpy as np
import pytest
import torch

from oracle import schedule_model as SM
from paper_2411_02820_amd import synth

pytestmark = pytest.mark.gpu

# E cache and one layer's KV have the same size (T*d = 2*T*Hkv*dh), as in the figure's unit-cost setting
SHAPE = synth.ModelShape(8, 512, 4, 2, 128, 1536, 10000.0, 1e-5, "bf16")
T = 2048
LO, HI = 2, 6
LINK_GBPS = 2.0


def timed(fn, reps=5):
    best = float("inf")
    for _ in range(reps):
        s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        s.record()
        fn()
        e.record()
        torch.cuda.synchronize()
        best = min(best, s.elapsed_time(e))
    return best


def test_strategies_over_a_slow_link_follow_the_schedule_model():
    from paper_2411_02820_amd import binding as B
    from tests import gpu_util as G
    hidden_pinned = G.to_dev(synth.hidden_states(SHAPE, T), SHAPE, pinned=True)
    hidden_dev = G.to_dev(synth.hidden_states(SHAPE, T), SHAPE)
    kv_pinned = G.to_dev(synth.kv_cache(SHAPE, T), SHAPE, pinned=True)
    kv_dev = G.to_dev(synth.kv_cache(SHAPE, T), SHAPE)
    layer_bytes = 2 * T * SHAPE.kv_width * 2
    assert layer_bytes == T * SHAPE.hidden * 2
    with G.GpuModel(SHAPE, T) as m:
        m.load_from_generator(0, scale=2.0)
        kv_out = m.new_cache(T, fill=0.0)
        # per-layer recompute time: everything device-resident and aliased, so nothing is loaded
        for _ in range(2):
            m.partial(hidden_dev, LO, HI, kv_dev, [T], kv_out=kv_dev)
        t_compute = timed(lambda: m.partial(hidden_dev, LO, HI, kv_dev, [T], kv_out=kv_dev)) / (HI - LO)
        # per-layer transfer time over the emulated link: a pure splice of all layers from host memory
        B.dsk_set_load_throttle(m.handle, LINK_GBPS)
        t_load = timed(lambda: m.partial(hidden_dev, 0, 0, kv_pinned, [T], kv_out=kv_out)) / SHAPE.n_layers
        assert t_load == pytest.approx(layer_bytes / (LINK_GBPS * 1e9) * 1e3, rel=0.25), "pacing misses the chosen rate"

        job = [SM.Job(0.0, SHAPE.n_layers, HI - LO, True)]
        measured, outs, modelled = {}, {}, {}
        for name, mode in (("all_then_compute", B.DSK_LOAD_ALL_FIRST), ("reused_then_compute", B.DSK_LOAD_REUSED_FIRST),
                           ("pipelined", B.DSK_LOAD_PIPELINED)):
            B.dsk_set_load_mode(m.handle, mode)
            res = []
            measured[name] = timed(lambda: res.append(m.partial(hidden_pinned, LO, HI, kv_pinned, [T], kv_out=kv_out)))
            outs[name] = (res[-1][0].clone(), res[-1][1].clone())
            modelled[name] = SM.total_ttft(job, name, unit_load=t_load, unit_compute=t_compute)
        B.dsk_set_load_throttle(m.handle, 0.0)
        B.dsk_set_load_mode(m.handle, B.DSK_LOAD_PIPELINED)
        print("measured ms:", {k: round(v, 3) for k, v in measured.items()}, "model ms:", {k: round(v, 3) for k, v in modelled.items()})
        assert measured["pipelined"] < measured["reused_then_compute"] < measured["all_then_compute"]
        for name in ("reused_then_compute", "pipelined"):
            got = measured[name] / measured["all_then_compute"]
            want = modelled[name] / modelled["all_then_compute"]
            assert got == pytest.approx(want, abs=0.2 * want), f"{name}: measured ratio {got:.3f}, model ratio {want:.3f}"
        # the link does not change a single bit, whatever the strategy
        ref_kv, ref_h = m.partial(hidden_pinned, LO, HI, kv_pinned, [T])
        torch.cuda.synchronize()
        for name in outs:
            assert torch.equal(outs[name][0], ref_kv) and torch.equal(outs[name][1], ref_h), name


# Device-resident layers: one launch per run of layers, but in full reuse with a deferred join, where nothing else covers the
# loads, the suffix pass follows launches of 1, 2, 4, .. layers; the result is the same either way
@pytest.mark.parametrize("lo,hi,deferred,launches", [(0, 0, True, 4), (3, 3, True, 4), (0, 0, False, 1), (2, 3, True, 2), (0, 5, True, 1)])
def test_launches_of_device_resident_layers(lo, hi, deferred, launches):
    from paper_2411_02820_amd import binding as B
    from tests import gpu_util as G
    n, s = 300, 20
    hidden = G.to_dev(synth.hidden_states(SHAPE, n), SHAPE)
    xs = G.to_dev(synth.hidden_states(SHAPE, s, seed=synth.SEED_SUFFIX), SHAPE)
    kv = G.to_dev(synth.kv_cache(SHAPE, n), SHAPE)
    with G.GpuModel(SHAPE, n, n + s) as m:
        m.init_random(3)
        ref_kv, _ = m.partial(hidden, lo, hi, kv, [n], n_rows=n + s)
        torch.cuda.synchronize()
        ref = m.suffix(xs, ref_kv, [n], [s])
        out_kv = m.new_cache(n + s, fill=float("nan"))
        torch.cuda.synchronize()
        B.dsk_set_option("reset_stats", 0)
        m.partial(hidden, lo, hi, kv, [n], kv_out=out_kv, flags=B.DSK_DEFER_JOIN if deferred else 0)
        out = m.suffix(xs, out_kv, [n], [s])
        torch.cuda.synchronize()
        assert B.dsk_get_stat("splice_launches") == launches
    assert torch.equal(out, ref) and torch.equal(out_kv, ref_kv)


def test_cache_that_is_not_this_devices_memory_is_copied():
    # a peer's cache, which a copy reaches without peer access and a kernel does not; here page-locked host memory stands for
    # it, which both can address
    from paper_2411_02820_amd import binding as B
    from tests import gpu_util as G
    n = 40
    kv = G.to_dev(synth.kv_cache(SHAPE, n), SHAPE, pinned=True)
    desc = B.kv_desc(kv)
    desc.mem = B.DSK_MEM_DEVICE
    batch = B.Batch(synth.cu_seqlens([n]), synth.packed_positions([n]))
    with G.GpuModel(SHAPE, n) as m:
        out = m.new_cache(n, fill=float("nan"))
        torch.cuda.synchronize()
        B.dsk_set_option("reset_stats", 0)
        B.dsk_partial_prefill_groups(m.handle, [], desc, B.kv_desc(out), batch.desc)
        torch.cuda.synchronize()
        assert B.dsk_get_stat("splice_launches") == 0
    assert torch.equal(out.cpu(), kv)


# a layer behind a host-resident E cache: the shortest contexts that are chunked, a rest that is not a multiple of a tile, and
# whole chunks of 4096 rows behind the first; against the layer in one piece, bit for bit.  The 8B shape; expert layers (a chunk
# groups its own rows by expert); 64 heads of 64; a width whose first chunk is not the 8B one's
WIDTHS = {"8b": (4096, 32, 8, 128, 14336), "experts": (4096, 32, 8, 128, 1536), "heads of 64": (4096, 64, 8, 64, 1536),
          "3072": (3072, 24, 8, 128, 1536)}


@pytest.mark.parametrize("width,T,chunks", [("8b", 4607, 0), ("8b", 4608, 2), ("8b", 5001, 2), ("8b", 8191, 2), ("8b", 9001, 2), ("8b", 12288, 3),
                                            ("experts", 4095, 0), ("experts", 4096, 2), ("experts", 5001, 2), ("experts", 9001, 2),
                                            ("heads of 64", 5001, 2), ("3072", 5631, 0), ("3072", 5632, 2), ("3072", 9001, 2)])
def test_chunked_first_layer_keeps_its_bits(width, T, chunks):
    from paper_2411_02820_amd import binding as B
    from tests import gpu_util as G
    shape = synth.ModelShape(1, *WIDTHS[width], 500000.0, 1e-5, "bf16", *((8, 2) if width == "experts" else ()))
    x = torch.randn((T, shape.hidden), generator=torch.Generator().manual_seed(T)).to(torch.bfloat16).pin_memory()
    with G.GpuModel(shape, T) as m:
        m.init_random(synth.SEED_RECEIVER)
        B.dsk_set_option("reset_stats", 0)
        kv_c, h_c = m.partial(x, 0, 1, None, [T])
        torch.cuda.synchronize()
        assert B.dsk_get_stat("e_cache_chunks") == chunks
        kv_1, h_1 = m.partial(x.cuda(), 0, 1, None, [T])
        torch.cuda.synchronize()
        assert torch.equal(kv_c, kv_1) and torch.equal(h_c, h_1)
