"""Decode calls by the number of work-groups they make: few (two pairs of waves per work-group, the last one merges the splits, a
single split writes the outputs) and many (one pair, a merge launch).  Bars of the parity tests: max 2e-3, relative L2 1e-3."""
import ctypes
from ctypes import c_void_p

import numpy as np
import pytest
import torch

import kvq_workloads as W
from test_gpu_parity import PAIRS, assert_outputs_close, kvq_mod  # noqa: F401

pytestmark = pytest.mark.gpu


def _filled(kvq_mod, oracle_mod, w, residual=32, stale=None, **options):
    g = kvq_mod.KVQ(1, w.batch, w.n_q_heads, w.n_kv_heads, 128, w.context + 40, w.kbits, w.vbits, residual=residual, **options)
    if stale is not None:
        g.workspace.fill_(stale)                        # whatever the memory held before
    o = oracle_mod.OracleCache(1, w.batch, w.n_q_heads, w.n_kv_heads, 128, w.kbits, w.vbits, residual=residual,
                               scale_fp16=bool(options.get("meta_dtype")), key_per_token=bool(options.get("key_mode")))
    K, V = W.kv_tokens(w, 0, 0, w.context)
    g.quantize_append(0, K.cuda(), V.cuda())
    o.quantize_append(0, K.numpy(), V.numpy())
    return g, o


@pytest.mark.parametrize("options", [{}, {"meta_dtype": 1}, {"key_mode": 1}], ids=["", "fp16 scales", "per-token keys"])
@pytest.mark.parametrize("gq", [4, 7])
@pytest.mark.parametrize("kb,vb", PAIRS)
def test_many_work_groups(kvq_mod, oracle_mod, kb, vb, gq, options):
    """More work-groups than are resident at once (400 caches of two splits): one pair each, merged by a launch of its own."""
    w = W.Workload("many", 1, 100, 4 * gq, 4, 128, 32 * 2 + 45, [kb], [vb], seed=40 + kb * 17 + vb, outlier_channels=3)
    g, o = _filled(kvq_mod, oracle_mod, w, **options)
    q = W.query(w, 0)
    assert_outputs_close(g.decode_attention(0, q.cuda()), *o.decode_attention(0, q.numpy()), "K%dV%d" % (kb, vb))
    g.close()


@pytest.mark.parametrize("gq,hkv,T,residual,splits", [
    (4, 2, 1, 32, 0), (4, 2, 63, 32, 0), (4, 2, 200, 500, 0),        # a single split: window of 1, 2 and 7 chunks
    (4, 2, 96, 0, 1), (4, 1, 32 * 7, 32, 1),                         # blocks only; both
    (4, 2, 32 * 2 + 5, 0, 0),                                        # a pair without units
    (4, 2, 32 * 66 + 40, 32, 48), (4, 2, 32 * 66 + 40, 32, 49),      # most splits that the last work-group merges, one more
    (8, 1, 32 * 40 + 40, 32, 16), (8, 1, 32 * 40 + 40, 32, 17),      # the same of a tile of 8 heads
    (7, 2, 32 * 40 + 40, 128, 9),                                    # five chunks of window beside blocks
    (12, 1, 32 * 20 + 3, 32, 0),                                     # two tiles of heads, the second with 4
    (1, 3, 32 * 12 + 40, 32, 0),
    (176, 1, 32 * 3 + 8, 32, 3), (177, 1, 32 * 3 + 8, 32, 3),        # as many tiles as the kernel has arrival counters, one more
])
@pytest.mark.parametrize("kb,vb", [(4, 2), (16, 16)])
def test_few_work_groups(kvq_mod, oracle_mod, gq, hkv, T, residual, splits, kb, vb):
    """Edges of the units' deal between the pairs and of the merge; repeated calls and calls between prefill attention (whose area
    the counters lie in) give the same bits, on a workspace full of ones."""
    w = W.Workload("few", 1, 1, gq * hkv, hkv, 128, T, [kb], [vb], seed=80 + T, outlier_channels=3)
    g, o = _filled(kvq_mod, oracle_mod, w, residual, stale=0xff)
    q = W.query(w, 0)
    qp = W.prefill_queries(w, 0, min(T, 40)).cuda()
    o16, o64 = o.decode_attention(0, q.numpy())
    g.set_decode_options(0, splits)
    out = g.decode_attention(0, q.cuda())
    assert_outputs_close(out, o16, o64, "first")
    for _ in range(3):
        g.prefill_attention(0, qp)
        assert torch.equal(out, g.decode_attention(0, q.cuda()))
        noalloc = torch.empty_like(out)
        g.decode_attention_noalloc(0, q.cuda(), noalloc)
        assert torch.equal(out, noalloc)
    g.reset()
    K, V = W.kv_tokens(w, 0, 0, T)
    g.quantize_append(0, K.cuda(), V.cuda())
    assert torch.equal(out, g.decode_attention(0, q.cuda()))
    g.close()


def test_layers_and_captured_calls_share_the_counters(kvq_mod):
    """Two layers of different lengths in turn, their steps recorded into a graph and replayed between eager calls: every call
    leaves the counters as it found them."""
    side = torch.cuda.Stream()
    lens, pairs = (32 * 9 + 40, 32 * 30 + 33), ([4, 8], [2, 4])
    with torch.cuda.stream(side):
        g = kvq_mod.KVQ(2, 2, 8, 2, 128, 2048, *pairs, stream=side)
        for layer, T in enumerate(lens):
            w = W.Workload("graph", 2, 2, 8, 2, 128, T, *pairs, seed=7, outlier_channels=3)
            g.quantize_append(layer, *W.kv_tokens(w, layer, 0, T, device="cuda:0"))
        q = W.query(w, 0, 0, device="cuda:0").clone()
        outs, refs = torch.empty(2, *q.shape, dtype=q.dtype, device=q.device), torch.empty(2, *q.shape, dtype=q.dtype, device=q.device)
        for layer in range(2):
            g.decode_attention(layer, q, outs[layer])
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        for layer in range(2):
            g.decode_attention(layer, q, outs[layer])
    g.set_decode_options(1, 0)                          # the vector-ALU kernel as the reference
    for step in range(1, 5):
        with torch.cuda.stream(side):
            q.copy_(W.query(w, 0, step, device="cuda:0"))
            outs.fill_(float("nan"))
            graph.replay()
            for layer in range(2):
                g.decode_attention(layer, q, refs[layer])
        side.synchronize()
        d = (outs.double() - refs.double()).cpu().numpy()
        assert np.all(np.isfinite(d)) and np.linalg.norm(d) <= 1e-3 * np.linalg.norm(refs.double().cpu().numpy()), step
    g.close()


def test_one_pass_over_many_layers_of_single_splits(kvq_mod, oracle_mod):
    """Single splits of many caches (more work-groups than are resident at once) write their outputs themselves."""
    w = W.Workload("single", 1, 300, 16, 4, 128, 61, [4], [2], seed=11, outlier_channels=3)
    g, o = _filled(kvq_mod, oracle_mod, w)
    s = ctypes.c_int32()
    from paper_2502_04420_amd.binding import make_config
    cfg, keep = make_config(1, 300, 16, 4, 128, 61, [4], [2])
    assert g._lib.kvq_debug_split_plan(ctypes.byref(cfg), 0, 61, 2, 0, ctypes.byref(s), ctypes.byref(ctypes.c_int32()), ctypes.byref(ctypes.c_int32())) == 0
    assert s.value == 1
    q = W.query(w, 0)
    qd = q.cuda()
    out = torch.full_like(qd, float("nan"))
    assert g._lib.kvq_decode_attention(g._h, 0, c_void_p(qd.data_ptr()), c_void_p(out.data_ptr())) == 0
    torch.cuda.synchronize()
    assert_outputs_close(out, *o.decode_attention(0, q.numpy()), "single")
    g.close()


@pytest.mark.parametrize("batch,hq,hkv,T,kb,vb,pairs", [
    (1024, 4, 2, 32 * 3 + 40, 4, 2, 1), (1024, 4, 2, 32 * 3 + 40, 16, 16, 2), (770, 2, 2, 32 * 16 + 37, 8, 8, 2), (520, 14, 2, 32 * 5 + 33, 8, 4, 1),
    (3, 8, 2, 32 * 40 + 45, 4, 2, 2), (3, 8, 2, 32 * 40 + 45, 16, 4, 2),
])
def test_long_single_splits(kvq_mod, oracle_mod, batch, hq, hkv, T, kb, vb, pairs):
    """One split over several blocks: of so many caches that there is one each (one pair of waves and a merge launch, or two pairs that write
    the outputs), or forced."""
    from paper_2502_04420_amd.binding import make_config
    w = W.Workload("long single", 1, batch, hq, hkv, 128, T, [kb], [vb], seed=900 + kb + vb, outlier_channels=3)
    forced = 1 if batch < 100 else 0
    cfg, keep = make_config(1, batch, hq, hkv, 128, T, [kb], [vb])
    p, s = ctypes.c_int32(), ctypes.c_int32()
    lib = kvq_mod.load_library()
    assert lib.kvq_debug_split_plan(ctypes.byref(cfg), 0, T, 2, forced, ctypes.byref(s), ctypes.byref(ctypes.c_int32()), ctypes.byref(ctypes.c_int32())) == 0
    assert lib.kvq_debug_decode_form(ctypes.byref(cfg), 0, T, forced, ctypes.byref(p), ctypes.byref(ctypes.c_int32())) == 0
    assert (s.value, p.value) == (1, pairs)
    g, o = _filled(kvq_mod, oracle_mod, w)
    g.set_decode_options(0, forced)
    q = W.query(w, 0)
    assert_outputs_close(g.decode_attention(0, q.cuda()), *o.decode_attention(0, q.numpy()), "K%dV%d" % (kb, vb))
    g.close()


@pytest.mark.parametrize("batch,hkv,T,residual", [(15, 1, 32 * 9 + 40, 32), (8, 2, 32 * 9, 0), (17, 1, 32 * 9 + 1, 0), (11, 3, 32 * 5 + 60, 32)])
def test_counters_of_every_cache_start_at_zero(kvq_mod, oracle_mod, batch, hkv, T, residual):
    """Numbers of caches on either side of what one clearing wave takes, with and without window rows in the same launch, on a workspace
    full of ones: every cache's splits are merged, in the first call and in the next."""
    w = W.Workload("counters", 1, batch, 4 * hkv, hkv, 128, T, [4], [2], seed=50 + batch, outlier_channels=3)
    g, o = _filled(kvq_mod, oracle_mod, w, residual, stale=0xff)
    q = W.query(w, 0)
    out = torch.full(q.shape, float("nan"), dtype=q.dtype, device="cuda:0")
    g.decode_attention(0, q.cuda(), out)
    assert_outputs_close(out, *o.decode_attention(0, q.numpy()), "first")
    assert torch.equal(out, g.decode_attention(0, q.cuda()))
    g.close()
