"""Prefill attention by the form its launch takes: work-groups of 4 waves and 128 rows or of 8 waves and 256, rows of one query head or of
several, whole tiles (started in pairs or in turn) or pieces."""
import ctypes

import numpy as np
import pytest
import torch

import kvq_workloads as W
from paper_2502_04420_amd.binding import make_config
from test_gpu_prefill import _run, assert_prefill_close, kvq_mod  # noqa: F401

pytestmark = pytest.mark.gpu

BY_CACHE, BY_LENGTH, PAIRED = 0, 1, 2


def forms(g, T, n_q):
    """Per pass of a prefill-attention call: caches, waves per work-group, query heads that share its rows, order of whole tiles, most
    pieces of a tile."""
    cfg, keep = make_config(1, g.batch, g.n_q_heads, g.n_kv_heads, 128, g.max_tokens, g.kbits, g.vbits, residual=g.residual,
                            meta_dtype=g.meta_dtype, key_mode=g.key_mode)
    caches, n, waves, heads, order = (ctypes.c_int32() for _ in range(5))
    out = []
    while True:
        most = 0
        for tile in range((n_q + 255) // 256):
            assert g._lib.kvq_debug_prefill_plan(ctypes.byref(cfg), g.workspace.numel(), T, n_q, len(out), tile, ctypes.byref(caches), ctypes.byref(n)) == 0
            most = max(most, n.value)
        assert g._lib.kvq_debug_prefill_form(ctypes.byref(cfg), g.workspace.numel(), T, n_q, len(out), ctypes.byref(waves), ctypes.byref(heads), ctypes.byref(order)) == 0
        if caches.value == 0:
            return out
        out.append((caches.value, waves.value, heads.value, order.value, most))


# room: tokens that the caches are configured for (they decide how many caches a pass takes), 0 for T
@pytest.mark.parametrize("T,n_q,batch,hq,hkv,residual,kb,vb,room,form", [
    # whole tiles, 4 waves, one head per work-group: few units, few work-groups
    (300, 300, 1, 8, 2, 32, 4, 2, 0, [(2, 4, 1, PAIRED, 1)]),            # caches that do not divide by 8
    (225, 225, 4, 8, 2, 32, 8, 4, 0, [(8, 4, 1, PAIRED, 1)]),            # caches that do
    (64, 64, 3, 12, 1, 500, 4, 2, 0, [(3, 4, 1, PAIRED, 1)]),            # window only
    (257, 129, 2, 3, 3, 32, 16, 16, 0, [(6, 4, 1, PAIRED, 1)]),          # one head per cache, fp16 keys; one row more than a work-group has
    (1, 1, 1, 4, 2, 32, 4, 4, 0, [(2, 4, 1, PAIRED, 1)]), (33, 2, 1, 16, 1, 0, 4, 4, 0, [(1, 4, 1, PAIRED, 1)]),
    # whole tiles, 4 waves, the group's heads together
    (400, 400, 1, 8, 2, 32, 4, 2, 0, [(2, 4, 4, PAIRED, 1)]),            # fewer work-groups than compute units, caches that do not divide by 8
    (330, 330, 4, 8, 2, 32, 8, 4, 0, [(8, 4, 4, PAIRED, 1)]),            # caches that do
    (160, 160, 12, 24, 1, 500, 4, 2, 0, [(12, 4, 24, PAIRED, 1)]),       # window only
    (500, 500, 8, 14, 2, 32, 4, 4, 0, [(16, 4, 7, PAIRED, 1)]),          # more than one work-group per compute unit; rows that do not divide by the heads
    (600, 480, 5, 21, 3, 0, 2, 2, 0, [(15, 4, 7, PAIRED, 1)]),           # the same of 15 caches, no window
    (700, 700, 8, 14, 2, 32, 4, 4, 0, [(16, 4, 7, BY_LENGTH, 1)]),       # more than two per compute unit
    (700, 650, 5, 21, 3, 0, 2, 2, 0, [(15, 4, 7, BY_LENGTH, 1)]),
    (400, 400, 40, 4, 2, 32, 4, 2, 2000, [(80, 4, 2, BY_LENGTH, 1)]),
    (390, 390, 27, 6, 3, 100, 4, 2, 2000, [(81, 4, 2, BY_LENGTH, 1)]),   # ... of 81 caches, several window chunks
    (700, 700, 40, 4, 2, 32, 4, 2, 4000, [(80, 4, 2, BY_CACHE, 1)]),     # caches that exceed the XCDs' L2
    (700, 690, 39, 6, 2, 0, 4, 4, 4000, [(78, 4, 3, BY_CACHE, 1)]),      # ... whose number does not divide by 8
    (400, 400, 17, 4, 2, 32, 4, 2, 0, [(16, 4, 2, PAIRED, 1)] * 2 + [(2, 4, 2, PAIRED, 1)]),         # several passes
    # whole tiles, 8 waves
    (6300, 5, 25, 32, 1, 32, 4, 2, 11000, [(25, 8, 32, BY_CACHE, 1)]),   # several heads' queries together
    (6300, 9, 32, 24, 1, 0, 8, 4, 14000, [(32, 8, 24, BY_CACHE, 1)]),
    # pieces, 4 waves
    (1600, 300, 4, 4, 2, 32, 4, 2, 0, [(8, 4, 1, BY_CACHE, 4)]),         # second tile: the second work-group of every piece has no rows
    (1500, 897, 1, 8, 2, 32, 4, 2, 0, [(2, 4, 1, BY_CACHE, 3)]),         # last tile: ... one row
    (2100, 33, 16, 28, 4, 32, 4, 2, 0, [(16, 4, 7, BY_CACHE, 4)] * 4),   # a tile of several heads' queries
    # pieces, 8 waves
    (1600, 385, 4, 4, 2, 32, 4, 2, 0, [(8, 8, 1, BY_CACHE, 4)]),
    (2000, 5, 1, 8, 2, 32, 4, 2, 0, [(2, 8, 1, BY_CACHE, 5)]), (3000, 17, 2, 14, 2, 0, 8, 2, 0, [(4, 8, 1, BY_CACHE, 7)]),
    (3000, 64, 8, 8, 2, 32, 4, 4, 0, [(16, 8, 1, BY_CACHE, 4)]),
    (5000, 60, 16, 8, 2, 32, 4, 4, 0, [(16, 8, 2, BY_CACHE, 8)] * 2),    # a tile of several heads' queries
])
def test_rows_and_waves(kvq_mod, oracle_mod, T, n_q, batch, hq, hkv, residual, kb, vb, room, form):
    w = W.Workload("rows", 1, batch, hq, hkv, 128, T, [kb], [vb], seed=1200 + T + n_q, outlier_channels=3)
    g = kvq_mod.KVQ(1, batch, hq, hkv, 128, room or T, [kb], [vb], residual=residual)
    assert forms(g, T, n_q) == form
    o = oracle_mod.OracleCache(1, batch, hq, hkv, 128, [kb], [vb], residual=residual)
    K, V = W.kv_tokens(w, 0, 0, T)
    g.quantize_append(0, K.cuda(), V.cuda())
    o.quantize_append(0, K.numpy(), V.numpy())
    q = W.prefill_queries(w, 0, n_q)
    out = torch.full(q.shape, float("nan"), dtype=q.dtype, device="cuda:0")
    g.prefill_attention(0, q.cuda(), out)
    assert_prefill_close(out, o.prefill_attention(0, q.numpy())[1], "T%d nq%d" % (T, n_q))
    assert torch.equal(out, g.prefill_attention(0, q.cuda()))
    g.close()


def test_prompts_by_cache_in_work_groups_of_four_waves_sampled_rows(kvq_mod, oracle_mod):
    """Four prompts of 4000 tokens, 32 / 8 heads: whole tiles of the group's heads together, started cache by cache, two passes.  Sampled
    (batch, kv head) pairs at sampled positions against the oracle."""
    w = W.Workload("by cache", 1, 4, 32, 8, 128, 4000, [4], [2], seed=1210, outlier_channels=3)
    T, gq = w.context, 4
    g = kvq_mod.KVQ(1, 4, 32, 8, 128, T, [4], [2])
    assert forms(g, T, T) == [(16, 4, 4, BY_CACHE, 1)] * 2
    K, V = W.kv_tokens(w, 0, 0, T, device="cuda:0")
    g.quantize_append(0, K, V)
    q = W.prefill_queries(w, 0, T, device="cuda:0")
    out = g.prefill_attention(0, q)
    pos = [0, 1, 15, 16, 31, 32, 33, 127, 128, 255, 256, 1023, 1999, 2000, 3935, 3936, 3967, 3968, 3998, 3999]
    for bh in (0, 15, 16, 31):                      # the first and last of either pass
        b, h = divmod(bh, 8)
        o = oracle_mod.OracleCache(1, 1, gq, 1, 128, [4], [2])
        o.quantize_append(0, K[b:b + 1, h:h + 1].cpu().numpy(), V[b:b + 1, h:h + 1].cpu().numpy())
        assert o.tokens(0) == g.layer_tokens(0)
        qs = q[b, h * gq:(h + 1) * gq][:, pos].cpu().numpy()[None]
        o16, o64 = o.prefill_attention_at(0, np.ascontiguousarray(qs), pos)
        assert_prefill_close(out[b, h * gq:(h + 1) * gq][:, pos][None], o64, "bh %d" % bh)
        o.close()
    g.close()


@pytest.mark.parametrize("form", ["low parts of all channels", "wide keys", "offset on every channel", "fp16 scales", "per-token keys", "fp16 values"])
@pytest.mark.parametrize("T,n_q,batch,hq,hkv,launch", [
    (420, 420, 4, 8, 2, [(8, 4, 4, PAIRED, 1)]),
    (2500, 33, 8, 14, 2, [(16, 4, 7, BY_CACHE, 4)]),                     # pieces
])
def test_forms_of_the_units_in_work_groups_of_four_waves(kvq_mod, oracle_mod, form, T, n_q, batch, hq, hkv, launch):
    vb = 16 if "values" in form else 4
    n, mult, offs = {"wide keys": (128, 12.0, 0.0), "offset on every channel": (0, 1.0, 20.0)}.get(form, (3, 12.0, 0.0))
    meta = kvq_mod.META_FP16 if "fp16 scales" in form else kvq_mod.META_FP32
    keys = kvq_mod.KEYS_PER_TOKEN if "per-token" in form else kvq_mod.KEYS_PER_CHANNEL
    w = W.Workload("row forms", 1, batch, hq, hkv, 128, T, [4], [vb], seed=1300 + T, outlier_channels=n, outlier_scale=mult, key_bias_std=offs)
    out, o64, g, o, q = _run(kvq_mod, oracle_mod, w, n_q, meta=meta, keys=keys, max_tokens=T, low_parts=1 if form.startswith("low") else None)
    assert forms(g, T, n_q) == launch
    assert_prefill_close(out, o64, form)
    g.close()


@pytest.mark.parametrize("vb", [16, 8, 2])
@pytest.mark.parametrize("T,n_q,batch,hq,hkv,launch", [
    (257, 129, 2, 3, 3, [(6, 4, 1, PAIRED, 1)]), (420, 420, 4, 8, 2, [(8, 4, 4, PAIRED, 1)]),       # whole tiles, 4 waves
    (2500, 33, 8, 14, 2, [(16, 4, 7, BY_CACHE, 4)]),                     # pieces, 4 waves
    (1600, 385, 4, 4, 2, [(8, 8, 1, BY_CACHE, 4)]), (3000, 17, 2, 14, 2, [(4, 8, 1, BY_CACHE, 7)]),  # pieces, 8 waves: one head's rows
    (5000, 60, 16, 8, 2, [(16, 8, 2, BY_CACHE, 8)] * 2),                 # ... several heads'
])
def test_half_precision_keys(kvq_mod, oracle_mod, T, n_q, batch, hq, hkv, launch, vb):
    """Value rows of fp16-key layers lie in another order for 4 waves than for 8 (value_shift), packed values and the window's rows alike, and
    4 waves fetch a unit at the top of a step."""
    w = W.Workload("half keys", 1, batch, hq, hkv, 128, T, [16], [vb], seed=1350 + T + n_q, outlier_channels=3)
    out, o64, g, o, q = _run(kvq_mod, oracle_mod, w, n_q, max_tokens=T)
    assert forms(g, T, n_q) == launch
    assert_prefill_close(out, o64, "V%d" % vb)
    g.close()


@pytest.mark.parametrize("T,n_q,batch,hq,hkv,room,form", [
    (6300, 9, 100, 8, 1, 60000, [(100, 8, 8, BY_CACHE, 1)]),             # whole tiles of several heads' queries, 8 waves
    (6300, 200, 96, 8, 2, 50000, [(128, 8, 1, BY_CACHE, 1), (64, 8, 1, BY_CACHE, 1)]),      # ... of one head
    (6300, 9, 96, 8, 2, 0, [(16, 8, 2, BY_CACHE, 6)] * 12), (6300, 200, 96, 8, 2, 0, [(16, 8, 1, BY_CACHE, 4)] * 12),     # the same in pieces
    (6200, 6200, 1, 8, 2, 0, [(2, 4, 1, BY_CACHE, 4)]),                  # a prompt in pieces
    (6400, 6400, 1, 32, 8, 0, [(8, 8, 1, BY_CACHE, 1)]),                 # a prompt past the line to 8 waves
])
def test_long_caches_against_decode_steps(kvq_mod, T, n_q, batch, hq, hkv, room, form):
    """The last query attends to everything, like a decode step; the query before it like the decode step of a cache that is one
    token shorter (checked on a second cache)."""
    gen = torch.Generator(device="cuda:0").manual_seed(T + n_q)
    g = kvq_mod.KVQ(1, batch, hq, hkv, 128, room or T, [4], [4])
    assert forms(g, T, n_q) == form
    K = torch.randn((batch, hkv, T, 128), generator=gen, device="cuda:0", dtype=torch.float16)
    V = torch.randn((batch, hkv, T, 128), generator=gen, device="cuda:0", dtype=torch.float16)
    q = torch.randn((batch, hq, n_q, 128), generator=gen, device="cuda:0", dtype=torch.float16)
    g.quantize_append(0, K, V)
    out = g.prefill_attention(0, q).double().cpu().numpy()
    assert np.all(np.isfinite(out))
    for back in (0, 1, 7):                  # (the window holds at least 32 tokens: both caches hold the same ones quantized)
        if T - back - 32 < 32 * ((T - 32) // 32):
            continue
        g.reset()
        g.quantize_append(0, K[:, :, :T - back].contiguous(), V[:, :, :T - back].contiguous())
        ref = g.decode_attention(0, q[:, :, n_q - 1 - back].contiguous()).double().cpu().numpy()
        assert np.linalg.norm(out[:, :, n_q - 1 - back] - ref) <= 1.5e-3 * np.linalg.norm(ref), back
    g.close()


@pytest.mark.parametrize("batch,hq,hkv,units,n_q,meta16", [
    (5, 5, 1, 257, 3, False), (3, 4, 2, 300, 3, True),              # 8 work-groups per cache; heads in two rounds
    (33, 2, 1, 290, 2, False), (33, 1, 1, 257, 1, True),            # 4
    (65, 1, 1, 258, 2, True),                                       # 2
    (129, 1, 1, 257, 1, False),                                     # 1: more than one round of loads
    (2, 12, 2, 256, 70, False), (2, 4, 2, 65, 5, True), (1, 4, 2, 64, 64, False), (1, 3, 1, 3, 4, True),   # 1: whole rounds, one unit more, few units
])
def test_selection_by_several_work_groups(kvq_mod, oracle_mod, batch, hq, hkv, units, n_q, meta16):
    """Channel selection of caches on either side of the line to several work-groups per cache: keys with large channels and an
    offset on every channel, which only come out right if every unit counts once in the centres."""
    w = W.Workload("parts", 1, batch, hq, hkv, 128, 32 * units + 33, [4], [4], seed=1400 + batch + units, outlier_channels=4, outlier_scale=12.0, key_bias_std=6.0)
    out, o64, g, o, q = _run(kvq_mod, oracle_mod, w, n_q, meta=kvq_mod.META_FP16 if meta16 else None)
    assert_prefill_close(out, o64, "%d caches of %d units" % (batch * hkv, units))
    assert torch.equal(out, g.prefill_attention(0, q.cuda()))
    g.close()
