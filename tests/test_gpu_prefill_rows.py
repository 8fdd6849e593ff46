"""Prefill attention by the form its launch takes: work-groups of 4 waves and 128 rows or of 8 waves and 256, rows of one query head or of
several, whole tiles (started in pairs or in turn) or pieces."""
import numpy as np
import pytest
import torch

import kvq_workloads as W
from test_gpu_prefill import _run, assert_prefill_close, kvq_mod  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,n_q,batch,hq,hkv,residual,kb,vb", [
    # whole tiles, 4 waves, the group's heads together
    (300, 300, 1, 8, 2, 32, 4, 2),          # fewer work-groups than compute units, caches that do not divide by 8
    (225, 225, 4, 8, 2, 32, 8, 4),          # caches that divide by 8
    (700, 700, 8, 14, 2, 32, 4, 4),         # more than one work-group per compute unit, paired; rows that do not divide by the heads
    (700, 650, 5, 21, 3, 0, 2, 2),          # the same of 15 caches, no window
    (400, 400, 40, 4, 2, 32, 4, 2),         # more than two per compute unit
    (390, 390, 27, 6, 3, 100, 4, 2),        # ... of 81 caches, several window chunks
    (64, 64, 3, 12, 1, 500, 4, 2),          # window only
    (257, 129, 2, 3, 3, 32, 16, 16),        # one head per cache, fp16 keys; one row more than a work-group has
    (1, 1, 1, 4, 2, 32, 4, 4), (33, 2, 1, 16, 1, 0, 4, 4),
    # pieces
    (1600, 300, 4, 4, 2, 32, 4, 2),         # second tile: the second work-group of every piece has no rows
    (1600, 385, 4, 4, 2, 32, 4, 2),         # ... one row
    (2000, 5, 1, 8, 2, 32, 4, 2), (3000, 17, 2, 14, 2, 0, 8, 2), (3000, 64, 8, 8, 2, 32, 4, 4),      # a tile of several heads' queries
    (5000, 60, 16, 8, 2, 32, 4, 2),
    (2100, 33, 16, 28, 4, 32, 4, 2),
])
def test_rows_and_waves(kvq_mod, oracle_mod, T, n_q, batch, hq, hkv, residual, kb, vb):
    w = W.Workload("rows", 1, batch, hq, hkv, 128, T, [kb], [vb], seed=1200 + T + n_q, outlier_channels=3)
    g = kvq_mod.KVQ(1, batch, hq, hkv, 128, T, [kb], [vb], residual=residual)
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


@pytest.mark.parametrize("form", ["low parts of all channels", "wide keys", "offset on every channel", "fp16 scales", "per-token keys", "fp16 values"])
@pytest.mark.parametrize("T,n_q,hq,hkv", [(420, 420, 8, 2), (2500, 40, 8, 2)])
def test_forms_of_the_units_in_work_groups_of_four_waves(kvq_mod, oracle_mod, form, T, n_q, hq, hkv):
    vb = 16 if "values" in form else 4
    n, mult, offs = {"wide keys": (128, 12.0, 0.0), "offset on every channel": (0, 1.0, 20.0)}.get(form, (3, 12.0, 0.0))
    meta = kvq_mod.META_FP16 if "fp16 scales" in form else kvq_mod.META_FP32
    keys = kvq_mod.KEYS_PER_TOKEN if "per-token" in form else kvq_mod.KEYS_PER_CHANNEL
    w = W.Workload("row forms", 1, 4, hq, hkv, 128, T, [4], [vb], seed=1300 + T, outlier_channels=n, outlier_scale=mult, key_bias_std=offs)
    out, o64, g, o, q = _run(kvq_mod, oracle_mod, w, n_q, meta=meta, keys=keys, max_tokens=T, low_parts=1 if form.startswith("low") else None)
    assert_prefill_close(out, o64, form)
    g.close()


@pytest.mark.parametrize("T,n_q,batch,hq,hkv", [
    (6300, 9, 96, 8, 2),                    # whole tiles of several heads' queries, 8 waves
    (6300, 200, 96, 8, 2),                  # ... of one head
    (6200, 6200, 1, 8, 2),                  # a prompt past the line to 8 waves
])
def test_long_caches_against_decode_steps(kvq_mod, T, n_q, batch, hq, hkv):
    """The last query attends to everything, like a decode step; the query before it like the decode step of a cache that is one
    token shorter (checked on a second cache)."""
    gen = torch.Generator(device="cuda:0").manual_seed(T + n_q)
    g = kvq_mod.KVQ(1, batch, hq, hkv, 128, T, [4], [4])
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
