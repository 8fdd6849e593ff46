"""GPU parity: the HIP library (through its C ABI) against the CPU oracle on the same seeded inputs.

Bars: packed codes, scales, zero-points and the fp16 window are compared bit for bit through the
canonical export; attention outputs must satisfy max|gpu - oracle| <= 2e-3 and
||gpu - oracle||_2 / ||oracle||_2 <= 1e-3 per layer tensor (fp16 outputs, fp32 accumulation).
"""
import numpy as np
import pytest
import torch

import kvq_workloads as W

pytestmark = pytest.mark.gpu

MAX_ABS = 2e-3
REL_L2 = 1e-3


@pytest.fixture(scope="module")
def kvq_mod():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_04420_amd as pkg

    pkg.load_library()          # raises if the HIP library is not built: no fallback
    return pkg


@pytest.fixture(params=[1, 2], ids=["valu", "mfma"])
def variant(request):
    """Decode kernel variant: 1 = vector ALU, 2 = matrix core."""
    return request.param


def _np(t):
    t = t.cpu()
    return t.view(torch.uint16).numpy() if t.dtype == torch.float16 else t.numpy()


def assert_export_equal(gpu_dump, ora_dump, where=""):
    assert gpu_dump["n_packed"] == ora_dump["n_packed"] and gpu_dump["n_residual"] == ora_dump["n_residual"], where
    for key in ("k_codes", "k_scale", "k_zero", "v_codes", "v_scale", "v_zero", "k_res", "v_res"):
        if key not in ora_dump:
            assert key not in gpu_dump
            continue
        g, o = _np(gpu_dump[key]), ora_dump[key]
        assert g.shape == o.shape, (where, key, g.shape, o.shape)
        gb, ob = g.view(np.uint8), o.view(np.uint8)
        if not np.array_equal(gb, ob):
            bad = np.argwhere(gb != ob)
            raise AssertionError("%s %s: %d differing bytes, first at %s" % (where, key, len(bad), bad[0]))


def assert_outputs_close(gpu_out, ora_out16, ora_out64, where=""):
    g = gpu_out.float().cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(g)), where
    err = np.abs(g - ora_out64)
    rel = np.linalg.norm(g - ora_out64) / max(np.linalg.norm(ora_out64), 1e-30)
    assert err.max() <= MAX_ABS, (where, "max abs", err.max())
    assert rel <= REL_L2, (where, "rel l2", rel)
    return err.max(), rel


def _pair(kvq_mod, oracle_mod, w, max_tokens, kbits=None, vbits=None, residual=32, variant=0):
    kb = w.kbits if kbits is None else kbits
    vb = w.vbits if vbits is None else vbits
    g = kvq_mod.KVQ(len(kb), w.batch, w.n_q_heads, w.n_kv_heads, w.head_dim, max_tokens, kb, vb, residual=residual)
    g.set_decode_options(variant, 0)
    o = oracle_mod.OracleCache(len(kb), w.batch, w.n_q_heads, w.n_kv_heads, w.head_dim, kb, vb, residual=residual)
    return g, o


def test_generator_is_bit_identical_on_cpu_and_gpu(kvq_mod):
    w = W.config4(batch=2, context=200)
    for layer in (0, 3):
        kc, vc = W.kv_tokens(w, layer, 0, 200)
        kg, vg = W.kv_tokens(w, layer, 0, 200, device="cuda:0")
        assert torch.equal(kc, kg.cpu()) and torch.equal(vc, vg.cpu())
        assert torch.equal(W.query(w, layer, 5), W.query(w, layer, 5, device="cuda:0").cpu())


def test_config1_every_element(kvq_mod, oracle_mod, variant):
    """The small correctness configuration: 1 layer, 8 q / 2 kv heads, 512 tokens, K8V4, 4 outlier channels."""
    w = W.config1()
    g, o = _pair(kvq_mod, oracle_mod, w, 1024, variant=variant)
    K, V = W.kv_tokens(w, 0, 0, w.context)
    q = W.query(w, 0)
    g.quantize_append(0, K.cuda(), V.cuda())
    o.quantize_append(0, K.numpy(), V.numpy())
    assert g.layer_tokens(0) == (480, 32)
    assert_export_equal(g.debug_export(0), o.export(0), "cfg1")
    out = g.decode_attention(0, q.cuda())
    o16, o64 = o.decode_attention(0, q.numpy())
    assert_outputs_close(out, o16, o64, "cfg1")


PAIRS = [(8, 8), (8, 4), (8, 2), (4, 8), (4, 4), (4, 2), (2, 8), (2, 4), (2, 2), (16, 16), (16, 4), (2, 16), (8, 16), (16, 8)]


@pytest.mark.parametrize("kb,vb", PAIRS)
def test_all_precision_pairs(kvq_mod, oracle_mod, kb, vb, variant):
    """Several blocks plus a ragged fp16 tail (5 blocks + 51 window tokens), batch 2, g_q = 4."""
    w = W.Workload("pairs", 1, 2, 8, 2, 128, 32 * 6 + 19, [kb], [vb], seed=100 + kb * 17 + vb, outlier_channels=3)
    g, o = _pair(kvq_mod, oracle_mod, w, 512, variant=variant)
    K, V = W.kv_tokens(w, 0, 0, w.context)
    q = W.query(w, 0)
    g.quantize_append(0, K.cuda(), V.cuda())
    o.quantize_append(0, K.numpy(), V.numpy())
    assert_export_equal(g.debug_export(0), o.export(0), "K%dV%d" % (kb, vb))
    out = g.decode_attention(0, q.cuda())
    o16, o64 = o.decode_attention(0, q.numpy())
    assert_outputs_close(out, o16, o64, "K%dV%d" % (kb, vb))


@pytest.mark.parametrize("kb,vb", [(8, 8), (8, 4), (4, 4), (4, 2), (2, 2), (16, 4), (2, 16)])
def test_fp16_scale_variant(kvq_mod, oracle_mod, kb, vb, variant):
    """Narrow metadata (scales rounded to fp16 and used that way): same bars against the oracle in the same mode,
    through chunked appends with window flushes, g_q = 7, a tiny-range channel whose scale underflows in fp16."""
    w = W.Workload("meta16", 1, 2, 14, 2, 128, 32 * 7 + 11, [kb], [vb], seed=900 + kb * 17 + vb, outlier_channels=3)
    g = kvq_mod.KVQ(1, w.batch, w.n_q_heads, w.n_kv_heads, w.head_dim, 512, [kb], [vb], meta_dtype=kvq_mod.META_FP16)
    g.set_decode_options(variant, 0)
    o = oracle_mod.OracleCache(1, w.batch, w.n_q_heads, w.n_kv_heads, w.head_dim, [kb], [vb], scale_fp16=True)
    K, V = W.kv_tokens(w, 0, 0, w.context)
    K[:, :, :, 9] = (K[:, :, :, 9] * 2.0 ** -22).to(torch.float16)        # subnormal fp16 inputs: scale ~ 2^-24 .. 0 in fp16
    V[:, :, 40:80, 32:64] = (V[:, :, 40:80, 32:64] * 2.0 ** -21).to(torch.float16)
    pos = 0
    for n in (100, 1, 31, 64, w.context - 196):
        g.quantize_append(0, K[:, :, pos:pos + n].contiguous().cuda(), V[:, :, pos:pos + n].contiguous().cuda())
        o.quantize_append(0, np.ascontiguousarray(K[:, :, pos:pos + n].numpy()), np.ascontiguousarray(V[:, :, pos:pos + n].numpy()))
        pos += n
    gd, od = g.debug_export(0), o.export(0)
    assert_export_equal(gd, od, "meta16 K%dV%d" % (kb, vb))
    for key in ("k_scale", "v_scale"):
        if key in od:          # every scale in use is an fp16 number
            assert np.array_equal(od[key].astype(np.float16).astype(np.float32), od[key])
    q = W.query(w, 0)
    out = g.decode_attention(0, q.cuda())
    o16, o64 = o.decode_attention(0, q.numpy())
    assert_outputs_close(out, o16, o64, "meta16 K%dV%d" % (kb, vb))


@pytest.mark.parametrize("meta16", [False, True], ids=["fp32scales", "fp16scales"])
@pytest.mark.parametrize("kb,vb,gq", [(8, 8, 4), (8, 4, 7), (4, 4, 4), (4, 2, 2), (2, 2, 8), (4, 16, 4), (2, 8, 5), (16, 4, 4)])
def test_per_token_key_grouping(kvq_mod, oracle_mod, kb, vb, gq, meta16, variant):
    """Keys grouped per token like the values (the paper's per-token-asym mode): canonical export (its key arrays have
    the value arrays' form) and outputs against the oracle in the same mode; chunked appends, biased keys."""
    hkv = 2
    w = W.Workload("kpt", 1, 2, gq * hkv, hkv, 128, 32 * 6 + 27, [kb], [vb], seed=1200 + kb * 17 + vb, outlier_channels=3,
                   key_bias_std=4.0)
    g = kvq_mod.KVQ(1, w.batch, w.n_q_heads, hkv, 128, 512, [kb], [vb], key_mode=kvq_mod.KEYS_PER_TOKEN,
                    meta_dtype=kvq_mod.META_FP16 if meta16 else kvq_mod.META_FP32)
    g.set_decode_options(variant, 0)
    o = oracle_mod.OracleCache(1, w.batch, w.n_q_heads, hkv, 128, [kb], [vb], key_per_token=True, scale_fp16=meta16)
    K, V = W.kv_tokens(w, 0, 0, w.context)
    pos = 0
    for n in (70, 1, 1, 95, w.context - 167):
        g.quantize_append(0, K[:, :, pos:pos + n].contiguous().cuda(), V[:, :, pos:pos + n].contiguous().cuda())
        o.quantize_append(0, np.ascontiguousarray(K[:, :, pos:pos + n].numpy()), np.ascontiguousarray(V[:, :, pos:pos + n].numpy()))
        pos += n
    gd, od = g.debug_export(0), o.export(0)
    if kb < 16:
        assert tuple(gd["k_scale"].shape) == (2, hkv, od["n_packed"], 4)
    assert_export_equal(gd, od, "per-token keys K%dV%d" % (kb, vb))
    for step in range(2):
        q = W.query(w, 0, step)
        out = g.decode_attention(0, q.cuda())
        o16, o64 = o.decode_attention(0, q.numpy())
        assert_outputs_close(out, o16, o64, "per-token keys K%dV%d step %d" % (kb, vb, step))


@pytest.mark.parametrize("gq,hkv", [(1, 3), (2, 2), (3, 1), (4, 2), (5, 1), (7, 4), (8, 1), (12, 1), (16, 1)])
def test_query_group_sizes(kvq_mod, oracle_mod, gq, hkv, variant):
    w = W.Workload("gq", 1, 2, gq * hkv, hkv, 128, 32 * 4 + 7, [4], [2], seed=200 + gq, key_bias_std=20.0)
    g, o = _pair(kvq_mod, oracle_mod, w, 256, variant=variant)
    K, V = W.kv_tokens(w, 0, 0, w.context)
    q = W.query(w, 0)
    g.quantize_append(0, K.cuda(), V.cuda())
    o.quantize_append(0, K.numpy(), V.numpy())
    assert_export_equal(g.debug_export(0), o.export(0), "gq%d" % gq)
    out = g.decode_attention(0, q.cuda())
    o16, o64 = o.decode_attention(0, q.numpy())
    assert_outputs_close(out, o16, o64, "gq%d" % gq)


@pytest.mark.parametrize("T", [1, 2, 31, 32, 33, 63, 64, 65, 95, 96, 97, 128])
def test_short_and_ragged_lengths(kvq_mod, oracle_mod, T, variant):
    w = W.Workload("short", 1, 1, 4, 1, 128, T, [2], [4], seed=300 + T)
    g, o = _pair(kvq_mod, oracle_mod, w, 128, variant=variant)
    K, V = W.kv_tokens(w, 0, 0, T)
    q = W.query(w, 0)
    g.quantize_append(0, K.cuda(), V.cuda())
    o.quantize_append(0, K.numpy(), V.numpy())
    assert g.layer_tokens(0) == o.tokens(0)
    assert_export_equal(g.debug_export(0), o.export(0), "T%d" % T)
    out = g.decode_attention(0, q.cuda())
    o16, o64 = o.decode_attention(0, q.numpy())
    assert_outputs_close(out, o16, o64, "T%d" % T)


@pytest.mark.parametrize("residual", [0, 32, 64])
@pytest.mark.parametrize("chunks", [[1] * 70, [31, 33, 1, 64, 38, 30], [197], [63, 1, 1, 132]])
def test_chunked_appends_match_oracle_bulk(kvq_mod, oracle_mod, chunks, residual, variant):
    """However the tokens arrive, the cache equals the oracle's after one bulk append (window flush logic)."""
    T = sum(chunks)
    w = W.Workload("chunks", 1, 2, 4, 2, 128, T, [8], [2], seed=400 + len(chunks), outlier_channels=2)
    g, o = _pair(kvq_mod, oracle_mod, w, 256, residual=residual, variant=variant)
    K, V = W.kv_tokens(w, 0, 0, T)
    o.quantize_append(0, K.numpy(), V.numpy())
    Kd, Vd = K.cuda(), V.cuda()
    t = 0
    for n in chunks:
        g.quantize_append(0, Kd[:, :, t:t + n].contiguous(), Vd[:, :, t:t + n].contiguous())
        t += n
    assert_export_equal(g.debug_export(0), o.export(0), "chunks")
    q = W.query(w, 0)
    out = g.decode_attention(0, q.cuda())
    o16, o64 = o.decode_attention(0, q.numpy())
    assert_outputs_close(out, o16, o64, "chunks")


@pytest.mark.parametrize("residual", [0, 32, 100])
@pytest.mark.parametrize("chunks", [[63, 40, 90], [40, 24, 1, 128], [50, 45, 98], [95, 1, 97]])
def test_append_that_flushes_and_fills_the_window(kvq_mod, oracle_mod, chunks, residual):
    """Appends that quantize groups and put new tokens into the ring: in one launch, or in two where a new token takes the
    slot of one that is being quantized (63 + 40 tokens at a window of 32: positions 64.. over 0..).  State after each."""
    w = W.Workload("ring", 1, 3, 4, 2, 128, sum(chunks), [4], [4], seed=450 + len(chunks), outlier_channels=2)
    g, o = _pair(kvq_mod, oracle_mod, w, 256, residual=residual)
    K, V = W.kv_tokens(w, 0, 0, w.context)
    t = 0
    for n in chunks:
        k1, v1 = K[:, :, t:t + n].contiguous(), V[:, :, t:t + n].contiguous()
        g.quantize_append(0, k1.cuda(), v1.cuda())
        o.quantize_append(0, k1.numpy(), v1.numpy())
        t += n
        assert_export_equal(g.debug_export(0), o.export(0), "after %d tokens" % t)


def test_decode_loop_with_flushes(kvq_mod, oracle_mod, variant):
    """Prefill, then 70 decode steps that append one token each (two window flushes), checked every step."""
    w = W.Workload("loop", 2, 2, 8, 2, 128, 100, [4, 8], [2, 4], seed=500, outlier_channels=3)
    g, o = _pair(kvq_mod, oracle_mod, w, 256, variant=variant)
    for layer in range(2):
        K, V = W.kv_tokens(w, layer, 0, 100)
        g.quantize_append(layer, K.cuda(), V.cuda())
        o.quantize_append(layer, K.numpy(), V.numpy())
    for step in range(70):
        for layer in range(2):
            K, V = W.kv_tokens(w, layer, step, step + 1, stream=1, total=70)
            g.quantize_append(layer, K.cuda(), V.cuda())
            o.quantize_append(layer, K.numpy(), V.numpy())
            q = W.query(w, layer, step)
            out = g.decode_attention(layer, q.cuda())
            o16, o64 = o.decode_attention(layer, q.numpy())
            assert_outputs_close(out, o16, o64, "step %d layer %d" % (step, layer))
        if step in (0, 27, 28, 59, 60, 69):
            for layer in range(2):
                assert_export_equal(g.debug_export(layer), o.export(layer), "step %d layer %d" % (step, layer))


@pytest.mark.parametrize("splits", [1, 2, 3, 7, 16, 64, 128])
def test_result_does_not_depend_on_splits(kvq_mod, oracle_mod, variant, splits):
    w = W.Workload("splits", 1, 1, 8, 2, 128, 32 * 40 + 45, [4], [4], seed=600, outlier_channels=3)
    g, o = _pair(kvq_mod, oracle_mod, w, 2048)
    K, V = W.kv_tokens(w, 0, 0, w.context)
    g.quantize_append(0, K.cuda(), V.cuda())
    o.quantize_append(0, K.numpy(), V.numpy())
    q = W.query(w, 0)
    o16, o64 = o.decode_attention(0, q.numpy())
    g.set_decode_options(variant, splits)
    out = g.decode_attention(0, q.cuda())
    assert_outputs_close(out, o16, o64, "splits %d" % splits)
    # deterministic: same launch twice gives the same bits
    out2 = g.decode_attention(0, q.cuda())
    assert torch.equal(out, out2)


@pytest.mark.parametrize("kb,vb,gq,splits", [(4, 2, 4, 1), (2, 2, 7, 1), (8, 4, 4, 2), (4, 8, 8, 1), (8, 8, 3, 3)])
def test_one_group_sweeps_many_chunks(kvq_mod, oracle_mod, kb, vb, gq, splits):
    """The matrix-core kernel fetches per-block exponents for 48 steps of a group's sweep at a time and the keys'
    zero-points for 16: a group that owns 50..101 blocks crosses several chunk boundaries of both kinds, with a ragged
    last chunk (the bench shapes give a group 16 blocks)."""
    w = W.Workload("chunks", 1, 2, gq * 2, 2, 128, 32 * 101 + 45, [kb], [vb], seed=640 + kb + vb, outlier_channels=3, key_bias_std=4.0)
    g, o = _pair(kvq_mod, oracle_mod, w, 4096)
    K, V = W.kv_tokens(w, 0, 0, w.context)
    g.quantize_append(0, K.cuda(), V.cuda())
    o.quantize_append(0, K.numpy(), V.numpy())
    g.set_decode_options(2, splits)
    for step in range(2):
        q = W.query(w, 0, step)
        o16, o64 = o.decode_attention(0, q.numpy())
        assert_outputs_close(g.decode_attention(0, q.cuda()), o16, o64, "K%dV%d gq %d splits %d" % (kb, vb, gq, splits))


@pytest.mark.parametrize("gq,residual,splits", [(4, 150, 0), (7, 32, 1), (8, 0, 2), (3, 90, 3)])
@pytest.mark.parametrize("kb,vb", [(16, 16), (16, 4), (4, 16), (4, 2)])
def test_fp16_row_units_and_window_chunks(kvq_mod, oracle_mod, kb, vb, gq, residual, splits):
    """fp16 rows of the matrix-core kernel: 16-bit units of which the next is in flight (odd and even numbers of them, one
    group or several), windows of one to six chunks that wrap around the ring, the appended row in the last of them."""
    w = W.Workload("rows", 1, 2, gq * 2, 2, 128, 32 * 9 + residual + 21, [kb], [vb], seed=660 + kb + vb + gq, outlier_channels=2)
    g, o = _pair(kvq_mod, oracle_mod, w, w.context + 20, residual=residual)
    K, V = W.kv_tokens(w, 0, 0, w.context)
    g.quantize_append(0, K.cuda(), V.cuda())
    o.quantize_append(0, K.numpy(), V.numpy())
    g.set_decode_options(2, splits)
    Kn, Vn = W.kv_tokens(w, 0, 0, 14, stream=1, total=14)
    for step in range(14):                                   # 21 + 14 > 32: one flush on the way
        k1, v1, q = Kn[:, :, step:step + 1].contiguous(), Vn[:, :, step:step + 1].contiguous(), W.query(w, 0, step)
        out = g.append_decode_attention(0, k1.cuda(), v1.cuda(), q.cuda())
        o.quantize_append(0, k1.numpy(), v1.numpy())
        if step in (0, 9, 10, 11, 13):
            o16, o64 = o.decode_attention(0, q.numpy())
            assert_outputs_close(out, o16, o64, "step %d" % step)
            assert torch.equal(out, g.decode_attention(0, q.cuda()))
    assert_export_equal(g.debug_export(0), o.export(0), "after the steps")


def test_biased_keys_gq7_mixed_layers(kvq_mod, oracle_mod, variant):
    """Shape of the Qwen configuration in small: g_q = 7, keys with a large per-channel offset, K8V2 / K4V2 layers."""
    w = W.config4(batch=2, context=32 * 20 + 32)
    w.n_layers, w.kbits, w.vbits = 2, [8, 4], [2, 2]
    g, o = _pair(kvq_mod, oracle_mod, w, 1024, variant=variant)
    for layer in range(2):
        K, V = W.kv_tokens(w, layer, 0, w.context)
        g.quantize_append(layer, K.cuda(), V.cuda())
        o.quantize_append(layer, K.numpy(), V.numpy())
        assert_export_equal(g.debug_export(layer), o.export(layer), "layer %d" % layer)
        q = W.query(w, layer)
        out = g.decode_attention(layer, q.cuda())
        o16, o64 = o.decode_attention(layer, q.numpy())
        assert_outputs_close(out, o16, o64, "layer %d" % layer)


def test_tie_heavy_keys_are_coded_identically(kvq_mod, oracle_mod):
    """Keys on a coarse dyadic grid (many exact .5 quotients) and constant groups: codes still match bit for bit."""
    torch.manual_seed(7)
    B, H, T, D = 1, 2, 96, 128
    K = (torch.randint(-40, 40, (B, H, T, D)).float() * 0.25).to(torch.float16)
    K[:, :, :, 5] = 3.0                      # constant channel -> s = 0
    V = (torch.randint(-6, 7, (B, H, T, D)).float() * 0.5).to(torch.float16)
    V[:, :, 10, 32:64] = -2.0                # constant value group
    for kb, vb in ((2, 2), (4, 4), (8, 8)):
        w = W.Workload("ties", 1, B, 4, H, D, T, [kb], [vb], seed=1)
        g, o = _pair(kvq_mod, oracle_mod, w, 128)
        g.quantize_append(0, K.cuda(), V.cuda())
        o.quantize_append(0, K.numpy(), V.numpy())
        assert_export_equal(g.debug_export(0), o.export(0), "ties K%dV%d" % (kb, vb))


def test_quotients_next_to_ties_are_coded_identically(kvq_mod, oracle_mod):
    """Adversarial groups for the encoder: inputs whose quotient (x - z) / s lies within a few fp32 ulp of k + 1/2
    without being a tie, found by search over fp16 values.  A rounding shortcut that is not exact fails here."""
    rng = np.random.default_rng(11)
    B, H, T, D = 1, 1, 64, 128
    for bits in (8, 4, 2):
        levels = (1 << bits) - 1
        K = np.zeros((B, H, T, D), dtype=np.float16)
        found = 0
        for d in range(D):
            # a channel = two key groups (tokens 0..31, 32..63) sharing min 0 and max R
            R = np.float16(rng.uniform(0.5, 60.0))
            s32 = np.float32(R) / np.float32(levels)
            xs = np.arange(1, int(np.float16(R).view(np.uint16)), dtype=np.uint16).view(np.float16)   # all fp16 in (0, R)
            q = xs.astype(np.float64) / np.float64(s32)
            dist = np.abs(q - np.floor(q) - 0.5)
            near = xs[(dist < 3e-5 * np.maximum(q, 1.0)) & (dist > 0)]
            if len(near) == 0:
                near = xs[np.argsort(dist)[:30]]
            found += len(near)
            col = rng.choice(near, size=T)
            col[0] = col[32] = 0.0
            col[1] = col[33] = R
            K[0, 0, :, d] = col
        assert found >= D
        V = K.copy()          # value groups (32 channels of a token) see the same numbers grouped differently
        w = W.Workload("near-ties", 1, B, 4, H, D, T, [bits], [bits], seed=1)
        g, o = _pair(kvq_mod, oracle_mod, w, 128, residual=0)
        g.quantize_append(0, torch.from_numpy(K).cuda(), torch.from_numpy(V).cuda())
        o.quantize_append(0, K, V)
        assert_export_equal(g.debug_export(0), o.export(0), "near ties %d bit" % bits)


@pytest.mark.parametrize("residual", [0, 32, 64])
@pytest.mark.parametrize("kb,vb", [(4, 2), (8, 8), (16, 4), (2, 16)])
def test_fused_append_decode_step(kvq_mod, oracle_mod, kb, vb, residual, variant):
    """kvq_append_decode_attention over 70 decode steps (window flushes included) against the oracle's append + decode,
    and bit for bit against the two separate calls on a second cache; the cache state at the end is compared too."""
    w = W.Workload("fused", 1, 2, 8, 2, 128, 32 * 3 + 5, [kb], [vb], seed=1500 + kb * 17 + vb + residual, outlier_channels=3)
    g, o = _pair(kvq_mod, oracle_mod, w, 256, residual=residual, variant=variant)
    g2, _ = _pair(kvq_mod, oracle_mod, w, 256, residual=residual, variant=variant)
    K, V = W.kv_tokens(w, 0, 0, w.context)
    for c in (g, g2):
        c.quantize_append(0, K.cuda(), V.cuda())
    o.quantize_append(0, K.numpy(), V.numpy())
    steps = 70
    Kn, Vn = W.kv_tokens(w, 0, 0, steps, stream=1, total=steps)
    for s_ in range(steps):
        k1, v1 = Kn[:, :, s_:s_ + 1].contiguous(), Vn[:, :, s_:s_ + 1].contiguous()
        q = W.query(w, 0, s_)
        out = g.append_decode_attention(0, k1.cuda(), v1.cuda(), q.cuda())
        g2.quantize_append(0, k1.cuda(), v1.cuda())
        out2 = g2.decode_attention(0, q.cuda())
        assert torch.equal(out, out2), "step %d: fused call differs from append + decode" % s_
        o.quantize_append(0, k1.numpy(), v1.numpy())
        if s_ % 7 == 0 or s_ == steps - 1:
            o16, o64 = o.decode_attention(0, q.numpy())
            assert_outputs_close(out, o16, o64, "fused step %d" % s_)
    assert g.layer_tokens(0) == g2.layer_tokens(0) == o.tokens(0)
    assert_export_equal(g.debug_export(0), o.export(0), "after fused steps")
    with pytest.raises(kvq_mod.KVQError):            # capacity: 101 + 70 = 171 tokens held, 256 allowed
        for _ in range(100):
            g.append_decode_attention(0, k1.cuda(), v1.cuda(), q.cuda())
    assert g.layer_tokens(0)[0] + g.layer_tokens(0)[1] == 256


def test_sixteen_bit_mode_equals_exact_attention(kvq_mod, oracle_mod, variant):
    w = W.Workload("fp16", 1, 2, 8, 2, 128, 300, [16], [16], seed=700)
    g, _ = _pair(kvq_mod, oracle_mod, w, 512, variant=variant)
    K, V = W.kv_tokens(w, 0, 0, 300)
    q = W.query(w, 0)
    g.quantize_append(0, K.cuda(), V.cuda())
    out = g.decode_attention(0, q.cuda())
    e16, e64 = oracle_mod.attention_exact(q.numpy(), K.numpy(), V.numpy())
    assert_outputs_close(out, e16, e64, "fp16 exact")


def test_reset_and_reuse(kvq_mod, oracle_mod):
    w = W.Workload("reset", 1, 1, 4, 1, 128, 80, [4], [4], seed=800)
    g, o = _pair(kvq_mod, oracle_mod, w, 128)
    K, V = W.kv_tokens(w, 0, 0, 80)
    g.quantize_append(0, K.cuda(), V.cuda())
    g.reset(0)
    assert g.layer_tokens(0) == (0, 0)
    with pytest.raises(kvq_mod.KVQError):
        g.decode_attention(0, W.query(w, 0).cuda())
    K2, V2 = W.kv_tokens(w, 0, 0, 70, stream=1, total=70)
    g.quantize_append(0, K2.cuda(), V2.cuda())
    o.quantize_append(0, K2.numpy(), V2.numpy())
    assert_export_equal(g.debug_export(0), o.export(0), "after reset")
    with pytest.raises(kvq_mod.KVQError):
        g.quantize_append(0, K.cuda(), V.cuda())       # 70 + 80 > 128 tokens


@pytest.mark.parametrize("meta16", [False, True], ids=["fp32scales", "fp16scales"])
@pytest.mark.parametrize("per_token", [False, True], ids=["keys-per-channel", "keys-per-token"])
@pytest.mark.parametrize("kb,vb", [(4, 2), (8, 8), (2, 4)])
def test_signed_zero_extremes(kvq_mod, oracle_mod, kb, vb, per_token, meta16):
    """Groups whose minimum (or maximum) is zero and that hold +0 and -0 in both orders, only -0, or zeros only:
    the zero-point and the scale are stored with a zero extreme as +0, so k_zero / v_zero / k_scale / v_scale agree
    with the oracle bit for bit whatever order the kernel's reduction meets the zeros in."""
    rng = np.random.default_rng(77)
    B, H, T, D = 2, 2, 128, 128
    K = (np.abs(rng.standard_normal((B, H, T, D))) + 0.25).astype(np.float16)
    V = K.copy()
    pz, nz = np.float16(0.0), np.float16(-0.0)
    # key groups over tokens (per channel): block 0 (+0 before -0), block 1 (-0 before +0), block 2 (-0 only, rest
    # negative: zero maximum), block 3 (all zeros of mixed sign) -- on some channels each, at several lane rows
    for ch in (0, 1, 17, 64, 127):
        K[:, :, 2, ch], K[:, :, 29, ch] = pz, nz
        K[:, :, 32 + 1, ch], K[:, :, 32 + 30, ch] = nz, pz
        K[:, :, 64:96, ch] = -K[:, :, 64:96, ch]
        K[:, :, 64 + 7, ch] = nz
        K[:, :, 96:128:2, ch], K[:, :, 97:128:2, ch] = nz, pz
    # groups over channels (values, and keys when grouped per token): the same four cases on several tokens
    for X in (V, K):
        for t in (0, 5, 40, 77, 127):
            X[:, :, t, 3], X[:, :, t, 30] = pz, nz
            X[:, :, t, 32 + 4], X[:, :, t, 32 + 9] = nz, pz
            X[:, :, t, 64:96] = -np.abs(X[:, :, t, 64:96])
            X[:, :, t, 64 + 21] = nz
            X[:, :, t, 96:128:2], X[:, :, t, 97:128:2] = pz, nz
    g = kvq_mod.KVQ(1, B, 4 * H, H, D, 256, [kb], [vb], residual=0,
                    key_mode=kvq_mod.KEYS_PER_TOKEN if per_token else kvq_mod.KEYS_PER_CHANNEL,
                    meta_dtype=kvq_mod.META_FP16 if meta16 else kvq_mod.META_FP32)
    o = oracle_mod.OracleCache(1, B, 4 * H, H, D, [kb], [vb], residual=0, key_per_token=per_token, scale_fp16=meta16)
    # in two chunks, so that the second one is encoded out of the window ring
    for a, b in ((0, 50), (50, T)):
        g.quantize_append(0, torch.from_numpy(np.ascontiguousarray(K[:, :, a:b])).cuda(), torch.from_numpy(np.ascontiguousarray(V[:, :, a:b])).cuda())
        o.quantize_append(0, np.ascontiguousarray(K[:, :, a:b]), np.ascontiguousarray(V[:, :, a:b]))
    gd, od = g.debug_export(0), o.export(0)
    assert_export_equal(gd, od, "signed zeros K%dV%d" % (kb, vb))
    for key in ("k_zero", "v_zero", "k_scale", "v_scale"):
        assert not np.any(od[key].view(np.uint32) == 0x80000000), key       # the cases are really there and canonical
        assert np.any(od[key].view(np.uint32) == 0), key


@pytest.mark.parametrize("kb,vb", [(4, 2), (2, 2), (8, 4), (4, 8)])
def test_groups_spanning_the_fp16_range(kvq_mod, oracle_mod, kb, vb, variant):
    """Keys and values whose groups span most of the fp16 range (about -6e4 .. 6e4) next to groups of ordinary and of
    tiny magnitude in the same block: the scales of one block then differ by more than 2^30, which is the stress for
    the lifting of the matrix-core operands by the block's largest scale exponent.  Codes, scales and zero-points bit
    for bit; outputs within the bars (queries are small on the huge channels so that the logits stay finite)."""
    w = W.Workload("span", 1, 2, 8, 2, 128, 32 * 5 + 9, [kb], [vb], seed=1700 + kb * 17 + vb, outlier_channels=3)
    g, o = _pair(kvq_mod, oracle_mod, w, 512, variant=variant)
    K, V = W.kv_tokens(w, 0, 0, w.context)
    q = W.query(w, 0)
    big = torch.tensor([7, 40, 41, 100])
    K[:, :, :, big] = (K[:, :, :, big].float() * 2.0e4).clamp(-6.0e4, 6.0e4).to(torch.float16)
    K[:, :, :, 8] = (K[:, :, :, 8].float() * 2.0 ** -18).to(torch.float16)               # subnormal-range channel
    q[:, :, big] = (q[:, :, big].float() * 2.0 ** -14).to(torch.float16)
    V[:, :, 3::7, 32:64] = (V[:, :, 3::7, 32:64].float() * 2.0e4).clamp(-6.0e4, 6.0e4).to(torch.float16)
    V[:, :, 5::11, 96:128] = (V[:, :, 5::11, 96:128].float() * 2.0 ** -16).to(torch.float16)
    g.quantize_append(0, K.cuda(), V.cuda())
    o.quantize_append(0, K.numpy(), V.numpy())
    assert_export_equal(g.debug_export(0), o.export(0), "span K%dV%d" % (kb, vb))
    out = g.decode_attention(0, q.cuda())
    o16, o64 = o.decode_attention(0, q.numpy())
    # Outputs reach the magnitude of the large values, so the absolute bar grows with the output's own fp16 spacing.
    # The matrix-core kernel gets one more term.  Its products p s c of a block's 32 tokens are summed by the matrix
    # core, which aligns them to the largest one and drops what lies more than about 24 bits below that product's
    # nominal exponent (the codes are fp16 subnormals: up to 6 leading zero bits); 32 products, truncated: the sum of a
    # block is off by up to 2^-13, typically 2^-14, of the largest product p s c <= p * (group range), and the output,
    # a weighted mean over blocks, by that fraction of the largest value-group range in the cache.  For N(0,1) values
    # (range about 5) that is 3e-4, inside the 2e-3 bar that all other tests apply unchanged; here the range is 1.2e5.
    gpu = out.float().cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(gpu))
    od = o.export(0)
    largest_range = float(od["v_scale"].max()) * ((1 << vb) - 1)
    bar = MAX_ABS + 2.0 ** -10 * np.abs(o64) + (2.0 ** -14 * largest_range if variant == 2 else 0.0)
    excess = float((np.abs(gpu - o64) - bar).max())
    assert excess <= 0.0, ("worst element exceeds its bar by", excess, "largest value-group range", largest_range)
    rel = float(np.linalg.norm(gpu - o64) / np.linalg.norm(o64))
    assert rel <= REL_L2, ("rel l2", rel)
