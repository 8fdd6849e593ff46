"""CPU-only checks of the product's host side: the C ABI loads and exports what include/kvq.h declares,
argument validation returns the documented codes without touching a GPU, and the schedule helpers."""
import ctypes
import os
import re
import time

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    from paper_2502_04420_amd import binding

    if not os.path.exists(binding.library_path()):
        from paper_2502_04420_amd.build import build

        build(verbose=False)
    return binding.load_library()


def _declared_functions():
    text = open(os.path.join(ROOT, "include", "kvq.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(kvq_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol(lib):
    names = _declared_functions()
    assert {"kvq_configure", "kvq_quantize_append", "kvq_decode_attention", "kvq_workspace_bytes"} <= set(names)
    for name in names:
        assert getattr(lib, name) is not None, name
    from paper_2502_04420_amd import binding

    assert sorted(binding.EXPORTED) == names


def _cfg(**over):
    from paper_2502_04420_amd import binding

    kw = dict(n_layers=2, batch=2, n_q_heads=8, n_kv_heads=2, head_dim=128, max_tokens=256, kbits=[8, 4], vbits=[4, 2])
    kw.update(over)
    return binding.make_config(**kw)


def test_workspace_bytes_and_config_validation(lib):
    cfg, keep = _cfg()
    need = lib.kvq_workspace_bytes(ctypes.byref(cfg))
    assert need > 0 and need % 256 == 0
    # codes + metadata of 8 blocks per (b, h) for both layers must fit
    assert need >= 4 * 8 * ((4096 + 2048 + 2 * 768) + (2048 + 1024 + 2 * 768))
    c16, k16 = _cfg(meta_dtype=1)          # fp16 scales: 256 bytes less per block and tensor
    need16 = lib.kvq_workspace_bytes(ctypes.byref(c16))
    assert 0 < need16 < need and need - need16 >= 4 * 8 * 4 * 256
    for bad in (dict(head_dim=64), dict(group=16), dict(n_q_heads=7), dict(kbits=[8, 3]), dict(vbits=[1, 2]),
                dict(max_tokens=0), dict(batch=0), dict(residual=-1), dict(meta_dtype=2), dict(key_mode=2), dict(batch=32768)):
        c, k = _cfg(**bad)
        assert lib.kvq_workspace_bytes(ctypes.byref(c)) == 0, bad
        h = ctypes.c_void_p()
        assert lib.kvq_configure(ctypes.byref(h), ctypes.byref(c), ctypes.c_void_p(256), 1 << 40, None) == -1, bad
    assert lib.kvq_workspace_bytes(None) == 0


def test_configure_and_call_errors_without_gpu(lib):
    cfg, keep = _cfg()
    need = lib.kvq_workspace_bytes(ctypes.byref(cfg))
    h = ctypes.c_void_p()
    assert lib.kvq_configure(ctypes.byref(h), ctypes.byref(cfg), None, need, None) == -4          # no workspace
    assert lib.kvq_configure(ctypes.byref(h), ctypes.byref(cfg), ctypes.c_void_p(256 + 8), need, None) == -4   # misaligned
    assert lib.kvq_configure(ctypes.byref(h), ctypes.byref(cfg), ctypes.c_void_p(256), need - 1, None) == -4   # too small
    assert lib.kvq_configure(None, ctypes.byref(cfg), ctypes.c_void_p(256), need, None) == -1
    # a fake (never dereferenced) workspace pointer is enough for the host-side checks below
    assert lib.kvq_configure(ctypes.byref(h), ctypes.byref(cfg), ctypes.c_void_p(256), need, None) == 0
    try:
        fake = ctypes.c_void_p(4096)
        assert lib.kvq_decode_attention(h, 0, fake, fake) == -3          # no token yet
        assert lib.kvq_decode_attention(h, 2, fake, fake) == -1          # bad layer
        assert lib.kvq_decode_attention(h, 0, None, fake) == -1
        assert lib.kvq_quantize_append(h, -1, fake, fake, 1) == -1
        assert lib.kvq_quantize_append(h, 0, fake, fake, 0) == -1
        assert lib.kvq_quantize_append(h, 0, fake, None, 1) == -1
        assert lib.kvq_quantize_append(h, 0, fake, fake, 257) == -2      # beyond max_tokens
        assert lib.kvq_append_decode_attention(h, 0, fake, fake, None, fake) == -1
        assert lib.kvq_append_decode_attention(h, 7, fake, fake, fake, fake) == -1
        a, b = ctypes.c_int32(-1), ctypes.c_int32(-1)
        assert lib.kvq_layer_tokens(h, 1, ctypes.byref(a), ctypes.byref(b)) == 0 and (a.value, b.value) == (0, 0)
        assert lib.kvq_layer_tokens(h, 5, ctypes.byref(a), ctypes.byref(b)) == -1
        assert lib.kvq_reset(h, -1) == 0 and lib.kvq_reset(h, 2) == -1
        assert lib.kvq_set_decode_options(h, 3, 0) == -1 and lib.kvq_set_decode_options(h, 1, 129) == -1
        assert lib.kvq_set_kernel_events(h, ctypes.c_void_p(8), None) == -1     # exactly one event
        assert lib.kvq_set_kernel_events(h, None, None) == 0
        assert lib.kvq_set_decode_options(h, 2, 8) == 0
        assert lib.kvq_debug_export(h, 0, *([None] * 8)) == 0              # empty layer: nothing to do
    finally:
        lib.kvq_destroy(h)
    for code in (0, -1, -2, -3, -4, -5, -99):
        assert len(lib.kvq_strerror(code)) > 0
    assert lib.kvq_last_error() is not None


def _bytes_without_pieces(layers, batch, hq, hkv, tokens, kb, vb, unit, residual=32):
    """The workspace without room for partial results of prefill pieces, worked out from the layout:
    packed blocks, window rings, split records, dequantized units of `unit` bytes, one selection record per cache."""
    up = lambda x: -(-x // 256) * 256                                    # noqa: E731
    caches, blocks, rows = batch * hkv, tokens // 32, batch * hq
    total = 0
    for bits in (kb, vb):
        total += layers * (up(caches * blocks * 512 * bits) + up(caches * blocks * (768 if bits < 16 else 0)) + up(caches * (residual + 32) * 256))
    total += layers * up(caches * blocks * 4)
    total += up(rows * 128 * 128 * 4) + up(rows * 128 * 2 * 4)
    return total + up(min(caches, 16) * blocks * unit) + up(caches * 768)


@pytest.mark.parametrize("layers,batch,hq,hkv,tokens,kb,vb", [
    (28, 1, 28, 4, 4096, 4, 2), (32, 1, 32, 8, 4133, 4, 2), (1, 1, 8, 2, 800, 4, 2), (4, 1, 32, 8, 24576, 16, 16),
    (2, 8, 32, 8, 2048, 8, 4), (2, 64, 32, 8, 2048, 4, 4), (1, 1, 1, 1, 700, 2, 2)])
def test_workspace_of_the_former_size_is_accepted(lib, layers, batch, hq, hkv, tokens, kb, vb):
    """Room for the partial results of prefill pieces is asked for but not insisted on: a workspace of the size that was
    enough before there were any (27 KiB per dequantized unit, no records) is taken, down to the layout without them."""
    cfg, keep = _cfg(n_layers=layers, batch=batch, n_q_heads=hq, n_kv_heads=hkv, max_tokens=tokens, kbits=[kb] * layers, vbits=[vb] * layers)
    need = lib.kvq_workspace_bytes(ctypes.byref(cfg))
    former = _bytes_without_pieces(layers, batch, hq, hkv, tokens, kb, vb, 27 * 1024)
    least = _bytes_without_pieces(layers, batch, hq, hkv, tokens, kb, vb, 26 * 1024)
    assert least <= need <= least + 512 * 256 * 130 * 4
    for have, expected in ((former, 0), (least, 0), (least + 133120, 0), (need, 0), (need + 4096, 0), (least - 1, -4)):
        h = ctypes.c_void_p()
        assert lib.kvq_configure(ctypes.byref(h), ctypes.byref(cfg), ctypes.c_void_p(256), have, None) == expected, (have - least, need - least)
        lib.kvq_destroy(h)


def _prefill_passes(lib, cfg, have, T, n_q):
    """[(caches, [pieces of each query tile])] of the passes of a prefill-attention call."""
    i32 = ctypes.c_int32
    passes = []
    while True:
        c, n, row = i32(), i32(), []
        for tile in range((n_q + 255) // 256):
            assert lib.kvq_debug_prefill_plan(ctypes.byref(cfg), have, T, n_q, len(passes), tile, ctypes.byref(c), ctypes.byref(n)) == 0
            row.append(n.value)
        if c.value == 0:
            assert row == [0] * len(row)
            return passes
        passes.append((c.value, row))


@pytest.mark.parametrize("batch,hq,hkv", [(1, 1, 1), (1, 2, 1), (1, 7, 1), (1, 32, 8), (2, 8, 4), (3, 28, 4), (17, 1, 1), (20, 2, 1)])
@pytest.mark.parametrize("residual", [0, 32, 500])
def test_prefill_plan_covers_every_tile_within_the_slots(lib, batch, hq, hkv, residual):
    """kvq_debug_prefill_plan over lengths, query counts and workspaces: the passes cover the caches; every piece of a cut
    tile holds at least 12 units and begins with one that lies in front of the tile's first query (so that every query sees a
    token of it); the partial results fit the records the workspace has room for."""
    seen = set()
    for T in (5, 700, 799, 800, 801, 1600, 2027, 3000, 6700, 24576, 33000):
        cfg, keep = _cfg(n_layers=1, batch=batch, n_q_heads=hq, n_kv_heads=hkv, max_tokens=T, kbits=[4], vbits=[2], residual=residual)
        need = lib.kvq_workspace_bytes(ctypes.byref(cfg))
        least = _bytes_without_pieces(1, batch, hq, hkv, T, 4, 2, 26 * 1024, residual)
        area = batch * hq * 128 * 130 * 4                                # split records: their room counts as well
        n_blocks = max(T - residual, 0) // 32
        for n_q in {1, min(T, 30), min(T, 257), min(T, 900), T}:
            for have in (need, least, min(need, least + 5 * 133120)):
                slots = min(512, (area + have - least) // 133120)
                passes = _prefill_passes(lib, cfg, have, T, n_q)
                assert sum(c for c, _ in passes) == batch * hkv
                for caches, row in passes:
                    heads = caches * (hq // hkv)
                    assert sum(n for n in row if n > 1) * heads <= slots, (T, n_q, have - least)
                    for tile, n in enumerate(row):
                        first, last = T - n_q + 256 * tile, T - n_q + min(256 * tile + 255, n_q - 1)
                        units = min(n_blocks, last // 32 + 1)
                        assert n >= 1 and (n == 1 or units >= 24), (T, n_q, tile, n)
                        for i in range(n if n > 1 else 0):
                            u0, u1 = units * i // n, units * (i + 1) // n
                            assert u1 - u0 >= 12 and 32 * u0 + 31 <= first, (T, n_q, tile, n)
                        seen.add(n)
    assert len(seen) >= 3
    c, n = ctypes.c_int32(), ctypes.c_int32()
    for bad in ((0, 1, 0, 0), (T + 1, 1, 0, 0), (T, 0, 0, 0), (T, T + 1, 0, 0), (T, 5, -1, 0), (T, 5, 0, 1), (T, 5, 0, -1)):
        assert lib.kvq_debug_prefill_plan(ctypes.byref(cfg), need, *bad, ctypes.byref(c), ctypes.byref(n)) == -1, bad
    assert lib.kvq_debug_prefill_plan(ctypes.byref(cfg), need, T, 5, 0, 0, None, ctypes.byref(n)) == -1
    assert lib.kvq_debug_prefill_plan(ctypes.byref(cfg), least - 1, T, 5, 0, 0, ctypes.byref(c), ctypes.byref(n)) == -4


@pytest.mark.parametrize("batch,hq,hkv,residual", [(1, 1, 1, 32), (1, 32, 8, 0), (2, 8, 4, 32), (3, 28, 4, 500), (17, 6, 1, 32), (40, 24, 1, 32)])
def test_prefill_form_goes_with_the_plan(lib, batch, hq, hkv, residual):
    """kvq_debug_prefill_form next to kvq_debug_prefill_plan: a known kernel form for every pass, heads that divide the group, and
    several heads in a launch of pieces or of 8 waves only where their rows fit one tile."""
    i32 = ctypes.c_int32
    w, h, o = i32(), i32(), i32()
    seen = set()
    for T in (1, 33, 300, 800, 2027, 6000, 6500, 12000, 33000):
        for room in (T, 4 * T):
            cfg, keep = _cfg(n_layers=1, batch=batch, n_q_heads=hq, n_kv_heads=hkv, max_tokens=room, kbits=[4], vbits=[2], residual=residual)
            need = lib.kvq_workspace_bytes(ctypes.byref(cfg))
            for n_q in {1, min(T, 9), min(T, 130), min(T, 400), T}:
                passes = _prefill_passes(lib, cfg, need, T, n_q)
                for i, (caches, row) in enumerate(passes):
                    assert lib.kvq_debug_prefill_form(ctypes.byref(cfg), need, T, n_q, i, ctypes.byref(w), ctypes.byref(h), ctypes.byref(o)) == 0
                    assert w.value in (4, 8) and o.value in (0, 1, 2) and h.value >= 1 and (hq // hkv) % h.value == 0
                    pieces = max(row) > 1
                    assert o.value == 0 or (w.value == 4 and not pieces)
                    assert h.value == 1 or n_q * h.value <= 256 or (w.value == 4 and not pieces), (T, n_q)
                    seen.add((w.value, h.value > 1, pieces))
                assert lib.kvq_debug_prefill_form(ctypes.byref(cfg), need, T, n_q, len(passes), ctypes.byref(w), ctypes.byref(h), ctypes.byref(o)) == 0
                assert (w.value, h.value, o.value) == (0, 0, 0)
    assert len(seen) >= 3
    for bad in ((0, 1, 0), (room + 1, 1, 0), (T, 0, 0), (T, T + 1, 0), (T, 5, -1)):
        assert lib.kvq_debug_prefill_form(ctypes.byref(cfg), need, *bad, ctypes.byref(w), ctypes.byref(h), ctypes.byref(o)) == -1, bad
    assert lib.kvq_debug_prefill_form(ctypes.byref(cfg), need, T, 5, 0, ctypes.byref(w), ctypes.byref(h), None) == -1
    assert lib.kvq_debug_prefill_form(ctypes.byref(cfg), 0, T, 5, 0, ctypes.byref(w), ctypes.byref(h), ctypes.byref(o)) == -4


def test_prefill_plan_is_quick_next_to_the_launch_it_divides(lib):
    """Few queries over a long cache: calls of some tens of us, in a loop over the layers, whose plan compares many numbers of pieces
    for every number of heads that share a work-group.  Each plan may take 10 us here (1 to 3 measured; the search took 21 to 38)."""
    i32 = ctypes.c_int32
    c, n = i32(), i32()
    for hq, T, n_q, pieces in ((24, 32000, 8, 21), (120, 32000, 8, 4), (120, 32000, 2, 4)):
        cfg, keep = _cfg(n_layers=1, batch=1, n_q_heads=hq, n_kv_heads=1, max_tokens=T, kbits=[4], vbits=[2])
        need = lib.kvq_workspace_bytes(ctypes.byref(cfg))

        def least(tokens, queries):
            best = 1.0
            for _ in range(300):
                t = time.perf_counter()
                lib.kvq_debug_prefill_plan(ctypes.byref(cfg), need, tokens, queries, 0, 0, ctypes.byref(c), ctypes.byref(n))
                best = min(best, time.perf_counter() - t)
            return best * 1e6

        call = least(5, 1)                      # (nothing to divide)
        assert least(T, n_q) - call < 10.0, (hq, n_q)
        assert n.value == pieces


def test_library_load_brings_torch_first():
    """The library must bind to the HIP runtime that torch ships (the one that owns torch's streams and allocations):
    loading it in a fresh interpreter, before anything imported torch, has to import torch on the way."""
    import subprocess
    import sys

    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    code = ("import sys; sys.path.insert(0, %r); import paper_2502_04420_amd as p; "
            "assert 'torch' not in sys.modules; p.load_library(); assert 'torch' in sys.modules" % root)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]


def test_binding_refuses_cpu_device(lib):
    import paper_2502_04420_amd as pkg

    with pytest.raises(ValueError):
        pkg.KVQ(1, 1, 4, 1, 128, 64, [8], [8], device="cpu")


def test_equivalent_precision_matches_the_papers_printed_values():
    import kvq_workloads as W
    from paper_2502_04420_amd import bytes_per_token, equivalent_precision, parse_pairs

    gold = {}
    with open(os.path.join(ROOT, "tests", "golden", "equivalent_precision.txt")) as f:
        for line in f:
            if line.strip() and not line.startswith("#"):
                name, val = [p.strip() for p in line.split("|")]
                gold[name] = float(val)
    for name, printed in gold.items():
        kb, vb = getattr(W, name)()
        assert round(equivalent_precision(kb, vb), 2) in (printed, round(printed + 0.01, 2)), name   # 4.906 prints as 4.90 / 4.91
    assert equivalent_precision(*W.llama_mix_325()) == 3.25
    assert equivalent_precision(*W.qwen_mix_40()) == 4.0
    assert equivalent_precision([4], [4]) == 4.0 and 16 / equivalent_precision([4], [2]) == pytest.approx(5.33, abs=0.01)
    # bytes per token per kv head (head_dim 128, group 32): as stored (fp32 scales, fp16 zero-points), all fp32
    pairs = ((8, 8), (8, 4), (8, 2), (4, 4), (4, 2), (2, 2), (16, 16))
    assert [bytes_per_token(k, v) for k, v in pairs] == [304, 240, 208, 176, 144, 112, 512]
    assert [bytes_per_token(k, v, zero_bytes=4) for k, v in pairs] == [320, 256, 224, 192, 160, 128, 512]
    assert parse_pairs("K8V4, KV4,K4V2") == ([8, 4, 4], [4, 4, 2])
    with pytest.raises(ValueError):
        parse_pairs("K3V4")


def _split_ranges(n_blocks, n_res, splits, units, rem):
    """The units [u0, u1) of every split as the kernels read the plan: blocks first, the window's chunks on the last."""
    out = []
    for s in range(splits):
        big = splits - rem                                   # the last `rem` splits take one unit more
        u0 = min(s * units + max(0, s - big), n_blocks)
        u1 = min(u0 + units + (1 if s >= big else 0), n_blocks)
        if s == splits - 1:
            u1 = n_blocks + (n_res + 31) // 32
        out.append((u0, u1))
    return out


def test_split_plan_covers_every_unit_once_and_leaves_no_split_empty(lib):
    """kvq_debug_split_plan over many shapes, lengths, widths, kernel variants and forced split counts: the splits'
    ranges tile the blocks in order, the window sits on the last split, no split is empty (an empty split would hand
    the merge a record without a maximum), blocks per split differ by at most one in front of the window's units, and
    a forced split count is never exceeded."""
    i32 = ctypes.c_int32
    seen_uneven = False
    for batch, hq, hkv in ((1, 1, 1), (2, 8, 2), (16, 32, 8), (8, 28, 4), (64, 32, 8)):
        for kb, vb in ((2, 2), (4, 2), (8, 8), (16, 4), (16, 16)):
            max_tokens = 40000
            cfg, keep = _cfg(n_layers=1, batch=batch, n_q_heads=hq, n_kv_heads=hkv, max_tokens=max_tokens, kbits=[kb], vbits=[vb])
            for T in (1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 160, 200, 1000, 4005, 8192, 8200, 8223, 32768, 32800, 39999):
                over = T - 32
                n_p = 32 * (over // 32) if over > 0 else 0
                n_blocks, n_res = n_p // 32, T - n_p
                for variant in (1, 2):
                    for forced in (0, 1, 2, 3, 7, 16, 100, 128):
                        s, u, r = i32(), i32(), i32()
                        assert lib.kvq_debug_split_plan(ctypes.byref(cfg), 0, T, variant, forced, ctypes.byref(s), ctypes.byref(u), ctypes.byref(r)) == 0
                        splits, units, rem = s.value, u.value, r.value
                        where = (batch, hkv, kb, vb, T, variant, forced, splits, units, rem)
                        assert 1 <= splits <= 128 and (forced == 0 or splits <= forced), where
                        assert units >= 0 and 0 <= rem < splits, where
                        ranges = _split_ranges(n_blocks, n_res, splits, units, rem)
                        assert ranges[0][0] == 0 and ranges[-1][1] == n_blocks + (n_res + 31) // 32, where
                        for (a0, a1), (b0, b1) in zip(ranges, ranges[1:]):
                            assert a1 == b0, where                       # in order, no gap, no overlap
                        assert all(u1 > u0 for u0, u1 in ranges), where  # nobody is empty
                        # the splits that lie in front of the window's virtual units
                        blocks = [u1 - u0 for k, (u0, u1) in enumerate(ranges[:-1]) if k * units + max(0, k - (splits - rem)) + units + (k >= splits - rem) <= n_blocks]
                        if blocks:
                            assert max(blocks) - min(blocks) <= 1, where
                            seen_uneven |= max(blocks) != min(blocks)
    assert seen_uneven
    s, u, r = i32(), i32(), i32()
    cfg, keep = _cfg()
    for bad in ((5, 10, 2, 0), (0, 0, 2, 0), (0, 257, 2, 0), (0, 10, 3, 0), (0, 10, 2, 129), (-1, 10, 2, 0)):
        assert lib.kvq_debug_split_plan(ctypes.byref(cfg), bad[0], bad[1], bad[2], bad[3], ctypes.byref(s), ctypes.byref(u), ctypes.byref(r)) == -1, bad
    assert lib.kvq_debug_split_plan(ctypes.byref(cfg), 0, 10, 2, 0, None, ctypes.byref(u), ctypes.byref(r)) == -1


@pytest.mark.parametrize("batch,hq,hkv,residual,T,expected", [
    # (work-groups with 4 / 5 blocks per group; a split is one per cache and 8 query heads)
    (1, 32, 8, 32, 128 * 32 + 37, 27),       # 264 / 216, two chunks of window: 5 blocks
    (1, 32, 8, 32, 155 * 32 + 60, 32),       # 320 / 256
    (1, 32, 8, 32, 156 * 32 + 60, 40),       # 320 / 264: 5 blocks are too many groups as well
    (1, 32, 8, 32, 124 * 32 + 60, 32),       # 256: one group per compute unit with 4 blocks
    (3, 32, 8, 32, 46 * 32 + 60, 13),        # 312 / 264
    (3, 32, 8, 128, 47 * 32 + 137, 11),      # 312 / 264, five chunks of window: 5 blocks all the same
    (3, 32, 8, 128, 52 * 32 + 137, 14),      # 336 / 288
    (1, 28, 4, 32, 255 * 32 + 41, 52),       # 260 / 208
    (1, 32, 8, 32, 127 * 32 + 32, 33),       # 264 / 216, one chunk: less than 32 groups over
    (1, 32, 8, 32, 139 * 32 + 32, 29),       # 288 / 232, one chunk
    (1, 32, 8, 0, 143 * 32, 29),             # 288 / 232, no window
    (1, 8, 2, 32, 15 * 32 + 32, 9),          # 2 blocks per group: one chunk, 16 groups
    (1, 8, 2, 32, 15 * 32 + 41, 5),          # two chunks: 4 blocks
    (1, 8, 2, 32, 62 * 32 + 32, 32),         # 64 groups with 2 blocks
    (1, 8, 2, 32, 64 * 32 + 32, 17),         # 66
    (2, 8, 1, 128, 20 * 32 + 137, 6),        # five chunks
])
def test_split_plan_of_short_caches(lib, batch, hq, hkv, residual, T, expected):
    """Blocks per group of short caches on either side of the lines that measurements drew."""
    i32 = ctypes.c_int32
    cfg, keep = _cfg(n_layers=1, batch=batch, n_q_heads=hq, n_kv_heads=hkv, max_tokens=40000, kbits=[4], vbits=[2], residual=residual)
    s, u, r = i32(), i32(), i32()
    assert lib.kvq_debug_split_plan(ctypes.byref(cfg), 0, T, 2, 0, ctypes.byref(s), ctypes.byref(u), ctypes.byref(r)) == 0
    assert s.value == expected


@pytest.mark.parametrize("batch,hq,hkv,kb,vb,residual,T,forced,expected", [
    # a single split: up to three work-groups per compute unit, at any length
    (1, 32, 8, 4, 2, 32, 4128, 1, (2, 1)), (96, 32, 8, 8, 8, 32, 1056, 1, (2, 1)), (192, 28, 4, 4, 2, 32, 288, 1, (2, 1)),
    # four, with tiles of 4 heads and narrow or fp16 pairs
    (128, 32, 8, 4, 2, 0, 128, 0, (2, 1)), (128, 32, 8, 16, 4, 32, 1056, 0, (2, 1)),
    (128, 32, 8, 8, 4, 32, 288, 0, (1, 0)), (256, 28, 4, 4, 2, 32, 288, 1, (1, 0)),
    # beyond: blocks go to one pair, except of fp16 pairs and many blocks of K8V8
    (256, 32, 8, 4, 2, 32, 288, 0, (1, 0)), (256, 32, 8, 2, 2, 32, 4128, 0, (1, 0)), (256, 32, 8, 8, 4, 32, 1056, 0, (1, 0)),
    (256, 32, 8, 16, 16, 32, 288, 0, (2, 1)), (256, 32, 8, 16, 4, 32, 288, 0, (1, 0)), (256, 32, 8, 8, 8, 32, 288, 0, (1, 0)), (256, 32, 8, 8, 8, 32, 1056, 0, (2, 1)),
    (512, 28, 4, 4, 2, 32, 1000, 0, (1, 0)),
    # a window alone: by its chunks
    (256, 32, 8, 4, 2, 64, 60, 0, (2, 1)), (256, 32, 8, 4, 2, 32, 30, 0, (1, 0)), (256, 32, 8, 16, 16, 32, 30, 0, (1, 0)),
    (256, 32, 8, 8, 4, 128, 90, 0, (1, 0)), (256, 32, 8, 8, 4, 128, 120, 0, (2, 1)), (128, 32, 8, 8, 4, 128, 120, 0, (1, 0)), (512, 28, 4, 8, 4, 128, 120, 0, (2, 1)),
    # several splits: as long as all work-groups are resident
    (1, 32, 8, 4, 2, 32, 4133, 0, (2, 1)), (4, 32, 8, 4, 2, 32, 3090, 0, (1, 0)), (8, 32, 8, 8, 8, 32, 1056, 8, (2, 1)), (8, 32, 8, 8, 8, 32, 1056, 9, (1, 0)),
    (18, 32, 8, 4, 2, 0, 32 * 2 + 7, 0, (1, 0)), (15, 32, 8, 4, 2, 0, 32 * 2 + 7, 0, (2, 1)), (18, 32, 8, 4, 2, 32, 32 * 2 + 40, 0, (2, 1)), (18, 32, 8, 4, 2, 0, 32 * 3 + 7, 0, (2, 1)),
    (1, 8, 2, 4, 2, 32, 32 * 188 + 43, 48, (2, 1)), (1, 8, 2, 4, 2, 32, 32 * 188 + 43, 49, (2, 0)),
    # tiles of 8 heads
    (11, 28, 4, 4, 4, 32, 1655, 0, (2, 1)), (48, 28, 4, 4, 2, 32, 32 * 12 + 40, 0, (2, 1)), (26, 28, 4, 8, 4, 32, 32 * 16 + 40, 0, (1, 0)),
    (18, 28, 4, 4, 2, 32, 352, 0, (2, 1)), (26, 28, 4, 4, 2, 32, 320, 0, (1, 0)), (26, 28, 4, 4, 2, 32, 416, 0, (2, 1)), (38, 28, 4, 4, 2, 32, 416, 0, (1, 0)),
    (1, 28, 4, 4, 2, 32, 8592, 0, (2, 0)),
])
def test_decode_form(lib, batch, hq, hkv, kb, vb, residual, T, forced, expected):
    """Pairs of waves per work-group of the decode kernel on either side of the lines that measurements drew, and who merges."""
    cfg, keep = _cfg(n_layers=1, batch=batch, n_q_heads=hq, n_kv_heads=hkv, max_tokens=40000, kbits=[kb], vbits=[vb], residual=residual)
    p, m = ctypes.c_int32(), ctypes.c_int32()
    assert lib.kvq_debug_decode_form(ctypes.byref(cfg), 0, T, forced, ctypes.byref(p), ctypes.byref(m)) == 0
    assert (p.value, m.value) == expected
    for bad in ((1, T, 0), (-1, T, 0), (0, 0, 0), (0, 40001, 0), (0, T, -1), (0, T, 129)):
        assert lib.kvq_debug_decode_form(ctypes.byref(cfg), *bad, ctypes.byref(p), ctypes.byref(m)) == -1, bad
    assert lib.kvq_debug_decode_form(ctypes.byref(cfg), 0, T, 0, None, ctypes.byref(m)) == -1
