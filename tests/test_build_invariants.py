"""Properties of the generated code that the sources rely on but the compiler does not promise."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2502_04420_amd", "csrc")


def _assembly(src, tmp_path, extra=()):
    hipcc = shutil.which("hipcc")
    if hipcc is None:
        pytest.skip("hipcc not available")
    out = tmp_path / (src + ".s")
    cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-w", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-S", "--cuda-device-only", *extra,
           os.path.join(CSRC, src), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=900)
    assert r.returncode == 0, r.stderr[-2000:]
    return out.read_text()


def _kernels(asm, name):
    """Bodies of the kernels whose mangled name contains `name`."""
    bodies = []
    for m in re.finditer(r"^(_Z\w*%s\w*):.*?^\.Lfunc_end\d+:" % name, asm, re.S | re.M):
        bodies.append((m.group(1), m.group(0)))
    return bodies


def test_prefill_attention_writes_m0_only_for_its_own_fetches(tmp_path):
    """The attention kernel sets M0 in inline assembly (LDS base of a global-to-LDS load).  M0 is named as clobbered,
    and on top of that the build refuses to link a library in whose generated code M0 is written anywhere but in front
    of those loads, read by anything else, or in which a kernel of the file spills: the same check, run here."""
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    from paper_2502_04420_amd import build as B

    asm = B.device_assembly("kvq_prefill_attn.hip")
    B.check_prefill_attention_code(asm)
    # the check is not vacuous: a second user of M0, or an M0 write away from a fetch, is refused
    name, body = B.kernel_bodies(asm, "prefill_attention")[0]
    planted = asm.replace(body, body.replace("global_load_lds_dwordx4", "s_mov_b32 m0, s5\n\tglobal_load_lds_dwordx4", 1), 1)
    with pytest.raises(RuntimeError):
        B.check_prefill_attention_code(planted)
    planted = asm.replace(body, body.replace("s_nop 0", "v_readlane_b32 s4, v0, m0\n\ts_nop 0", 1), 1)
    with pytest.raises(RuntimeError):
        B.check_prefill_attention_code(planted)


def test_assembly_can_be_taken_before_anything_is_built(tmp_path, monkeypatch):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    from paper_2502_04420_amd import build as B

    monkeypatch.setattr(B, "OBJ", str(tmp_path / "not there yet"))
    assert "amdgcn" in B.device_assembly("kvq_api.hip")


def test_uncut_prefill_launches_take_no_piece_table():
    """A prefill launch too short for a cut of its query tiles runs a kernel that knows no pieces: its arguments are a few pointers
    and sizes, not the 520 bytes of the table, whose reading shows in the time of prompts of a few dozen tokens."""
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    from paper_2502_04420_amd import build as B

    asm = B.device_assembly("kvq_prefill_attn.hip")
    sizes = []
    for block in re.split(r"\n  - \.agpr_count", asm)[1:]:
        if "prefill_attention" in re.findall(r"\.name:\s+(_Z\S+)", block)[-1]:
            sizes.append(int(re.search(r"\.kernarg_segment_size:\s+(\d+)", block).group(1)))
    assert len(sizes) == 4 and sorted(s > 512 for s in sizes) == [False, False, True, True], sizes


def test_quantize_kernel_keeps_the_fused_widen_and_subtract(tmp_path):
    """x - z is meant to be one mixed-precision instruction per element (both fp16 operands widened inside it); the
    multiplier 1.0 is hidden from the optimiser for that.  If a compiler folds it after all, the code is still right
    but slower: this test tells."""
    asm = _assembly("kvq_quantize.hip", tmp_path, extra=("-ffp-contract=off",))
    kernels = [b for n, b in _kernels(asm, "quantize_blocks") if "ILi4ELi2ELb0E" in n]
    assert len(kernels) == 1
    assert len(re.findall(r"^\s*v_fma_mix_f32 ", kernels[0], re.M)) >= 128      # 2 tensors x 64 elements per lane


def test_quantize_kernels_keep_their_tokens_in_registers(tmp_path):
    """No quantize kernel uses scratch memory, and the one that stores fp16 rows as they are uses no LDS: an array the
    compiler cannot keep in registers (the window rows a launch takes along) ends up in the one or the other without any
    message, and the launch takes two to four times as long."""
    asm = _assembly("kvq_quantize.hip", tmp_path, extra=("-ffp-contract=off",))
    kernels = 0
    for block in re.split(r"\n  - \.agpr_count", asm)[1:]:
        name = re.findall(r"\.name:\s+(_Z\S+)", block)[-1]
        size = {k: int(v) for k, v in re.findall(r"\.(private_segment_fixed_size|group_segment_fixed_size):\s+(\d+)", block)}
        if "quantize_blocks" in name:
            kernels += 1
            assert size["private_segment_fixed_size"] == 0, name
            if "ILi16ELi16E" in name:
                assert size["group_segment_fixed_size"] == 0, name
    assert kernels == 32                                          # 4 x 4 bit widths, two scale precisions


def test_builtin_scratch_array_is_visible_to_the_loader():
    """kvq_decode_attention_noalloc asks the runtime for the device address of the library's built-in scratch array.
    That only works if the device code object exports the array as a global symbol (an attribute such as `used` keeps
    a static device variable local, the lookup then yields an address that is not the array's, and the first kernel
    that uses it faults).  Checked on the object the build produced."""
    tools = "/opt/rocm/llvm/bin"
    obj = os.path.join(ROOT, "paper_2502_04420_amd", "_build", "kvq_api.o")
    if not (os.path.exists(obj) and all(os.path.exists(os.path.join(tools, t)) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-readelf"))):
        pytest.skip("needs the built object and the LLVM binary tools")
    import tempfile

    with tempfile.TemporaryDirectory() as tmp:
        fat, co = os.path.join(tmp, "fat.bin"), os.path.join(tmp, "api.co")
        subprocess.check_call([os.path.join(tools, "llvm-objcopy"), "-O", "binary", "--only-section=.hip_fatbin", obj, fat])
        subprocess.check_call([os.path.join(tools, "clang-offload-bundler"), "--type=o", "--input=" + fat,
                               "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--output=" + co, "--unbundle"])
        syms = subprocess.check_output([os.path.join(tools, "llvm-readelf"), "-s", co], text=True)
    rows = [l.split() for l in syms.splitlines() if l.strip().endswith("scratch")]
    assert rows, "no scratch symbol in the device code object"
    assert all(r[4] == "GLOBAL" and r[3] == "OBJECT" and int(r[2]) == 16384 * 130 * 4 for r in rows), rows


def test_decode_kernels_leave_hand_issued_loads_alone():
    """The matrix-core decode kernels issue their block loads in inline assembly and wait for them with hand-written
    counts.  The build refuses a library in whose generated code an instruction of the compiler's own touches a
    register such a load may still be writing: the same check, run here on one instantiation, and shown not to be
    vacuous by planting a copy of an in-flight register."""
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    from paper_2502_04420_amd import build as B

    asm = B.device_assembly("kvq_decode_mfma.hip")
    assert B.check_decode_code(asm) > 1000                               # every instantiation streams through these loads
    name, body = [kb for kb in B.kernel_bodies(asm, "decode_mfma") if "ILi4ELi2ELi4ELb0ELb0E" in kb[0]][0]
    m = re.search(r"buffer_load_dwordx4 (v\[(\d+):\d+\]), [^\n]*\n\s*;;#ASMEND\n", body)
    assert m
    planted = body[:m.end()] + "\tv_mov_b32_e32 v200, v%s\n" % m.group(2) + body[m.end():]
    with pytest.raises(RuntimeError):
        B.check_decode_code(asm.replace(body, planted, 1))


def test_decode_check_follows_every_path_to_the_streaming_loop():
    """The loads issued in front of the streaming loop are pending on both ways out of the prologue: into the loop, and past
    it (a group without packed blocks).  A copy over one of their registers is refused wherever it is planted: behind the
    last of them; in the key wave, whose queries are fetched first, also in front of the loop and in front of the wait of
    the other way (the value wave waits for its queries, and with them for everything, before the two part)."""
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    from paper_2502_04420_amd import build as B

    asm = B.device_assembly("kvq_decode_mfma.hip")
    plants = 0
    for tag in ("ILi4ELi2ELi4ELb0ELb0E", "ILi8ELi8ELi4ELb1ELb0E", "ILi4ELi2ELi8ELb0ELb0E", "ILi2ELi4ELi4ELb0ELb1E"):
        lines = [kb for kb in B.kernel_bodies(asm, "decode_mfma") if tag in kb[0]][0][1].split("\n")
        by_hand = lambda i, start: lines[i].strip().startswith(start) and "ASMSTART" in lines[i - 1]     # noqa: E731
        assert B.check_decode_code("\n".join(lines)) > 0
        loops = [i for i, l in enumerate(lines) if l.strip() == "s_setprio 3"]
        assert len(loops) == 2                                           # the value wave's, then the key wave's
        for k, loop in enumerate(loops):
            first = loops[0] if k else 0
            waits = [i for i in range(first, loop) if re.search(r"vmcnt\(0\)", lines[i])]
            drain = [i for i in waits if by_hand(i, "s_waitcnt vmcnt(0)")][-1]      # of a group without packed blocks
            issued = [i for i in range(max(i for i in waits if i < drain) if k else 0, drain) if by_hand(i, "buffer_load")]
            regs = [re.search(r"v\[?(\d+)", lines[i]).group(1) for i in issued]
            assert len(regs) >= 3
            spots = [(issued[-1] + 2, r) for r in regs]
            if k:
                spots += [(drain - 1, r) for r in regs] + [(loop, r) for r in regs[-2:]]
            for spot, r in spots:
                plants += 1
                with pytest.raises(RuntimeError, match="hand-issued load"):
                    B.check_decode_code("\n".join(lines[:spot] + ["\tv_mov_b32_e32 v%s, 0" % r] + lines[spot:]))
    assert plants >= 4 * (3 + 3 + 3 + 2)


@pytest.mark.parametrize("src", ["kvq_decode_mfma.hip", "kvq_decode_short.hip"])
def test_decode_kernels_wait_for_nothing_between_queries_and_first_blocks(src):
    """The key wave asks for its queries, then for the first blocks, and the wait for the queries leaves exactly the blocks' loads in
    flight.  A wait of the compiler's in between (it knows of none of these loads) would put a memory round trip in front of the
    blocks; a count that is one too high would let the queries be read before they are there."""
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    from paper_2502_04420_amd import build as B

    kernels = 0
    for name, body in B.kernel_bodies(B.device_assembly(src), "decode_mfma"):
        kb, vb, gq = (int(x) for x in re.search(r"ILi(\d+)ELi(\d+)ELi(\d+)E", name).groups())
        if 16 in (kb, vb):                                               # (their queries are ordinary loads)
            continue
        queries, behind, by_hand = 0, 0, False
        for line in (l.strip() for l in body.split("\n")):
            if line.startswith(";;#ASM"):
                by_hand = line.startswith(";;#ASMSTART")
            elif by_hand and line.startswith("global_load"):
                queries += 1
            elif by_hand and queries and line.startswith("buffer_load"):
                behind += 1
            elif queries and (by_hand or "vmcnt" in line) and line.startswith("s_waitcnt"):
                assert by_hand and line == "s_waitcnt vmcnt(%d)" % behind, (name, line, behind)
                assert queries == gq and behind > 3, (name, queries, behind)
                queries, behind, kernels = 0, 0, kernels + 1
        assert queries == 0, name
    assert kernels == 3 * 3 * 2 * 2 * 2                                  # key and value bits, head tiles, scale precisions, key groupings


def test_merge_of_the_splits_reads_at_checked_offsets():
    """The work-group that merges asks for a fixed number of records and has the absent ones read as zero: their place must be in the offset that
    the buffer resource checks, so the loads past the caches (the merge's, all of them) have no scalar offset."""
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    from paper_2502_04420_amd import build as B

    kernels = B.kernel_bodies(B.device_assembly("kvq_decode_short.hip"), "decode_mfma")
    assert kernels
    for name, body in kernels:
        loads = re.findall(r"buffer_load_dwordx[24] \S+ (\S+), (s\[[0-9:]+\]), (\S+) offen( offset:\d+)? sc0 sc1", body)
        assert len(loads) >= 17 and len(loads) == len(re.findall(r"buffer_load\w* [^\n]*sc0 sc1", body)), (name, len(loads))
        assert {x[2] for x in loads} == {"0"}, name


def _record_bytes(asm, name):
    """Bytes of the argument records of the kernels whose mangled name contains `name` (implicit arguments included)."""
    return {int(n) for n in re.findall(r"\.amdhsa_kernel _Z\w*%s\w*\n(?:(?!\.end_amdhsa_kernel).*\n)*?\s*\.amdhsa_kernarg_size (\d+)" % name, asm)}


def test_decode_launches_carry_only_their_own_arguments():
    """What only the short-cache form of the decode kernel needs is not part of the record of the streaming form and of the merge,
    whose calls it made longer; no kernel of a decode call asks for implicit arguments."""
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    from paper_2502_04420_amd import build as B

    assert _record_bytes(B.device_assembly("kvq_decode_mfma.hip"), "decode_mfma") == {176}
    assert _record_bytes(B.device_assembly("kvq_decode_valu.hip"), "combine_splits") == {176}
    assert _record_bytes(B.device_assembly("kvq_decode_short.hip"), "decode_mfma") == {192}


def test_quantize_waves_read_two_lines_of_their_arguments(tmp_path):
    """A block's wave of the quantize kernels reads the first 128 bytes of the argument record only (what the waves that copy window
    rows or clear counters need lies behind them, and is asked for behind the branch that tells the waves apart)."""
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    from paper_2502_04420_amd import build as B

    kernels = B.kernel_bodies(B.device_assembly("kvq_quantize.hip"), "quantize_blocks")
    assert len(kernels) == 32
    for name, body in kernels:
        branch = re.search(r"s_cbranch_\w+ (\.LBB\d+_\d+)", body)
        near, far = body.split("\n" + branch.group(1) + ":")              # the other waves' code is the branch's target
        assert branch.start() < len(near) and len(far) < len(near)
        loads = re.findall(r"s_load_dword(x\d+)? \S+ s\[0:1\], (0x[0-9a-f]+)", near)
        ends = [int(off, 16) + 4 * int(n[1:] or 1) for n, off in loads]
        assert ends and max(ends) <= 128, (name, loads)
        # of the other waves, those that copy window rows do not wait for the third line either: it holds the counters' place only
        first = far.index("s[0:1], 0x80")
        assert "s_cbranch" in far[:first] and "global_load" not in far[:first] and "lgkmcnt" not in far[:first], name
        third = [(off, n) for n, off in re.findall(r"s_load_dword(x\d+)? \S+ s\[0:1\], (0x[0-9a-f]+)", far) if int(off, 16) >= 128]
        assert sorted(third) == [("0x80", "x2"), ("0x88", "")], (name, third)


def test_prefill_launches_ask_for_their_arguments_at_once():
    """The kernels of a prefill call share an argument record of two and a half 64-byte lines, without implicit arguments, and what a
    launch adds to it begins on the third; the 8-wave attention kernels and the channel selection wait for them once, in front
    of their first branch, and the dequantization asks for all of its lines in front of its first wait."""
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    from paper_2502_04420_amd import build as B

    asm = B.device_assembly("kvq_prefill_attn.hip")
    assert _record_bytes(asm, "prefill_dequantize") == {160}
    assert _record_bytes(asm, "prefill_select") == {164}
    assert _record_bytes(asm, "prefill_attention") | _record_bytes(asm, "prefill_attend_long") | _record_bytes(asm, "prefill_merge") == {176, 160 + 24 + 4 * 128}
    kernels = B.kernel_bodies(asm, "prefill_attend_long") + B.kernel_bodies(asm, "prefill_select")
    assert len(kernels) == 6
    for name, body in kernels:
        assert body.split("s_cbranch", 1)[0].count("lgkmcnt(0)") == 1, name
    kernels = B.kernel_bodies(asm, "prefill_dequantize")
    assert len(kernels) == 4
    assert _record_bytes(asm, "units_of_half_keys") == {160} and len(B.kernel_bodies(asm, "units_of_half_keys")) == 2
    kernels += B.kernel_bodies(asm, "units_of_half_keys")
    for name, body in kernels:                          # every line of the record is on its way at the first wait
        loads = re.findall(r"s_load_dword(x\d+)? \S+ s\[0:1\], (0x[0-9a-f]+)", body.split("lgkmcnt(0)", 1)[0])
        assert {(int(off, 16) + 4 * int(n[1:] or 1) - 1) // 64 for n, off in loads} == {0, 1, 2}, (name, loads)
