"""Build the HIP library for gfx950: one hipcc compile per translation unit (in parallel), one link.

    python -m paper_2502_04420_amd.build

Produces paper_2502_04420_amd/libkvq.so next to this file.  The objects go to
paper_2502_04420_amd/_build/.  hipcc cross-compiles, so no GPU is needed to build.
"""
from __future__ import annotations

import functools
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

from .decode_check import check_decode_code, kernel_bodies

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libkvq.so")
OBJ = os.path.join(HERE, "_build")

COMMON = ["--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-Wall", "-Wno-unused-function",
          # packed fp32 instructions are kept out of the generated code on purpose
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# the encode path must not contract or reassociate anything: its results are compared bit for bit
PER_FILE = {"kvq_quantize.hip": ["-ffp-contract=off"],
            # M0 is named as clobbered by the global-to-LDS fetch; the compiler notes that it reserves that register
            "kvq_prefill_attn.hip": ["-Wno-inline-asm"]}


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    cmd = ["hipcc"] + COMMON + PER_FILE.get(src, []) + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "not a recognized feature" not in l)
    if r.returncode:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


@functools.lru_cache(maxsize=None)
def device_assembly(src: str, extra=()) -> str:
    """The gfx950 assembly hipcc generates for one source file with the library's flags (once per process and source)."""
    os.makedirs(OBJ, exist_ok=True)
    out = os.path.join(OBJ, src.replace(".hip", ".s"))
    cmd = (["hipcc"] + COMMON + ["-w"] + PER_FILE.get(src, []) + list(extra)
           + ["-S", "--cuda-device-only", os.path.join(CSRC, src), "-o", out])
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode:
        raise RuntimeError("hipcc -S failed for %s:\n%s" % (src, r.stderr[-2000:]))
    with open(out) as f:
        return f.read()


def check_prefill_attention_code(asm: str) -> None:
    """The prefill attention kernels set M0 in inline assembly (LDS base of their global-to-LDS fetches).  The library
    is only linked if, in the generated code, every M0 write is the one in front of such a fetch, nothing else reads or
    writes M0, and no kernel of the file spills registers (two waves per SIMD is what its pipelining assumes)."""
    # keys quantized / fp16; 4 waves: tiles cut / whole, 8 waves: rows of one head / of several
    kernels = kernel_bodies(asm, "prefill_attention") + kernel_bodies(asm, "prefill_attend_long")
    if len(kernels) != 8:
        raise RuntimeError("expected 8 prefill attention kernels in the generated code, found %d" % len(kernels))
    for name, body in kernels:
        lines = [l.strip() for l in body.splitlines()]
        code = [l for l in lines if l and not l.startswith((";", ".", "_Z")) and not l.endswith(":")]
        writes = [i for i, l in enumerate(code) if re.match(r"s_mov_b32 m0,", l)]
        fetches = [i for i, l in enumerate(code) if l.startswith("global_load_lds_dwordx4")]
        if not fetches or len(writes) != len(fetches):
            raise RuntimeError("%s: %d writes of M0 for %d fetches" % (name, len(writes), len(fetches)))
        for w, f in zip(writes, fetches):
            if not w < f <= w + 3:                                         # s_mov m0 ; s_nop ; load
                raise RuntimeError("%s: M0 write not in front of a fetch: %s" % (name, code[w:w + 4]))
        others = [l for l in code if re.search(r"\bm0\b", l) and not re.match(r"s_mov_b32 m0,", l)]
        if others:
            raise RuntimeError("%s: M0 used outside the fetches: %s" % (name, others[:3]))
    spills = re.findall(r"\.vgpr_spill_count:\s+(\d+)", asm)
    if not spills or any(int(x) for x in spills):
        raise RuntimeError("kvq_prefill_attn.hip: register spills %s" % spills)


def _check_prefill() -> None:
    check_prefill_attention_code(device_assembly("kvq_prefill_attn.hip"))


def _check_decode(src: str) -> None:
    if check_decode_code(device_assembly(src)) == 0:
        raise RuntimeError("%s: no hand-issued loads found in the generated code" % src)


def build(verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    srcs = sources()
    with ThreadPoolExecutor(max_workers=8) as ex:
        # alongside the compiles; a failure refuses the link
        checked = [ex.submit(_check_decode, src) for src in srcs if src.startswith(("kvq_decode_mfma", "kvq_decode_short"))]
        objs = list(ex.map(_compile, srcs))
        checked.append(ex.submit(_check_prefill))
        for c in checked:
            c.result()
    tmp = OUT + ".tmp.%d" % os.getpid()
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs,
                       capture_output=True, text=True)
    if r.returncode:
        raise RuntimeError("link failed:\n" + r.stderr)
    os.replace(tmp, OUT)
    if verbose:
        print("built", OUT)
    return OUT


if __name__ == "__main__":
    build()
