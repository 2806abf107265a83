"""Builds libscalebits.so (gfx950) in-tree with hipcc: one object per .hip file, then a link.

Variants (compile-time switches of the arithmetic, one library each):
  ""   -> libscalebits.so      cost = sum s * d^2
  "l1" -> libscalebits_l1.so   cost = sum s * |d|   (-DSBITS_COST_POWER=1)
For the tests only (--tests):
  "impatient" -> libscalebits_impatient.so   the search's workgroups give up waiting for each other at once, so that
                                             the single-workgroup search behind it is reached
  "masked" -> libscalebits_masked.so         takes the device for one whose 16-bit loads leave half of a register as it was
  "noretry" -> libscalebits_noretry.so       a search that was given up is not repeated: what it finds, the resident
                                             workgroups have found
"""
from __future__ import annotations

import os
import re
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
VARIANTS = {"": [], "l1": ["-DSBITS_COST_POWER=1"]}
TEST_VARIANTS = {"impatient": ["-DSBITS_SPIN_LIMIT=0"],
                 "masked": ["-DSBITS_D16_ZERO_FILL=0"],
                 "noretry": ["-DSBITS_SECOND_TRY=0"]}
ONLY = {v: ["api.hip" if v == "masked" else "alloc.hip"] for v in TEST_VARIANTS}       # sources a variant compiles anew; the rest are the default build's objects
SOURCES = ["api.hip", "reorder.hip", "cost.hip", "fused.hip", "fused_copies.hip", "fused_wide.hip", "alloc.hip", "pack.hip", "mpgemm.hip", "dequant.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-ffp-contract=off",                       # no implicit FMA: only the fmaf() the method names
         "-Xarch_device", "-fno-honor-nans",        # device code only: inputs are finite by contract,
                                                    # spares the NaN-quieting ops around min/max
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I" + INCLUDE, "-I" + CSRC, "-Wall", "-Wno-unused-function"]


def lib_path(variant: str = "") -> str:
    return os.path.join(HERE, "libscalebits%s.so" % ("_" + variant if variant else ""))


def _compile(src: str, force: bool, variant: str) -> str:
    if src not in ONLY.get(variant, SOURCES):
        force, variant = False, ""
    objdir = os.path.join(HERE, "_build" + ("_" + variant if variant else ""))
    obj = os.path.join(objdir, src.replace(".hip", ".o"))
    deps = [os.path.join(CSRC, src)] + [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hpp")]
    deps.append(os.path.join(INCLUDE, "scalebits.h"))
    if not force and os.path.exists(obj) and os.path.getmtime(obj) >= max(os.path.getmtime(d) for d in deps):
        return obj
    cmd = [HIPCC, *FLAGS, *{**VARIANTS, **TEST_VARIANTS}[variant], "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout)
        raise RuntimeError("hipcc failed on " + src)
    if src == "mpgemm.hip":
        try:
            listing = device_listing(obj)
            if check_block_waits(listing) == 0:
                raise RuntimeError("no kernel with counted waits found in " + src)
        except Exception:
            os.remove(obj)                          # not taken by a later build either
            raise
    return obj


def device_listing(obj: str) -> str:
    """The gfx950 assembly of an object file of this build."""
    def tool(name):
        return subprocess.check_output([HIPCC, "-print-prog-name=" + name], text=True).strip()
    with tempfile.TemporaryDirectory() as d:
        bundle, code = os.path.join(d, "bundle"), os.path.join(d, "code")
        subprocess.check_call([tool("llvm-objcopy"), "--dump-section", ".hip_fatbin=" + bundle, obj, os.path.join(d, "rest")])
        subprocess.check_call([tool("clang-offload-bundler"), "--type=o", "--unbundle", "--input=" + bundle, "--output=" + code,
                               "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"])
        return subprocess.check_output([tool("llvm-objdump"), "-d", "--no-show-raw-insn", code], text=True)


def check_block_waits(listing: str) -> int:
    """In the product of many rows a wave waits for the x of a block by counting the loads of codes and scales, 4 a tile, that it requested
    behind it.  A compiler that made fewer of them, out of a scalar load or out of two neighbouring ones, would let it read x too early.
    They may be requested before the loop or at its end, and in part at its beginning, in front of the
    wait; each way there are exactly as many between one block's loads to LDS and the wait.  Returns how many kernels were checked."""
    kernels = re.findall(r"([0-9a-f]+) <(\w*mp_gemm_many_kernelILi(\d+)ELi(\d+)ELi(\d+)E\w*)>:\n(.*?)(?=\n\n|\Z)", listing, re.S)
    for start, name, n_cols, batch_tiles, tiles, text in kernels:
        behind, x_loads = 4 * int(tiles), int(batch_tiles) * int(n_cols) // 32
        lines = text.split("\n")
        vector = [bool(re.match(r"\s*(?:buffer|global|flat)_load_", s)) for s in lines]
        lds = [v and re.search(r"\blds\b", s.split("//")[0]) is not None for v, s in zip(vector, lines)]
        to_lds = [i for i, v in enumerate(lds) if v]
        waits = [i for i, s in enumerate(lines) if re.search(r"s_waitcnt vmcnt\(%d\)\s" % behind, s + " ")
                 and any("ds_read_b128" in t for t in lines[i:i + 24])]
        waits = [i for i in waits if len(to_lds) == 2 * x_loads and to_lds[x_loads - 1] < i < to_lds[x_loads]]
        if len(waits) != 1:
            raise RuntimeError("%s: %d loads to LDS and %d waits between them, %d and 1 expected" % (name, len(to_lds), len(waits), 2 * x_loads))
        wait, end = waits[0], next(i for i, s in enumerate(lines) if i > to_lds[-1] and "s_barrier" in s)
        address = [int(m.group(1), 16) if (m := re.search(r"// ([0-9A-F]+):", s)) else -1 for s in lines]
        heads = [int(start, 16) + int(m.group(1), 16) for s in lines[to_lds[-1]:end]
                 if (m := re.search(r"s_c?branch\w* .*\+0x([0-9a-f]+)>", s))]
        heads = [i for i in range(to_lds[x_loads - 1], wait + 1) if address[i] in heads]
        if len(heads) != 1:
            raise RuntimeError("%s: %d loops around the wait" % (name, len(heads)))

        def count(a, b):
            return sum(vector[i] and not lds[i] for i in range(a, b))
        first, again = count(to_lds[x_loads - 1], wait), count(to_lds[-1], end) + count(heads[0], wait)
        if first != behind or again != behind or count(wait, to_lds[-1]):
            raise RuntimeError("%s: %d and %d loads behind the x of a block, %d expected" % (name, first, again, behind))
    return len(kernels)


def build(force: bool = False, variant: str = "") -> str:
    LIB = lib_path(variant)
    os.makedirs(os.path.join(HERE, "_build" + ("_" + variant if variant else "")), exist_ok=True)
    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(lambda s: _compile(s, force, variant), SOURCES))
    if force or not os.path.exists(LIB) or os.path.getmtime(LIB) < max(os.path.getmtime(o) for o in objs):
        tmp = LIB + ".tmp%d" % os.getpid()
        subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs])
        os.replace(tmp, LIB)
    return LIB


def build_all(force: bool = False, tests: bool = False) -> list:
    return [build(force, v) for v in [*VARIANTS, *(TEST_VARIANTS if tests else [])]]


if __name__ == "__main__":
    for path in build_all(force="--force" in sys.argv, tests="--tests" in sys.argv):
        print(path)
