"""Build libteno.so (HIP, gfx950) in-tree with hipcc.

Every HIP source is compiled with -ffp-contract=off (each + - * / sqrt of the
kernels is one IEEE operation in source order, so results are reproducible
bit for bit) and with packed FP32 instructions disabled.  The translation
units are compiled in parallel into _build/ and linked into one library.

A build ends in an error when a kernel that is not named in SPILLING keeps
vector registers in scratch memory, or when a kernel stores one where its lanes
have not rejoined yet (see narrow_stores).
"""
from __future__ import annotations

import glob
import os
import re
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libteno.so")
OBJ = os.path.join(ROOT, "_build")
ARCH = os.environ.get("TENO_OFFLOAD_ARCH", "gfx950")

FLAGS = [
    "-O3", "-std=c++17", "-fPIC",
    f"--offload-arch={ARCH}",
    "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


# Kernels that are known to spill vector registers (mangled-name prefixes): the 2D
# and 3D adjoint chunks, the fused z sweep of the march and the 2D TENO5-A x sweep
# of long lines.
SPILLING = ("_ZN4teno7k_sweepILi2ELi0ELi4ELb0ELi264ELb1E",
            "_ZN4teno11k_adj_chunkILi2E", "_ZN4teno11k_adj_chunkILi3E",
            "_ZN4teno7k_marchILi3ELi2ELb0ELi2E", "_ZN4teno7k_marchILi3ELi2ELb1ELi2E")


def sources():
    return sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    # hipcc's host pass does not know the packed-FP32 feature and says so
    noise = "'-packed-fp32-ops' is not a recognized feature"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if err.strip():
        print(err, file=sys.stderr, flush=True)
    if r.returncode != 0:
        raise subprocess.CalledProcessError(r.returncode, cmd)


def narrow_stores(asm: str) -> dict:
    """Scratch stores of a disassembly (llvm-objdump -d) that lie in a block before
    the instruction that widens the lane mask again, by kernel.  hipcc has placed a
    spill's store there, at a join of diverged lanes, and its reload under the wide
    mask: the lanes that rejoined read what was never stored."""
    line = re.compile(r"^\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):.*?(?:<(\S+?)(?:\+0x([0-9a-f]+))?>)?$")
    kernels, cur = {}, None
    for text in asm.splitlines():
        head = re.match(r"^([0-9a-f]+) <(\S+)>:$", text)
        if head:
            cur = kernels.setdefault(head[2], (int(head[1], 16), []))
            continue
        m = line.match(text)
        if m and cur is not None:
            cur[1].append((int(m[3], 16), m[1], m[2], m[5]))
    bad = {}
    for name, (start, code) in kernels.items():
        targets = {start + int(off, 16) for _, op, _, off in code if "branch" in op and off}
        stores, found = 0, 0
        for at, op, args, _ in code:
            if at in targets:
                stores = 0
            if op.startswith("scratch_store"):
                stores += 1
            elif op == "s_or_b64" and args.replace(" ", "").startswith("exec,exec,"):
                found += stores
                stores = 0
            elif "branch" in op:
                stores = 0
        if found:
            bad[name] = found
    return bad


def check_spills(objects):
    """({kernel: vector registers spilled}, {kernel: narrow_stores}) of built objects."""
    rocm = os.environ.get("ROCM_PATH") or os.path.dirname(os.path.dirname(
        os.path.realpath(shutil.which("hipcc") or "/opt/rocm/bin/hipcc")))
    tool = lambda name: os.path.join(rocm, "llvm", "bin", name)
    out = lambda cmd: subprocess.run(cmd, check=True, capture_output=True, text=True).stdout

    def one(obj):
        with tempfile.TemporaryDirectory() as d:
            fat, co = os.path.join(d, "fat"), os.path.join(d, "co")
            out([tool("llvm-objcopy"), "--dump-section", f".hip_fatbin={fat}", obj, os.path.join(d, "o")])
            out([tool("clang-offload-bundler"), "-type=bc", "-unbundle", f"-input={fat}",
                 f"-targets=hipv4-amdgcn-amd-amdhsa--{ARCH}", f"-output={co}"])
            notes = out([tool("llvm-readelf"), "--notes", co])
            counts = re.findall(r"\.name:\s+(_Z\w+).*?\.vgpr_spill_count:\s+(\d+)", notes, re.S)
            spills = {k: int(n) for k, n in counts if int(n) > 0}
            return spills, narrow_stores(out([tool("llvm-objdump"), "-d", co])) if spills else {}

    spills, narrow = {}, {}
    with ThreadPoolExecutor(4) as ex:
        for s, n in ex.map(one, objects):
            spills.update(s)
            narrow.update(n)
    return spills, narrow


def build(verbose: bool = False, extra=None) -> str:
    os.makedirs(OBJ, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include")]
    jobs = []
    objs = []
    for src in sources():
        obj = os.path.join(OBJ, os.path.basename(src) + ".o")
        objs.append(obj)
        jobs.append(["hipcc", *FLAGS, *(extra or []), *inc, "-c", "-o", obj, src])
    workers = min(len(jobs), max(1, min(8, os.cpu_count() or 1)))
    with ThreadPoolExecutor(workers) as ex:
        list(ex.map(lambda c: _run(c, verbose), jobs))
    spills, narrow = check_spills(objs)
    if verbose:
        for k, n in sorted(spills.items()):
            print(f"{n} vector registers spilled: {k}", flush=True)
    unexpected = sorted(k for k in spills if not k.startswith(SPILLING))
    if unexpected or narrow:
        raise RuntimeError(f"vector register spills in {unexpected}; stored before the lanes rejoin: {narrow}")
    _run(["hipcc", "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", LIB + ".tmp", *objs],
         verbose)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True, extra=sys.argv[1:])
