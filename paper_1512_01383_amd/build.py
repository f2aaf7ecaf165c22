"""Build libsublabel.so (HIP, gfx950) in-tree with hipcc."""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import re
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libsublabel.so")
SOURCES = ["capi.hip", "pdhg_iter.hip", "aux.hip", "adjoint.hip", "steps.hip", "stereo.hip", "temporal.hip"]
ARCH = os.environ.get("SUBLABEL_OFFLOAD_ARCH", "gfx950")

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    # FMA contraction only within one source expression (never across statements), so
    # every template variant of a kernel rounds the same way
    "-ffp-contract=on",
    # keep the compiler from forming packed FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-Wall", "-Wno-unused-function",
]


def _hipcc() -> str:
    for cand in ("/opt/rocm/bin/hipcc", "hipcc"):
        if os.path.exists(cand) or cand == "hipcc":
            return cand
    return "hipcc"


def _vector_registers(text: str) -> set:
    out = {int(x) for x in re.findall(r"\bv(\d+)\b", text)}
    for a, b in re.findall(r"\bv\[(\d+):(\d+)\]", text):
        out |= set(range(int(a), int(b) + 1))
    return out


def misplaced_spills(asm: str) -> list:
    """Vector spills and reloads that the compiler put at the end of a divergent region ahead of
    the instruction that turns the other lanes on again, for a register that the region itself
    does not use: (kernel, line) pairs.

    Where many scalar registers are spilled too, the register allocator has been seen to put a
    spill there that is read back with all lanes on, so the lanes outside the region read what
    was never written (a kernel's addresses among it). Correct code has none of these.
    """
    found = []
    for part in re.split(r"\n(?=_Z\S+:)", asm)[1:]:
        name = part.split(":")[0]
        block = None   # instructions since the block's start; None once its exec mask has changed
        for line in part.split(".Lfunc_end")[0].splitlines():
            t = line.strip()
            if re.match(r"\.LBB\S+:", t) or t.startswith("; %bb"):
                block = []
            elif not t or t[0] in ";." or block is None:
                continue
            elif re.match(r"s_\S+ exec,|s_\S+saveexec", t):
                if re.match(r"s_or_b64 exec, exec", t):
                    written = set()
                    for j, x in enumerate(block):
                        own = _vector_registers(x.split(";")[0])
                        if "Folded Spill" in x and not own & written:
                            found.append((name, x))
                        if "Folded Reload" in x and not any(own & _vector_registers(y) for y in block[j + 1:]):
                            found.append((name, x))
                        written |= _vector_registers(x.split(",")[0])
                block = None
            else:
                block.append(t)
    return found


def build(verbose: bool = False, jobs: int = 8) -> str:
    objdir = os.path.join(PKG, "_build")
    os.makedirs(objdir, exist_ok=True)
    hipcc = _hipcc()

    def compile_one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        temps = os.path.join(objdir, "temps_" + src.replace(".hip", ""))   # the assembly among them
        os.makedirs(temps, exist_ok=True)
        made = os.path.join(temps, os.path.basename(obj))
        cmd = [hipcc] + HIPCC_FLAGS + ["-save-temps=obj", "-c", os.path.join(CSRC, src), "-o", made]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        msgs = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                         if "packed-fp32-ops" not in l and l.strip())
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed for {src}:\n{msgs}")
        if msgs and verbose:
            print(msgs, file=sys.stderr)
        listings = glob.glob(os.path.join(temps, "*-hip-amdgcn-*.s"))
        if not listings:
            raise RuntimeError(f"no assembly of {src} to check")
        for path in listings:
            with open(path) as f:
                bad = misplaced_spills(f.read())
            if bad:
                raise RuntimeError(f"{src}: the compiler misplaced spills of {len(bad)} registers, e.g. {bad[0]}: "
                                   "lower the kernel's register pressure or leave the instance out")
        os.replace(made, obj)
        shutil.rmtree(temps)
        return obj

    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [hipcc, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
