"""Build step: compile the HIP sources under csrc/ into paper_2602_04879_amd/libdppo.so for
gfx950 with hipcc (one object per source, compiled side by side, then linked).
`python -m paper_2602_04879_amd.build` or build() from Python."""
from __future__ import annotations

import glob
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
LIB_PATH = os.path.join(PKG_DIR, "libdppo.so")
OBJ_DIR = os.path.join(PKG_DIR, "_build")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


# Sources whose kernels name accumulation registers in assembly statements without telling the compiler
# (dppo_gemm.hip: 256 accumulators per lane).  It must keep nothing of its own there, spilled vector registers
# included; the generated assembly, which the object is made from, is looked through for that.
NAMED_ACCUMULATORS = {"dppo_gemm.hip": "dppo_gemm_nt_kernel"}
NAMED_ACCUMULATORS_FLAGS = [
    "-mllvm", "-amdgpu-spill-vgpr-to-agpr=0",
    # keep the assembly; written from there, a warning (a clobbered m0) would quote binary files
    "--save-temps=obj", "-Wno-inline-asm",
]


def check_named_accumulators(asm: str, kernel: str) -> None:
    """Raise RuntimeError unless, in the assembly text `asm`, every kernel whose name contains `kernel` has all 256 accumulation
    registers, mentions them nowhere but in its own assembly statements, and spills no vector register.
    (Others would not fault: their results would be silently wrong.)"""
    faults, bodies, entries, name, own = [], set(), set(), None, False
    for n, line in enumerate(asm.splitlines(), 1):
        if m := re.match(r"(\w+):", line):
            name = m[1] if kernel in m[1] else None
            bodies.add(name)
        elif line.startswith(".Lfunc_end"):
            name = None
        elif "#ASMSTART" in line or "#ASMEND" in line:
            own = "#ASMSTART" in line
        elif name and not own:
            code = line.split(";")[0].strip()
            if not code.startswith(".") and re.search(r"\ba(\d+|\[\d)", code):
                faults.append(f"line {n}, {name}: {code}")
    for entry in asm.partition("amdhsa.kernels:")[2].split("\n  - ")[1:]:
        f = dict(re.findall(r"^(?: {4})?\.(\w+): +(\S+)$", entry, re.M))
        if kernel in f.get("name", ""):
            entries.add(f["name"])
            if (f["agpr_count"], f["vgpr_spill_count"], f["private_segment_fixed_size"]) != ("256", "0", "0"):
                faults.append("{name}: {agpr_count} accumulation registers, {vgpr_spill_count} spilled vector registers, "
                              "{private_segment_fixed_size} bytes of scratch memory".format(**f))
    bodies.discard(None)
    if not bodies or bodies != entries:
        faults.append(f"kernels named {kernel}: {len(bodies)} bodies, {len(entries)} entries")
    if faults:
        raise RuntimeError("accumulation registers named in assembly statements are not safe:\n" + "\n".join(faults[:20]))


def sources() -> list[str]:
    return sorted(glob.glob(os.path.join(PKG_DIR, "csrc", "*.hip")))


def _run(cmd: list[str], verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass warns that it does not know the packed-fp32 feature: harmless
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        sys.stderr.write(err + "\n")
        raise RuntimeError("hipcc failed building libdppo.so: " + " ".join(cmd))
    if verbose and err.strip():
        print(err)


def _compile(hipcc: str, flags: list[str], src: str, obj: str, verbose: bool) -> None:
    kernel = NAMED_ACCUMULATORS.get(os.path.basename(src))
    _run([hipcc, *flags, *(NAMED_ACCUMULATORS_FLAGS if kernel else []), "-c", src, "-o", obj], verbose)
    if kernel:
        with open(obj[:-2] + "-hip-amdgcn-amd-amdhsa-gfx950.s") as f:
            asm = f.read()
        for temp in glob.glob(glob.escape(obj[:-2]) + "[-.]*"):
            if temp != obj:
                os.remove(temp)
        check_named_accumulators(asm, kernel)


def build(verbose: bool = True, jobs: int | None = None) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ_DIR, exist_ok=True)
    inc = ["-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(PKG_DIR, "csrc")]
    srcs = sources()
    objs = [os.path.join(OBJ_DIR, os.path.basename(s)[:-4] + ".o") for s in srcs]
    jobs = jobs or min(len(srcs), os.cpu_count() or 1, 8)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        list(ex.map(lambda so: _compile(hipcc, HIPCC_FLAGS + inc, so[0], so[1], verbose), zip(srcs, objs)))
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB_PATH], verbose)
    return LIB_PATH


if __name__ == "__main__":
    build()
