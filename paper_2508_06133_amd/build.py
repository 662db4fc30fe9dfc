"""Compile libkvsched.so (hand-written HIP, gfx950 only) and the Python module over it next to this file.

hipcc cross-compiles without a GPU, so this runs anywhere the ROCm toolchain is installed.

timeline_reg.hip and predicted.hip keep per-timeline state in a block of physical VGPRs (v30 / v60 upward) that
only their inline-assembly blocks touch.  That is sound only while everything the compiler allocates in those
kernels (its own code and the operand registers it hands to the assembly statements) stays below the block,
so the build emits the device assembly of these files and fails if such a kernel names a VGPR of
the block anywhere but in the hand-written row code, or if it did not see every instantiation.
"""
from __future__ import annotations

import importlib.util
import os
import re
import shutil
import subprocess
import sys
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libkvsched.so")
# csrc/host.cpp, a Python module over the library and torch (its name says for which interpreter, so that another one leaves it alone)
HOST = os.path.join(HERE, "kvsched_host" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
SOURCES = ["api.hip", "simulate.hip", "timeline_reg.hip", "sortedf.hip", "localswap.hip", "exactdp.hip", "horizon.hip", "permute.hip", "prefix.hip", "shortrows.hip", "eventrows.hip", "online.hip", "predicted.hip"]
DEVICE_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    # packed fp32 instructions are kept off for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]
# Branches that all lanes of a wavefront take together stay branches: by default every way out of a loop becomes a flag in
# scalar registers, tested later.  For the files whose kernels have main loops without other branches (4096 candidates of
# predicted_reg_kernel 5.9 ms without, 5.1 with it; predicted_ring_kernel, whose passes over the ring do branch by the lane, has it too);
# elsewhere it makes no difference.
UNIFORM_BRANCHES = ["-mllvm", "-structurizecfg-skip-uniform-regions"]
SOURCE_FLAGS = {name: UNIFORM_BRANCHES for name in ("localswap.hip", "predicted.hip", "online.hip", "eventrows.hip")}
FLAGS = DEVICE_FLAGS + ["-fPIC", "-Wall"]
RESERVED_VGPR_BASE = 30  # KVS_PB in timeline_reg.hip
PREDICTED_VGPR_BASE = 60  # KVP_PB in predicted.hip


def lib_path() -> str:
    return LIB


def is_stale() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(HOST):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(HOST))
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC)] + [os.path.join(HERE, "..", "include", "kvsched.h"), os.path.abspath(__file__)]
    return any(os.path.getmtime(d) > t for d in deps)


def timeline_reg_instantiations() -> int:
    """Kernel instantiations kvs_launch_simulate_reg can reach: one per launch statement of launch_reg
    and profile-file size."""
    src = open(os.path.join(CSRC, "timeline_reg.hip")).read()
    launches = len(re.findall(r"hipLaunchKernelGGL\(\(timeline_reg_kernel<NR, (?:WPB|1),", src))
    sizes = len(re.findall(r"return launch_reg<\d+, \d+>\(p, st\);", src))
    return launches * sizes


def predicted_reg_instantiations() -> int:
    src = open(os.path.join(CSRC, "predicted.hip")).read()
    return len(re.findall(r"\(const void \*\)predicted_reg_kernel<\d+>", src))


def reserved_vgpr_scan(asm_text: str, base: int = RESERVED_VGPR_BASE,
                       kernel: str = "timeline_reg_kernel") -> tuple[list[str], int]:
    """(offending lines, kernel bodies scanned) for the bodies of `kernel` in a device assembly.

    The profile block of an instantiation with NR rows (read off the kernel's mangled name) is
    v[base, base + NR).  It belongs to the hand-written assembly alone, which names it only as
    v[<base>+...].  Offending are therefore: a compiler-generated line that names a VGPR of the block in
    any form, and a line INSIDE an assembly statement that names one as plain vN or v[a:b] -- an operand
    register the compiler substituted (temporaries and inputs of the statements must lie outside the
    block as well).  A body runs from the kernel's label to its .Lfunc_end label (s_endpgm may come
    early, for the exits in the prologue); inline assembly sits between the ASMSTART / ASMEND (or APP /
    NO_APP) comment lines the compiler emits around it.
    """
    bad = []
    bodies = 0
    in_kernel = in_asm = False
    top = base
    for line in asm_text.splitlines():
        s = line.strip()
        m = re.match(r"^_Z\w*" + kernel + r"ILi(\d+)E\w*:", s)
        if m:
            in_kernel, in_asm = True, False
            top = base + int(m.group(1))
            bodies += 1
            continue
        if not in_kernel:
            continue
        if s.startswith(".Lfunc_end"):
            in_kernel = False
            continue
        if s.startswith((";;#ASMSTART", ";APP", "#APP")):
            in_asm = True
            continue
        if s.startswith((";;#ASMEND", ";NO_APP", "#NO_APP")):
            in_asm = False
            continue
        if not s or s.startswith(";") or (not in_asm and s.startswith(".")):
            continue
        code = s.split(";", 1)[0]
        regs = [(int(m), int(m)) for m in re.findall(r"\bv(\d+)\b", code)]
        regs += [(int(lo), int(hi)) for lo, hi in re.findall(r"\bv\[(\d+):(\d+)\]", code)]
        if any(lo < top and hi >= base for lo, hi in regs):
            bad.append(s)
    return bad, bodies


def reserved_vgpr_violations(asm_text: str, base: int = RESERVED_VGPR_BASE) -> list[str]:
    return reserved_vgpr_scan(asm_text, base)[0]


def emit_assembly(hipcc: str, source: str) -> str:
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "device.s")
        cmd = [hipcc, *DEVICE_FLAGS, *SOURCE_FLAGS.get(source, []), "-S", "--cuda-device-only", os.path.join(CSRC, source), "-o", out]
        subprocess.check_call(cmd, stderr=subprocess.DEVNULL)
        return open(out).read()


def emit_timeline_reg_assembly(hipcc: str) -> str:
    return emit_assembly(hipcc, "timeline_reg.hip")


def check_reserved_vgprs(hipcc: str, verbose: bool = False) -> None:
    for source, kernel, base, want in (
            ("timeline_reg.hip", "timeline_reg_kernel", RESERVED_VGPR_BASE, timeline_reg_instantiations()),
            ("predicted.hip", "predicted_reg_kernel", PREDICTED_VGPR_BASE, predicted_reg_instantiations())):
        bad, bodies = reserved_vgpr_scan(emit_assembly(hipcc, source), base, kernel)
        if bodies != want or want == 0:
            raise RuntimeError(f"scanned {bodies} {kernel} bodies, the launcher can reach {want}")
        if bad:
            raise RuntimeError("the reserved VGPR block (v%d..) is named outside the hand-written row code:\n  "
                               % base + "\n  ".join(bad[:10]))
        if verbose:
            print(f"reserved VGPR block untouched in all {bodies} {kernel} bodies", flush=True)


def build_host(run, lib: str, out: str) -> None:
    torch = os.path.dirname(importlib.util.find_spec("torch").origin)
    run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", os.path.join(CSRC, "host.cpp"), "-o", out,
         "-isystem", os.path.join(torch, "include"), "-isystem", os.path.join(torch, "include", "torch", "csrc", "api", "include"),
         "-I", sysconfig.get_paths()["include"],
         "-L", os.path.join(torch, "lib"), "-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10",
         "-L", os.path.dirname(lib), "-l:" + os.path.basename(lib), "-Wl,-rpath,$ORIGIN"])


def build(verbose: bool = False) -> str:
    """Both files, put in place together once everything has been built and checked."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)

    with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(min(len(SOURCES), os.cpu_count() or 1, 8)) as pool:
        built = [os.path.join(tmp, f + ".o") for f in SOURCES]
        lib, host = os.path.join(tmp, os.path.basename(LIB)), os.path.join(tmp, os.path.basename(HOST))
        list(pool.map(run, [[hipcc, *FLAGS, *SOURCE_FLAGS.get(f, []), "-c", os.path.join(CSRC, f), "-o", o]
                            for f, o in zip(SOURCES, built)]))
        run([hipcc, *DEVICE_FLAGS[:1], "-fPIC", "-shared", *built, "-o", lib])
        check_reserved_vgprs(hipcc, verbose)
        build_host(run, lib, host)
        for new, place in ((lib, LIB), (host, HOST)):
            beside = place + f".tmp{os.getpid()}"
            shutil.copy(new, beside)
            os.replace(beside, place)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    print(LIB)
