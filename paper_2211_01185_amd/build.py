"""Compile the HIP sources into paper_2211_01185_amd/lib/libcfddem.so (gfx950).

hipcc cross-compiles for gfx950 without a GPU.  Packed FP32 instructions are
disabled for every device pass.  The compiler's report of each kernel's
resources is read, and a kernel of NO_SPILLS that keeps vector registers in
scratch memory fails the build.
"""
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIBDIR = os.path.join(HERE, "lib")
LIB = os.path.join(LIBDIR, "libcfddem.so")
SOURCES = ["api.hip", "dem_kernels.hip", "couple_kernels.hip", "smooth_kernels.hip"]
ARCH = os.environ.get("CFDDEM_ARCH", "gfx950")

# Builds of the contact-force kernels that spilled vector registers have given
# results that differed from run to run, for a reason that was not found.  Not
# spilling is the way round it, so it is checked here.  The split element
# kernel, which came in with spills at that time, is held to the same; the other
# element kernels have spilled since they were written and repeat to the bit.
NO_SPILLS = re.compile(r"force_kick|couple_occupied_few")


def kernel_resources(report):
    """{mangled kernel name: {resource: number}} of the compiler's remarks."""
    out, cur = {}, None
    for line in report.splitlines():
        m = re.search(r"remark: .*?(?:Function )?Name: (\S+)", line)
        if m:
            cur = out.setdefault(m.group(1), {})
            continue
        m = re.search(r"remark: .*?([A-Za-z][A-Za-z ]*?)(?: \[[^\]]*\])?: (\d+)", line)
        if m and cur is not None:
            cur[m.group(1)] = int(m.group(2))
    return out


def check_resources(report):
    """Raises RuntimeError for a kernel of NO_SPILLS with spilled vector
    registers, and where the report lacks the count.  Returns the number of
    kernels looked at."""
    seen = 0
    for name, r in kernel_resources(report).items():
        if not NO_SPILLS.search(name):
            continue
        seen += 1
        if r.get("VGPRs Spill", -1) != 0:
            raise RuntimeError(f"{name}: {r.get('VGPRs Spill', 'unknown')} vector registers spilled")
    return seen


def hipcc_flags():
    return ["--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-Wall",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def build(verbose: bool = False, jobs: int = 3) -> str:
    os.makedirs(LIBDIR, exist_ok=True)
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []

    def finish(src, log, p):
        rc = p.wait()
        with open(log) as fh:
            report = fh.read()
        other = [ln for ln in report.splitlines() if "[-Rpass-analysis=kernel-resource-usage]" not in ln]
        if other:
            print("\n".join(other), file=sys.stderr, flush=True)
        if rc != 0:
            raise RuntimeError("hipcc failed on " + src)
        if check_resources(report) == 0 and src in ("dem_kernels.hip", "couple_kernels.hip"):
            raise RuntimeError("no resource report of the kernels of " + src)

    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        log = os.path.join(objdir, src.replace(".hip", ".report"))
        objs.append(obj)
        cmd = ["hipcc", "-c", *hipcc_flags(), "-Rpass-analysis=kernel-resource-usage", "-fno-caret-diagnostics",
               "-o", obj, os.path.join(CSRC, src)]
        if verbose:
            print(" ".join(cmd), flush=True)
        with open(log, "w") as fh:
            procs.append((src, log, subprocess.Popen(cmd, stderr=fh)))
        if len(procs) >= jobs:
            finish(*procs.pop(0))
    for p in procs:
        finish(*p)
    cmd = ["hipcc", "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", LIB + ".tmp", *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
