"""Build libodwf.so (HIP, gfx950) in-tree from paper_1811_08095_amd/csrc.

Every source is compiled with hipcc for gfx950 only, with packed FP32 vector
instructions disabled, and linked into a shared library with a plain C ABI
(include/odwf.h).
"""
import concurrent.futures as cf
import json
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libodwf.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCES = ["hop_fp64.hip", "hop_fp32.hip", "hop_fp16.hip", "hop_bf16.hip", "hop.hip", "force.hip", "pack.hip",
           "blas.hip", "m5.hip", "noalloc.hip", "runtime.cpp", "api.cpp", "solver.cpp", "batch.cpp"]
COMMON = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-Wall",
          "-Wno-unused-function", "-Wno-unused-variable",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-I" + CSRC, "-I" + os.path.join(os.path.dirname(HERE), "include"),
          "-Rpass-analysis=kernel-resource-usage"]


def check_usage(messages: str) -> dict:
    """Scratch bytes a lane of every kernel, from the compiler's resource-usage
    remarks, refusing kernels that hold values in accumulation registers.  Every kernel here fits the
    256 vector registers that its launch bounds leave it.  Builds of the four-wave hopping
    kernel with a larger budget, in which the matrix results went to accumulation
    registers, gave wrong results for a reason that is not known (the generated
    code shows none: LDS accesses in order, matrix results waited for as in the
    right builds), so no such kernel is let into the library."""
    name, scratch = None, {}
    for line in messages.splitlines():
        m = re.search(r"remark: .*?(Function Name|AGPRs|ScratchSize)(?: \[bytes/lane\])?: (\S+)", line)
        if not m:
            continue
        if m[1] == "Function Name":
            name = m[2]
        elif m[1] == "ScratchSize":
            scratch[name] = int(m[2])
        elif int(m[2]) > 0:
            raise RuntimeError(f"{name} uses {m[2]} accumulation registers: give it a launch bound "
                               "that keeps it within 256 vector registers")
    return scratch


def _without_remarks(messages: str) -> str:
    """The compiler's messages but for the resource-usage remarks, their source
    lines and the include lines that lead to them."""
    out, lead, remark = [], [], False
    for line in messages.splitlines():
        if line.startswith("In file included from"):
            lead.append(line)
        elif "[-Rpass-analysis=kernel-resource-usage]" in line:
            lead, remark = [], True
        elif not (remark and re.match(r"\s*\d* \|", line)):
            out += lead + [line]
            lead, remark = [], False
    return "\n".join(out)


def _compile(src: str, verbose: bool, build_dir: str, defines) -> str:
    obj = os.path.join(build_dir, os.path.splitext(src)[0] + ".o")
    lang = ["-x", "hip"]
    cmd = [HIPCC] + lang + COMMON + ["-D" + d for d in defines] + \
        ["-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
    messages = _without_remarks(r.stderr)
    if messages:
        print(messages, file=sys.stderr, flush=True)
    r.check_returncode()
    with open(os.path.splitext(obj)[0] + ".scratch.json", "w") as f:
        json.dump(check_usage(r.stderr), f)
    return obj


def build(verbose: bool = False, jobs: int = 8, out: str = LIB, defines=()) -> str:
    """Compile every source and link `out` (default: the in-tree libodwf.so).
    `defines` are extra preprocessor definitions (tuning builds)."""
    build_dir = BUILD if out == LIB else out + ".objs"
    os.makedirs(build_dir, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose, build_dir, defines), SOURCES))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", out + ".tmp"] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(out + ".tmp", out)
    return out


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
