"""Builds libpackinfer.so (gfx950) in-tree with hipcc.

    python -m paper_2602_06072_amd.build
"""
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(CSRC, "_build")
LIB = os.path.join(HERE, "libpackinfer.so")

SOURCES = ["planner.cpp", "schedule.cpp", "api.cpp", "trie.cpp", "debug_f32.hip", "upload.hip", "reorg.hip",
           "decode.hip", "prefill.hip", "prefill_pipe.hip", "padded_decode.hip", "mixed_step.hip"]

HIP_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option"]


# Kernels whose inline assembly copies through buffer descriptors without wait states (copy_16 in prefill_body.hip.h): the words come
# from scalar instructions a turn earlier.  A spilled scalar register is read back by v_readlane right before its use, which the compiler's
# hazard recogniser cannot see in front of a statement of ours: such a build must not run.
NO_SCALAR_SPILLS = {"prefill_pipe.hip", "mixed_step.hip"}
USAGE = "-Rpass-analysis=kernel-resource-usage"


def scalar_spills(remarks):
    """[(kernel, spilled scalar registers)] of the kernels that spill any, from the compiler's resource-usage remarks.  Text
    without a count for every kernel is an error: the check would pass for want of something to look at."""
    names = re.findall(r"Function Name: (\S+)", remarks)
    counts = [int(x) for x in re.findall(r"SGPRs Spill: (\d+)", remarks)]
    if not names or len(names) != len(counts):
        raise RuntimeError(f"resource usage of {len(names)} kernels with {len(counts)} spill counts: cannot tell whether scalar registers spill")
    return [(n, c) for n, c in zip(names, counts) if c > 0]


def _compile(src):
    obj = os.path.join(OBJ, src + ".o")
    cmd = ["hipcc"] + HIP_FLAGS + (["-x", "hip"] if src.endswith(".cpp") else []) + \
          ([USAGE] if src in NO_SCALAR_SPILLS else []) + ["-c", os.path.join(CSRC, src), "-o", obj]
    p = subprocess.run(cmd, capture_output=True, text=True)
    if p.returncode == 0 and src in NO_SCALAR_SPILLS:
        spills = scalar_spills(p.stderr)
        if spills:
            os.remove(obj)
            raise RuntimeError(f"{src}: scalar registers spill in {spills}; the copies of these kernels rely on none (see NO_SCALAR_SPILLS)")
        p.stderr = "\n".join(l for l in p.stderr.splitlines() if "warning:" in l)
    err = "\n".join(l for l in p.stderr.splitlines()
                    if "packed-fp32-ops" not in l and "is not a recognized feature" not in l)
    if p.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(verbose=True):
    os.makedirs(OBJ, exist_ok=True)
    srcs = [s for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.run(cmd, check=True)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()
