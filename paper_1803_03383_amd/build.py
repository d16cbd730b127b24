"""Build libhalp.so (HIP, gfx950 only) in-tree with hipcc.

    python -m paper_1803_03383_amd.build

Object files go to csrc/_build/ (git-ignored); the shared library lands next
to this file so that it travels with the source tree.
"""
import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(CSRC, "_build")
OUT = os.path.join(HERE, "libhalp.so")
SOURCES = ["halp_api.hip", "fullgrad.hip", "recenter.hip", "inner_generic.hip", "inner_reg.hip",
           "inner_reg_b8.hip", "inner_reg_b16.hip", "inner_reg_helped_b8.hip", "inner_reg_helped_b16.hip", "inner_reg_lone_b8.hip", "inner_reg_lone_b16.hip",
           "inner_reg_lone_b8_l2.hip", "inner_reg_lone_b16_l2.hip", "inner_softmax.hip", "inner_softmax_b8.hip", "inner_softmax_batch.hip", "inner_softmax_split.hip", "inner_softmax_mfma.hip", "softmax_ahead.hip", "fullgrad_softmax.hip", "fullgrad_wide.hip", "inner_svrg.hip", "inner_batch.hip", "inner_batch_cut.hip", "step_latency.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    # packed fp32 instructions are kept out of the generated code on this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def _compile(src):
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj, r.stderr


def build(verbose=False):
    os.makedirs(OBJ, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        results = list(ex.map(_compile, SOURCES))
    if verbose:
        for _, err in results:
            if err.strip():
                sys.stderr.write(err)
    objs = [o for o, _ in results]
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", OUT, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    return OUT


if __name__ == "__main__":
    print(build(verbose=True))
