"""Compile the HIP sources under csrc/ into the in-tree shared library
``libglide.so`` for gfx950 (hipcc, one object per source or part of one, built in parallel)."""
import concurrent.futures as cf
import glob
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libglide.so")
BUILD_DIR = os.path.join(ROOT, "_build")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC,
         # no packed-fp32 instructions (v_pk_*_f32) anywhere in device code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


# Per-source extra flags.  The prefill kernels never produce or consume NaNs
# (masked scores are -inf, 0/0 is tested explicitly), so their max
# reductions need no NaN quieting of matrix-core results.
EXTRA = {"prefill.hip": ["-fno-honor-nans"]}
# Sources compiled in several parts (one object each, built in parallel):
# the prefill kernels once per element type and head dim.
PARTS = {"prefill.hip": ("GLIDE_PREFILL_PART", 4)}


def _compile(job):
    src, part = job
    name = os.path.basename(src)
    extra, obj = list(EXTRA.get(name, [])), os.path.join(BUILD_DIR, name + ".o")
    if part is not None:
        extra.append(f"-D{PARTS[name][0]}={part}")
        obj = os.path.join(BUILD_DIR, f"{name}.{part}.o")
    r = subprocess.run([HIPCC, *FLAGS, *extra, "-c", src, "-o", obj], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def _jobs(src):
    name = os.path.basename(src)
    return [(src, p) for p in range(PARTS[name][1])] if name in PARTS else [(src, None)]


def build(verbose=False):
    os.makedirs(BUILD_DIR, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    jobs = [j for s in srcs for j in _jobs(s)]
    with cf.ThreadPoolExecutor(max_workers=min(8, len(jobs))) as ex:
        objs = list(ex.map(_compile, jobs))
    tmp = LIB + ".tmp"
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
