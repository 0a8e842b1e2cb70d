"""Compile the HIP sources under csrc/ into libmg_gemm.so (gfx950 only) and the Python calls into _mg_call.so, in-tree.

hipcc cross-compiles without a GPU.  Objects are rebuilt when a source or header is newer.
"""
import concurrent.futures
import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmg_gemm.so")
CALL = os.path.join(HERE, "_mg_call.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-early-inline-all=true"]


def _compile(src, obj, extra):
    cmd = [HIPCC, *FLAGS, *extra, "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    return src, r.returncode, (r.stdout + r.stderr)


def build(force: bool = True, verbose: bool = False, extra_flags=()) -> str:
    os.makedirs(OBJ, exist_ok=True)
    sources = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    headers = glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(HERE, "..", "include", "*.h"))
    newest_header = max(os.path.getmtime(h) for h in headers)
    jobs, objs = [], []
    for src in sources:
        obj = os.path.join(OBJ, os.path.basename(src)[:-4] + ".o")
        objs.append(obj)
        stale = force or not os.path.exists(obj) or os.path.getmtime(obj) < max(os.path.getmtime(src), newest_header)
        if stale:
            jobs.append((src, obj))
    workers = min(8, max(1, len(jobs)))
    with concurrent.futures.ThreadPoolExecutor(workers) as pool:
        for src, code, out in pool.map(lambda j: _compile(j[0], j[1], list(extra_flags)), jobs):
            if verbose or code != 0:
                sys.stderr.write(out)
            if code != 0:
                raise RuntimeError(f"hipcc failed on {src}")
    if jobs or not os.path.exists(LIB):
        cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
        subprocess.run(cmd, check=True)
    source = os.path.join(CSRC, "python_call.cpp")
    if force or not os.path.exists(CALL) or os.path.getmtime(CALL) < max(os.path.getmtime(source), newest_header):
        subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I", sysconfig.get_paths()["include"],
                        source, "-o", CALL], check=True)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv, verbose=True))
