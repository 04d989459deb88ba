"""Build the HIP library libnco.so in-tree for gfx950.

Every source under ``csrc/`` is compiled by hipcc for gfx950 only, with
packed float32 instructions disabled, and linked into
``paper_2412_08229_amd/libnco.so`` next to this file.
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(ROOT, "_build", "obj")
LIB = os.path.join(HERE, "libnco.so")
SOURCES = ["api.hip", "kernels.hip", "spectrum.hip", "nco_mfma.hip", "nco_mfma_full.hip",
           "nco_mfma_split.hip", "nco_mfma_bf16.hip", "nco_f64.hip", "nco_adjoint.hip", "adjoint.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # Matrix-core results in ordinary VGPRs: the activations read them
         # directly instead of copying out of the accumulation registers.
         "-mllvm", "-amdgpu-mfma-vgpr-form",
         "-I" + os.path.join(ROOT, "include"), "-Wall", "-Wno-unused-function"]


def _newest_header():
    heads = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    heads += [os.path.join(ROOT, "include", f) for f in os.listdir(os.path.join(ROOT, "include"))]
    return max(os.path.getmtime(h) for h in heads)


def build(verbose=False, out=None, extra_flags=(), obj_dir=None, incremental=False):
    """Compile and link.  ``out``/``extra_flags``/``obj_dir`` build a variant
    library elsewhere (tuning experiments); the defaults build libnco.so.
    ``incremental`` skips sources whose object is newer than the source and
    every header (a development shortcut; the default compiles everything)."""
    out = out or LIB
    obj_dir = obj_dir or OBJ
    os.makedirs(obj_dir, exist_ok=True)
    procs = []
    objs = []
    newest_header = _newest_header()
    for src in SOURCES:
        obj = os.path.join(obj_dir, src.replace(".hip", ".o"))
        objs.append(obj)
        if incremental and os.path.exists(obj):
            t = os.path.getmtime(obj)
            if t > os.path.getmtime(os.path.join(CSRC, src)) and t > newest_header:
                continue
        cmd = [HIPCC] + FLAGS + list(extra_flags) + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
    failed = []
    for src, p in procs:
        log, _ = p.communicate()
        text = log.decode(errors="replace")
        if p.returncode != 0:
            failed.append(src)
            sys.stderr.write(text)
        elif verbose and text.strip():
            sys.stderr.write(text)
    if failed:
        raise RuntimeError("hipcc failed for: " + ", ".join(failed))
    tmp = out + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    subprocess.check_call(cmd)
    os.replace(tmp, out)
    return out


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv, incremental="-i" in sys.argv))
