"""Build in-tree with hipcc: libmaskkv.so (the product, gfx950), libmaskkv_bench.so (measurement probes and stage marks for
benchmark harnesses; it links against the product library) and the CPython extension that marshals the binding's
arguments (host code against torch's headers)."""
from __future__ import annotations

import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmaskkv.so")
BENCH_LIB = os.path.join(HERE, "libmaskkv_bench.so")
SOURCES = ["api.hip", "score.hip", "sweep.hip", "rows.hip", "select.hip", "compact.hip", "attend.hip", "attend_tiles.hip", "layer.hip"]
MARSHAL = os.path.join(HERE, "_marshal" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
BENCH_SOURCES = [os.path.join("bench", "probe.hip")]
FLAGS = [
    "-shared", "-fPIC", "-O3", "-std=c++17", "--offload-arch=gfx950",
    # packed fp32 arithmetic is kept off for every kernel in this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # MFMA accumulators in ordinary VGPRs: the exponentials read them directly (no v_accvgpr_read copies)
    "-mllvm", "-amdgpu-mfma-vgpr-form=1",
]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)


def _build_marshal(hipcc, verbose):
    import torch
    from torch.utils import cpp_extension
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    # torch's own warnings are not ours to see (-isystem); its libraries are already loaded when the extension is imported
    inc = [x for d in cpp_extension.include_paths() + [sysconfig.get_paths()["include"], "/opt/rocm/include"] for x in ("-isystem", d)]
    _run([hipcc, "-x", "c++", "-shared", "-fPIC", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
          "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)] + inc +
         [os.path.join(CSRC, "python.cpp"), "-L" + lib, "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip",
          "-Wl,-rpath," + lib, "-o", MARSHAL + ".tmp"], verbose)
    os.replace(MARSHAL + ".tmp", MARSHAL)


def build(verbose: bool = False) -> str:
    """Compile every kernel file into paper_2510_09309_amd/libmaskkv.so (+ libmaskkv_bench.so, _marshal); returns the product's path."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    _run([hipcc] + FLAGS + [os.path.join(CSRC, s) for s in SOURCES] + ["-o", LIB + ".tmp"], verbose)
    os.replace(LIB + ".tmp", LIB)
    _run([hipcc] + FLAGS + [os.path.join(CSRC, s) for s in BENCH_SOURCES] +
         ["-L" + HERE, "-l:libmaskkv.so", "-Wl,-rpath,$ORIGIN", "-o", BENCH_LIB + ".tmp"], verbose)
    os.replace(BENCH_LIB + ".tmp", BENCH_LIB)
    _build_marshal(hipcc, verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
