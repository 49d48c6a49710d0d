"""Builds the HIP decode library (libsprout.so, gfx950) and the host-only
bookkeeping test library (libsprout_host.so) in the package directory."""
import concurrent.futures
import os
import subprocess
import sys
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libsprout.so")
HOST_LIB = os.path.join(PKG, "libsprout_host.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
HIP_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # Packed fp32 instructions stay off: ordinary float code only.
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # MFMA accumulators in VGPRs: epilogues and the softmax rescale operate on
    # them with VALU instructions, which cannot address AGPRs.
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    # The leading scalar kernel arguments (pointers, sizes) arrive preloaded in
    # SGPRs, so a kernel's first loads need not wait for its argument fetch.
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wno-unused-result",
]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)


# Translation units of libsprout.so, the slowest to compile first; compiled in parallel.
SOURCES = ["panel_qkv.hip", "panel_qkv_rows.hip", "panel_mlp.hip", "sprout.hip", "panel_resid.hip", "tile_qkv.hip",
           "tile_resid.hip", "tile_mlp.hip", "host_state.cpp"]


def build(verbose: bool = True) -> None:
    with tempfile.TemporaryDirectory() as d:
        objs = [os.path.join(d, s + ".o") for s in SOURCES]
        with concurrent.futures.ThreadPoolExecutor(len(SOURCES)) as ex:
            list(ex.map(lambda so: _run([HIPCC, *HIP_FLAGS, "-c", os.path.join(CSRC, so[0]), "-o", so[1]], verbose),
                        zip(SOURCES, objs)))
        tmp = LIB + ".tmp"
        _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp], verbose)
        os.replace(tmp, LIB)
    tmp = HOST_LIB + ".tmp"
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
          os.path.join(CSRC, "host_state.cpp"), os.path.join(CSRC, "host_test_api.cpp"), "-o", tmp], verbose)
    os.replace(tmp, HOST_LIB)


if __name__ == "__main__":
    build(verbose="-q" not in sys.argv)
