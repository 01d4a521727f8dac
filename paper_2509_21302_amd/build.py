"""Compile the HIP sources in csrc/ into libqvggt.so (gfx950 only), and csrc/call.cpp into the Python module _call, in-tree.

    python -m paper_2509_21302_amd.build          # build (always recompiles)

Objects and compiler temporaries go to paper_2509_21302_amd/_build/; the shared libraries are
written next to this file so that they travel with the source tree.
"""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libqvggt.so")
CALL = os.path.join(HERE, "_call" + sysconfig.get_config_var("EXT_SUFFIX"))       # another Python does not find it
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
SOURCES = ["api.hip", "rotate_quant.hip", "rotate_quant_mfma.hip", "gemm_w4a4.hip", "nfds.hip",
           "rotate_quant_general.hip", "rotate_quant_paley.hip", "gemm_e2m3.hip", "gemm_e2m3_256.hip", "gemm_resident.hip",
           "gemm_resident_1024_wide.hip", "gemm_resident_1280_2048.hip", "gemm_resident_1536_1792.hip", "gemm_resident_affine.hip", "linear_small.hip", "ceilings.hip", "calib.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # no packed-fp32 instructions: some of their forms are unreliable on this hardware
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", INCLUDE, "-Wall", "-Wno-unused-function",
    # the global -> LDS transfer wrappers name M0 (a register the compiler reserves) as clobbered, which it reports for every use
    "-Wno-inline-asm",
]
# results of the matrix instructions in ordinary registers, where the epilogue reads them without a copy
FLAGS_OF = {s: ["-mllvm", "-amdgpu-mfma-vgpr-form=1"] for s in SOURCES if s.startswith("gemm_resident")}


def _compile(src: str, save_temps: bool) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, *FLAGS_OF.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    if save_temps:
        cmd.append("-save-temps=obj")
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _compile_call() -> None:
    """csrc/call.cpp against torch's headers (host code).  It reads torch's objects through inlined accessors, so it is for this torch only and
    says which that is."""
    import torch
    top = os.path.dirname(torch.__file__)
    tmp = CALL + ".tmp"
    cmd = [os.environ.get("CXX", "g++"), "-std=c++17", "-O2", "-fPIC", "-shared", "-Wall", "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__",
           f'-DQVGGT_TORCH_VERSION="{torch.__version__}"',
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-isystem", os.path.join(top, "include"), "-isystem", "/opt/rocm/include",
           "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "call.cpp"), "-o", tmp, "-L" + os.path.join(top, "lib"),
           "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed on call.cpp:\n{r.stderr}")
    if r.stderr.strip():
        sys.stderr.write(r.stderr)
    os.replace(tmp, CALL)


def build(save_temps: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as ex:
        call = ex.submit(_compile_call)
        objs = list(ex.map(lambda s: _compile(s, save_temps), SOURCES))
        try:
            call.result()
        except (ImportError, OSError, RuntimeError) as e:       # the library does without it: no torch headers, no host compiler
            if os.path.exists(CALL):
                os.remove(CALL)                                 # of an older source
            sys.stderr.write(f"{e}\n{os.path.basename(CALL)} was not built: DsfqLinear's calls will go through Python, some microseconds slower\n")
    tmp = LIB + ".tmp"
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(save_temps="--save-temps" in sys.argv))
