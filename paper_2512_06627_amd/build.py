"""Build the exact-simulation library for gfx950 in-tree (hipcc; no GPU needed).

Produces paper_2512_06627_amd/_lib/libfastlec_es.so from csrc/.  Sources are
compiled in parallel to objects under _build/, then linked with hipRTC; the compile
helper program _lib/fastlec_es_rtc is built from rtc/.
"""
import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT_DIR = os.path.join(HERE, "_lib")
LIB = os.path.join(OUT_DIR, "libfastlec_es.so")
BUILD = os.path.join(ROOT, "_build")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-result",
          "-I" + os.path.join(ROOT, "include"), "-I/opt/rocm/include"]
# Packed FP32 instructions are disabled for all device code.
DEVICE = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    if src.endswith(".hip"):
        cmd = [HIPCC, "-x", "hip"] + DEVICE + COMMON + ["-c", src, "-o", obj]
    else:  # host-only C++ that calls the HIP runtime
        cmd = [HIPCC, "-x", "c++", "-D__HIP_PLATFORM_AMD__"] + COMMON + ["-c", src, "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {src}\n{r.stdout}\n{r.stderr}")
    return obj


def _native_template(verbose: bool) -> str:
    """Object file that embeds the code object of native/es_native.hip, the host kernel of the
    passes that the library encodes at run time."""
    code = os.path.join(BUILD, "es_native.co")
    cmd = [HIPCC, "-x", "hip"] + DEVICE + COMMON + ["--cuda-device-only", "--no-gpu-bundle-output", "-fuse-cuid=none",
           "-c", os.path.join(HERE, "native", "es_native.hip"), "-o", code]
    src = os.path.join(BUILD, "es_native_template.S")
    obj = src + ".o"
    with open(src, "w") as f:
        f.write('.section .rodata\n.globl fes_native_template\n.hidden fes_native_template\n'
                '.globl fes_native_template_end\n.hidden fes_native_template_end\n.balign 64\n'
                f'fes_native_template:\n.incbin "{code}"\nfes_native_template_end:\n.byte 0\n'
                '.section .note.GNU-stack,"",@progbits\n')
    for c in (cmd, ["gcc", "-c", src, "-o", obj]):
        if verbose:
            print(" ".join(c), flush=True)
        r = subprocess.run(c, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"native template failed\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    os.makedirs(OUT_DIR, exist_ok=True)
    srcs = sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".cpp", ".hip")))
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        template = ex.submit(_native_template, verbose)
        objs = list(ex.map(lambda s: _compile(s, verbose), srcs)) + [template.result()]
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs + [
        "-L/opt/rocm/lib", "-lhiprtc", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    # The compile helper program (grouped hipRTC compiles in child processes), next to the library.
    helper = os.path.join(OUT_DIR, "fastlec_es_rtc")
    cmd = [HIPCC, "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-O2", "-std=c++17", "-I/opt/rocm/include",
           os.path.join(HERE, "rtc", "fastlec_es_rtc.cpp"), "-o", helper + ".tmp",
           "-L/opt/rocm/lib", "-lhiprtc", "-Wl,-rpath,/opt/rocm/lib"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile helper failed\n{r.stdout}\n{r.stderr}")
    os.replace(helper + ".tmp", helper)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
