"""Builds the library's host sources, the native tier among them, against the host stand-in of a GPU
(tests/sanitize/): as a shared library for the package, or as a program with a sanitizer.

The stand-in runs interpreter launches from the descriptors and streams that the kernels read, native
launches by executing the generated machine code, and the finish kernel on a thread of its own.  Its
simulations and hashes plan and build like the library's and then fail, and it has no autotuning.
"""
import concurrent.futures
import os
import subprocess

from paper_2512_06627_amd import build as lib_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_06627_amd", "csrc")
SAN = os.path.join(ROOT, "tests", "sanitize")
CLANG = "/opt/rocm/llvm/bin/clang++"
HOST_SOURCES = ("aig", "batch", "capi", "cofactor", "emit_block", "lut", "model", "native", "native_build",
                "native_emit", "native_sim", "native_sim_emit", "plan", "runtime", "server", "sweep")
# Functions of fake_device.cpp that native_device.cpp replaces and calls, by their second name.
SECOND_NAMES = {"launch_interp(": "standin_interp", "launch_interp_regs(": "standin_regs",
                "jit_prepare(": "standin_prepare", "jit_enqueue(": "standin_enqueue"}


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, (cmd[:3], r.stderr[-3000:])
    return r.stdout


def build(out_dir, sanitize=None, drivers=(), opt="-O2"):
    """The shared library's path, or with driver sources (of tests/sanitize/) the programs' paths."""
    template = lib_build._native_template(False)
    san = [f"-fsanitize={sanitize}", "-fno-omit-frame-pointer"] if sanitize else []
    flags = ["-std=c++17", opt, "-g", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROOT, "include"),
             "-I/opt/rocm/include", "-I" + CSRC]
    srcs = [os.path.join(CSRC, f + ".cpp") for f in HOST_SOURCES] + [
        os.path.join(SAN, f) for f in ("fake_device.cpp", "native_device.cpp", "native_emulator.cpp")]
    srcs += [os.path.join(SAN, d) for d in drivers]

    def compile_one(src):
        obj = os.path.join(str(out_dir), os.path.basename(src) + ".o")
        extra = ["-O2"] if src.endswith("native_emulator.cpp") else san
        _run([CLANG] + flags + extra + ["-c", src, "-o", obj])
        return obj

    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        objs = list(ex.map(compile_one, srcs))
    fake = next(o for o in objs if o.endswith("fake_device.cpp.o"))
    mangled = {}
    for line in _run(["nm", fake]).splitlines():
        name = line.split()[-1]
        plain = _run(["c++filt", name]).strip() if "_ZN3fes" in name and " T " in line else ""
        for start, second in SECOND_NAMES.items():
            if plain.startswith("fes::" + start):
                mangled[name] = second
    assert len(mangled) == len(SECOND_NAMES), mangled
    _run(["objcopy", "--weaken"] + [f"--redefine-sym={a}={b}" for a, b in mangled.items()] + [fake])
    if not drivers:
        out = os.path.join(str(out_dir), "libstandin.so")
        # -Bsymbolic: in a process with the HIP runtime the stand-in's own functions are meant.
        _run([CLANG, "-shared", "-Wl,-Bsymbolic", "-Wl,-z,defs", "-o", out] + objs + [template, "-lpthread"])
        return out
    common, outs = objs[:len(objs) - len(drivers)], []
    for obj in objs[len(common):]:
        outs.append(obj[:-len(".cpp.o")])
        _run([CLANG] + san + ["-o", outs[-1]] + common + [obj, template, "-lpthread"])
    return outs
