"""The generated simulation pass, executed on the host and compared with what the assembler makes of it.

The driver (tests/native/sim_driver.cpp) encodes a circuit's pass with the library's own sources, runs
the words one instruction at a time from registers full of rubbish, with every address checked, and
compares each row with a plain evaluation, for whole and ragged waves and for few registers and many.
"""
import os
import subprocess

import numpy as np
import pytest

import miters

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_06627_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang"


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = tmp_path_factory.mktemp("native") / "sim_driver"
    srcs = [os.path.join(CSRC, f) for f in ("aig.cpp", "native_sim_emit.cpp")]
    r = subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=all", "-I" + CSRC,
                        os.path.join(ROOT, "tests", "native", "sim_driver.cpp"), *srcs, "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return str(exe)


def special():
    """Gates that read the constant, one input twice, and gates that nothing reads."""
    g = miters.Aig(5)
    g.ands += [(3, 0), (3, 1), (5, 4), (4, 4), (2 * 9 + 1, 2 * 6), (2 * 7, 2 * 8 + 1)]
    g.add_output(2 * 10)
    return g


CASES = [("special", special), ("mult6", lambda: miters.mult_miter(6, "booth")),
         ("layered", lambda: miters.layered_cone_miter(3, 17, 900)), ("wide", lambda: miters.layered_cone_miter(4, 40, 2500))]


@pytest.mark.parametrize("name,make", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("vgprs,words", [(112, 64), (240, 1), (240, 37), (240, 64), (8, 64)])
def test_rows(driver, tmp_path, name, make, vgprs, words):
    f = tmp_path / "c.aig"
    f.write_bytes(make().to_aag())
    r = subprocess.run([driver, str(f), str(vgprs), str(words)], capture_output=True, text=True)
    other = [x for x in r.stdout.split("\n") if not x.startswith("asm")]
    assert r.returncode == 0, (other[:3], r.stderr[-2000:])
    if vgprs == 240:
        assert "does not fit" not in other
    if "does not fit" in other or words != 64:
        return
    lines = [x.split(maxsplit=1)[1] for x in r.stdout.split("\n") if x.startswith("asm")]
    hexes, text = [], []
    for x in lines:
        t = x.split()
        k = 2 if len(t[1]) == 8 and all(c in "0123456789abcdef" for c in t[1]) else 1
        hexes += t[:k]
        text.append(" ".join(t[k:]))
    src, obj, raw = tmp_path / "p.s", tmp_path / "p.o", tmp_path / "p.bin"
    src.write_text("\n".join(text) + "\n")
    subprocess.run([CLANG, "-c", "-x", "assembler", "-target", "amdgcn-amd-amdhsa", "-mcpu=gfx950", str(src), "-o",
                    str(obj)], check=True)
    subprocess.run(["/opt/rocm/llvm/bin/llvm-objcopy", "-O", "binary", "-j", ".text", str(obj), str(raw)], check=True)
    assert np.array_equal(np.frombuffer(raw.read_bytes(), dtype=np.uint32)[:len(hexes)],
                          np.array([int(h, 16) for h in hexes], dtype=np.uint32))
