"""The native tier's generated machine code, executed on the host against the oracle.

The driver (tests/native/native_driver.cpp) plans, maps and encodes a circuit's pass with the
library's own sources and runs the words one instruction at a time, with every register that a
pass may not read before writing filled with rubbish.  Every assignment's miter word of every lane
must equal the oracle's, for no inner input and for several, in ample registers and in so few that
values go through LDS.  The words themselves must be what the assembler makes of their text.
"""
import os
import subprocess

import numpy as np
import pytest

import miters
import oracle
from miters.miter import mult_circuit

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_06627_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang"


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = tmp_path_factory.mktemp("native") / "native_driver"
    srcs = [os.path.join(CSRC, f) for f in ("aig.cpp", "plan.cpp", "lut.cpp", "cofactor.cpp", "native_emit.cpp")]
    r = subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=all", "-I" + CSRC,
                        os.path.join(ROOT, "tests", "native", "native_driver.cpp"), *srcs, "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return str(exe)


def product_bit(w, j):
    """Output j of a w x w multiplier: a function with both values everywhere (no miter)."""
    c = mult_circuit("array", w)
    g = miters.Aig(2 * w)
    g.add_output(miters.import_into(g, c)[j])
    return g


def run_pass(driver, tmp_path, g, k, vgprs, slots, bases):
    f = tmp_path / "c.aig"
    f.write_bytes(g.to_aig())
    r = subprocess.run([driver, str(f), str(k), str(vgprs), str(slots), *map(str, bases)], capture_output=True,
                       text=True)
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])
    return r.stdout.split("\n")


def check(driver, tmp_path, g, k, vgprs=240, slots=255, passes=2, seed=1):
    n = g.num_inputs
    packed = max(1, 1 << max(0, n - k - 11))
    rng = miters.SplitMix64(seed)
    bases = sorted({0, 64 * (packed - 1)} | {64 * rng.below(packed) for _ in range(passes)})
    lines = run_pass(driver, tmp_path, g, k, vgprs, slots, bases)
    if lines[0] == "does not fit":
        return None
    inner = [int(x) for x in lines[0].split()[1:]]
    assert len(inner) == k and all(b >= 6 for b in inner)
    size = [int(x) for x in lines[1].split()[1:]]
    o = oracle.Circuit(g.to_aag())
    seen = {}
    base = None
    for line in lines[2:]:
        t = line.split()
        if not t or t[0] == "asm":
            continue
        if t[0] == "pass":
            base = int(t[1])
            seen[base] = set()
            continue
        assert t[0] == "word"
        off = int(t[1])
        seen[base].add(off)
        real = base
        for b in inner:  # zero bits at the inner positions, lowest first
            real = ((real >> b) << (b + 1)) | (real & ((1 << b) - 1))
        hw = (real | off) + np.arange(64, dtype=np.uint64)
        ps = hw[:, None] * np.uint64(32) + np.arange(32, dtype=np.uint64)[None, :]
        if n < 11:
            ps = ps % np.uint64(1 << n)
        want = o.miter(ps.reshape(-1)).reshape(64, 32).astype(np.uint64)
        got = np.array([int(x, 16) for x in t[2:]], dtype=np.uint64)
        assert np.array_equal((want << np.arange(32, dtype=np.uint64)).sum(axis=1), got), (k, base, off)
    offs = {sum(1 << b for i, b in enumerate(inner) if (c >> i) & 1) for c in range(1 << k)}
    for base, got in seen.items():
        # an assignment that folds to constant 0 has no word to compare
        assert got <= offs
    return size, lines, seen, offs


@pytest.mark.parametrize("k", [0, 1, 3, 5])
def test_words_match_oracle(driver, tmp_path, k):
    fit = 0
    for g in (product_bit(9, 10), product_bit(8, 7), miters.workload("mult12_array_booth_f2"),
              miters.layered_cone_miter(31, 17, 700, fault_seed=5), miters.minterm_miter(16, [0, 4000, 65535])):
        r = check(driver, tmp_path, g, k, seed=k + 1)
        if r:  # a refused pass is never run; multipliers and minterms always fit
            assert all(got == r[3] for got in r[2].values())
            fit += 1
    assert fit >= 4


@pytest.mark.parametrize("vgprs,slots", [(24, 255), (14, 255), (60, 80)])
def test_spills_match_oracle(driver, tmp_path, vgprs, slots):
    """Few registers: LUT results through LDS slots, words and wave-uniform copies made again."""
    spilled = 0
    for g, k in ((product_bit(9, 9), 2), (miters.workload("mult12_array_booth_f1"), 1),
                 (miters.layered_cone_miter(77, 15, 900, fault_seed=3), 0)):
        r = check(driver, tmp_path, g, k, vgprs, slots, passes=1)
        if r:
            assert r[0][4] <= slots
            spilled += r[0][3]
    assert spilled > 0


def test_small_spaces_and_fixed_outputs(driver, tmp_path):
    for n, t in ((1, [1]), (4, [7, 9]), (6, [40]), (9, [300]), (11, [2047]), (13, [8000, 77])):
        check(driver, tmp_path, miters.minterm_miter(n, t), 0)
    for lit in (0, 1, 2, 3, 15, 24, 27):  # constants, a word input, a lane input, wave-uniform inputs
        g = miters.Aig(14)
        g.add_output(lit)
        check(driver, tmp_path, g, 0)
        check(driver, tmp_path, g, 2)
    g = miters.Aig(13)  # several outputs: their OR
    for lit in (g.AND(2, 5), g.AND(26, 24) ^ 1, 12):
        g.add_output(lit)
    check(driver, tmp_path, g, 1)


def test_refuses_what_does_not_fit(driver, tmp_path):
    lines = run_pass(driver, tmp_path, miters.workload("mult12_array_booth"), 3, 40, 0, [0])
    assert lines[0] == "does not fit"


def test_words_are_what_the_assembler_writes(driver, tmp_path):
    """The encoder against LLVM's assembler, over passes with every instruction form."""
    for g, k, vgprs, slots in ((miters.workload("mult12_array_booth_f2"), 2, 240, 0),
                               (miters.layered_cone_miter(78, 40, 900, fault_seed=3), 3, 20, 255)):
        lines = [x[4:] for x in run_pass(driver, tmp_path, g, k, vgprs, slots, []) if x.startswith("asm ")]
        text = [x.split(" | ")[0] for x in lines]
        words = [int(w, 16) for x in lines for w in x.split(" | ")[1].split()]
        assert {"v_bitop3_b32", "v_mov_b32", "s_bfe_i32", "v_cmp_ne_u32", "s_cbranch_vccnz", "s_branch", "s_mov_b32",
                "s_setpc_b64", "s_swappc_b64"} <= {x.split()[0] for x in text}
        src, obj, raw = tmp_path / "p.s", tmp_path / "p.o", tmp_path / "p.bin"
        src.write_text("\n".join(text) + "\n")
        subprocess.run([CLANG, "-c", "-x", "assembler", "-target", "amdgcn-amd-amdhsa", "-mcpu=gfx950", str(src), "-o",
                        str(obj)], check=True)
        subprocess.run(["/opt/rocm/llvm/bin/llvm-objcopy", "-O", "binary", "-j", ".text", str(obj), str(raw)],
                       check=True)
        assert np.array_equal(np.frombuffer(raw.read_bytes(), dtype=np.uint32)[:len(words)],
                              np.array(words, dtype=np.uint32))
