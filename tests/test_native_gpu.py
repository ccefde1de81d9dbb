"""Native kernels (generated machine code) on the GPU against the oracle: every number of inner
inputs, spaces below one wave, ragged word ranges, chunked checks, and many kernels in one launch.
Answers are the verdict and the lowest failing pattern, compared exactly."""
import os

import pytest

import miters
import oracle
import paper_2512_06627_amd as es

pytestmark = pytest.mark.gpu


def answer(r):
    assert r["verdict"] in (es.FASTLEC_EQUIVALENT, es.FASTLEC_NONEQUIVALENT)
    return r["cex"] if r["verdict"] == es.FASTLEC_NONEQUIVALENT else None


def circuits():
    rng = miters.SplitMix64(61)
    out = [miters.mult_miter(7, "booth"), miters.mult_miter(8, "wallace", fault_seed=2),
           miters.minterm_miter(17, [131071, 90000]), miters.minterm_miter(20, [1 << 19, 999999]),
           miters.layered_cone_miter(611, 18, 1500, fault_seed=3), miters.layered_cone_miter(612, 19, 900)]
    for i in range(3):  # the only failing pattern anywhere in the space
        g = miters.Aig(21)
        base = miters.import_into(g, miters.layered_cone_miter(620 + i, 21, 700))
        t = 1
        p = rng.below(1 << 21)
        for j in range(21):
            t = g.AND(t, g.input(j) ^ (0 if (p >> j) & 1 else 1))
        for o in base:
            g.add_output(o)
        g.add_output(t)
        out.append(g)
    return out


@pytest.mark.parametrize("inner", range(6))
def test_inner_inputs_match_oracle(monkeypatch, inner):
    monkeypatch.setenv("FASTLEC_ES_NATIVE_INNER", str(inner))
    for i, g in enumerate(circuits()):
        c = es.fastlec_es_load_aig(g.to_aig())
        print("inner", inner, "circuit", i, flush=True)
        assert answer(es.fastlec_es_check(c, kernel="specialized")) == oracle.check(g.to_aag(), threads=8)


@pytest.mark.parametrize("inner", [0, 1, 3])
def test_word_ranges_match_oracle(monkeypatch, inner):
    """Ranges that start and end inside a wave, inside a block of inner inputs, or hold one word."""
    monkeypatch.setenv("FASTLEC_ES_NATIVE_INNER", str(inner))
    rng = miters.SplitMix64(62 + inner)
    for g in (miters.minterm_miter(20, [70000, 500000, 1048000]), miters.mult_miter(9, "booth", fault_seed=5),
              miters.layered_cone_miter(631, 19, 1200, fault_seed=2)):
        c = es.fastlec_es_load_aig(g.to_aig())
        o = oracle.Circuit(g.to_aag())
        W = 1 << (g.num_inputs - 6)
        ranges = [(0, 1), (W - 1, W), (0, W), (1, W - 1), (33, 34), (70000 // 64, 70000 // 64 + 1)]
        for _ in range(8):
            a, b = sorted((rng.below(W), rng.below(W)))
            ranges.append((a, b + 1))
        for a, b in ranges:
            want = o.lowest_failure(64 * a, 64 * b, threads=8)[0]
            print("inner", inner, "range", a, b, flush=True)
            r = es.fastlec_es_check(c, kernel="specialized", begin_word=a, end_word=b)
            assert answer(r) == want
            if want is None:
                assert r["patterns_evaluated"] == 64 * (b - a)


def test_small_spaces_match_oracle():
    for n in range(1, 13):
        for t in {0, (1 << n) - 1, (1 << n) // 3}:
            c = es.fastlec_es_load_aig(miters.minterm_miter(n, [t]).to_aig())
            assert answer(es.fastlec_es_check(c, kernel="specialized")) == t


def test_chunked_check_matches_whole():
    g = miters.workload("mult12_array_booth_f1")
    c = es.fastlec_es_load_aig(g.to_aig())
    whole = es.fastlec_es_check(c, kernel="specialized")
    chunked = es.fastlec_es_check(c, kernel="specialized", deadline_s=60.0)
    assert answer(whole) == answer(chunked) == oracle.check(g.to_aag(), threads=8)


def test_batch_of_native_kernels_matches_oracle():
    """One launch per register tier over many kernels, twice (the second from the kept code object);
    a subset next (another set of kernels), then the rest."""
    rng = miters.SplitMix64(63)
    gs = [miters.layered_cone_miter(640 + i, rng.between(8, 18), rng.between(60, 3500),
                                    fault_seed=(i + 1 if i % 3 == 0 else None)) for i in range(40)]
    gs.append(miters.layered_cone_miter(690, 16, 14000, fault_seed=4))  # two waves per SIMD, LDS slots
    want = [oracle.check(g.to_aag(), threads=8) for g in gs]
    cs = [es.fastlec_es_load_aig(g.to_aig()) for g in gs]
    for part in (slice(0, 41), slice(0, 41), slice(5, 20), slice(0, 41)):
        res = es.fastlec_es_check_batch(cs[part], kernel="specialized")
        assert [answer(r) for r in res] == want[part]


def test_repeated_auto_checks_keep_the_answer():
    """AUTO starts a small check on the interpreter and moves to a native kernel once that pays: the
    same answer before and after."""
    g = miters.mult_miter(9, "booth", fault_seed=8)
    c = es.fastlec_es_load_aig(g.to_aig())
    want = oracle.check(g.to_aag(), threads=8)
    assert all(answer(es.fastlec_es_check(c)) == want for _ in range(300))
