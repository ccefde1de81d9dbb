"""Checks whose kernel changes from call to call, on the GPU: built beside pieces of a check with a deadline
or cancel flag, made for a few words before the whole space is checked, or not to be had at all.  Every
answer follows from where the circuits differ.
"""
import ctypes

import pytest

import miters
import oracle
import paper_2512_06627_amd as es

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def differs_at(g, pattern):
    """The miter's outputs and one more that is true at a single pattern (None: nowhere)."""
    m = miters.Aig(g.num_inputs)
    for o in miters.import_into(m, g):
        m.add_output(o)
    if pattern is not None:
        t = 1
        for j in range(g.num_inputs):
            t = m.AND(t, m.input(j) ^ (0 if (pattern >> j) & 1 else 1))
        m.add_output(t)
    return es.fastlec_es_load_aig(m.to_aig())


def check(c, where, n, begin=0, end=None, **kw):
    words = 1 << (n - 6)
    end = words if end is None else end
    r = es.fastlec_es_check(c, begin_word=begin, end_word=end, **kw)
    inside = where is not None and begin <= where // 64 < end
    assert r["verdict"] == (es.FASTLEC_NONEQUIVALENT if inside else es.FASTLEC_EQUIVALENT), (where, begin, end, kw)
    assert r["patterns_evaluated"] == (where - 64 * begin + 1 if inside else 64 * (end - begin))
    if inside:
        assert r["cex"] == where


@pytest.mark.parametrize("how", ["deadline", "cancel", "scratch"])
@pytest.mark.parametrize("where", [None, 5, (1 << 29) + 777])
def test_built_beside_pieces(how, where):
    c = differs_at(miters.mac_miter(8), where)
    flag = ctypes.c_int(0)
    kw = {"deadline": {"deadline_s": 120.0}, "cancel": {"cancel_flag": flag},
          "scratch": {"deadline_s": 120.0, "scratch": torch.zeros(4096, dtype=torch.uint8, device="cuda"),
                      "stream": torch.cuda.current_stream()}}[how]
    for _ in range(3):
        check(c, where, 32, **kw)
        check(c, where, 32, 12345, (1 << 25) + 77, **kw)
    check(c, where, 32)


@pytest.mark.parametrize("kernel", ["auto", "specialized"])
@pytest.mark.parametrize("where", [None, 64 * 9 + 3, (1 << 28) - 2])
def test_few_words_before_the_whole_space(kernel, where):
    c = differs_at(miters.mult_miter(14, "booth"), where)
    for _ in range(3):
        check(c, where, 28, 8, 10, kernel=kernel)
    for _ in range(60):  # more than its own kernel's building
        check(c, where, 28, kernel=kernel)
    check(c, where, 28, 3, 70001, kernel=kernel)
    inside = where is not None
    for r in es.fastlec_es_check_batch([c, c], kernel=kernel):
        assert (r["verdict"], r["cex"]) == ((1, where) if inside else (0, 0))


def test_no_kernel_to_be_had():
    g = miters.layered_cone_miter(1, 14, 27000, fault_seed=3)
    want = oracle.check(g.to_aag(), threads=8)
    cs = [es.fastlec_es_load_aig(g.to_aig()) for _ in range(4)]
    answer = lambda r: r["cex"] if r["verdict"] == es.FASTLEC_NONEQUIVALENT else None
    with pytest.raises(es.EsError):
        es.fastlec_es_native_info(cs[0])
    for _ in range(5):
        assert answer(es.fastlec_es_check(cs[0])) == want
        assert answer(es.fastlec_es_check(cs[0], deadline_s=60.0)) == want
        assert [answer(r) for r in es.fastlec_es_check_batch(cs)] == [want] * 4
    srv = es.Server(1 << 34)
    assert [answer(srv.poll(t, wait=True)) for t in [srv.submit(c) for c in cs]] == [want] * 4
    srv.close()
