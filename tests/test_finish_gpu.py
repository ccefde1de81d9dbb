"""Checks that learn of their end by polling the finish kernel's last store.

Behind a long fill on the same stream (the poll gives up and the stream is waited for), many
times in a row, from several threads on their own streams at once, alone and as a batch: every
answer is the oracle's, and the kernel time is that of the kernel, not of the wait.
"""
import threading

import pytest

import miters
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NAMES = ["mult6_array_wallace", "mult6_array_wallace_f1"]


def es():
    import paper_2512_06627_amd as m
    return m


def load(name):
    return es().fastlec_es_load_aig(miters.workload(name).to_aig())


def want_of(name):
    return oracle.check(miters.workload(name).to_aag())


def answer(r):
    assert r["verdict"] in (es().FASTLEC_EQUIVALENT, es().FASTLEC_NONEQUIVALENT)
    return r["cex"] if r["verdict"] == es().FASTLEC_NONEQUIVALENT else None


@pytest.mark.parametrize("kernel", ["interp", "specialized"])
@pytest.mark.parametrize("batch", [False, True])
def test_behind_a_long_fill(kernel, batch):
    cs = [load(n) for n in NAMES]
    stream = torch.cuda.current_stream()

    def run():
        if batch:
            return es().fastlec_es_check_batch(cs, stream=stream, kernel=kernel)
        return [es().fastlec_es_check(c, stream=stream, kernel=kernel) for c in cs]

    want = [want_of(n) for n in NAMES]
    assert [answer(r) for r in run()] == want
    big = torch.zeros(1 << 31, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    for _ in range(4):
        big.fill_(1)
    got = run()
    assert [answer(r) for r in got] == want
    assert all(0 < r["kernel_ms"] < 0.5 for r in got)


@pytest.mark.parametrize("threads", [1, 4])
def test_many_calls(threads):
    want = [want_of(n) for n in NAMES]
    errors = []

    def work(i):
        try:
            cs = [load(n) for n in NAMES]
            stream = torch.cuda.Stream()
            for k in range(1000 // threads):
                kernel = ("interp", "specialized")[k & 1]
                one = es().fastlec_es_check(cs[k % 2], stream=stream, kernel=kernel)
                many = es().fastlec_es_check_batch(cs, stream=stream, kernel=kernel)
                assert answer(one) == want[k % 2] and [answer(r) for r in many] == want
        except BaseException as e:  # noqa: BLE001
            errors.append((i, e))

    ts = [threading.Thread(target=work, args=(i,)) for i in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors
