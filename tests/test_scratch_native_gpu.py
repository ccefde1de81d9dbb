"""Checks in the caller's device memory on native kernels, which need only the control block: a
large AUTO check builds its kernel first instead of starting on the interpreter, whose value
files and descriptors may not fit.
"""
import pytest

import miters

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", ["auto", "specialized"])
@pytest.mark.parametrize("words", [None, (1 << 20, (1 << 25) + 77)])
def test_small_scratch(kernel, words):
    import paper_2512_06627_amd as es
    c = es.fastlec_es_load_aig(miters.workload("mac8_fused_separate").to_aig())
    scratch = torch.zeros(4096, dtype=torch.uint8, device="cuda")
    rng = {} if words is None else {"begin_word": words[0], "end_word": words[1]}
    for _ in range(2):
        r = es.fastlec_es_check(c, kernel=kernel, scratch=scratch, stream=torch.cuda.current_stream(), **rng)
        assert r["verdict"] == es.FASTLEC_EQUIVALENT
        assert r["patterns_evaluated"] == (1 << 32 if words is None else 64 * (words[1] - words[0]))
