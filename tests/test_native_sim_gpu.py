"""Repeated simulations of a circuit, which the library moves to a native pass once it pays: new
input words in every call, word counts that change on the way (whole and ragged waves, several
waves a workgroup, a second round), every row against the plain CPU oracle.
"""
import numpy as np
import pytest

import miters
from oracle import rsim

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = {
    "layered27": (lambda: miters.layered_cone_miter(41, 27, 3000), [1003, 1, 64, 65, 16384, 16385]),
    "mult12": (lambda: miters.workload("mult12_array_booth"), [200, 4096, 70001]),
    "wide": (lambda: miters.layered_cone_miter(42, 14, 9000), [322, 33]),
    "small": (lambda: miters.mult_miter(4, "booth"), [77, 131072 + 64 * 3072 + 5]),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_repeated(name):
    import paper_2512_06627_amd as es
    make, sizes = CASES[name]
    g = make()
    c = es.fastlec_es_load_aig(g.to_aig())
    rows, n = g.max_var + 1, g.num_inputs
    rng = np.random.default_rng(1)
    for call in range(30):  # 15 or so calls are enough
        W = sizes[0]
        pi = torch.zeros((n, W), dtype=torch.int32, device="cuda")
        sig = torch.empty((rows, W), dtype=torch.int32, device="cuda")
        es.fastlec_es_simulate(c, pi, W, sig, stream=torch.cuda.current_stream())
    for W in sizes + sizes[:1]:
        w = rng.integers(0, 2**32, (n, W), dtype=np.uint32)
        pi = torch.from_numpy(w.view(np.int32).copy()).cuda()
        sig = torch.full((rows * W + 64,), -1, dtype=torch.int32, device="cuda")
        print(name, W, flush=True)
        es.fastlec_es_simulate(c, pi, W, sig, stream=torch.cuda.current_stream())
        got = sig.cpu().numpy().view(np.uint32)
        assert np.array_equal(got[:-64].reshape(rows, W), rsim.simulate(g.to_aag(), w)), W
        assert np.all(got[-64:] == 0xFFFFFFFF)
