"""Calls on torch's default stream wait for the work that torch has put there.

A fill of several gigabytes is still running when the call is made; the call's results are
those of the filled buffer, and are not overwritten by the fill.
"""
import numpy as np
import pytest

import miters
from oracle import rsim

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("entry", ["simulate", "hash"])
def test_ordered_after_torch(entry):
    import paper_2512_06627_amd as es
    g = miters.workload("mult6_array_wallace")
    c = es.fastlec_es_load_aig(g.to_aig())
    W, n = 1 << 14, g.num_inputs
    words = np.random.default_rng(5).integers(0, 2**32, (n, W), dtype=np.uint32)
    pi = torch.from_numpy(words.view(np.int32).copy()).cuda()
    rows = g.max_var + 1
    out = torch.zeros((2, rows), dtype=torch.int64, device="cuda")
    sig = torch.zeros((rows, W), dtype=torch.int32, device="cuda")
    stream = torch.cuda.current_stream()
    es.fastlec_es_simulate(c, pi, W, sig, stream=stream)  # plans and buffers are there
    es.fastlec_es_signature_hash(sig, rows, W, out[0], out[1], stream=stream)
    big = torch.zeros(1 << 30, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    big.fill_(3)
    sig.fill_(-1)
    if entry == "simulate":
        es.fastlec_es_simulate(c, pi, W, sig, stream=stream)
        assert np.array_equal(sig.cpu().numpy().view(np.uint32), rsim.simulate(g.to_aag(), words))
    else:
        es.fastlec_es_signature_hash(sig, rows, W, out[0], out[1], stream=stream)
        assert torch.all(out[1] == 32 * W) and torch.all(out[0] == 0)
