"""The register tier's simulation pass at the edges of its groups, blocks and rounds.

Gate counts around the groups of 8 and the record blocks of 64; word counts around a
wave, a workgroup per CU, several waves a workgroup and a second round of workgroups, odd
ones among them; compared bit for bit with the plain CPU oracle.
"""
import numpy as np
import pytest

from miters.aig import Aig
from oracle import rsim

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def chain(n, gates, seed):
    """`gates` AND gates over `n` inputs with random operands and complements."""
    rng = np.random.default_rng(seed)
    g = Aig(n)
    lits = [g.input(i) for i in range(n)]
    while len(g.ands) < gates:
        a, b = rng.choice(len(lits), 2, replace=False)
        x = g.AND(lits[a] ^ int(rng.integers(2)), lits[b] ^ int(rng.integers(2)))
        if x > 1 and (x >> 1) not in {v >> 1 for v in lits}:
            lits.append(x)
    g.add_output(lits[-1])
    return g


@pytest.mark.parametrize("gates,words", [
    (1, 1), (7, 63), (8, 64), (9, 65), (63, 129), (64, 16384), (65, 16385), (72, 3 * 16384 + 1),
    (128, 33000), (129, 65537), (200, 100003), (9, 262144), (17, 262145), (65, 300007),
])
def test_edges(gates, words):
    import paper_2512_06627_amd as es
    n = 12
    g = chain(n, gates, seed=gates)
    w = np.random.default_rng(words).integers(0, 2**32, (n, words), dtype=np.uint32)
    c = es.fastlec_es_load_aig(g.to_aig())
    pi = torch.from_numpy(w.view(np.int32).copy()).cuda()
    guard = 64
    sig = torch.full(((n + 1 + gates) * words + guard,), -1, dtype=torch.int32, device="cuda")
    es.fastlec_es_simulate(c, pi, words, sig, stream=torch.cuda.current_stream())
    got = sig.cpu().numpy().view(np.uint32)
    assert np.array_equal(got[:-guard].reshape(-1, words), rsim.simulate(g.to_aag(), w))
    assert np.all(got[-guard:] == 0xFFFFFFFF)
