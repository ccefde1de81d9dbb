"""Sub-miter texts around the binding's first guess at their length (64 KB), against the oracle."""
import numpy as np
import pytest

import miters
import paper_2512_06627_amd as es
from oracle import sweep


@pytest.mark.parametrize("gates", [40, 3000, 4500, 9000])
def test_text_lengths(gates):
    g = miters.layered_cone_miter(gates, 30, gates)
    rows = g.max_var + 1
    cls = np.arange(rows, dtype=np.uint32)
    pol = np.random.default_rng(gates).integers(0, 2, rows).astype(np.uint8)
    target = rows - 1
    cls[target] = rows // 2 + g.num_inputs // 2  # a gate well below
    want = sweep.submiter_aag(g.to_aag(), cls.tolist(), pol.tolist(), target)
    got = es.fastlec_es_submiter_aag(es.fastlec_es_load_aig(g.to_aig()), cls, pol, target)
    assert got[0] == (want[0] if isinstance(want[0], bytes) else want[0].encode())
    assert list(got[1]) == list(want[1])
    assert gates < 4500 or len(got[0]) > 1 << 16
