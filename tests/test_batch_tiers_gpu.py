"""Batches whose cones need different register files: few passes share one launch at the larger
file, many keep their own; workgroups of eight waves with whole and partial last groups, fewer
items than waves and more.  Every answer is the oracle's.
"""
import pytest

import miters
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [
    [(6, 60)] * 2,
    [(8, 100)] * 7 + [(9, 900)],
    [(10, 120)] * 9 + [(12, 2600), (13, 9000)],
    [(14, 400)] * 33 + [(16, 3000)] * 3 + [(11, 8000)] * 2,
    [(18, 500)] * 40 + [(17, 6000)] * 4,
    [(20, 300)] * 17 + [(19, 9000), (12, 16000)],
])
def test_mixed_files(sizes):
    import paper_2512_06627_amd as es
    gs = [miters.layered_cone_miter(900 + i, n, k, fault_seed=i if i % 3 == 0 else None)
          for i, (n, k) in enumerate(sizes)]
    cs = [es.fastlec_es_load_aig(g.to_aig()) for g in gs]
    want = [oracle.check(g.to_aag(), threads=8) for g in gs]
    for kernel in ("interp", "auto", "auto"):
        got = es.fastlec_es_check_batch(cs, kernel=kernel, stream=torch.cuda.current_stream())
        assert [r["cex"] if r["verdict"] == es.FASTLEC_NONEQUIVALENT else None for r in got] == want, kernel
