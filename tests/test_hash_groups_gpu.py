"""The hash kernel's row groups (1 or 2 rows, by how many rows there are) and its column
chunks of 256 words shared among 1 to 16 waves: rows and words at their edges, rows at every
alignment, both polarities and extreme words, exact against the plain CPU oracle.
"""
import numpy as np
import pytest

from oracle import rsim

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,words", [
    (1, 1), (1, 255), (2, 256), (3, 257), (5, 100003), (255, 511), (511, 1023), (512, 4096), (513, 4099),
    (1023, 769), (1024, 1), (1025, 255), (1027, 2049), (3111, 1001), (4097, 64), (9001, 3),
])
@pytest.mark.parametrize("offset", [0, 1, 3])
def test_groups(rows, words, offset):
    import paper_2512_06627_amd as es
    sig = np.random.default_rng(rows * 7 + words).integers(0, 2**32, (rows, words), dtype=np.uint32)
    sig[rows // 2] = 0xFFFFFFFF
    sig[rows // 3] = 0
    buf = torch.zeros(rows * words + offset, dtype=torch.int32, device="cuda")
    buf[offset:] = torch.from_numpy(sig.reshape(-1).view(np.int32).copy()).cuda()
    out = torch.full((2, rows + 8), -1, dtype=torch.int64, device="cuda")
    es.fastlec_es_signature_hash(buf[offset:], rows, words, out[0], out[1], stream=torch.cuda.current_stream())
    got = out.cpu().numpy()
    wh, wones = rsim.signature_hash(sig)
    assert np.array_equal(got[0, :rows].view(np.uint64), wh)
    assert np.array_equal(got[1, :rows].view(np.uint64), wones)
    assert np.all(got[:, rows:] == -1)
