"""Device packing at the edges of its work split: units per tile on both sides
of a round of eight (ternarize + pack) for every number of rows per workgroup,
and unit counts on both sides of a workgroup of four (the lane-interleaving
converter).  Bytes equal the host packers'; alpha within one fp32 unit of the
oracle's fp64 mean; nothing outside the outputs is written."""
import sys

import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GUARD = 4096


@pytest.fixture(scope="module")
def dev():
    d = torch.device("cuda:0")
    torch.cuda.set_device(d)
    return d


def _guarded(nbytes, dev):
    return torch.full((nbytes + 2 * GUARD,), 0xA5, dtype=torch.uint8, device=dev)


def _inside(buf):
    b = buf.cpu().numpy()
    assert (b[:GUARD] == 0xA5).all() and (b[-GUARD:] == 0xA5).all()
    return b[GUARD:-GUARD]


# tiles: 1 and 15 (4 rows per workgroup), 16 (8), 64 (16), 65 (8), 119 and 129
# (8 on either side of 16)
@pytest.mark.parametrize("n", [61, 15 * 64 - 1, 16 * 64 - 33, 63 * 64 + 5, 65 * 64, 119 * 64, 120 * 64 - 7,
                               128 * 64 + 2])
@pytest.mark.parametrize("units", [1, 7, 8, 9, 17])
def test_ternarize_and_interleave_edges(dev, n, units):
    import paper_2601_07892_amd as sh
    print("[case] pack edges", n, units, file=sys.stderr, flush=True)
    k = 128 * units - 4 * (n % 3)
    w = synth.dense_weights(n, k, 91, "edges", n, units)
    nbytes = sh.sherry_packed_bytes(n, k)
    packed, il = _guarded(nbytes, dev), _guarded(nbytes, dev)
    alpha = torch.full((n,), float("nan"), dtype=torch.float32, device=dev)
    view = lambda b: b[GUARD:GUARD + nbytes]  # noqa: E731
    sh.sherry_ternarize_pack(torch.from_numpy(w).to(dev), n, k, view(packed), alpha)
    sh.sherry_interleave(view(packed), view(il), n, k)
    torch.cuda.synchronize()
    t_ref, alpha_ref = oracle.ternarize_rows(w)
    assert np.array_equal(_inside(packed), sh.sherry_pack(t_ref))
    assert np.array_equal(_inside(il), sh.sherry_pack_il(t_ref))
    a, r = alpha.cpu().numpy().astype(np.float64), alpha_ref.astype(np.float32)
    assert (np.abs(a - r) <= np.spacing(np.maximum(np.abs(a).astype(np.float32), r))).all()
