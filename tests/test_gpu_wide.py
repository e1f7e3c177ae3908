"""GPU parity of the register-decoded product of five and more tokens in each
of its workgroup shapes (128 x 4, 64 x 4, 64 x 2, 32 x 1 tokens x tiles; K
whole or in 2, 4 or 8 parts), lone and grouped, against the CPU oracle: int32
sums bit-exact, fp32 outputs equal to the fp32 epilogue of those sums."""
import sys

import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    d = torch.device("cuda:0")
    torch.cuda.set_device(d)
    return d


def _epilogue(acc, sx, sw):
    # y = float(acc) * (sx * sw) in fp32; the sums are exact in fp32
    s = (sx[:, None] * np.broadcast_to(np.float32(sw), acc.shape[1:])[None, :]).astype(np.float32)
    return (acc.astype(np.float32) * s).astype(np.float32)


def _inputs(dev, m, n, k, tag):
    t = synth.ternary_34(n, k, 9, "wide", tag)
    q = synth.int8_any(m, k, 9, "wide", tag, m)
    sx = (np.random.default_rng(m + n).random(m) + 0.01).astype(np.float32)
    import paper_2601_07892_amd as sh
    w = torch.from_numpy(sh.sherry_pack(t)).to(dev)
    return t, q, sx, w, torch.from_numpy(q).to(dev), torch.from_numpy(sx).to(dev)


# by the launch's cost model: 32 x 1 (K in 4), 32 x 1 (K in 8), 64 x 2 (K in
# 2), 64 x 2 (K in 4), 64 x 4, 128 x 4; token, row and K remainders of each
# (k % 128 and k % 16 of every kind, parts of K that are shorter or empty)
LONE = [(5, 1, 4), (33, 65, 68), (70, 130, 1028), (300, 330, 644), (257, 1030, 1540), (31, 64, 384),
        (65, 70, 8196), (100, 130, 12292), (16, 3072, 3072),
        (513, 2052, 132), (257, 4100, 136), (65, 12300, 260), (700, 2100, 276),
        (8193, 70, 8196), (193, 5122, 8200),
        (385, 5122, 132), (6145, 300, 4), (129, 12300, 140), (513, 4104, 388),
        (193, 16390, 2052), (1025, 4100, 2056)]


@pytest.mark.parametrize("m,n,k", LONE)
@pytest.mark.parametrize("channel", [False, True])
def test_lone(dev, m, n, k, channel):
    import paper_2601_07892_amd as sh
    print("[case] wide", m, n, k, channel, file=sys.stderr, flush=True)
    t, q, sx, w, qd, sxd = _inputs(dev, m, n, k, "lone")
    y = torch.full((m, n), float("nan"), dtype=torch.float32, device=dev)
    acc = torch.full((m, n), -7, dtype=torch.int32, device=dev)
    if channel:
        sw = (np.random.default_rng(n).random(n) * 0.05 + 0.001).astype(np.float32)
        sh.sherry_gemm_channel(w, qd, sxd, torch.from_numpy(sw).to(dev), y, acc, m, n, k,
                               sh.SHERRY_KERNEL_SKINNY)
    else:
        sw = np.float32(0.0173)
        sh.sherry_gemm_ex(w, qd, sxd, float(sw), y, acc, m, n, k, sh.SHERRY_KERNEL_SKINNY)
    torch.cuda.synchronize()
    ref = oracle.gemm_i32(q, t, threads=16)
    assert np.array_equal(acc.cpu().numpy(), ref)
    assert np.array_equal(y.cpu().numpy(), _epilogue(ref, sx, sw))
    # without sums, and an output that only 4-byte stores can write
    y2 = torch.full((m * n + 1,), float("nan"), dtype=torch.float32, device=dev)
    if not channel:
        sh.sherry_gemm_ex(w, qd, sxd, float(sw), y2[1:].view(m, n), None, m, n, k,
                          sh.SHERRY_KERNEL_SKINNY)
        torch.cuda.synchronize()
        assert torch.equal(y2[1:].view(m, n), y) and bool(torch.isnan(y2[0]))


# (m, n, k) of the products of one launch, by prepared blocks (8 tiles x 64
# tokens): up to 32, 64, 128 and more; odd and even numbers of token blocks,
# one token, a single tile, ragged rows
FEW = [(33, 70, 132), (64, 1030, 260), (129, 300, 1540), (1, 64, 128)]
MORE = FEW + [(128, 4100, 132), (257, 520, 388)]
MANY = MORE + [(700, 1030, 260), (64, 16390, 136)]
MOST = MANY + [(257, 4100, 132), (129, 2052, 516)]


@pytest.mark.parametrize("shapes,low,high", [(FEW, 1, 32), (MORE, 33, 64), (MANY, 65, 128),
                                             (MOST, 129, 256)])
@pytest.mark.parametrize("channel", [False, True])
def test_grouped(dev, shapes, low, high, channel):
    import paper_2601_07892_amd as sh
    descs = (sh.sherry_gemm_desc * len(shapes))()
    cases, keep = [], []
    for i, (m, n, k) in enumerate(shapes):
        t, q, sx, w, qd, sxd = _inputs(dev, m, n, k, "grouped%d" % i)
        y = torch.full((m, n), float("nan"), dtype=torch.float32, device=dev)
        acc = torch.full((m, n), -7, dtype=torch.int32, device=dev)
        sw = (np.random.default_rng(n).random(n) * 0.05 + 0.001).astype(np.float32) if channel \
            else np.float32(0.0173)
        swd = torch.from_numpy(np.atleast_1d(sw)).to(dev)
        d = descs[i]
        d.w, d.x, d.x_scale, d.y = w.data_ptr(), qd.data_ptr(), sxd.data_ptr(), y.data_ptr()
        d.acc = acc.data_ptr() if i % 2 == 0 else None
        d.w_scales = swd.data_ptr() if channel else None
        d.n, d.k, d.m, d.w_scale = n, k, m, float(np.float32(0.0173))
        keep.append((w, qd, sxd, swd))
        cases.append((t, q, sx, sw, y, acc))
    total, value = sh.sherry_gemm_batched_prepare(descs)
    print("[case] wide grouped", len(shapes), total, value, file=sys.stderr, flush=True)
    assert low <= total <= high and value > 32
    sh.sherry_gemm_batched(torch.from_numpy(sh.descs_to_bytes(descs)).to(dev), len(shapes), total,
                           value)
    torch.cuda.synchronize()
    for i, (t, q, sx, sw, y, acc) in enumerate(cases):
        ref = oracle.gemm_i32(q, t, threads=16)
        if i % 2 == 0:
            assert np.array_equal(acc.cpu().numpy(), ref)
        assert np.array_equal(y.cpu().numpy(), _epilogue(ref, sx, sw))
