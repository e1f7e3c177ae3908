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


# the cost model's shapes, every one of which some case takes (checked on the CPU
# beside the launch rules): 32 x 1 (K in 4), 32 x 1 (K in 8), 64 x 2 (K in 2), 64 x
# 2 (K in 4), 64 x 4, 128 x 4; token, row and K remainders of each
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
# tokens): up to 32, 64, 128, 256 and more; odd and even numbers of token blocks,
# one token, a single tile, ragged rows
FEW = [(33, 70, 132), (64, 1030, 260), (129, 300, 1540), (1, 64, 128)]
MORE = FEW + [(128, 4100, 132), (257, 520, 388)]
MANY = MORE + [(700, 1030, 260), (64, 16390, 136)]
MOST = MANY + [(257, 4100, 132), (129, 2052, 516)]
LONGEST = MOST + [(1090, 7000, 132), (193, 1030, 4)]
GROUPED = [(FEW, 1, 32), (MORE, 33, 64), (MANY, 65, 128), (MOST, 129, 256), (LONGEST, 385, 512)]


@pytest.mark.parametrize("shapes,low,high", GROUPED)
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


# ---- per-group scales, and launches of 32-token blocks --------------------------

def _group_scales(n, k, seed):
    return (np.random.default_rng(seed).random((n, -(-k // 128))) * 0.04 + 0.01).astype(np.float32)


def _group_ok(y, q, t, sx, gs, k):
    y_ref, mag, acc = oracle.product_groups(q, t, sx, gs, threads=16)
    G = -(-k // 128)
    assert not (np.abs(y.astype(np.float64) - y_ref) > (G + 4) * 2.0 ** -24 * mag).any()
    return acc


# by the cost model, with 4-byte and (rows of whole aligned pieces) 16-byte
# scale loads: 32 x 2, 32 x 1 (K in 4), 32 x 1 (K in 8), 64 x 2, 64 x 4
LONE_GROUP = [(5, 64, 128), (33, 70, 132), (37, 130, 1028), (31, 300, 516), (100, 70, 8196),
              (385, 8190, 132), (641, 5122, 388), (385, 8190, 1028), (17, 66, 4),
              (5, 70, 512), (65, 130, 2044), (40, 300, 3584), (33, 580, 8192), (513, 2900, 2044),
              (385, 5122, 508), (257, 8190, 512), (226, 4100, 1540)]


@pytest.mark.parametrize("m,n,k", LONE_GROUP)
@pytest.mark.parametrize("aligned", [True, False])
def test_lone_group(dev, m, n, k, aligned):
    import paper_2601_07892_amd as sh
    print("[case] wide group", m, n, k, aligned, file=sys.stderr, flush=True)
    t, q, sx, w, qd, sxd = _inputs(dev, m, n, k, "group")
    gs = _group_scales(n, k, n + k)
    # a scale matrix that starts 4 bytes past a 16-byte boundary takes the
    # 4-byte loads
    buf = torch.zeros(gs.size + 1, dtype=torch.float32, device=dev)
    gsd = (buf[:-1] if aligned else buf[1:]).view(gs.shape)
    gsd.copy_(torch.from_numpy(gs))
    y = torch.full((m, n), float("nan"), dtype=torch.float32, device=dev)
    acc = torch.full((m, n), -7, dtype=torch.int32, device=dev)
    sh.sherry_gemm_group(w, qd, sxd, gsd, y, acc if aligned else None, m, n, k,
                         sh.SHERRY_KERNEL_SKINNY)
    torch.cuda.synchronize()
    ref = _group_ok(y.cpu().numpy(), q, t, sx, gs, k)
    if aligned:
        assert np.array_equal(acc.cpu().numpy(), ref)


def test_lone_group_infinite_scale_stays_in_its_group(dev):
    # a unit past a part's end must not meet another row's scales: an infinite
    # scale reaches its own row and nothing else
    import paper_2601_07892_amd as sh
    for k in (132, 1408, 2176):
        m, n = 40, 130
        t, q, sx, w, qd, sxd = _inputs(dev, m, n, k, "inf")
        q[:] = np.abs(q) + (q == 0)
        gs = _group_scales(n, k, 3)
        ref, _, _ = oracle.product_groups(q, t, sx, gs, threads=16)
        gs[77, 0] = np.inf
        y = torch.empty((m, n), dtype=torch.float32, device=dev)
        sh.sherry_gemm_group(w, torch.from_numpy(q).to(dev), sxd, torch.from_numpy(gs).to(dev), y,
                             None, m, n, k, sh.SHERRY_KERNEL_SKINNY)
        torch.cuda.synchronize()
        yn = y.cpu().numpy()
        rows = np.arange(n) != 77
        assert np.isfinite(yn[:, rows]).all() and not np.isfinite(yn[:, 77]).any()
        assert np.allclose(yn[:, rows], ref[:, rows], rtol=1e-4, atol=1e-3)


# (m, n, k, per-group) of the products of one launch; prepared blocks of 8
# tiles (4 with per-group scales) x 32 tokens
SMALL32 = [(17, 70, 132, False), (32, 1030, 1540, False), (5, 300, 260, False)]
MIXED32 = [(33, 70, 132, True), (300, 4100, 260, True), (65, 520, 1540, False), (97, 1000, 388, True)]
GROUPED32 = [
    (SMALL32, 1, 96),
    (SMALL32 + [(20, 51000, 68, False)], 97, 192),
    (SMALL32 + [(31, 86000, 68, False)], 161, 192),
    (SMALL32 + [(31, 98000, 68, False)], 193, 256),
    ([(33, 70, 132, True), (17, 130, 1540, False), (5, 1030, 260, True), (1, 64, 128, True)], 1, 64),
    ([(33, 70, 132, True), (64, 1030, 260, True), (129, 300, 1540, True), (1, 64, 128, True)], 1, 192),
    (MIXED32, 193, 256),
    ([(33, 70, 132, True), (500, 4100, 260, True), (65, 520, 644, False), (97, 1000, 388, True)], 257,
     384),
    ([(33, 70, 132, True), (700, 4100, 260, True), (65, 520, 644, False), (97, 1000, 388, True)], 385,
     512),
    # odd and even last token blocks of 32 under 64-token workgroups
    (MIXED32 + [(1030, 5000, 132, True), (64, 130, 4, True), (31, 300, 260, True)], 769, 1536),
    (MIXED32 + [(2050, 5130, 132, True), (64, 130, 4, True), (31, 300, 260, True)], 1537, 2048),
]


@pytest.mark.parametrize("shapes,low,high", GROUPED32)
def test_grouped32(dev, shapes, low, high):
    import paper_2601_07892_amd as sh
    descs = (sh.sherry_gemm_desc * len(shapes))()
    cases, keep = [], []
    for i, (m, n, k, group) in enumerate(shapes):
        t, q, sx, w, qd, sxd = _inputs(dev, m, n, k, "grouped32_%d" % i)
        y = torch.full((m, n), float("nan"), dtype=torch.float32, device=dev)
        acc = torch.full((m, n), -7, dtype=torch.int32, device=dev)
        gs = _group_scales(n, k, i)
        gsd = torch.from_numpy(gs).to(dev)
        d = descs[i]
        d.w, d.x, d.x_scale, d.y = w.data_ptr(), qd.data_ptr(), sxd.data_ptr(), y.data_ptr()
        d.acc = None if group else acc.data_ptr()
        d.w_group_scales = gsd.data_ptr() if group else None
        d.n, d.k, d.m, d.w_scale = n, k, m, float(np.float32(0.0173))
        keep.append((w, qd, sxd, gsd))
        cases.append((t, q, sx, gs, y, acc, group, k))
    total, value = sh.sherry_gemm_batched_prepare(descs)
    print("[case] wide grouped32", len(shapes), total, value, file=sys.stderr, flush=True)
    assert low <= total <= high and 17 <= (value & ~sh.SHERRY_LAUNCH_GROUPS) <= 32
    sh.sherry_gemm_batched(torch.from_numpy(sh.descs_to_bytes(descs)).to(dev), len(shapes), total,
                           value)
    torch.cuda.synchronize()
    for t, q, sx, gs, y, acc, group, k in cases:
        if group:
            _group_ok(y.cpu().numpy(), q, t, sx, gs, k)
        else:
            ref = oracle.gemm_i32(q, t, threads=16)
            assert np.array_equal(acc.cpu().numpy(), ref)
            assert np.array_equal(y.cpu().numpy(), _epilogue(ref, sx, np.float32(0.0173)))
