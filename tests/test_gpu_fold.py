"""Grouped launches of few blocks, which run several workgroups per prepared
block (each tile's units over up to 2, 4 or 8 times as many waves): every
grouped M <= 4 call around the block counts where that factor changes, on
products whose rows are one unit, ragged, and split over all 8 waves already.
int32 sums bit-exact against the oracle; fp32 outputs bit-identical to the
lone products' (per-group scales: within the fp32-sum bound)."""
import sys

import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# total blocks of the launch: 8, 4, 2 and 1 workgroups per block on each side
# of 32 | 33, 64 | 65, 128 | 129
TOTALS = [3, 32, 33, 64, 65, 128, 129]


@pytest.fixture(scope="module")
def dev():
    d = torch.device("cuda:0")
    torch.cuda.set_device(d)
    return d


def _products(total):
    # one unit per row: ceil(tiles / 8) blocks; 65 units: 8 waves per tile, so
    # two tiles are two blocks
    b = total - 2
    return [(512 * b - 3, 132), (70, 8196)]


@pytest.mark.parametrize("total", TOTALS)
@pytest.mark.parametrize("call", ["gemv", "f32", "f32_il", "tok", "tok_il", "f32_group", "tok_group"])
def test_few_blocks(dev, total, call):
    import paper_2601_07892_amd as sh
    print("[case] fold", total, call, file=sys.stderr, flush=True)
    m = 3 if call.startswith("tok") else 1
    il, group = call.endswith("_il"), call.endswith("_group")
    fused = call.startswith("f32")
    Desc = sh.sherry_gemv_desc if call == "gemv" else sh.sherry_gemv_f32_desc if fused else \
        sh.sherry_gemm_desc
    shapes = _products(total)
    descs = (Desc * len(shapes))()
    keep, cases = [], []
    for i, (n, k) in enumerate(shapes):
        t = synth.ternary_34(n, k, 5, "fold", i, total)
        w = torch.from_numpy(sh.sherry_pack_il(t) if il else sh.sherry_pack(t)).to(dev)
        x = synth.activations(m, k, 5, "fold", i)
        q, sx = oracle.quantize_act(x)
        xd = torch.from_numpy(x if fused else q).to(dev)
        sxd = torch.from_numpy(np.zeros(1, np.float32) if fused else sx).to(dev)
        G = -(-k // 128)
        gs = np.random.default_rng(i).random((n, G)).astype(np.float32)
        gsd = torch.from_numpy(gs).to(dev)
        y = torch.full((m, n), float("nan"), dtype=torch.float32, device=dev)
        acc = torch.full((m, n), -7, dtype=torch.int32, device=dev)
        d = descs[i]
        d.w, d.x, d.x_scale, d.y = w.data_ptr(), xd.data_ptr(), sxd.data_ptr(), y.data_ptr()
        d.acc = None if (group and not fused) else acc.data_ptr()
        d.w_group_scales = gsd.data_ptr() if group else None
        d.n, d.k, d.w_scale = n, k, 0.0173
        if not fused and call != "gemv":
            d.m = m
        keep.append((w, xd, gsd))
        cases.append((n, k, t, q, sx, gs, y, acc, sxd))
    if call == "gemv":
        blocks = sh.sherry_gemv_batched_prepare(descs)
        run = lambda b: sh.sherry_gemv_batched(b, len(shapes), blocks)  # noqa: E731
    elif fused:
        prep = sh.sherry_gemv_f32_il_batched_prepare if il else sh.sherry_gemv_f32_batched_prepare
        go = sh.sherry_gemv_f32_il_batched if il else sh.sherry_gemv_f32_batched
        blocks = prep(descs)
        run = lambda b: go(b, len(shapes), blocks)  # noqa: E731
    else:
        prep = sh.sherry_gemm_il_batched_prepare if il else sh.sherry_gemm_batched_prepare
        go = sh.sherry_gemm_il_batched if il else sh.sherry_gemm_batched
        blocks, value = prep(descs)
        assert value & ~sh.SHERRY_LAUNCH_GROUPS <= 4
        run = lambda b: go(b, len(shapes), blocks, value)  # noqa: E731
    assert blocks == total
    run(torch.from_numpy(sh.descs_to_bytes(descs)).to(dev))
    torch.cuda.synchronize()
    for n, k, t, q, sx, gs, y, acc, sxd in cases:
        acc_ref = oracle.gemm_i32(q, t, threads=16)
        if fused:
            assert np.array_equal(sxd.cpu().numpy(), sx)
        if not group or fused:
            assert np.array_equal(acc.cpu().numpy(), acc_ref)
        yn = y.cpu().numpy().astype(np.float64)
        if group:
            y_ref, mag, _ = oracle.product_groups(q, t, sx, gs, threads=16)
            G = -(-k // 128)
            assert not (np.abs(yn - y_ref) > (G + 4) * 2.0 ** -24 * mag).any()
        else:
            # the epilogue of every kernel: fp32 product of the scales, then of
            # the exactly converted sum
            s = (sx * np.float32(0.0173)).astype(np.float32)
            assert np.array_equal(y.cpu().numpy(), acc_ref.astype(np.float32) * s[:, None])
