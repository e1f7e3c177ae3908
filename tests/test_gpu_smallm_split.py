"""Grouped launches of 5 to 16 tokens with few blocks, whose tiles' K is split
over the four waves of a workgroup where the rows are long enough: on both sides
of the block counts where that line moves and where the split ends, products of
one unit per row, of 5 units (parts of 2, 2, 1 and 0), of 8 and 12 (split or
whole by the blocks; with per-group scales parts of 4, 4 and 0), of 17 (two
windows per part) and of 4-byte-aligned rows, split and whole ones in one
launch; ragged last tiles and blocks.  int32 sums bit-exact against the oracle,
fp32 outputs bit-identical to its epilogue (per-group scales: within the
fp32-sum bound)."""
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


@pytest.mark.parametrize("total", [9, 128, 129, 192, 193, 257])
@pytest.mark.parametrize("call", ["tiled", "il", "group"])
@pytest.mark.parametrize("m", [5, 16])
def test_split_k(dev, total, call, m):
    import paper_2601_07892_amd as sh
    print("[case] smallm split", total, call, m, file=sys.stderr, flush=True)
    group = call == "group"
    # the last product fills the launch up to `total` blocks of 256 rows
    shapes = ([(70, 512), (130, 2560), (257, 1536), (66, 1024)] if group else
              [(70, 128), (130, 644), (257, 2176), (3, 132), (66, 1024), (130, 1536)])
    used = sum(-(-n // 256) for n, _ in shapes)
    shapes.append((256 * (total - used) - 63, 512))
    descs = (sh.sherry_gemm_desc * len(shapes))()
    keep, cases = [], []
    for i, (n, k) in enumerate(shapes):
        t = synth.ternary_34(n, k, 6, "split", i, total)
        w = torch.from_numpy(sh.sherry_pack_il(t) if call == "il" else sh.sherry_pack(t)).to(dev)
        q, sx = oracle.quantize_act(synth.activations(m, k, 6, "split", i))
        ws = np.random.default_rng(i).random(n).astype(np.float32)
        G = -(-k // 128)
        gs = np.random.default_rng(i).random((n, G)).astype(np.float32)
        wsd, gsd, qd, sxd = (torch.from_numpy(a).to(dev) for a in (ws, gs, q, sx))
        y = torch.full((m, n), float("nan"), dtype=torch.float32, device=dev)
        acc = torch.full((m, n), -7, dtype=torch.int32, device=dev)
        d = descs[i]
        d.w, d.x, d.x_scale, d.y = w.data_ptr(), qd.data_ptr(), sxd.data_ptr(), y.data_ptr()
        d.acc = None if group else acc.data_ptr()
        d.w_group_scales = gsd.data_ptr() if group else None
        d.w_scales = None if group else wsd.data_ptr()
        d.n, d.k, d.m = n, k, m
        keep.append((w, wsd, gsd, qd, sxd))
        cases.append((t, q, sx, ws, gs, y, acc))
    prep = sh.sherry_gemm_il_batched_prepare if call == "il" else sh.sherry_gemm_batched_prepare
    go = sh.sherry_gemm_il_batched if call == "il" else sh.sherry_gemm_batched
    blocks, value = prep(descs)
    assert blocks == total
    go(torch.from_numpy(sh.descs_to_bytes(descs)).to(dev), len(shapes), blocks, value)
    torch.cuda.synchronize()
    for t, q, sx, ws, gs, y, acc in cases:
        if group:
            y_ref, mag, _ = oracle.product_groups(q, t, sx, gs, threads=16)
            # every fp32 fma, partial sum and scale product rounds once
            bound = (gs.shape[1] + 8) * 2.0 ** -24 * mag
            assert not (np.abs(y.cpu().numpy().astype(np.float64) - y_ref) > bound).any()
        else:
            acc_ref = oracle.gemm_i32(q, t, threads=16)
            assert np.array_equal(acc.cpu().numpy(), acc_ref)
            s = (sx[:, None] * ws[None, :]).astype(np.float32)
            assert np.array_equal(y.cpu().numpy(), acc_ref.astype(np.float32) * s)
