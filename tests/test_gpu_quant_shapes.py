"""Activation quantization at the row lengths where its workgroup changes (256
threads holding 2, 4 or 8 pieces each, 512 holding 8 or 16, two passes), lone
and grouped, and lone where the inputs are read past the caches (64 MB and
more), bit-exact against the oracle: ragged ends, ties, all-zero rows and a
wide range of scales."""
import sys

import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

KS = [4, 1020, 2048, 2052, 4096, 4100, 8192, 8196, 16384, 16388, 32768, 32772]


def _rows(m, k):
    x = synth.activations(m, k, 17, "shapes", k, outlier_frac=0.01)
    x *= (10.0 ** np.linspace(-30, 25, m, dtype=np.float64)).astype(np.float32)[:, None]
    if m > 2:
        x[1] = 0.0
        x[2, :] = 0.0
        x[2, :4] = [0.5, 1.5, 2.5, -127.0]  # ties after scaling by absmax 127
        x[2, -1] = -126.5
    return x


@pytest.mark.parametrize("m,k", [(5, k) for k in KS] + [(1, 2048), (3073, 8192), (3073, 8196),
                                                        (1537, 16388)])
def test_lone(m, k):
    import paper_2601_07892_amd as sh
    print("[case] quant", m, k, file=sys.stderr, flush=True)
    x = _rows(m, k)
    xd = torch.from_numpy(x).cuda()
    q = torch.full((m * k + 8,), 99, dtype=torch.int8, device="cuda")
    sx = torch.full((m + 1,), -1.0, dtype=torch.float32, device="cuda")
    sh.sherry_quantize_act(xd, q[:m * k].view(m, k), sx[:m])
    torch.cuda.synchronize()
    q_ref, sx_ref = oracle.quantize_act(x)
    assert np.array_equal(sx[:m].cpu().numpy(), sx_ref) and float(sx[m]) == -1.0
    assert np.array_equal(q[:m * k].view(m, k).cpu().numpy(), q_ref)
    assert bool((q[m * k:] == 99).all())  # nothing past the last row


@pytest.mark.parametrize("k", [1028, 2052, 4100, 8196, 16388, 32772])
def test_lone_past_the_caches(k):
    import paper_2601_07892_amd as sh
    base = _rows(61, k)
    m = (64 << 20) // (4 * k) + 1
    print("[case] quant streamed", m, k, file=sys.stderr, flush=True)
    xd = torch.from_numpy(base).cuda().repeat(-(-m // 61), 1)[:m]
    q = torch.empty((m, k), dtype=torch.int8, device="cuda")
    sx = torch.empty(m, dtype=torch.float32, device="cuda")
    sh.sherry_quantize_act(xd, q, sx)
    torch.cuda.synchronize()
    q_ref, sx_ref = (torch.from_numpy(a).cuda() for a in oracle.quantize_act(base))
    row = torch.arange(m, device="cuda") % 61
    assert torch.equal(sx, sx_ref[row]) and torch.equal(q, q_ref[row])


@pytest.mark.parametrize("k", [1024, 4100, 8196, 16388, 32772])
def test_grouped(k):
    import paper_2601_07892_amd as sh
    shapes = [(3, k), (4, 132), (1, max(4, k // 2 // 4 * 4)), (2, 4)]
    descs = (sh.sherry_quant_desc * len(shapes))()
    keep = []
    for d, (m, kk) in zip(descs, shapes):
        x = _rows(m, kk)
        xd = torch.from_numpy(x).cuda()
        q = torch.empty((m, kk), dtype=torch.int8, device="cuda")
        sx = torch.empty(m, dtype=torch.float32, device="cuda")
        d.x, d.q, d.x_scale, d.m, d.k = xd.data_ptr(), q.data_ptr(), sx.data_ptr(), m, kk
        keep.append((x, xd, q, sx))
    rows, mk = sh.sherry_quantize_act_batched_prepare(descs)
    sh.sherry_quantize_act_batched(torch.from_numpy(sh.descs_to_bytes(descs)).cuda(), len(shapes),
                                   rows, mk)
    torch.cuda.synchronize()
    for x, _, q, sx in keep:
        q_ref, sx_ref = oracle.quantize_act(x)
        assert np.array_equal(sx.cpu().numpy(), sx_ref)
        assert np.array_equal(q.cpu().numpy(), q_ref)


@pytest.mark.parametrize("k", [8196, 16388])
def test_grouped_many_rows(k):
    # one long row among 2^23 short ones: 512 threads per row would not fit a grid
    import paper_2601_07892_amd as sh
    print("[case] quant many rows", k, file=sys.stderr, flush=True)
    long_row, base, m = _rows(1, k), _rows(61, 4), 1 << 23
    xs = [torch.from_numpy(long_row).cuda(),
          torch.from_numpy(base).cuda().repeat(-(-m // 61), 1)[:m].contiguous()]
    qs = [torch.empty(x.shape, dtype=torch.int8, device="cuda") for x in xs]
    sxs = [torch.full((x.shape[0],), -1.0, device="cuda") for x in xs]
    descs = (sh.sherry_quant_desc * 2)()
    for d, x, q, sx in zip(descs, xs, qs, sxs):
        d.x, d.q, d.x_scale = x.data_ptr(), q.data_ptr(), sx.data_ptr()
        d.m, d.k = x.shape
    rows, mk = sh.sherry_quantize_act_batched_prepare(descs)
    sh.sherry_quantize_act_batched(torch.from_numpy(sh.descs_to_bytes(descs)).cuda(), 2, rows, mk)
    torch.cuda.synchronize()
    row = torch.arange(m, device="cuda") % 61
    for (q, sx), (ref, pick) in zip(zip(qs, sxs), ((long_row, None), (base, row))):
        q_ref, sx_ref = (torch.from_numpy(a).cuda() for a in oracle.quantize_act(ref))
        assert torch.equal(q, q_ref if pick is None else q_ref[pick])
        assert torch.equal(sx, sx_ref if pick is None else sx_ref[pick])
