"""SHERRY_KERNEL_AUTO past 8192 tokens, on both sides of the lines between the
LDS-tiled and the register-decoded kernel (k <= 1024, k <= n): int32 sums
bit-exact against the oracle, outputs equal to their fp32 epilogue, and both
equal to those of the kernel that sherry_gemm_kernel_for names."""
import sys

import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k,kernel", [(1036, 1024, "MFMA"), (1036, 1028, "SKINNY"),
                                        (132, 132, "MFMA"), (128, 132, "SKINNY")])
def test_long_products(n, k, kernel):
    import paper_2601_07892_amd as sh
    print("[case] auto", n, k, file=sys.stderr, flush=True)
    m, dev = 8197, torch.device("cuda:0")
    assert sh.sherry_gemm_kernel_for(m, n, k) == getattr(sh, "SHERRY_KERNEL_" + kernel)
    t = synth.ternary_34(n, k, 3, "auto")
    q = synth.int8_any(m, k, 3, "auto")
    sx = (np.random.default_rng(n + k).random(m) + 0.01).astype(np.float32)
    w, qd, sxd = (torch.from_numpy(a).to(dev) for a in (sh.sherry_pack(t), q, sx))
    outs = []
    for kern in (sh.SHERRY_KERNEL_AUTO, sh.sherry_gemm_kernel_for(m, n, k)):
        y = torch.full((m, n), float("nan"), dtype=torch.float32, device=dev)
        acc = torch.full((m, n), -7, dtype=torch.int32, device=dev)
        sh.sherry_gemm_ex(w, qd, sxd, 0.0173, y, acc, m, n, k, kern)
        outs.append((y, acc))
    torch.cuda.synchronize()
    ref = oracle.gemm_i32(q, t, threads=16)
    s = (sx * np.float32(0.0173)).astype(np.float32)
    assert np.array_equal(outs[0][1].cpu().numpy(), ref)
    assert np.array_equal(outs[0][0].cpu().numpy(), ref.astype(np.float32) * s[:, None])
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
