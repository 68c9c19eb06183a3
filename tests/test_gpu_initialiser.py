"""GPU: the initialiser's fallback (R vec(I_q) when the block sums vanish) and
the diagonal entries of the time factor, per kernel shape.

Every training snapshot alternates in sign over the q samples, so the block
sums of Eq. (18) are exactly zero; one pixel carries a generic snapshot, and
its statistic (that pixel is in its own guard band, so its training set is
purely alternating) is compared with the FP64 oracle.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SHAPES = [(2, 8, "fp32"), (2, 32, "fp32"), (3, 8, "fp32"), (3, 12, "fp32"), (3, 16, "fp32"), (4, 16, "fp32"),
          (6, 8, "fp32"), (3, 8, "bf16x3"), (3, 12, "bf16x3"), (3, 16, "bf16x3"),
          (3, 16, "fp32_f64"), (5, 24, "fp32"), (6, 16, "fp32"), (5, 24, "bf16x3")]


@pytest.mark.parametrize("p,q,precision", SHAPES)
def test_vanishing_block_sums(p, q, precision):
    import torch

    import paper_1604_03622_amd as kstap
    rng = np.random.default_rng(p * 100 + q)
    H, W, n = 24, 25, 64
    cn = lambda *s: (rng.standard_normal(s) + 1j * rng.standard_normal(s)) / np.sqrt(2)  # noqa: E731
    z = cn(p, 1, 1) * cn(1, H, W) * 3 + 0.3 * cn(p, H, W)
    x = (z[..., None] * (-1.0) ** np.arange(q)).astype(np.complex64)
    r, c = 12, 11
    x[:, r, c, :] = cn(p, q).astype(np.complex64)
    cfg = oracle.OracleConfig(p=p, q=q, n=n, r_a=1, r_b=1)
    ref = oracle.kron_stap.kron_stap_pixels(x, np.array([[r, c]]), cfg)
    plan = kstap.Plan(p=p, q=q, n=n, r_a=1, r_b=1, precision=precision)
    xd = torch.from_numpy(x).cuda()
    T = float(kstap.run(plan, xd)[0][r, c])
    Tp = float(kstap.probe(plan, xd, [(r, c)])["T"][0])
    want = float(ref["T"][0])
    assert want > 0.1
    # the FP32 paths' bar against the oracle
    assert abs(T - want) <= 1e-4 * max(want, 1.0)
    assert abs(Tp - want) <= 1e-4 * max(want, 1.0)
