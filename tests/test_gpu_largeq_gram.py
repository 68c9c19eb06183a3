"""GPU: the many-workgroup Gram sums of the large-covariance solve.

With the time factor asked for and enough samples (q from 256, 32 768 entries
x samples) the Gram sums come from many workgroups; without it one workgroup
forms them.  Both sum FP32 products in
FP64, so the factor A agrees to FP32 rounding and the statistics to FP64
rounding of sums of at most 4 100 terms (4 100 * 2^-53 < 1e-12).  Sizes: both
sides of the threshold, ends of 64-sample chunks, more than 512 entries, and a
span of more than one chunk per workgroup.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,q,n", [(3, 255, 5), (3, 256, 5), (3, 257, 5), (3, 319, 5), (6, 320, 4), (2, 260, 3), (2, 4097, 2),
                                   (8, 300, 8), (4, 513, 16), (5, 1000, 12)])
def test_gram_paths_agree(p, q, n):
    import torch

    import paper_1604_03622_amd as kstap
    rng = np.random.default_rng(p * q + n)
    cn = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)  # noqa: E731
    X = torch.from_numpy((10 * cn(p, 1) * cn(n, 1, q) + cn(n, p, q)).astype(np.complex64)).cuda()
    one = kstap.lrkron(X, with_B=False)
    many = kstap.lrkron(X)
    a, b = one["A"].cpu().numpy(), many["A"].cpu().numpy()
    assert np.max(np.abs(a - b)) <= 2 ** -23 * np.max(np.abs(a))
    s, t = one["stats"].cpu().numpy(), many["stats"].cpu().numpy()
    assert s[1] == t[1]
    assert np.all(np.abs(s[1:] - t[1:]) <= 1e-12 * np.abs(s[1:]))
    # eta is a root of a difference of sums of size 1: 1e-12 of eta^2
    assert abs(s[0] ** 2 - t[0] ** 2) <= 1e-12
    # B-hat = (1 / (n ||A||^2)) sum_m X_m^T conj(A) conj(X_m)
    x, A = X.cpu().numpy().astype(np.complex128), b.astype(np.complex128)
    B = np.einsum("mik,ij,mjl->kl", x, A.conj(), x.conj(), optimize=True) / (n * np.sum(np.abs(A) ** 2))
    assert np.max(np.abs(many["B"].cpu().numpy() - B)) <= 1e-5 * np.max(np.abs(B))
