"""Qudit gate updates on both sides of the rule that sends environments of fewer products than
rows straight to the SVD, and on spectra that the polynomials leave to it after some stages."""
import numpy as np
import pytest
import torch

from paper_2405_12866_amd import inputs as I
from paper_2405_12866_amd import qfs as Q

pytestmark = pytest.mark.gpu


def _sweep(d, n, psi, phi, u, precision, beta):
    D = d * d
    gates = torch.as_tensor(np.ascontiguousarray(u.reshape(1, 1, D, D))).cuda()
    Q.qfs_qudit_sweep(d, n, [(0, 1)], torch.as_tensor(psi).cuda(), torch.as_tensor(phi).cuda(), gates, precision,
                      beta=beta)
    return gates.cpu().numpy()[0, 0]


@pytest.mark.parametrize("precision", [Q.QFS_PREC_FP64, Q.QFS_PREC_MIXED])
@pytest.mark.parametrize("beta", [0.0, 0.3])
@pytest.mark.parametrize("d,n,M", [(3, 2, 1), (3, 2, 8), (3, 2, 9), (3, 3, 2), (3, 3, 3), (4, 2, 15), (4, 2, 16), (4, 3, 3)])
def test_products_and_rows(d, n, M, beta, precision):
    """A unitary that attains the sum of the singular values of (1 - beta) Gamma + beta u. A value
    below the rounding of the matrix, 16 x 1e-16 of it, may come as it likes."""
    g = np.random.default_rng(10 * d + M)
    D = d * d
    psi, phi = ((lambda z: (z / np.linalg.norm(z, axis=1, keepdims=True)).astype(np.complex64).astype(np.complex128))(
        g.standard_normal((M, d ** n)) + 1j * g.standard_normal((M, d ** n))) for _ in range(2))
    u0 = I.haar_unitary(D, g)
    x = (1 - beta) * np.einsum("jqr,jpr->qp", phi.reshape(M, D, -1), psi.reshape(M, D, -1).conj()) + beta * u0
    u = _sweep(d, n, psi, phi, u0, precision, beta)
    s = np.linalg.svd(x, compute_uv=False)
    assert np.max(np.abs(u.conj().T @ u - np.eye(D))) < 1e-13 * min(s[0] / max(s[-1], 1e-300), 10)
    assert abs(np.sum(x.conj() * u).real - s.sum()) < 1e-13 * s.sum()


@pytest.mark.parametrize("d", [3, 4])
@pytest.mark.parametrize("small", [(1e-2,), (1e-3,), (3e-4,), (1e-4,), (1e-6,), (1e-3, 1e-5), (0.3, 1e-2, 1e-4), (1e-5, 1e-5)])
def test_slow_directions(d, small):
    D = d * d
    g = np.random.default_rng(int(-1e3 * np.log(small[-1])) + D)
    a = (I.haar_unitary(D, g) * np.r_[np.ones(D - len(small)), small]) @ I.haar_unitary(D, g)
    u = _sweep(d, 2, np.eye(D, dtype=complex), np.ascontiguousarray(a.T), I.haar_unitary(D, g), Q.QFS_PREC_FP64, 0.0)
    w, s, vh = np.linalg.svd(a)
    assert np.max(np.abs(u - w @ vh)) < 1e-13 * s[0] / s[-1]
    assert np.max(np.abs(u.conj().T @ u - np.eye(D))) < 1e-13 * 10
