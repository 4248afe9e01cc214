"""The qudit gate update of complex64 sweeps and of single complex128 ones (polar factor by matrix products, the SVD where
those do not converge) on environments of given singular values, against numpy's SVD. With the
computational basis as the sample set of one gate on two qudits, the environment is the
transposed output set itself."""
import numpy as np
import pytest
import torch

from paper_2405_12866_amd import inputs as I
from paper_2405_12866_amd import qfs as Q

pytestmark = pytest.mark.gpu


def _update(d, a, precision=Q.QFS_PREC_MIXED):
    D = d * d
    psi = torch.eye(D, dtype=torch.complex128, device="cuda")
    phi = torch.as_tensor(np.ascontiguousarray(a.T)).cuda()
    gates = torch.eye(D, dtype=torch.complex128, device="cuda").reshape(1, 1, D, D).contiguous()
    Q.qfs_qudit_sweep(d, 2, [(0, 1)], psi, phi, gates, precision=precision)
    return gates.cpu().numpy()[0, 0]


def _environment(d, sigma, seed):
    g = np.random.default_rng(seed)
    a = (I.haar_unitary(d * d, g) * np.asarray(sigma)[None, :]) @ I.haar_unitary(d * d, g)
    return a.astype(np.complex64).astype(np.complex128)  # as the sweep holds it


# 0.25 = the line between the first stage's two polynomials in |D Y - I|_F^2; about 1e3 is
# where the products give up
@pytest.mark.parametrize("kappa", [1.0, 1.2, 1.5, 5.0, 100.0, 700.0, 2000.0, 1e4])
@pytest.mark.parametrize("d", [2, 3, 4])
def test_full_rank(d, kappa):
    """W V^dagger to 1e-13 times the condition number (of the rounded matrix), unitary as well."""
    D = d * d
    a = _environment(d, np.exp(-np.linspace(0, np.log(kappa), D)) * 37.0, seed=int(kappa * 10) + d)
    w, s, vh = np.linalg.svd(a)
    got = _update(d, a)
    assert np.max(np.abs(got - w @ vh)) < 1e-13 * s[0] / s[-1]
    assert np.max(np.abs(got.conj().T @ got - np.eye(D))) < 1e-13 * s[0] / s[-1]


@pytest.mark.parametrize("d,rank", [(2, 0), (2, 2), (3, 0), (3, 1), (3, 8), (4, 0), (4, 5), (4, 15)])
def test_rank_deficient(d, rank):
    """Unitary, and Re Tr(G^dagger u) the sum of the singular values to the matrix's rounding
    (whose null part, 1e-7 of it, the update may take as it comes)."""
    D = d * d
    a = _environment(d, [1.0] * rank + [0.0] * (D - rank), seed=rank + 10 * d)
    got = _update(d, a)
    assert np.max(np.abs(got.conj().T @ got - np.eye(D))) < 1e-11
    f = np.sum(a.conj() * got).real
    assert abs(f - np.sum(np.linalg.svd(a, compute_uv=False))) < 1e-6 * max(1, rank)


@pytest.mark.parametrize("kappa", [1.0, 1.5, 100.0, 700.0, 1e4])
@pytest.mark.parametrize("d", [2, 3, 4])
def test_full_rank_fp64(d, kappa):
    a = _environment(d, np.exp(-np.linspace(0, np.log(kappa), d * d)) * 37.0, seed=int(kappa * 10) + d + 1)
    w, s, vh = np.linalg.svd(a)
    got = _update(d, a, Q.QFS_PREC_FP64)
    assert np.max(np.abs(got - w @ vh)) < 1e-13 * s[0] / s[-1]
    assert np.max(np.abs(got.conj().T @ got - np.eye(d * d))) < 1e-13 * s[0] / s[-1]
