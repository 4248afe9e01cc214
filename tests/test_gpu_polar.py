"""The gate update's polar factor on both sides of the rule that picks its method (Newton
for well-conditioned environments, Jacobi SVD for the others), against numpy's SVD."""
import numpy as np
import pytest
import torch

from paper_2405_12866_amd import inputs as I
from paper_2405_12866_amd import qfs as Q

pytestmark = pytest.mark.gpu


def _matrices(sigma, count, seed):
    g = np.random.default_rng(seed)
    u = np.stack([I.haar_unitary(4, g) for _ in range(count)])
    v = np.stack([I.haar_unitary(4, g) for _ in range(count)])
    return (u * np.asarray(sigma)[None, None, :]) @ v


def _update(m, beta=0.0, u=None):
    du = None if u is None else torch.as_tensor(np.ascontiguousarray(u)).cuda()
    return Q.qfs_polar_update(torch.as_tensor(np.ascontiguousarray(m)).cuda(), beta, du).cpu().numpy()


# |X|_F |X^-1|_F is 4 for a unitary matrix; the rule's line is 64
@pytest.mark.parametrize("sigma", [(1, 1, 1, 1), (256, 256, 256, 256), (1, 1 + 1e-9, 1, 1 - 1e-9), (1, 1, 1, 0.999),
                                   (1, 1, 1, 1 / 36.5), (1, 1, 1, 1 / 37.5), (1, 1 / 37, 1 / 37, 1 / 37),
                                   (1, 0.3, 0.03, 0.016), (1, 1, 1, 1e-6), (3e-40, 2e-40, 1e-40, 1e-40),
                                   (3e90, 2e90, 1e90, 1e90)])
@pytest.mark.parametrize("count", [1, 65])
def test_full_rank(sigma, count):
    """u = W V^dagger within 1e-13 times the condition number (backward error of a few
    hundred roundings), unitary to 1e-13 times it as well."""
    m = _matrices(sigma, count, seed=int(1e6 * np.log10(max(sigma)) + count) & 0xFFFF)
    w, s, vh = np.linalg.svd(m)
    kappa = max(sigma) / min(sigma)
    got = _update(m)
    assert np.max(np.abs(got - w @ vh)) < 1e-13 * kappa
    assert np.max(np.abs(got.conj().swapaxes(1, 2) @ got - np.eye(4))) < 1e-13 * kappa


@pytest.mark.parametrize("sigma", [(1, 1, 1, 0), (5, 1, 0, 0), (2, 0, 0, 0), (0, 0, 0, 0)])
def test_rank_deficient(sigma):
    """Unitary, and Re Tr(G^dagger u) equals the sum of the singular values."""
    m = _matrices(sigma, 9, seed=3)
    got = _update(m)
    assert np.max(np.abs(got.conj().swapaxes(1, 2) @ got - np.eye(4))) < 1e-12
    f = np.einsum("kij,kij->k", m.conj(), got).real
    assert np.max(np.abs(f - sum(sigma))) < 1e-12 * max(1, sum(sigma))


@pytest.mark.parametrize("beta", [0.25, 1.0])
def test_beta(beta):
    """The mix (1 - beta) G + beta u is what is factored; beta = 1 keeps the gate."""
    g = np.random.default_rng(5)
    m = _matrices((4, 3, 2, 1), 7, seed=4)
    u = np.stack([I.haar_unitary(4, g) for _ in range(7)])
    w, s, vh = np.linalg.svd((1 - beta) * m + beta * u)
    assert np.max(np.abs(_update(m, beta, u) - w @ vh)) < 1e-13 * np.max(s[:, 0] / s[:, 3])
