"""The gate update's polar factor for environments at the ends of the range of a double."""
import numpy as np
import pytest
import torch

from paper_2405_12866_amd import inputs as I
from paper_2405_12866_amd import qfs as Q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [1e-309, 1e-315, 2.2e-308, 1e-300, 1e300])
@pytest.mark.parametrize("sigma", [(3, 2, 1, 1), (4, 1, 0.01, 0.001), (1, 1, 0, 0)])
def test_extreme_scale(sigma, size):
    """Unitary to rounding and, where the matrix has full rank, the factor of the same matrix
    scaled by a power of two (exact): to 1e-13 times its condition number."""
    g = np.random.default_rng(7)
    m = np.stack([I.haar_unitary(4, g) * np.asarray(sigma) @ I.haar_unitary(4, g) for _ in range(5)]) * size
    x = m * 2.0 ** (1000 if size < 1 else -1000)
    got = Q.qfs_polar_update(torch.as_tensor(m).cuda()).cpu().numpy()
    assert np.max(np.abs(got.conj().swapaxes(1, 2) @ got - np.eye(4))) < 1e-12
    w, s, vh = np.linalg.svd(x)
    if min(sigma) > 0:
        assert np.max(np.abs(got - w @ vh)) < 1e-13 * np.max(s[:, 0] / s[:, 3])


@pytest.mark.parametrize("size", [1e-160, 1e-80, 1.0, 1e80, 1e120])
@pytest.mark.parametrize("sigma", [(2, 1), (1, 1e-6), (1, 0)])
@pytest.mark.parametrize("backward", [Q.QFS_BWD_GROUPED, Q.QFS_BWD_PER_GATE])
def test_one_qubit_extreme_scale(sigma, size, backward):
    """A variable one-qubit gate (x) I whose environment is A (x) I / 2 times a scale: with the
    computational basis as inputs the environment is the transposed output set itself."""
    g = np.random.default_rng(8)
    a = I.haar_unitary(2, g) * np.asarray(sigma) @ I.haar_unitary(2, g)
    phi = torch.as_tensor(np.ascontiguousarray(np.kron(a, np.eye(2)).T) * size).cuda()
    psi = torch.eye(4, dtype=torch.complex128, device="cuda")
    gates = torch.eye(4, dtype=torch.complex128, device="cuda").reshape(1, 1, 4, 4).contiguous()
    Q.qfs_sweep(2, [(0, 1)], psi, phi, gates, Q.QFS_PREC_FP64, kinds=[Q.QFS_GATE_1Q], backward=backward)
    u = gates.cpu().numpy()[0, 0]
    v = u[::2, ::2]
    assert np.array_equal(u, np.kron(v, np.eye(2)))
    assert np.max(np.abs(v.conj().T @ v - np.eye(2))) < 1e-14
    assert abs(np.sum(a.conj() * v).real - sum(sigma)) < 1e-14
    if sigma[1] > 0:
        w, s, vh = np.linalg.svd(a)
        assert np.max(np.abs(v - w @ vh)) < 1e-14 * s[0] / s[1]
