"""qfs_apply_gates in one launch (2 to 13 qubits) and gate by gate (above), against the oracle's
simulation: work-groups of several samples and of one, ragged sample counts, more gates than
one launch takes, gates on the lowest and highest bits, both directions."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2405_12866_amd import inputs as I
from paper_2405_12866_amd import qfs as Q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,M,L", [(2, 1, 1), (2, 5, 130), (5, 70, 7), (8, 513, 6), (9, 3, 121), (11, 5, 241),
                                   (12, 2, 9), (12, 259, 3), (13, 3, 5), (14, 2, 3)])
def test_apply_gates(n, M, L):
    """Within 2 L eps sqrt(4) of a unit state per gate: 1e-15 (L + 1), forward and back."""
    g = np.random.default_rng(n * 1000 + M + L)
    pairs = np.asarray([g.choice(n, size=2, replace=False) for _ in range(L)], dtype=np.int32)
    pairs[0], pairs[-1] = (n - 1, n - 2), (0, 1)
    gates = I.haar_gates(L, g)
    x = g.standard_normal((M, 1 << n)) + 1j * g.standard_normal((M, 1 << n))
    x /= np.linalg.norm(x, axis=1, keepdims=True)
    dx, dg = torch.as_tensor(x).cuda(), torch.as_tensor(gates).cuda()
    Q.qfs_apply_gates(n, dx, pairs, dg)
    assert np.max(np.abs(dx.cpu().numpy() - O.apply_circuit(n, x, pairs, gates))) < 1e-15 * (L + 1)
    Q.qfs_apply_gates(n, dx, pairs, dg, dagger=True)
    assert np.max(np.abs(dx.cpu().numpy() - x)) < 1e-15 * (2 * L + 1)
