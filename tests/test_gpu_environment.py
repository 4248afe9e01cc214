"""qfs_environment and its form without device memory of its own against a sum in numpy: fewer
items than a block, remainders of the blocks, one item a thread, and many."""
import numpy as np
import pytest
import torch

from paper_2405_12866_amd import qfs as Q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,M", [(2, 1), (2, 257), (3, 85), (4, 64), (6, 3), (9, 5), (10, 64), (13, 130)])
def test_environment_sizes(n, M):
    """Sums of M 2^(n-2) products of unit-norm rows: within a hundred eps of M."""
    r = np.random.default_rng(17 * n + M)
    a, b = (r.standard_normal((M, 1 << n)) + 1j * r.standard_normal((M, 1 << n)) for _ in range(2))
    a, b = (x / np.linalg.norm(x, axis=1, keepdims=True) for x in (a, b))
    da, db = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    for qa, qb in ((0, n - 1), (n - 1, n - 2), (n // 2, 0)):
        if qa == qb:
            continue
        want = np.empty((4, 4), dtype=np.complex128)
        x, y = (np.moveaxis(v.reshape((M,) + (2,) * n), (1 + qa, 1 + qb), (0, 1)).reshape(4, -1) for v in (a, b))
        want[:] = x @ y.conj().T
        g = torch.empty((4, 4), dtype=torch.complex128, device="cuda")
        for got in (Q.qfs_environment(n, da, db, qa, qb), Q.qfs_environment_noalloc(n, da, db, qa, qb, g)):
            assert np.max(np.abs(got.cpu().numpy() - want)) < 100 * 2.3e-16 * M
