"""qfs_dense_apply against torch's product in FP64: sizes below and off the tiles of 32 and the
blocks of eight k, and an output that is an input."""
import pytest
import torch

from paper_2405_12866_amd import qfs as Q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,M", [(1, 1), (2, 3), (3, 8), (5, 17), (5, 32), (6, 33), (8, 65), (9, 31), (11, 2)])
def test_dense_apply(n, M):
    """Sums of N products: within 2 N eps of the row and column norms' product."""
    g = torch.Generator().manual_seed(100 * n + M)
    N = 1 << n
    u = torch.view_as_complex(torch.randn(N, N, 2, generator=g, dtype=torch.float64)) / N ** 0.5
    x = torch.view_as_complex(torch.randn(M, N, 2, generator=g, dtype=torch.float64)) / N ** 0.5
    want = x @ u.T
    du, dx = u.cuda(), x.cuda()
    assert torch.max(torch.abs(Q.qfs_dense_apply(n, du, dx).cpu() - want)) < 2 * N * 2.3e-16 * 2
    lib = Q.load()
    assert lib.qfs_dense_apply(n, M, du.data_ptr(), dx.data_ptr(), dx.data_ptr(), None) == 0
    assert torch.max(torch.abs(dx.cpu() - want)) < 2 * N * 2.3e-16 * 2
