"""qfs_dense_apply with few rows of 32 x 32 tiles (fewer than the eight XCDs: a grid order of its
own) and with very many states."""
import pytest
import torch

from paper_2405_12866_amd import qfs as Q

pytestmark = pytest.mark.gpu


# rows of tiles: 1, 1, 2, 4 | 8; one and many columns of tiles
@pytest.mark.parametrize("n", [2, 5, 6, 7, 8])
@pytest.mark.parametrize("M", [1, 33, 3000])
def test_rows_of_tiles(n, M):
    """Sums of N products: within 4 N eps of the row and column norms' product."""
    g = torch.Generator(device="cuda").manual_seed(n + M)
    N = 1 << n
    u, x = (torch.view_as_complex(torch.randn(r, N, 2, generator=g, dtype=torch.float64, device="cuda")) / N ** 0.5
            for r in (N, M))
    assert torch.max(torch.abs(Q.qfs_dense_apply(n, u, x).cpu() - x.cpu() @ u.cpu().T)) < 4 * N * 2.3e-16


def test_many_states():
    """2^26 + 33 states of one qubit: more than 2^32 / 2048 tiles' columns."""
    M = (1 << 26) + 33
    g = torch.Generator(device="cuda").manual_seed(1)
    u = torch.view_as_complex(torch.randn(2, 2, 2, generator=g, dtype=torch.float64, device="cuda"))
    x = torch.view_as_complex(torch.randn(M, 2, 2, generator=g, dtype=torch.float64, device="cuda"))
    got = Q.qfs_dense_apply(1, u, x)
    for i in range(2):
        want = u[i, 0] * x[:, 0] + u[i, 1] * x[:, 1]
        assert torch.max(torch.abs(got[:, i] - want)) < 1e-13
