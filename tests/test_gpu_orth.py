"""The blocked Cholesky of the sample draw on the device, at sizes below, at and off its panels of
32 rows and 64 columns, against the draw's columns by the oracle."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2405_12866_amd import qfs as Q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,M", [(1, 1), (3, 2), (6, 31), (7, 32), (7, 33), (8, 64), (8, 97), (9, 129), (10, 300)])
def test_drawn_states(n, M):
    """Orthonormal to the rounding of sums of 2^n products; the columns themselves to that times
    the condition number of a Ginibre matrix of at most half as many columns as rows (below 6.9),
    with room for the solves of M steps."""
    got = Q.qfs_draw_states(n, M, seed=77 + n, device="cuda").cpu().numpy()
    assert np.max(np.abs(got @ got.conj().T - np.eye(M))) < 50 * 2.3e-16 * M ** 0.5
    assert np.max(np.abs(got - O.draw_states(n, M, seed=77 + n))) < 7 * 50 * 2.3e-16 * M ** 0.5
