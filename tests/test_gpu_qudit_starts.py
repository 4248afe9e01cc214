"""A qudit start's sweep does not depend on the starts beside it: bit for bit the same alone."""
import numpy as np
import pytest
import torch

from paper_2405_12866_amd import inputs as I
from paper_2405_12866_amd import qfs as Q

pytestmark = pytest.mark.gpu


# items of an environment over 256: 1 block, below and above 16, above 64 (kinds of the block rule)
@pytest.mark.parametrize("precision", [Q.QFS_PREC_FP64, Q.QFS_PREC_MIXED])
@pytest.mark.parametrize("d,n,M", [(3, 4, 5), (3, 6, 40), (4, 4, 45), (3, 7, 64), (4, 6, 70), (2, 10, 90)])
def test_alone_and_beside_others(d, n, M, precision):
    g = np.random.default_rng(d + n)
    D, N, starts = d * d, d ** n, 5
    pairs = [(0, 1), (n - 2, n - 1), (0, n - 1)]
    psi, phi = (torch.as_tensor(x / np.linalg.norm(x, axis=1, keepdims=True)).cuda()
                for x in (g.standard_normal((M, N)) + 1j * g.standard_normal((M, N)) for _ in range(2)))
    gates = torch.as_tensor(np.stack([np.stack([I.haar_unitary(D, g) for _ in pairs]) for _ in range(starts)])).cuda()
    all_, c_all = gates.clone(), None
    for _ in range(2):
        c_all = Q.qfs_qudit_sweep(d, n, pairs, psi, phi, all_, precision)
    for s in range(starts):
        one = gates[s:s + 1].clone()
        for _ in range(2):
            c = Q.qfs_qudit_sweep(d, n, pairs, psi, phi, one, precision)
        assert torch.equal(one[0], all_[s])
        assert c[0] == c_all[s]
