"""Costs of sweeps that run in stream parts of unequal size with an unfused forward pass (sets
too wide for LDS, so a part's block count follows its own number of starts): every start's
validation cost against that of the same run on one stream (timing = 1)."""
import numpy as np
import pytest
import torch

from paper_2405_12866_amd import inputs as I
from paper_2405_12866_amd import qfs as Q

pytestmark = pytest.mark.gpu


# complex64 sums of a thread hold 32 terms or fewer: 32 x 6e-8; complex128 ones likewise
@pytest.mark.parametrize("n,prec,starts,tol", [(13, Q.QFS_PREC_FP64, 5, 1e-13), (14, Q.QFS_PREC_MIXED, 5, 2e-6)])
@pytest.mark.parametrize("graphs", [0, 1])
def test_unequal_parts(n, prec, starts, tol, graphs):
    g = np.random.default_rng(n)
    pairs = [(int(a), int(b)) for a, b in I.brickwork_template(n, 2)]
    L = len(pairs)
    tg = np.stack([I.haar_unitary(4, g) for _ in range(L)])
    other = np.stack([np.stack([I.haar_unitary(4, g) for _ in range(L)]) for _ in range(starts)])
    dtg = torch.as_tensor(tg).cuda()
    base = dict(multistarts=starts, m_init=128, fixed_m=1, seed=3, precision=prec, dist_tol=0.0, diff_tol_r=0.0,
                plateau_window=1 << 20, refine_below=0.0, max_iter=1)
    for s in range(starts):  # start s leads: the run returns its costs
        init = other.copy()
        init[s, 1:] = tg[1:]
        dinit = torch.as_tensor(init).cuda()
        got = [Q.qfs_instantiate(n, pairs, target_pairs=pairs + [(0, 2)], target_gates=torch.cat([dtg, dtg[:1]]),
                                 gates_in=dinit, params=Q.qfs_default_params(**base, **kw))[1]
               for kw in (dict(timing=1), dict(graphs=graphs))]
        assert [r["best_start"] for r in got] == [s, s]
        assert got[0]["c_val"] > 0.1
        assert abs(got[1]["c_val"] - got[0]["c_val"]) < tol * got[0]["c_val"], s
        assert abs(got[1]["c_train"] - got[0]["c_train"]) < tol * got[0]["c_train"], s
