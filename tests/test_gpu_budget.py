"""Device memory of calls that go on with buffers of other sizes: a qudit run that doubles its
training set, or is split into groups of starts by a memory budget, holds its live buffers and
not those of its earlier stages; buffers of large calls take up what was asked for."""
import threading

import numpy as np
import pytest
import torch

from paper_2405_12866_amd import qfs as Q

pytestmark = pytest.mark.gpu

MB = 1 << 20


class Peak:
    """The device's most used memory above the level at entry, polled while a call runs."""

    def __enter__(self):
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        Q.qfs_release_device_cache()
        self.low = self.start = torch.cuda.mem_get_info()[0]
        self.stop = False
        self.t = threading.Thread(target=self.poll)
        self.t.start()
        return self

    def poll(self):
        while not self.stop:
            self.low = min(self.low, torch.cuda.mem_get_info()[0])

    def __exit__(self, *exc):
        self.stop = True
        self.t.join()
        self.used = self.start - self.low


def _states(N, M, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.view_as_complex(torch.randn(M, N, 2, generator=g, dtype=torch.float64, device="cuda"))
    return x / torch.linalg.vector_norm(x, dim=1, keepdim=True)


def _live(N, M, Mv, L, S):
    """Bytes of a complex64 run's sets and B lists."""
    return 8 * N * (M * (2 + (L - 1) * S + S) + Mv * (2 + S)) + 16 * S * 64 * 256


def _run(n, rows, val, S, **kw):
    """Validation outputs that no circuit gives: every generation over-trains and doubles."""
    N, pairs = 4 ** n, [(q, q + 1) for q in range(0, n - 1, 2)]
    psi, phi = _states(N, rows + val, 1), _states(N, rows + val, 2)
    phi[:rows] = psi[:rows]
    p = Q.qfs_default_params(multistarts=S, precision=Q.QFS_PREC_MIXED, refine_below=0.0, dist_tol=0.0, diff_tol_r=0.0,
                             plateau_window=1 << 20, min_iter=1, seed=4, **kw)
    # (first a small one: loaded code and the queues' scratch memory stay with the process)
    rows_w = list(range(4)) + list(range(rows, rows + 2))
    Q.qfs_qudit_instantiate(4, n, pairs, psi[rows_w].contiguous(), phi[rows_w].contiguous(), n_val=2,
                            params={**p, "m_init": 1})
    with Peak() as peak:
        _, info = Q.qfs_qudit_instantiate(4, n, pairs, psi, phi, n_val=val, params=p)
    return len(pairs), peak.used, info


@pytest.mark.parametrize("budget", [0, 4 << 30])
def test_doublings(budget):
    L, used, info = _run(7, 512, 16, 8, m_init=64, max_iter=8, device_mem_budget=budget)
    assert info["restarts"] == 3 and info["m_final"] == 512
    live = _live(4 ** 7, 512, 16, L, 8)
    # a quarter: blocks up to 64 MiB of the earlier stages, the library's own small buffers
    assert used < 1.25 * live, (used / MB, live / MB)


def test_groups_of_starts():
    """A budget that holds two of eight starts: four groups, one after the other."""
    N = 4 ** 7
    budget = _live(N, 512, 16, 3, 2) + MB
    L, used, info = _run(7, 512, 16, 8, m_init=512, fixed_m=1, max_iter=3, device_mem_budget=budget)
    assert L == 3 and info["start_groups"] == 4
    assert used < 1.25 * budget, (used / MB, budget / MB)


def test_block_sizes():
    """What one sweep's buffers are kept as, against their sizes: 2 % above at most (2 MiB a
    block and its small buffers; eighths would add 11 % to this one's B lists)."""
    d, n, M, S, L = 3, 9, 64, 15, 9
    N = d ** n
    pairs = [(q % (n - 1), q % (n - 1) + 1) for q in range(L)]
    psi, phi = _states(N, M, 1), _states(N, M, 2)
    gates = torch.eye(9, dtype=torch.complex128, device="cuda").repeat(S, L, 1, 1).contiguous()
    Q.qfs_release_device_cache()
    Q.qfs_qudit_sweep(d, n, pairs, psi, phi, gates, Q.QFS_PREC_MIXED)
    assert Q.qfs_release_device_cache() < 1.02 * _live(N, M, 0, L, S)
