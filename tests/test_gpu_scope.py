"""Entries whose device buffers are kept between calls: the same results on kept, fresh and
differently sized buffers, from one thread and from several on streams of their own."""
import threading

import numpy as np
import pytest
import torch

from paper_2405_12866_amd import inputs as I
from paper_2405_12866_amd import qfs as Q

pytestmark = pytest.mark.gpu


def _problem(n, M, starts, seed, d=2):
    g = np.random.default_rng(seed)
    pairs = I.brickwork_template(n, 3)
    psi = I.orthonormal_states(d ** n, M, g)
    phi = I.orthonormal_states(d ** n, M, g)
    gates = np.stack([np.stack([I.haar_unitary(d * d, g) for _ in pairs]) for _ in range(starts)])
    return [torch.as_tensor(x).cuda() for x in (psi, phi, gates)] + [pairs]


def _calls(n, M, starts, seed):
    psi, phi, gates, pairs = _problem(n, M, starts, seed)
    out = []
    for prec in (Q.QFS_PREC_FP64, Q.QFS_PREC_MIXED):
        g = gates.clone()
        out += [Q.qfs_sweep(n, pairs, psi, phi, g, prec), g.cpu().numpy()]
    x = psi.clone()
    out.append(Q.qfs_apply_gates(n, x, pairs, gates[0]).cpu().numpy())
    out.append(Q.qfs_environment(n, x, phi, 0, n - 1).cpu().numpy())
    out.append(Q.qfs_state_distance(n, x, phi))
    out.append(Q.qfs_draw_states(n, M, 5).cpu().numpy())
    psi, phi, gates, pairs = _problem(3, 9, starts, seed, d=3)
    out += [Q.qfs_qudit_sweep(3, 3, pairs, psi, phi, gates), gates.cpu().numpy()]
    return out


def _same(a, b):
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert np.array_equal(np.asarray(x), np.asarray(y))


@pytest.mark.parametrize("n,M,starts", [(3, 3, 1), (8, 33, 3), (11, 40, 2)])
def test_kept_buffers(n, M, starts):
    """Bitwise the same on fresh buffers, on kept ones, and after calls of other sizes."""
    Q.qfs_release_device_cache()
    first = _calls(n, M, starts, 7)
    _same(first, _calls(n, M, starts, 7))
    _calls(n - 1, M // 2 + 1, starts + 1, 9)
    _same(first, _calls(n, M, starts, 7))
    assert Q.qfs_release_device_cache() > 0
    assert Q.qfs_release_device_cache() == 0


def test_threads():
    """Two host threads on streams of their own get the one-at-a-time results."""
    want = [_calls(7, 20, 2, s) for s in (1, 2)]
    got = [[], []]

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(4):
                got[i].append(_calls(7, 20, 2, i + 1))

    ts = [threading.Thread(target=work, args=(i,)) for i in (0, 1)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for i in (0, 1):
        assert len(got[i]) == 4
        for r in got[i]:
            _same(want[i], r)
