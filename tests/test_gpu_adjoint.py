"""Parameter bilinear forms at the edges of their kernels: more bonds than one
launch holds, columns beyond the LDS, one-row and one-column sectors, segments
of 128 rows with a remainder; against the oracle."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hub():
    import torch
    import paper_1307_7542_amd as h
    h.lib()
    torch.cuda.set_device(0)
    return h


def _models():
    return {
        "bonds36": W.random_graph(9, 36, seed=11, site_U=True, n_up=4, n_dn=3),       # two bond groups, 126 rows
        "bonds72": W.random_graph(13, 72, seed=12, n_up=3, n_dn=2),                   # three, 286 rows
        "rows24310": W.ring(17, U=3.0, n_up=8, n_dn=1),                               # two chunks of a column
        "rows20349": W.ring(21, U=3.0, n_up=5, n_dn=1),                               # a column that just fits
        "rows1": W.ring(7, U=3.0, n_up=0, n_dn=3),
        "columns1": W.ring(7, U=3.0, n_up=3, n_dn=7),
        "sites25": W.ring(25, U=3.0, n_up=2, n_dn=1),
    }


@pytest.mark.parametrize("which", ["bonds36", "bonds72", "rows24310", "rows20349", "rows1", "columns1", "sites25"])
def test_bilinear_edges(hub, which):
    import torch
    m = _models()[which]
    s = hub.Sector(m)
    osec = oracle.Sector(m)
    g, x = oracle.start_vector(3, osec.dim), oracle.start_vector(4, osec.dim)
    db, du, de = s.param_bilinear(torch.from_numpy(g).cuda(), torch.from_numpy(x).cuda())
    rb, ru, re = osec.param_bilinear(g, x)
    # sums of up to dim products of entries below 1, each rounded to 2^-53 of the running sum
    tol = 64 * np.finfo(float).eps * float(np.sqrt(osec.dim)) * float(np.linalg.norm(g) * np.linalg.norm(x))
    assert np.max(np.abs(db - rb), initial=0.0) <= tol
    assert np.max(np.abs(du - ru)) <= tol and np.max(np.abs(de - re)) <= tol
    s.close()
