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
        "rows48620": W.ring(18, U=3.0, n_up=9, n_dn=1),                               # gathered, rows in parts
        "rows167960": W.random_graph(20, 40, seed=13, site_U=True, n_up=9, n_dn=0),         # the same, two bond groups
        "parts7": W.ring(16, U=3.0, n_up=7, n_dn=0),                                  # one staged column, rows in parts
    }


@pytest.mark.parametrize("which", ["bonds36", "bonds72", "rows24310", "rows20349", "rows1", "columns1", "sites25",
                                   "rows48620", "rows167960", "parts7"])
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


# a column with paired partners (70 rows), in two chunks (24310 rows), gathered (48620)
@pytest.mark.parametrize("M,n_up,n_dn", [(8, 4, 3), (17, 8, 1), (18, 9, 1)])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_bilinear_non_finite_entry(hub, M, n_up, n_dn, bad):
    """One infinite or NaN entry of g spoils the forms that contain it and no others."""
    import torch
    m = W.ring(M, U=3.0, n_up=n_up, n_dn=n_dn)
    s = hub.Sector(m)
    up, dn = s.basis(0), s.basis(1)
    a, b = s.count_up // 3, s.count_dn // 2
    g, x = s.start_vector(seed=3), s.start_vector(seed=4)
    ref = s.param_bilinear(g, x)
    g[b * s.count_up + a] = bad
    got = s.param_bilinear(g, x)
    bi, bj, _ = s.bonds()
    bit = lambda v, i: (int(v) >> int(i)) & 1  # noqa: E731
    hop = np.array([bit(up[a], i) != bit(up[a], j) or bit(dn[b], i) != bit(dn[b], j) for i, j in zip(bi, bj)])
    both = np.array([bit(up[a], i) & bit(dn[b], i) for i in range(M)], dtype=bool)
    assert hop.any() and not hop.all()
    for r, v, hit in ((ref[0], got[0], hop), (ref[1], got[1], both)):
        assert not np.isfinite(v[hit]).any()
        assert np.array_equal(v[~hit], r[~hit])
    s.close()


# one column of 2704156 rows, and 22 of 497420
@pytest.mark.parametrize("M,n_up,n_dn", [(24, 12, 0), (22, 9, 1)])
def test_bilinear_of_few_long_columns_uses_the_chip(hub, M, n_up, n_dn):
    """The forms of a sector with few columns take no more than 30 products' time
    (rows and bonds are read a few times, not once per part of a column, and by
    every CU)."""
    import time
    import torch
    s = hub.Sector(W.ring(M, U=3.0, n_up=n_up, n_dn=n_dn))
    g, x = s.start_vector(seed=3), s.start_vector(seed=4)
    y = torch.empty_like(x)

    def best(f):
        t = []
        for _ in range(4):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            f()
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return min(t)

    assert best(lambda: s.param_bilinear(g, x)) <= 30 * best(lambda: s.matvec(x, y))
    s.close()
