"""Vectors of more elements than one launch of a per-segment kernel holds."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hub():
    import torch
    import paper_1307_7542_amd as h
    h.lib()
    torch.cuda.set_device(0)
    return h


def _elements(m, s, x, a, b):
    """Elements (a, b) of H x and the sums of their terms' magnitudes, from the bonds."""
    import torch
    up, dn = s.basis(0).astype(np.int64), s.basis(1).astype(np.int64)
    cu = s.count_up

    def at(i, j):
        return x[torch.from_numpy(i + j * cu).to(x.device)].cpu().numpy()

    both = np.array([bin(int(v)).count("1") for v in up[a] & dn[b]])
    ref = m.U[0] * both * at(a, b)
    mag = np.abs(ref)
    for (i, j), t in zip(m.bonds, m.t):
        lo, hi = min(i, j), max(i, j)
        between = ((1 << hi) - 1) & ~((1 << (lo + 1)) - 1)
        for basis, idx, other in ((up, a, b), (dn, b, a)):
            v = basis[idx]
            hop = ((v >> lo) ^ (v >> hi)) & 1 == 1
            to = np.searchsorted(basis, v[hop] ^ ((1 << lo) | (1 << hi)))
            sign = np.array([1 - 2 * (bin(int(w)).count("1") & 1) for w in v[hop] & between])
            got = at(to, other[hop]) if basis is up else at(other[hop], to)
            ref[hop] -= t * sign * got
            mag[hop] += abs(t) * np.abs(got)
    return ref, mag


# 77520 x 125970 states of the 20-site ring: 9.8e9 elements, 78 GB a vector
def test_product_of_a_vector_beyond_one_launch(hub):
    """The tuned product and the one whose H_dn term has its own pass, element by
    element at random places and in the last rows and columns."""
    import torch
    m = W.ring(20, U=4.0, n_up=7, n_dn=8)
    if torch.cuda.mem_get_info()[0] < 175e9:
        torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 175e9:
        pytest.skip("needs 175 GB of device memory")
    s = hub.Sector(m)
    assert s.dim * 256 // (128 * 4) >= 1 << 32  # lanes of the H_dn pass: 128 rows and 4 columns a workgroup
    x = s.start_vector(seed=5, normalize=False)
    y = torch.empty_like(x)
    rng = np.random.default_rng(3)
    a = np.concatenate([rng.integers(0, s.count_up, 1500), np.arange(s.count_up - 150, s.count_up)])
    b = np.concatenate([rng.integers(0, s.count_dn, 1500), np.arange(s.count_dn - 150, s.count_dn)])
    ref, mag = _elements(m, s, x, a, b)
    where = torch.from_numpy(a + b * s.count_up).cuda()
    for order in (None, 2):
        if order is not None:
            s.set_schedule(hub.F64, hub.SCHED_CHUNKED, tile_cols=1, quads_per_lane=8, order=order)
        y.fill_(7.0)
        s.matvec(x, y)
        # 42 terms at most, each rounded to 2^-53 of the running sum
        assert np.all(np.abs(y[where].cpu().numpy() - ref) <= 42 * 2.0 ** -53 * 2 * mag), order
    s.close()
    del x, y
    torch.cuda.empty_cache()


# 31 x 7888725: more columns than workgroups of 1024 lanes that one launch holds,
# and a column length that is no multiple of four
def test_product_of_many_short_columns(hub):
    import torch
    m = W.ring(31, U=4.0, n_up=1, n_dn=8)
    s = hub.Sector(m)
    assert s.count_dn * 1024 >= 1 << 32 and s.count_up % 4
    x = s.start_vector(seed=5, normalize=False)
    y = s.matvec(x)
    rng = np.random.default_rng(3)
    a = np.concatenate([rng.integers(0, s.count_up, 1500), np.full(150, s.count_up - 1)])
    b = np.concatenate([rng.integers(0, s.count_dn, 1500), np.arange(s.count_dn - 150, s.count_dn)])
    ref, mag = _elements(m, s, x, a, b)
    got = y[torch.from_numpy(a + b * s.count_up).cuda()].cpu().numpy()
    assert np.all(np.abs(got - ref) <= 42 * 2.0 ** -53 * 2 * mag)
    s.close()


# 173686800 representatives (more than 2^27) of 32 sites with 13 electrons under i -> i - 16
def test_k0_sector_of_many_representatives(hub):
    """With one bond, H H = t^2 on the states whose ends differ there, and 0 else."""
    from types import SimpleNamespace
    import torch
    if torch.cuda.mem_get_info()[0] < 80e9:
        torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 80e9:
        pytest.skip("needs 80 GB of device memory")
    t = 1.5
    m = SimpleNamespace(n_sites=32, bonds=[(0, 16)], t=[t], U=[2.0] * 32, eps=[0.0] * 32, n_up=13, n_dn=0)
    s = hub.Sector(m, translation=16)
    reps, periods = s.k0_layout()
    assert len(reps) == 173686800 and s.dim == len(reps) and periods.min() == 2
    x = s.start_vector(seed=5, normalize=False)
    y = s.matvec(x)
    z = s.matvec(y)
    r = torch.from_numpy(reps.astype(np.int64)).cuda()
    hops = ((r ^ (r >> 16)) & 1).bool()
    assert torch.equal(z, torch.where(hops, t * (t * x), torch.zeros_like(x)))
    assert not torch.equal(y[hops], t * x[hops])   # the hops go somewhere
    s.close()
