"""The H_dn term in a pass of its own (order 2), and columns of any length in the
kernels with four rows per lane, against the row and CSR kernels (bit for bit)
and the oracle."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hub():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("needs a GPU")
    import paper_1307_7542_amd as h
    h.lib()
    return h


# count_up: 4 (one quad), 252 (partial group of 256 rows), 924 (several groups, partial last one)
@pytest.mark.parametrize("M,n_up,n_dn", [(4, 1, 2), (10, 5, 3), (12, 6, 2)])
def test_separate_dn_pass_bitwise(hub, M, n_up, n_dn):
    """Every two-pass shape gives the CSR kernel's product bit for bit, and a
    solve through it the energy and steps of the one-pass product."""
    import torch
    m = W.ring(M, U=3.0, n_up=n_up, n_dn=n_dn).with_params(eps=[0.07 * i for i in range(M)])
    s = hub.Sector(m)
    assert s.count_up % 4 == 0
    for dt in (hub.F64, hub.F32):
        x = s.start_vector(seed=3, dtype=dt)
        s.set_schedule(dt, hub.SCHED_CSR)
        y0 = s.matvec(x)
        s.set_schedule(dt, hub.SCHED_COLUMNS, tile_cols=1, block=512, order=1)
        g0 = s.ground_state(dtype=dt, want_vector=False)
        shapes = [(hub.SCHED_COLUMNS, dict(tile_cols=tb, block=bs)) for tb in (1, 2, 3) for bs in (512, 1024)]
        shapes += [(hub.SCHED_CHUNKED, dict(tile_cols=tb, quads_per_lane=q, chunk_rows=c))
                   for tb, q in ((1, 4), (2, 4), (1, 8)) for c in (0, 100)]
        for fam, kw in shapes:
            s.set_schedule(dt, fam, order=2, **kw)
            assert torch.equal(s.matvec(x), y0), (dt, fam, kw)
            g = s.ground_state(dtype=dt, want_vector=False)
            assert (g.e0, g.info["iters"]) == (g0.e0, g0.info["iters"]), (dt, fam, kw)
        s.set_schedule(dt, None)
    s.close()


# count_up % 4 = 1, 2, 3: 21 and 126 (less than one group of 256 rows), 715 (several),
# 20349 and 24310 (columns beyond the LDS in FP64: chunks, two passes)
@pytest.mark.parametrize("M,n_up,n_dn", [(7, 2, 3), (9, 4, 4), (13, 4, 2), (21, 5, 1), (17, 8, 1)])
def test_ragged_columns(hub, M, n_up, n_dn):
    """Tuned products of columns whose length is no multiple of four equal the
    CSR kernel's bit for bit; FP64 solves reach the oracle's energy."""
    import torch
    m = W.ring(M, U=2.0, n_up=n_up, n_dn=n_dn).with_params(eps=[0.05 * ((5 * i) % M) for i in range(M)])
    s = hub.Sector(m)
    assert s.count_up % 4 != 0
    for dt in (hub.F64, hub.F32):
        x = s.start_vector(seed=5, dtype=dt)
        y = s.matvec(x)
        s.set_schedule(dt, hub.SCHED_CSR)
        assert torch.equal(s.matvec(x), y), dt
        s.set_schedule(dt, None)
    xr = s.start_vector(seed=5, normalize=False)
    osec = oracle.Sector(m)
    ref = oracle.spmv(osec.csr(), oracle.start_vector(5, osec.dim))
    assert np.max(np.abs(s.matvec(xr).cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref))
    _, e_ref, _ = oracle.ground_state(m, want_vector=False)
    g = s.ground_state(want_vector=True, refine=True)
    assert abs(g.e0 - e_ref) <= 1e-10 * abs(e_ref)
    assert g.info["true_residual"] <= 1e-9 * abs(e_ref)
    s.close()


# 11440 x 12870: the order of the columns spans one component, or (sites 0-9 a
# chain, 10-13 a ring, 14 and 15 alone) many of different sizes
@pytest.mark.parametrize("whole", [True, False])
def test_column_order_of_dn_pass_bitwise(hub, whole):
    """The H_dn pass in breadth-first order of the columns reaches every column
    once: the two-pass product equals the one-pass one bit for bit."""
    import torch
    from types import SimpleNamespace
    M = 16
    bonds = [(i, (i + 1) % M) for i in range(M)]
    if not whole:
        bonds = [(i, i + 1) for i in range(9)] + [(10, 11), (11, 12), (12, 13), (10, 13)]
    m = SimpleNamespace(n_sites=M, bonds=bonds, t=[1.0 + 0.01 * i for i in range(len(bonds))], U=[4.0] * M,
                        eps=[0.0] * M, n_up=7, n_dn=8)
    s = hub.Sector(m)
    x = s.start_vector(seed=5, dtype=hub.F32)
    s.set_schedule(hub.F32, hub.SCHED_COLUMNS, tile_cols=1, block=1024, order=1)
    y0 = s.matvec(x)
    s.set_schedule(hub.F32, hub.SCHED_COLUMNS, tile_cols=2, block=1024, order=2)
    assert torch.equal(s.matvec(x), y0)
    s.close()


# count_up: 4 (one quad), 20 and 28, 220 and 252 (within one group of 256 rows),
# 276 and 816 (two and four groups); ragged 25, 231, 455 (tuned shapes)
@pytest.mark.parametrize("M,n_up,n_dn", [(4, 1, 2), (20, 1, 4), (8, 2, 3), (12, 3, 2), (10, 5, 4), (24, 2, 2), (18, 3, 2),
                                         (25, 1, 3), (22, 2, 3), (15, 3, 4)])
def test_short_columns_bitwise(hub, M, n_up, n_dn):
    """Workgroups of one or four wavefronts give the CSR kernel's product bit for
    bit, and a solve through them the energy and steps of 512 lanes."""
    import torch
    m = W.ring(M, U=3.0, n_up=n_up, n_dn=n_dn).with_params(eps=[0.07 * i for i in range(M)])
    s = hub.Sector(m)
    for dt in (hub.F64, hub.F32):
        x = s.start_vector(seed=3, dtype=dt)
        s.set_schedule(dt, hub.SCHED_CSR)
        y0 = s.matvec(x)
        s.set_schedule(dt, None)
        assert torch.equal(s.matvec(x), y0), dt
        assert s.schedule(dt)["block"] in (64, 256)
        assert s.count_dn > 512 or s.schedule(dt)["tile_cols"] == 1   # few columns: one a workgroup
        if s.count_up % 4:
            continue
        s.set_schedule(dt, hub.SCHED_COLUMNS, tile_cols=1, block=512, order=1)
        g0 = s.ground_state(dtype=dt, want_vector=False)
        for bs in (64, 256):
            for tb in (1, 2, 3):
                s.set_schedule(dt, hub.SCHED_COLUMNS, tile_cols=tb, block=bs, order=1)
                assert torch.equal(s.matvec(x), y0), (dt, bs, tb)
                g = s.ground_state(dtype=dt, want_vector=False)
                assert (g.e0, g.info["iters"]) == (g0.e0, g0.info["iters"]), (dt, bs, tb)
        s.set_schedule(dt, None)
    s.close()


def test_short_columns_take_no_idle_lanes(hub):
    """A product of 25 x 480700 states takes at most 45 times a copy of its vector
    (25 with one wavefront a column, 94 with eight)."""
    import time
    import torch
    s = hub.Sector(W.ring(25, U=4.0, n_up=1, n_dn=7))
    x = s.start_vector(seed=1)
    y = torch.empty_like(x)

    def best(f):
        t = []
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(20):
                f()
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return min(t)

    assert best(lambda: s.matvec(x, y)) <= 45 * best(lambda: y.copy_(x))
    s.close()


def test_sector_creation_leaves_the_column_order_to_the_product(hub):
    """Creating the 2x9 ladder's half-filled sector (one basis of 48620 states) takes
    less than twice that of its sector with one down electron (the same basis and a
    small one); the order is made by the first product that uses it."""
    import time

    def best(n_dn):
        m = W.config("ladder2x9").with_params(n_up=9, n_dn=n_dn)
        t = []
        for _ in range(6):
            t0 = time.perf_counter()
            hub.Sector(m).close()
            t.append(time.perf_counter() - t0)
        return min(t)

    best(1)
    assert best(9) <= 2 * best(1)


# the order is made outside a capture only: 11440 x 12870, two passes
def test_two_pass_product_captured_first(hub):
    """A product in two passes whose first call is captured replays to the eager one."""
    import torch
    m = W.ring(16, U=4.0, n_up=7, n_dn=8)
    s = hub.Sector(m)
    x = s.start_vector(seed=5, dtype=hub.F32)
    s.set_schedule(hub.F32, hub.SCHED_COLUMNS, tile_cols=2, block=1024, order=2)
    y, z = torch.empty_like(x), torch.empty_like(x)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        s.matvec(x, y)
    for seed in (5, 6, 7):
        x.copy_(s.start_vector(seed=seed, dtype=hub.F32))
        g.replay()
        s.matvec(x, z)
        torch.cuda.synchronize()
        assert torch.equal(y, z), seed
    s.close()


# count_up % 4 = 1, 2, 3: 21 (one group of 256 rows), 126, 715 and 455 (several groups)
@pytest.mark.parametrize("M,n_up,n_dn", [(7, 2, 3), (9, 4, 4), (13, 4, 2), (15, 3, 2)])
def test_every_ragged_shape_bitwise(hub, M, n_up, n_dn):
    """Every shape that columns of odd length can have gives the CSR kernel's product
    bit for bit and the fused solve's energy and steps, and what the tuner reports can
    be set again."""
    import torch
    m = W.ring(M, U=2.0, n_up=n_up, n_dn=n_dn).with_params(eps=[0.05 * ((5 * i) % M) for i in range(M)])
    s = hub.Sector(m)
    assert s.count_up % 4 != 0
    for dt in (hub.F64, hub.F32):
        x = s.start_vector(seed=5, dtype=dt)
        s.matvec(x)
        tuned = s.schedule(dt)
        s.set_schedule(dt, tuned["family"], tile_cols=tuned["tile_cols"], block=tuned["block"], order=tuned["order"])
        assert {**s.schedule(dt), "ms": 0} == {**tuned, "ms": 0}
        s.set_schedule(dt, hub.SCHED_CSR)
        y0 = s.matvec(x)
        g0 = None
        shapes = [(hub.SCHED_COLUMNS, dict(tile_cols=tb, block=bs, order=o)) for tb in (1, 2)
                  for bs, o in ((64, 1), (256, 1), (512, 1), (1024, 1), (512, 2), (1024, 2)) if (tb, bs, o) != (2, 1024, 1)]
        shapes += [(hub.SCHED_CHUNKED, dict(tile_cols=tb, quads_per_lane=q, chunk_rows=c, order=2))
                   for tb, q in ((1, 4), (2, 4), (1, 8)) for c in (0, 100)]
        for fam, kw in shapes:
            s.set_schedule(dt, fam, **kw)
            assert torch.equal(s.matvec(x), y0), (dt, fam, kw)
            g = s.ground_state(dtype=dt, want_vector=False)
            g0 = g0 or g
            assert (g.e0, g.info["iters"]) == (g0.e0, g0.info["iters"]), (dt, fam, kw)
        for fam, kw in ((hub.SCHED_COLUMNS, dict(tile_cols=1, block=512, order=0)),
                        (hub.SCHED_COLUMNS, dict(tile_cols=3, block=512, order=1)),
                        (hub.SCHED_COLUMNS, dict(tile_cols=2, block=1024, order=1)),
                        (hub.SCHED_COLUMNS, dict(tile_cols=1, block=64, order=2)),
                        (hub.SCHED_CHUNKED, dict(tile_cols=1, quads_per_lane=4, order=0))):
            with pytest.raises(hub.HubError) as e:
                s.set_schedule(dt, fam, **kw)
            assert e.value.status == 1, kw
        s.set_schedule(dt, None)
    s.close()
