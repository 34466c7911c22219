"""psi from kept Lanczos vectors, from a second run of the recurrence, and from both:
however many are kept, a solve gives the same energy, steps and vector."""
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


def _dtypes(hub):
    return hub.F64, hub.F32


# 63504 rows of quads, 44100 of odd columns, 20 rows (few steps), 28 x 8008
@pytest.mark.parametrize("M,n_up,n_dn", [(10, 5, 5), (10, 4, 4), (6, 3, 3), (8, 2, 3), (16, 2, 6)])
def test_kept_vectors_of_a_sector(hub, M, n_up, n_dn):
    m = W.ring(M, U=3.0, n_up=n_up, n_dn=n_dn).with_params(eps=[0.07 * i for i in range(M)])
    s = hub.Sector(m)
    for dt in _dtypes(hub):
        want = s.ground_state(dtype=dt, refine=True)
        it = want.info["iters"]
        for keep in sorted({0, 1, 2, 3, 8, it - 1, it, it + 5}):
            got = s.ground_state(dtype=dt, refine=True, keep_vectors=keep)
            assert got.info["iters"] == it and got.info["e0_ritz"] == want.info["e0_ritz"], (dt, keep)
            # the vectors come back bit for bit; psi sums `it` terms in FP64, each below |psi| <= 1
            assert float((got.psi - want.psi).abs().max()) <= 4 * it * 2.0 ** -53, (dt, keep)
            products = it if keep == 0 else max(it - max(keep, 1), 0)
            assert got.info["matvec_count"] - want.info["matvec_count"] in (products - 1, products), (dt, keep)
    s.close()


def test_kept_vectors_of_a_batch(hub):
    """Sectors that stop before, at and after the last kept vector."""
    models = [W.ring(M, U=U, n_up=u, n_dn=d) for M, U, u, d in
              [(4, 2.0, 2, 2), (6, 4.0, 3, 3), (8, 3.0, 4, 4), (9, 2.0, 4, 4), (10, 6.0, 5, 5), (10, 1.0, 4, 4), (7, 3.0, 0, 3)]]
    secs = [hub.Sector(m) for m in models]
    b = hub.Batch(secs)
    for dt in _dtypes(hub):
        e0, it, psi, _ = b.ground_state(dtype=dt, want_vector=True)
        assert it.min() < 30 < np.median(it) < it.max()
        for keep in sorted({0, 1, 2, 3, 8, 30, int(np.median(it)), int(it.max()) - 1, int(it.max())}):
            for graph in (True, False):
                f0, jt, phi, _ = b.ground_state(dtype=dt, want_vector=True, keep_vectors=keep, graph=graph)
                assert np.array_equal(f0, e0) and np.array_equal(jt, it), (dt, keep)
                assert float((phi - psi).abs().max()) <= 4 * int(it.max()) * 2.0 ** -53, (dt, keep, graph)
    b.close()
    for s in secs:
        s.close()
