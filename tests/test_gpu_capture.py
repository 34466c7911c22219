"""First products of a sector under stream capture."""
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


# columns of odd length, for which no product needed tuning before the four-row
# kernels took them: within the LDS (126, 715 rows) and beyond it (24310, 20349)
@pytest.mark.parametrize("M,n_up,n_dn", [(9, 4, 4), (13, 4, 2), (17, 8, 1), (21, 5, 1)])
@pytest.mark.parametrize("tuned_by_another", [False, True])
def test_first_product_of_ragged_columns_captured(hub, M, n_up, n_dn, tuned_by_another):
    """The very first product of a sector, captured, replays to the eager one for
    new inputs, also where a sector of the same structure was tuned before."""
    import torch
    m = W.ring(M, U=2.0, n_up=n_up, n_dn=n_dn)
    for dt in (hub.F64, hub.F32):
        if tuned_by_another:
            with hub.Sector(m) as o:
                o.matvec(o.start_vector(seed=1, dtype=dt))
        s = hub.Sector(m.with_params(eps=[0.01 * (tuned_by_another + dt * 2)] * M))
        x = s.start_vector(seed=5, dtype=dt)
        y, z = torch.empty_like(x), torch.empty_like(x)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            s.matvec(x, y)
        for seed in (5, 6, 7):
            x.copy_(s.start_vector(seed=seed, dtype=dt))
            g.replay()
            s.matvec(x, z)
            torch.cuda.synchronize()
            assert torch.equal(y, z), (dt, seed)
        s.close()
