"""What the first product of a sector costs beside the later ones."""
import time

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


def test_first_product_times_few_launches(hub):
    """The first product of a structure, which chooses the schedule (6435 x 6435, eight
    shapes), takes at most 75 products' time (two full rounds over every shape: 100)."""
    import torch
    with hub.Sector(W.ring(10, U=4.0, n_up=5, n_dn=5)) as o:
        o.matvec(o.start_vector(seed=1))   # code loaded
    s = hub.Sector(W.ring(15, U=4.0, n_up=7, n_dn=8))
    x = s.start_vector(seed=1)
    y = torch.empty_like(x)

    def run(n):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(n):
            s.matvec(x, y)
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) / n

    first = run(1)
    assert first <= 75 * min(run(10) for _ in range(3))
    s.close()
