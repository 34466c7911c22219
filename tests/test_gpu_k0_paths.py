"""The k = 0 product's paths against each other: the H_dn term in its own pass
(vectors above 16 MB) or gathered in the kernel, cycles staged in LDS or read
from global memory, one or four members per lane."""
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


# FP64: own pass, staged; FP32: in the kernel, staged (ring 15, 22 and 11 MB);
# FP64: own pass, not staged (194 KB a cycle); FP32: own pass, staged (ring 17);
# short cycles and a ragged last group of members (ring 18 with shift 3: q = 6, 2, 1)
@pytest.mark.parametrize("M,n_up,n_dn,shift", [(15, 7, 7, 1), (17, 8, 8, 1), (18, 4, 9, 3)])
def test_k0_product_paths_agree(hub, M, n_up, n_dn, shift):
    import torch
    s = hub.Sector(W.ring(M, U=3.0, n_up=n_up, n_dn=n_dn), translation=shift)
    x = s.start_vector(seed=21)
    y64 = s.matvec(x)
    y32 = s.matvec(x.float()).double()
    # rows of at most 2 M hops and a diagonal of 3 M: 35 terms rounded to FP32
    scale = float(y64.abs().max())
    assert float((y64 - y32).abs().max()) <= 35 * 6e-8 * 4 * scale
    # H is symmetric on the block
    z = s.start_vector(seed=22)
    a, b = float(torch.dot(z, y64)), float(torch.dot(s.matvec(z), x))
    assert abs(a - b) <= 1e-12 * float(torch.linalg.vector_norm(y64))
    assert np.isfinite(a)
    s.close()
