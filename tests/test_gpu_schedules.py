"""Launch paths that a schedule or a batch size selects give the bits of the
plain one-state launch."""
import numpy as np
import pytest

from paper_2302_10736_amd import gridgen, pf
from tests import _gpu

pytestmark = pytest.mark.gpu

METHODS = (pf.PF_METHOD_ELEMENTWISE, pf.PF_METHOD_YBUS, pf.PF_METHOD_ELEMENTWISE | pf.PF_JAC_CSC,
           pf.PF_METHOD_YBUS | pf.PF_JAC_CSC)


def _shifted(shape, fill=None):
    """A device tensor that starts 8 bytes past a 16-byte boundary."""
    import torch
    n = int(np.prod(shape))
    t = torch.zeros(n + 1, dtype=torch.float64, device="cuda:0")[1:].view(shape)
    if fill is not None:
        t.copy_(torch.as_tensor(fill))
    return t


@pytest.fixture(scope="module")
def grid_6k():
    """6,007 buses: at least eight tiles per XCD at every tile size."""
    _gpu.require_gpu()
    g = gridgen.make_grid(6_007, 10_200, 0.15, case=9)
    G = pf.Grid.from_grid(g)
    pf.pf_ybus(G)
    return G


# States below, at and past the first read-ahead, whole and cut bursts
# (256-record tiles: 10 or 14 per XCD, first at 34 or 27 states; 64: 14).
@pytest.mark.parametrize("tile,nstate", [(256, 2), (256, 26), (256, 27), (256, 34), (256, 41), (256, 61), (64, 13), (64, 14),
                                         (64, 31), (512, 50)])
def test_read_ahead_same_bits(grid_6k, tile, nstate):
    import torch
    G = grid_6k
    vm0, va0 = gridgen.states(G.nb, nstate, case=9, grid=nstate)
    vm, va = _shifted(vm0.shape, vm0), _shifted(va0.shape, va0)
    for method in METHODS:
        got = {}
        for order in (pf.PF_ORDER_GROUPED, pf.PF_ORDER_TILE_MAJOR):
            G.set_schedule(tile, 1, order)
            p, q = _shifted(vm0.shape), _shifted(vm0.shape)
            j = torch.empty((nstate, G.nnz_j), dtype=torch.float64, device="cuda:0")
            pf.pf_jacobian_values(G, method, vm, va, p, q, j)
            got[order] = (p, q, j)
        torch.cuda.synchronize()
        for a, b in zip(got[pf.PF_ORDER_GROUPED], got[pf.PF_ORDER_TILE_MAJOR]):
            assert torch.equal(a, b)
