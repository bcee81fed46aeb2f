"""The launches that the automatic schedule chooses, on host-only handles (a
device of 256 compute units is assumed; nothing is launched)."""
from __future__ import annotations

import pytest

from paper_2302_10736_amd import gridgen, pf

CALLS = [(pf.PF_OP_INJECTIONS, pf.PF_METHOD_ELEMENTWISE), (pf.PF_OP_INJECTIONS, pf.PF_METHOD_YBUS),
         (pf.PF_OP_JACOBIAN, pf.PF_METHOD_ELEMENTWISE), (pf.PF_OP_JACOBIAN, pf.PF_METHOD_YBUS),
         (pf.PF_OP_JACOBIAN, pf.PF_METHOD_ELEMENTWISE | pf.PF_JAC_CSC),
         (pf.PF_OP_JACOBIAN, pf.PF_METHOD_YBUS | pf.PF_JAC_CSC), (pf.PF_OP_VJP, pf.PF_METHOD_ELEMENTWISE)]
ORDERS = (pf.PF_ORDER_AUTO, pf.PF_ORDER_TILE_MAJOR, pf.PF_ORDER_STATE_MAJOR, pf.PF_ORDER_GROUPED)


def _plan(G, call, nstate):
    """states per workgroup, order, read-ahead, workgroups, threads"""
    return pf.pf_debug_launch(G, *call, nstate)


# A launch holds less than 2^32 threads however many states it has; the
# grouped order's grid is padded to eight equal shares of the tiles.
@pytest.mark.parametrize("nb,nl", [(2, 1), (500, 700), (2_500, 3_400)])
@pytest.mark.parametrize("tile", [64, 256, 512])
def test_launches_below_two_to_the_32_threads(nb, nl, tile):
    G = pf.Grid.from_grid(gridgen.make_grid(nb, nl, 0.15, case=9), host_only=True)
    for order in ORDERS:
        G.set_schedule(tile, 0, order)
        for call in CALLS:
            for nstate in (1, 3, (1 << 24) + 5, 1 << 26, (1 << 31) - 1):
                spb, _, _, blocks, threads = _plan(G, call, nstate)
                assert threads == tile and 1 <= spb <= nstate
                assert blocks * threads < 1 << 32, (order, call, nstate, spb, blocks)


def test_debug_launch_argument_checks():
    G = pf.Grid.from_grid(gridgen.make_grid(2, 1, 0.0, case=9), host_only=True)
    for op, nstate in ((7, 1), (pf.PF_OP_VJP, 0)):
        with pytest.raises(pf.PFError) as e:
            pf.pf_debug_launch(G, op, 0, nstate)
        assert e.value.code == pf.PF_EINVAL
