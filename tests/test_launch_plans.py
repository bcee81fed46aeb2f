"""The launches that the automatic schedule chooses, on host-only handles (a
device of 256 compute units is assumed; nothing is launched)."""
from __future__ import annotations

import pytest

import numpy as np

from paper_2302_10736_amd import gridgen, pf
from tests import _grids

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


# One long row leaves the other tiles' launch as it is; it only gets work items
# of its own, in front.
@pytest.mark.parametrize("nb,deg,tile", [(60_000, 513, 256), (60_000, 3_000, 256), (30_000, 140, 64)])
@pytest.mark.parametrize("nstate", [2, 7, 32, 128])
def test_a_long_row_leaves_the_other_tiles_launch(nb, deg, tile, nstate):
    g = gridgen.make_grid(nb, nb + nb // 3, 0.15, case=9)
    far = np.arange(1, deg + 1, dtype=np.int32) * (nb // (deg + 2))
    cat = lambda a, b: np.concatenate([a, np.full(deg, b)])  # noqa: E731
    h = gridgen.Grid(nb, g.nl + deg, cat(g.fbus, 0).astype(np.int32), np.concatenate([g.tbus, far]).astype(np.int32),
                     cat(g.r, 0.01), cat(g.x, 0.1), cat(g.b, 0.02), cat(g.tap, 1.0), cat(g.shift, 0.0), g.gs, g.bs)
    G, H = (pf.Grid.from_grid(x, host_only=True) for x in (g, h))
    G.set_schedule(tile)
    H.set_schedule(tile)
    for call in CALLS:
        a, b = _plan(G, call, nstate), _plan(H, call, nstate)
        assert a[:2] == b[:2] and abs(b[3] - a[3]) <= 0.1 * a[3] + 2 * nstate + 16


# The adjoint's split over a device of 1,024 resident workgroups: one round of
# equal walks where that is the shortest at any number of tiles (tile-major, never
# a workgroup more than the device holds), else 16 or 32 states per workgroup.
@pytest.mark.parametrize("nb,nstate,want", [(5_000, 1_000, 50), (5_000, 2_000, 100), (33_000, 64, 22), (33_000, 48, 16),
                                            (50_000, 40, 20), (96_500, 32, 32), (100_000, 32, 32), (105_000, 32, 16),
                                            (70_000, 37, 16), (20_000, 80, 20), (20_000, 128, 16), (20_000, 40, 10),
                                            (100_000, 100, 32), (100_000, 20, 20), (60_000, 20, 16)])
def test_adjoint_split(nb, nstate, want):
    G = pf.Grid.from_grid(gridgen.make_grid(nb, int(1.3 * nb), 0.15, case=9), host_only=True)
    spb, order, _, blocks, _ = _plan(G, CALLS[6], nstate)
    assert spb == want
    if order == pf.PF_ORDER_TILE_MAJOR:
        assert blocks <= 1_024 + 7


# Injections: tile-major for one grid or several, grouped from 64 states and 48 MB
# of grids larger than a tile.
@pytest.mark.parametrize("nb,grids,nstate,want", [(40, 200, 64, pf.PF_ORDER_TILE_MAJOR), (40, 200, 1_000, pf.PF_ORDER_TILE_MAJOR),
                                                  (3_000, 20, 4, pf.PF_ORDER_TILE_MAJOR), (3_000, 20, 63, pf.PF_ORDER_TILE_MAJOR),
                                                  (3_000, 20, 64, pf.PF_ORDER_GROUPED), (60_000, 1, 64, pf.PF_ORDER_GROUPED),
                                                  (60_000, 1, 63, pf.PF_ORDER_TILE_MAJOR), (40_000, 1, 64, pf.PF_ORDER_TILE_MAJOR)])
def test_order_of_injections(nb, grids, nstate, want):
    big, bo, ro = gridgen.concat([gridgen.make_grid(nb, int(1.3 * nb), 0.15, case=9, grid=k) for k in range(grids)])
    G = pf.Grid.from_grid(big, *((bo, ro) if grids > 1 else (None, None)), host_only=True)
    assert all(_plan(G, call, nstate)[1] == want for call in CALLS[:2])


# Jacobian launches of grids numbered at random: two states per workgroup from 8
# states on while the arrays of two stay in L2, never an uneven rest of few states.
@pytest.mark.parametrize("nb,nstate,csr,csc", [(60_000, 3, (1, 2), (1, 3)), (60_000, 7, (1, 2), (1, 3)), (60_000, 8, (2, 2), (2, 2)),
                                               (100_000, 3, (1, 2), (1, 2)), (100_000, 8, (2, 2), (2, 2)), (10_000, 24, (1, 2), (1, 2)),
                                               (140_000, 24, (1, 2), (1, 2))])
def test_scattered_jacobian_plans(nb, nstate, csr, csc):
    G = pf.Grid.from_grid(gridgen.relabel(gridgen.make_grid(nb, int(1.3 * nb), 0.15, case=9), 9, 1)[0], host_only=True)
    for call, want in zip(CALLS[2:6], (csr, csr, csc, csc)):
        assert _plan(G, call, nstate)[:2] == want


# Jacobian launches read later states ahead from 128 MB of inputs on, in the
# library's own order only.
@pytest.mark.parametrize("nb,nstate,want", [(20_000, 419, 0), (20_000, 420, 1), (60_000, 139, 0), (60_000, 140, 1), (130_000, 65, 1),
                                            (260_000, 60, 0)])
def test_read_ahead_plans(nb, nstate, want):
    G = pf.Grid.from_grid(gridgen.make_grid(nb, int(1.3 * nb), 0.15, case=9), host_only=True)
    assert all(_plan(G, call, nstate)[2] == want for call in CALLS[2:6])
    assert all(_plan(G, call, nstate)[2] == 0 for call in CALLS[:2] + CALLS[6:])
    G.set_schedule(256, 1, pf.PF_ORDER_GROUPED)
    assert all(_plan(G, call, nstate)[2] == 0 for call in CALLS)


# S+J of grids whose tables do not stay in L2: two states per workgroup for
# element-wise CSR launches whose inputs may be in the memory-side cache, else four.
@pytest.mark.parametrize("nb,nstate,ew,others", [(140_000, 8, 1, 1), (200_000, 8, 2, 4), (300_000, 4, 4, 4), (300_000, 5, 2, 4),
                                             (300_000, 55, 2, 4), (300_000, 56, 4, 4)])
def test_states_per_workgroup_with_large_tables(nb, nstate, ew, others):
    G = pf.Grid.from_grid(gridgen.make_grid(nb, int(1.3 * nb), 0.15, case=9), host_only=True)
    assert [_plan(G, call, nstate)[0] for call in CALLS[2:6]] == [ew, others, others, others]


# Parallel circuits lengthen the element-wise rows, not those of Ybus.
def test_long_rows_of_each_method():
    g = _grids.random_small(120, 119, 3)
    far = np.repeat(np.arange(1, 101, dtype=np.int32), 6)
    n = len(far)
    cat = lambda a, b: np.concatenate([a, np.full(n, b)])  # noqa: E731
    G = pf.Grid.from_grid(gridgen.Grid(g.nb, g.nl + n, cat(g.fbus, 0).astype(np.int32), np.concatenate([g.tbus, far]).astype(np.int32),
                                       cat(g.r, 0.01), cat(g.x, 0.1), cat(g.b, 0.02), cat(g.tap, 1.0), cat(g.shift, 0.0),
                                       g.gs, g.bs), host_only=True)
    G.set_schedule(256, 4, pf.PF_ORDER_TILE_MAJOR)
    ew, yb = (_plan(G, c, 64)[3] for c in CALLS[:2])
    assert ew >= 64 + 16 and yb <= 16 * 8  # 600 branch ends: 64 items more; 120 nonzeros a row: none


def test_debug_launch_argument_checks():
    G = pf.Grid.from_grid(gridgen.make_grid(2, 1, 0.0, case=9), host_only=True)
    for op, nstate in ((7, 1), (pf.PF_OP_VJP, 0)):
        with pytest.raises(pf.PFError) as e:
            pf.pf_debug_launch(G, op, 0, nstate)
        assert e.value.code == pf.PF_EINVAL
