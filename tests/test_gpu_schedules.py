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


# Inputs at and past the size from which states are read ahead (8,388,608
# values of a state array), whole and cut bursts (256-record tiles: first at 34
# or 27 states).  The last 20 states are compared, and the sums of all.
@pytest.mark.parametrize("tile,nb,nstate", [(256, 60_013, 139), (256, 60_013, 140), (256, 60_013, 143), (64, 41_002, 206),
                                            (512, 70_001, 121), (256, 8_101, 1_040)])
def test_read_ahead_same_bits(tile, nb, nstate):
    import torch
    _gpu.require_gpu()
    g = gridgen.make_grid(nb, nb + nb // 9, 0.15, case=9)
    G = pf.Grid.from_grid(g)
    pf.pf_ybus(G)
    gen = torch.Generator(device="cuda:0").manual_seed(nstate)
    vm, va = _shifted((nstate, nb)), _shifted((nstate, nb))
    vm.uniform_(0.95, 1.05, generator=gen)
    va.normal_(0.0, 0.2, generator=gen)
    p, q = _shifted((nstate, nb)), _shifted((nstate, nb))
    j = torch.empty((nstate, G.nnz_j), dtype=torch.float64, device="cuda:0")
    for method in METHODS:
        got = []
        for order in (pf.PF_ORDER_GROUPED, pf.PF_ORDER_TILE_MAJOR):
            G.set_schedule(tile, 1, order)
            for t in (p, q, j):
                t.fill_(-7.0)
            pf.pf_jacobian_values(G, method, vm, va, p, q, j)
            got.append([t[-20:].clone() for t in (p, q, j)] + [t.view(torch.int64).sum(dim=1) for t in (p, q, j)])
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(*got))


def _twins(g, every):
    """The grid with every ``every``-th branch doubled."""
    cat = lambda x: np.concatenate([x, x[::every]])  # noqa: E731
    return gridgen.Grid(g.nb, len(cat(g.fbus)), *[cat(x) for x in (g.fbus, g.tbus, g.r, g.x, g.b, g.tap, g.shift)], g.gs, g.bs)


# Launches that read ahead (one has a hub bus, whose row's items of their own take
# its place) against the plain one-state launch: tile sizes, parallel circuits,
# several grids, bursts of 4 (from 72 tiles per XCD) and 8, whole and cut ones.
@pytest.mark.parametrize("tile,nb,grids,nstate,kind", [(256, 60_013, 1, 143, ""), (128, 41_002, 1, 207, ""), (256, 40_001, 1, 211, "twins"),
                                                       (512, 50_003, 1, 170, "twins"), (256, 20_005, 3, 141, ""), (64, 30_001, 1, 285, ""),
                                                       (256, 82_001, 1, 105, ""), (256, 50_007, 1, 170, "hub")])
def test_read_ahead_launches_same_bits(tile, nb, grids, nstate, kind):
    import torch
    _gpu.require_gpu()
    parts = [gridgen.make_grid(nb, nb + nb // 9, 0.15, case=9, grid=k) for k in range(grids)]
    if kind == "twins":
        parts = [_twins(parts[0], 13)]
    if kind == "hub":
        far = np.arange(1, 701, dtype=np.int32) * 31
        cat = lambda a, b: np.concatenate([a, np.full(700, b)])  # noqa: E731
        g = parts[0]
        parts = [gridgen.Grid(nb, g.nl + 700, cat(g.fbus, 0).astype(np.int32), np.concatenate([g.tbus, far]), cat(g.r, 0.01),
                              cat(g.x, 0.1), cat(g.b, 0.02), cat(g.tap, 1.0), cat(g.shift, 0.0), g.gs, g.bs)]
    big, bo, ro = gridgen.concat(parts)
    G = pf.Grid.from_grid(big, *((bo, ro) if grids > 1 else (None, None)))
    pf.pf_ybus(G)
    gen = torch.Generator(device="cuda:0").manual_seed(nstate)
    vm, va = _shifted((nstate, G.nb)), _shifted((nstate, G.nb))
    vm.uniform_(0.95, 1.05, generator=gen)
    va.normal_(0.0, 0.2, generator=gen)
    p, q = _shifted((nstate, G.nb)), _shifted((nstate, G.nb))
    j = torch.empty((nstate, G.nnz_j), dtype=torch.float64, device="cuda:0")
    for method in METHODS:
        got = []
        for order, ahead in ((pf.PF_ORDER_AUTO, kind != "hub"), (pf.PF_ORDER_TILE_MAJOR, False)):
            G.set_schedule(tile, 1, order)
            assert pf.pf_debug_launch(G, pf.PF_OP_JACOBIAN, method, nstate)[2] == ahead
            for t in (p, q, j):
                t.fill_(-7.0)
            pf.pf_jacobian_values(G, method, vm, va, p, q, j)
            got.append([t[-20:].clone() for t in (p, q, j)] + [t.view(torch.int64).sum(dim=1) for t in (p, q, j)])
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(*got))


# Branches below, at and past a wave's 48 outputs and a workgroup's 192, with
# rows that start at every place of a 128-byte line (nl odd).
@pytest.mark.parametrize("nl,nstate,off", [(1, 2, 0), (47, 3, 1), (48, 17, 0), (49, 16, 5), (176, 2, 15), (177, 3, 0),
                                           (191, 9, 3), (193, 16, 2), (385, 5, 7)])
def test_flow_rows_any_alignment(nl, nstate, off):
    import oracle
    import torch
    _gpu.require_gpu()
    nb = max(2, int(nl / 1.3))
    g = gridgen.make_grid(nb, max(nl, nb - 1), 0.3, case=9, grid=nl)
    G = pf.Grid.from_grid(g)
    vm, va = gridgen.states(nb, nstate, case=9, grid=nl)
    pad = 64  # values around every output, which stay as they are
    def out(*shape):
        n = int(np.prod(shape))
        whole = torch.full((n + 2 * pad + off,), -7.0, dtype=torch.float64, device="cuda:0")
        return whole, whole[pad + off:pad + off + n].view(shape)
    outs = [out(nstate, g.nl) for _ in range(4)] + [out(nstate, 16, g.nl)]
    pf.pf_branch_flows(G, _gpu.to_dev(vm), _gpu.to_dev(va), *[o for _, o in outs])
    torch.cuda.synchronize()
    for whole, o in outs:
        assert (whole[:pad + off] == -7.0).all() and (whole[pad + off + o.numel():] == -7.0).all()
    got = [o.cpu().numpy() for _, o in outs]
    for s in range(nstate):
        want = oracle.branch_flows(g, vm[s], va[s])
        for a, b in zip(got[:4], want):
            assert _gpu.rel_err(a[s], b) <= _gpu.TOL
        assert _gpu.rel_err(got[4][s], np.asarray(oracle.branch_flow_jac(g, vm[s], va[s])).reshape(got[4][s].shape)) <= _gpu.TOL


# Every form of the launch: rows on whole lines, on half lines (40 states too few
# for the overlap, 55 enough) and anywhere (14 too few), sizes around a wave's 48 and
# a workgroup's 192 outputs, and more branches than an XCD's L2 keeps records of.
# Each state has the bits of its own launch, and nothing is written beside a row.
@pytest.mark.parametrize("nl,nstate,off", [(1, 79_000, 1), (47, 1_700, 0), (49, 1_630, 5), (177, 450, 3), (193, 420, 15),
                                           (385, 210, 0), (5_600, 55, 2), (5_608, 40, 0), (5_608, 60, 0), (5_601, 12, 0),
                                           (24_000, 5, 0), (24_000, 6, 0),
                                           (60_000, 2, 0), (60_001, 2, 0), (60_001, 1, 1), (60_008, 2, 8), (60_008, 6, 8)])
def test_flow_forms_same_bits(nl, nstate, off):
    import torch
    _gpu.require_gpu()
    nb = max(2, int(nl / 1.3))
    g = gridgen.make_grid(nb, max(nl, nb - 1), 0.3, case=9, grid=nl)
    G = pf.Grid.from_grid(g)
    few = min(nstate, 7)
    vm, va = (_gpu.to_dev(x).repeat(nstate // few + 1, 1)[:nstate].contiguous() for x in gridgen.states(nb, few, case=9, grid=nl))
    pad = 64
    def out(*shape):
        n = int(np.prod(shape))
        whole = torch.full((n + 2 * pad + off,), -7.0, dtype=torch.float64, device="cuda:0")
        return whole, whole[pad + off:pad + off + n].view(shape)
    one = [torch.empty((few, nl), dtype=torch.float64, device="cuda:0") for _ in range(4)]
    one.append(torch.empty((few, 16, nl), dtype=torch.float64, device="cuda:0"))
    for s in range(few):
        pf.pf_branch_flows(G, vm[s], va[s], *[o[s] for o in one])
    for partials in (False, True):
        outs = [out(nstate, nl) for _ in range(4)] + ([out(nstate, 16, nl)] if partials else [])
        pf.pf_branch_flows(G, vm, va, *[o for _, o in outs])
        for (whole, o), w in zip(outs, one):
            assert (whole[:pad + off] == -7.0).all() and (whole[pad + off + o.numel():] == -7.0).all()
            assert all(torch.equal(o[s::few], w[s].expand_as(o[s::few])) for s in range(few))


# More states than a launch of less than 2^32 threads holds workgroups of 256:
# every state of a repeating sequence of seven has the flows of its first turn.
def test_flows_of_many_states():
    import torch
    _gpu.require_gpu()
    g = gridgen.make_grid(2, 1, 0.0, case=9)
    G = pf.Grid.from_grid(g)
    nstate = (1 << 24) + 5
    vm, va = (_gpu.to_dev(x).repeat(nstate // 7 + 1, 1)[:nstate].contiguous() for x in gridgen.states(2, 7, case=9))
    outs = [torch.full((nstate, g.nl), -7.0, dtype=torch.float64, device="cuda:0") for _ in range(4)]
    pf.pf_branch_flows(G, vm, va, *outs)
    few = [torch.empty((7, g.nl), dtype=torch.float64, device="cuda:0") for _ in range(4)]
    pf.pf_branch_flows(G, vm[:7], va[:7], *few)
    for o, f in zip(outs, few):
        assert torch.equal(o, f.repeat(nstate // 7 + 1, 1)[:nstate])


# States per workgroup of the Jacobian loop: one, a few, more than there are.
@pytest.mark.parametrize("tile", [64, 256, 512])
@pytest.mark.parametrize("parallel", [False, True])
def test_jacobian_states_per_workgroup_same_bits(tile, parallel):
    import torch
    _gpu.require_gpu()
    g = gridgen.make_grid(1_501, 2_100, 0.15, case=9, grid=1)
    if parallel:
        cat = lambda x: np.concatenate([x, x[::7]])  # noqa: E731
        g = gridgen.Grid(g.nb, len(cat(g.fbus)), *[cat(x) for x in (g.fbus, g.tbus, g.r, g.x, g.b, g.tap, g.shift)], g.gs, g.bs)
    G = pf.Grid.from_grid(g)
    pf.pf_ybus(G)
    nstate = 7
    vm, va = (_gpu.to_dev(x) for x in gridgen.states(g.nb, nstate, case=9, grid=1))
    for method in METHODS:
        want = None
        for spb in (1, 2, 3, 4, 7, 9):
            G.set_schedule(tile, spb, pf.PF_ORDER_AUTO)
            p, q = torch.empty_like(vm), torch.empty_like(vm)
            j = torch.empty((nstate, G.nnz_j), dtype=torch.float64, device="cuda:0")
            pf.pf_jacobian_values(G, method, vm, va, p, q, j)
            torch.cuda.synchronize()
            if want is None:
                want = (p, q, j)
            assert all(torch.equal(a, b) for a, b in zip((p, q, j), want))


# Grids numbered at random take other work orders than those numbered along
# the network (2,500 buses: above the distance that counts as far; 900: below).
@pytest.mark.parametrize("nb,nstate", [(900, 9), (2_500, 2), (2_500, 33), (7_001, 19)])
def test_random_numbering_same_bits(nb, nstate):
    import torch
    _gpu.require_gpu()
    g, _ = gridgen.relabel(gridgen.make_grid(nb, int(1.35 * nb), 0.15, case=9, grid=nb), 9, nb)
    G = pf.Grid.from_grid(g)
    pf.pf_ybus(G)
    vm, va = (_gpu.to_dev(x) for x in gridgen.states(nb, nstate, case=9, grid=nb))
    lp, lq = (_gpu.to_dev(x) for x in gridgen.adjoint_seeds(nb, nstate, case=9, grid=nb))
    want = None
    for sched in ((256, 0, pf.PF_ORDER_AUTO), (256, 1, pf.PF_ORDER_TILE_MAJOR), (128, 5, pf.PF_ORDER_GROUPED)):
        G.set_schedule(*sched)
        out = [torch.empty_like(vm) for _ in range(6)]
        pf.pf_injections_elementwise(G, vm, va, out[0], out[1])
        pf.pf_injections_ybus(G, vm, va, out[2], out[3])
        pf.pf_injections_vjp(G, vm, va, lp, lq, out[4], out[5])
        for method in METHODS:
            out += [torch.empty_like(vm), torch.empty_like(vm),
                    torch.empty((nstate, G.nnz_j), dtype=torch.float64, device="cuda:0")]
            pf.pf_jacobian_values(G, method, vm, va, *out[-3:])
        torch.cuda.synchronize()
        want = want or out
        assert all(torch.equal(a, b) for a, b in zip(out, want))


# Rows longer than a tile among others, and (10 buses, tile 64) nearly alone, and
# packed rows of more than 64 terms: their states are work items of their own.
@pytest.mark.parametrize("tile,nb,nhub,deg,parallel,nstate", [(64, 400, 3, (65, 140), 0, 5), (64, 400, 9, (70, 399), 60, 7),
                                                              (128, 900, 1, (129, 129), 0, 2), (256, 2_000, 11, (257, 1_300), 300, 9),
                                                              (512, 2_500, 2, (513, 2_400), 0, 19), (64, 10, 0, (0, 0), 900, 6),
                                                              (128, 6_000, 2, (66, 120), 40, 5), (256, 9_000, 3, (100, 250), 0, 18)])
def test_long_rows_several_states_same_bits(tile, nb, nhub, deg, parallel, nstate):
    import torch
    from tests import _grids
    _gpu.require_gpu()
    G = pf.Grid.from_grid(_grids.random_hubs(nb, nhub, *deg, parallel, seed=nb + nhub))
    pf.pf_ybus(G)
    vm, va = (_gpu.to_dev(x) for x in gridgen.states(nb, nstate, case=9, grid=nb))
    lp, lq = (_gpu.to_dev(x) for x in gridgen.adjoint_seeds(nb, nstate, case=9, grid=nb))
    ph = [torch.empty(4 * nstate * nb, dtype=torch.float64, device="cuda:0") for _ in range(2)]
    for layout, buf in zip((pf.PF_PHASOR_SPLIT, pf.PF_PHASOR_INTERLEAVED), ph):
        pf.pf_phasors(G, layout, vm, va, buf)
    want = None
    for spb, order in ((1, pf.PF_ORDER_TILE_MAJOR), (0, pf.PF_ORDER_AUTO), (2, pf.PF_ORDER_TILE_MAJOR), (3, pf.PF_ORDER_STATE_MAJOR),
                       (4, pf.PF_ORDER_GROUPED), (nstate, pf.PF_ORDER_GROUPED), (nstate + 5, pf.PF_ORDER_AUTO)):
        G.set_schedule(tile, spb, order)
        new = lambda n: torch.full((nstate, n), -7.0, dtype=torch.float64, device="cuda:0")  # noqa: E731
        out = [new(nb) for _ in range(6)]
        pf.pf_injections_elementwise(G, vm, va, out[0], out[1])
        pf.pf_injections_ybus(G, vm, va, out[2], out[3])
        pf.pf_injections_vjp(G, vm, va, lp, lq, out[4], out[5])
        for method in METHODS:
            out += [new(nb), new(nb), new(G.nnz_j)]
            pf.pf_jacobian_values(G, method, vm, va, *out[-3:])
        for layout, buf in zip((pf.PF_PHASOR_SPLIT, pf.PF_PHASOR_INTERLEAVED), ph):
            out += [new(nb), new(nb), new(G.nnz_j)]
            pf.pf_ybus_from_phasors(G, layout, nstate, buf, *out[-3:])
        torch.cuda.synchronize()
        want = want or out
        assert all(torch.equal(a, b) for a, b in zip(out, want)), (spb, order)


# States below, at and past a thread's four; positions outside the target are
# skipped and entries that J does not cover stay as they are.
@pytest.mark.parametrize("nb,nstate", [(3, 1), (40, 4), (41, 5), (700, 3), (701, 13)])
def test_scatter_states_and_skips(nb, nstate):
    import torch
    _gpu.require_gpu()
    G = pf.Grid.from_grid(gridgen.make_grid(nb, max(nb - 1, int(1.3 * nb)), 0.15, case=9, grid=nb))
    rng = np.random.default_rng(nb)
    out_nnz = G.nnz_j + 37
    pos = rng.permutation(out_nnz)[:G.nnz_j].astype(np.int32)
    pos[::11] = -1
    pos[5::13] = out_nnz
    jval = rng.standard_normal((nstate, G.nnz_j))
    want = np.full((nstate, out_nnz), -7.0)
    ok = (pos >= 0) & (pos < out_nnz)
    want[:, pos[ok]] = jval[:, ok]
    out = torch.full((nstate, out_nnz), -7.0, dtype=torch.float64, device="cuda:0")
    pf.pf_jacobian_scatter(G, _gpu.to_dev(jval), torch.as_tensor(pos, device="cuda:0"), out)
    assert np.array_equal(out.cpu().numpy(), want)


# The same above 48 MB of targets, where stores of positions that lie apart are
# plain ones and others streaming ones.
@pytest.mark.parametrize("nb,nstate", [(12_000, 43), (101_001, 5)])
@pytest.mark.parametrize("apart", [True, False])
def test_scatter_into_large_targets(nb, nstate, apart):
    import torch
    _gpu.require_gpu()
    G = pf.Grid.from_grid(gridgen.make_grid(nb, int(1.3 * nb), 0.15, case=9, grid=nb))
    rng = np.random.default_rng(nb)
    out_nnz = G.nnz_j + G.nnz_j // 12
    pos = rng.permutation(out_nnz)[:G.nnz_j].astype(np.int32)
    if not apart:
        pos.sort()
        pos[64 * 1_001:64 * 1_002] = pos[64 * 1_001:64 * 1_002][::-1]
    pos[::11] = -1
    pos[5::13] = out_nnz
    pos, jval = torch.as_tensor(pos, device="cuda:0"), torch.randn((nstate, G.nnz_j), dtype=torch.float64, device="cuda:0")
    want = torch.full((nstate, out_nnz), -7.0, dtype=torch.float64, device="cuda:0")
    ok = (pos >= 0) & (pos < out_nnz)
    want[:, pos[ok].long()] = jval[:, ok]
    out = torch.full((nstate, out_nnz), -7.0, dtype=torch.float64, device="cuda:0")
    pf.pf_jacobian_scatter(G, jval, pos, out)
    assert torch.equal(out, want)
