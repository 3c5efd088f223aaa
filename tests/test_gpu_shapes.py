"""Launch shapes of the kernels at their edges: block and group remainders, both sizes of
a dispatch rule, against the general path or the oracle."""
import numpy as np
import pytest

import lj_inputs as li
from helpers import gpu_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return gpu_device()


def _gas(n, L, seed, ntypes=1):
    """n atoms no closer than about 0.8 (a jittered lattice with sites taken out)."""
    g = np.random.default_rng(seed)
    m = int(np.ceil(n ** (1.0 / 3.0)))
    sites = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)
    sites = sites[np.sort(g.permutation(m ** 3)[:n])]
    x = (sites + 0.5 + g.uniform(-0.05, 0.05, (n, 3))) * (L / m)
    return x, g.integers(0, ntypes, n).astype(np.int32)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 128, 129, 193, 1000])
@pytest.mark.parametrize("ntypes", [1, 2])
def test_chained_step_block_shapes(dev, n, ntypes):
    """Chained steps in blocks of 64 atoms (the full workspace) and of 128 (twice the
    force workspace) and ljmd_md_step: positions, velocities, forces and the sums of the
    rows bitwise the same; the sums formed by the next launch equal to rounding."""
    import torch
    from paper_2109_09056_amd import _lib, md, ops
    L = np.array([11.0, 12.0, 13.0])
    x, ty = _gas(n, L, 5 + n, ntypes)
    eps, sig = ([1.0], [1.0]) if ntypes == 1 else ([1.0, 0.9, 1.1], [1.0, 0.95, 0.9])
    T = lambda a, d=torch.float64: torch.as_tensor(a, dtype=d, device=dev).contiguous()
    xs, _, ts, _, cs = ops.bin(L, 2.8, T(x), None, T(ty, torch.int32))
    nl = md.NeighborList(L, 2.8, ops.FULL, device=dev).build(xs, cs)
    v0 = T(np.random.default_rng(n).normal(size=(n, 3)))
    full = ops.workspace_bytes(ops.OP_MD_CHAIN, n)
    small = 2 * ops.workspace_bytes(ops.OP_FORCES, n)
    assert small <= full
    got = []
    for nbytes in (None, full, small):
        a = (L, ops.FP64, 2.5, T(eps), T(sig), xs, ts, nl.nbr, nl.nnbr, nl.maxn, 0.005, 1.3)
        v, F = v0.clone(), torch.empty_like(xs)
        if nbytes is None:
            x1, _, ev = ops.md_step(*a, v, F=F)
            got.append((x1, v, F, ev))
            continue
        ws = torch.empty(nbytes, dtype=torch.uint8, device=dev)
        lib, p = _lib.load(), lambda t: t.data_ptr()
        x1, ev, prev = torch.empty_like(xs), torch.empty(8, dtype=torch.float64, device=dev), \
            torch.empty(8, dtype=torch.float64, device=dev)
        box = _lib.make_box(L)
        st = torch.cuda.current_stream(dev).cuda_stream
        args = lambda half, out, vel, xn: (
            box, ops.FP64, 2.5, ntypes, p(a[3]), p(a[4]), n, p(xs), p(ts), p(nl.nbr), p(nl.nnbr),
            nl.maxn, 0.005, 1.3, p(vel), p(xn), 1, p(F), None, half, out, p(ws), nbytes, st)
        _lib.check(lib.ljmd_md_step_chained(*args(0, None, v, x1)), "chained")
        _lib.check(lib.ljmd_md_step_sums(n, 0, p(ws), nbytes, p(ev), st), "sums")
        # the next step's launch sums half 0 as well
        F1 = F.clone()
        _lib.check(lib.ljmd_md_step_chained(*args(1, p(prev), v.clone(), torch.empty_like(xs))),
                   "chained")
        scale = ev.abs().max().item()
        assert (prev - ev).abs().max().item() <= 1e-13 * max(scale, 1.0)
        got.append((x1, v, F1, ev))
    for other in got[1:]:
        assert all(torch.equal(s, t) for s, t in zip(got[0], other))


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("cells", [4, 10, 26])
def test_csr_teams_of_two_and_four_bitwise_tiled(dev, cells, prec):
    """CSR with teams of two and of four gives bitwise the tiled kernel's forces and
    per-atom energies at every size, one and two types."""
    import torch
    from paper_2109_09056_amd import md, ops
    for ntypes in (1, 2):
        w = li.Workload("t", 9, cells=cells, ntypes=ntypes)
        s = li.make_system(w)
        P = ops.FP64 if prec == "fp64" else ops.MIXED
        sim = md.LJSim(w.box, eps=s["eps"], sigma=s["sigma"], precision=P, device=dev)
        sim.load(s["x"], None, s["types"])
        a = (sim.L, P, 2.5, sim.eps, sim.sigma, sim.x, sim.types)
        F, e, _ = ops.compute_forces(*a[:2], ops.FULL, *a[2:], sim.nl.nbr, sim.nl.nnbr, sim.nl.maxn)
        off, csr = ops.list_to_csr(sim.nl.nbr, sim.nl.nnbr, sim.nl.maxn)
        for team in (2, 4):
            F2, e2, _ = ops.compute_forces_csr(*a, off, csr, team=team)
            assert torch.equal(F, F2) and torch.equal(e, e2), (ntypes, team)


# every length of the three passes (x rows of 4..128 complex points), both the whole-row
# (8) and the two-step transforms, grids narrower than a block's columns
FFT_GRIDS = [(8, 8, 8), (8, 8, 256), (16, 256, 8), (32, 32, 16), (128, 16, 64), (64, 128, 32),
             (256, 64, 128)]


@pytest.mark.parametrize("K", FFT_GRIDS)
def test_spme_grid_shapes_vs_oracle(dev, orc, K):
    """Reciprocal forces and energy on grids of every pass length against the reference
    steps (same grid and order): rounding only, 1e-11 of the largest force and of the
    energy as for the other grids."""
    import torch
    from paper_2109_09056_amd import ops
    L = np.array([11.0, 12.0, 13.0])
    g = np.random.default_rng(18)
    q = g.uniform(-1.5, 1.5, 777)
    q -= q.mean()
    x = li.random_gas(777, L, 41)
    T = lambda a: torch.as_tensor(a, dtype=torch.float64, device=dev)
    F, E = ops.spme_recip(L, li.EWALD_ALPHA, 4, K, T(x), T(q), want_energy=True)
    E_o, F_o = orc.spme_recip(x, q, L, li.EWALD_ALPHA, K, 4)
    E_o += orc.ewald_self(q, li.EWALD_ALPHA)
    assert np.abs(F.cpu().numpy() - F_o).max() <= 1e-11 * np.abs(F_o).max()
    assert E.item() == pytest.approx(E_o, rel=1e-11)


def _spme_min_bytes(n, npts):
    half = npts // 2 + npts // 8
    return npts * 8 + half * 16 + 3 * 256 * 8 + 8 * (-(-half // 512) + max(1, -(-n // 256))) + 256


@pytest.mark.parametrize("order,K,n", [(4, (8, 8, 8), 1), (4, (8, 16, 8), 300),
                                       (4, (64, 32, 64), 5000), (4, (128, 128, 64), 9000),
                                       (6, (128, 64, 128), 3000), (6, (16, 32, 8), 500),
                                       (8, (128, 64, 128), 2000)])
def test_spme_tiles_against_direct_spreading(dev, order, K, n):
    """Reciprocal forces and energy with the tiles' workspace (both tile shapes, empty and
    crowded tiles, tiles that are their own neighbour, particles on cell corners, outside
    the box and in any order) and with the smaller one (no tiles): rounding only, a few
    hundred additions per point: 1e-13 of the largest force, 1e-12 of the energy."""
    import torch
    from paper_2109_09056_amd import _lib, ops
    L = np.array([17.0, 16.0, 18.0])
    g = np.random.default_rng(n)
    x = g.uniform(0, 1, (n, 3)) * L
    x[: n // 3] = L * 0.4 + g.uniform(0, 1, (n // 3, 3))  # a clump
    x[n // 3: n // 3 + 20] = np.floor(x[n // 3: n // 3 + 20] / L * K) * (L / K)  # on grid points
    x[-1] = L * np.array([1.02, -0.03, 0.5])
    q = g.uniform(-1.0, 1.0, n)
    T = lambda a: torch.as_tensor(a, dtype=torch.float64, device=dev).contiguous()
    xt, qt = T(x), T(q)
    npts = K[0] * K[1] * K[2]
    full, small = ops.workspace_bytes(ops.OP_SPME, n, ncells=npts), _spme_min_bytes(n, npts)
    assert small < full
    lib, out = _lib.load(), []
    import ctypes
    Kc = (ctypes.c_int32 * 3)(*K)
    for nbytes in (full, small, small - 8):
        ws = torch.full((nbytes,), 255, dtype=torch.uint8, device=dev)  # NaN everywhere
        F = torch.empty_like(xt)
        e = torch.empty(1, dtype=torch.float64, device=dev)
        rc = lib.ljmd_spme_recip(_lib.make_box(L), li.EWALD_ALPHA, order, Kc, n, xt.data_ptr(),
                                 qt.data_ptr(), F.data_ptr(), e.data_ptr(), 0, ws.data_ptr(),
                                 nbytes, torch.cuda.current_stream(dev).cuda_stream)
        if nbytes < small:
            assert rc == _lib.EWORKSPACE
            continue
        _lib.check(rc, "spme")
        out.append((F.cpu().numpy(), e.item()))
    (Fa, ea), (Fb, eb) = out
    assert np.isfinite(Fa).all()
    # the forces of a few particles are differences of terms about |q| alpha^2 large
    scale = max(np.abs(Fb).max(), li.EWALD_ALPHA ** 2)
    assert np.abs(Fa - Fb).max() <= 1e-13 * scale * max(1.0, n / 100.0)
    assert ea == pytest.approx(eb, rel=1e-12)


@pytest.mark.parametrize("n", [1, 63, 65, 1000])
def test_bin_counts_any_order(dev, orc, n):
    """Cell sort of atoms in random order (every lane of a wavefront its own cell) and of
    atoms all in one cell."""
    import torch
    from paper_2109_09056_amd import ops
    L = np.array([20.0, 23.0, 26.0])
    for x in (li.random_gas(n, L, n), np.tile(L * 0.3, (n, 1))):
        xs, _, _, ids, cs = ops.bin(L, 2.8, torch.as_tensor(x, device=dev))
        nc = ops.grid(L, 2.8)
        c = np.minimum(np.floor(x / (L / nc)).astype(int), np.array(nc) - 1)
        cell = (c[:, 2] * nc[1] + c[:, 1]) * nc[0] + c[:, 0]
        want = np.lexsort((np.arange(n), cell))
        assert np.array_equal(ids.cpu().numpy(), want)
        assert np.array_equal(xs.cpu().numpy(), x[want])
        assert np.array_equal(cs.cpu().numpy()[:-1], np.searchsorted(cell[want], np.arange(np.prod(nc))))


@pytest.mark.parametrize("alpha", [0.05, 1.2, 2.4])
@pytest.mark.parametrize("n", [2, 65, 1000])
def test_ewald_real_tables(dev, orc, alpha, n):
    """Real-space forces and energy for alpha rc from 0.125 to 6 (the tables' intervals from
    a 1000th to a 20th of a unit), pairs from 1e-3 apart to the cutoff, against the direct
    sum at the pair kernels' bar (1e-12 of the largest), with and without energies."""
    import torch
    from paper_2109_09056_amd import md, ops
    L = np.array([11.0, 12.0, 13.0])
    x = li.random_gas(n, L, 7 + n)
    x[1] = x[0] + np.array([1e-3, 0.0, 0.0])
    x = np.mod(x, L)
    g = np.random.default_rng(n)
    q = g.uniform(-1.5, 1.5, n)
    T = lambda a: torch.as_tensor(a, dtype=torch.float64, device=dev).contiguous()
    xs, _, _, ids, cs = ops.bin(L, 2.8, T(x))
    qs = ops.gather_rows(ids, T(q))
    nl = md.NeighborList(L, 2.8, ops.FULL, device=dev).build(xs, cs)
    F, E = ops.ewald_real(L, alpha, 2.5, xs, qs, nl.nbr, nl.nnbr, nl.maxn, want_energy=True)
    F2, _ = ops.ewald_real(L, alpha, 2.5, xs, qs, nl.nbr, nl.nnbr, nl.maxn)
    e_o, F_o = orc.ewald_direct(x, q, L, alpha, 2.5)
    for f in (F, F2):
        fg = ops.scatter_rows(ids, f).cpu().numpy()
        assert np.abs(fg - F_o).max() <= 1e-12 * np.abs(F_o).max()
    assert abs(E.item() - e_o.sum()) <= 1e-12 * np.abs(e_o).sum()

@pytest.mark.parametrize("n,ntypes", [(1, 1), (127, 2), (129, 1), (1000, 2), (1000, 3)])
def test_vjp_and_sph_at_block_edges(dev, orc, n, ntypes):
    """VJP of the forces (teams of four; one lane for three types) and the SPH passes on
    sizes around a block, rows of 0 to a few dozen entries: gradients against the oracle's
    (1e-12 of the largest), densities and accelerations against its sums."""
    import torch
    from paper_2109_09056_amd import md, ops
    L = np.array([11.0, 12.0, 13.0])
    x, ty = _gas(n, L, 3 + n, ntypes)
    p = ntypes * (ntypes + 1) // 2
    eps, sig = np.linspace(0.9, 1.1, p), np.linspace(0.9, 1.0, p)
    T = lambda a, d=torch.float64: torch.as_tensor(np.ascontiguousarray(a), dtype=d, device=dev)
    xs, _, ts, ids, cs = ops.bin(L, 2.8, T(x), None, T(ty, torch.int32))
    nl = md.NeighborList(L, 2.8, ops.FULL, device=dev).build(xs, cs)
    g = np.random.default_rng(n).normal(size=(n, 3))
    gs = ops.gather_rows(ids, T(g))
    gx, ge, gsig = ops.force_backward(L, ops.FP64, 2.5, T(eps), T(sig), xs, ts, nl.nbr, nl.nnbr,
                                      nl.maxn, gs)
    gx_o, ge_o, gs_o = orc.force_vjp(x, L, 2.5, g, eps, sig, ty if ntypes > 1 else None)
    near = lambda a, b: np.abs(a - b).max() <= 1e-12 * max(np.abs(b).max(), 1e-30)
    assert near(ops.scatter_rows(ids, gx).cpu().numpy(), gx_o)
    assert near(ge.cpu().numpy(), ge_o) and near(gsig.cpu().numpy(), gs_o)
    if ntypes > 1:
        return
    rho, _ = ops.sph_density(L, 1.2, 1.0, 10.0, 1.0, xs, nl.nbr, nl.nnbr, nl.maxn)
    acc = ops.sph_accel(L, 1.2, 1.0, 10.0, 1.0, xs, rho, nl.nbr, nl.nnbr, nl.maxn)
    rho_o = orc.sph_density(x, L, 1.2, 1.0)
    acc_o = orc.sph_accel(x, L, 1.2, 1.0, 10.0, 1.0, rho_o)
    assert near(ops.scatter_rows(ids, rho).cpu().numpy(), rho_o)
    assert near(ops.scatter_rows(ids, acc).cpu().numpy(), acc_o)


@pytest.mark.parametrize("kind", ["full", "half"])
@pytest.mark.parametrize("per_cell", [3, 9, 17, 20, 21, 24, 29, 36, 60])
def test_lists_by_slot_count(dev, kind, per_cell):
    """Lists over stencils of 2 to 13 and more register slots (every slot count the build
    has code for, and the unstaged one), with pairs at the cutoff to rounding and coincident
    atoms, rows cut at half their length, and the compressed rows: against all pairs in
    FP64; compressed rows equal to the tiled ones entry by entry."""
    import torch
    from helpers import decode_rows
    from paper_2109_09056_amd import ops
    rl = 2.8
    L = np.full(3, 3 * rl * 1.01)
    n = per_cell * 27
    g = np.random.default_rng(per_cell)
    x = g.uniform(0, 1, (n, 3)) * L
    x[1] = x[0] + np.array([rl, 0.0, 0.0])  # at the cutoff, to rounding
    x[2] = x[0] + np.array([0.0, rl * (1 - 1e-9), 0.0])
    x[3] = x[0]  # coincident atoms are neighbours
    x = np.mod(x, L)
    k = ops.FULL if kind == "full" else ops.HALF
    xs, _, _, ids, cs = ops.bin(L, rl, torch.as_tensor(x, device=dev))
    X = xs.cpu().numpy()
    d = X[:, None, :] - X[None, :, :]
    d = np.where(d > L / 2, d - L, np.where(d < -L / 2, d + L, d))
    r2 = (d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1]) + d[..., 2] * d[..., 2]
    hit = r2 < rl * rl
    np.fill_diagonal(hit, False)
    if kind == "half":
        hit = np.triu(hit)
    most = int(hit.sum(1).max())
    for maxn in (most, max(1, most // 2), most + 200):
        nbr, nnbr, mc = ops.build_neighbors(L, rl, k, xs, cs, maxn)
        assert int(mc.item()) == most
        rows = decode_rows(nbr.cpu().numpy(), nnbr.cpu().numpy(), maxn)
        for i, row in enumerate(rows):
            want = np.flatnonzero(hit[i])
            assert row.size == min(want.size, maxn)
            assert np.isin(row, want).all() and np.unique(row).size == row.size
        if maxn >= most:
            full = rows
    off, csr = ops.build_neighbors_csr(L, rl, k, xs, cs)
    off, csr = off.cpu().numpy(), csr.cpu().numpy()
    assert off[-1] == hit.sum()
    for i, row in enumerate(full):
        assert np.array_equal(csr[off[i]:off[i + 1]], row)
    # too small a capacity: the entries below it are the same
    cap = int(off[-1]) // 2
    off2, csr2 = ops.build_neighbors_csr(L, rl, k, xs, cs, cap=cap,
                                         csr=torch.full((cap,), -7, dtype=torch.int32, device=dev))
    assert np.array_equal(off2.cpu().numpy(), off)
    assert np.array_equal(csr2.cpu().numpy(), csr[:cap])


@pytest.mark.parametrize("nsteps", [1, 2, 3, 6])
@pytest.mark.parametrize("open_last", [True, False])
def test_md_steps_match_single_calls(dev, nsteps, open_last):
    """One call of several chained steps gives bitwise the positions, velocities, forces and
    sums of as many single ones, started fresh and after a chained step, and leaves the
    newest positions where it says."""
    import torch
    from paper_2109_09056_amd import md, ops
    L = np.array([11.0, 12.0, 13.0])
    n = 700
    x, ty = _gas(n, L, 77)
    T = lambda a, d=torch.float64: torch.as_tensor(a, dtype=d, device=dev).contiguous()
    xs, _, ts, _, cs = ops.bin(L, 2.8, T(x), None, T(ty, torch.int32))
    nl = md.NeighborList(L, 2.8, ops.FULL, device=dev).build(xs, cs)
    one = T([1.0])
    v0 = T(np.random.default_rng(1).normal(size=(n, 3)))
    a = lambda xx: (L, ops.MIXED, 2.5, one, one, xx)
    b = (ts, nl.nbr, nl.nnbr, nl.maxn, 0.005, 1.0)
    nb = ops.workspace_bytes(ops.OP_MD_CHAIN, n)
    out = []
    for native in (False, True):
        cur, alt, v, F = xs.clone(), torch.empty_like(xs), v0.clone(), torch.empty_like(xs)
        ws, ev = torch.empty(nb, dtype=torch.uint8, device=dev), T(np.zeros(8))
        ops.md_step_chained(*a(cur), *b, v, 1, ws, x_next=alt)  # half 1
        cur, alt = alt, cur
        if native:
            cur, alt = ops.md_steps(*a(cur), alt, *b, v, nsteps, 0, ws, ev, chained=True,
                                    open_last=open_last, F=F)
        else:
            for s in range(nsteps):
                op = open_last or s < nsteps - 1
                ops.md_step_chained(*a(cur), *b, v, s % 2, ws, x_next=alt, open_next=op, F=F,
                                    ev_prev=ev)
                if op:
                    cur, alt = alt, cur
        out.append((cur, v, F, ev, ops.md_step_sums(n, (nsteps - 1) % 2, ws)))
    assert all(torch.equal(p, q) for p, q in zip(*out))
    with pytest.raises(Exception):
        ops.md_steps(*a(xs), xs, *b, v0, 1, 0, ws, ev)  # aliased buffers


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 1024, 1025, 3000])
@pytest.mark.parametrize("maxn", [1, 15, 16, 17, 33])
def test_list_to_csr_shapes(dev, n, maxn):
    """Tiled rows of every length (also counted past their capacity) to compressed ones,
    whole and with half the room: equal entry by entry, nothing written past the room."""
    import torch
    from paper_2109_09056_amd import ops
    g = np.random.default_rng(n + 1000 * maxn)
    nbr = g.integers(0, n, ((n + 63) // 64, maxn, 64)).astype(np.int32)
    nnbr = g.integers(0, maxn + 4, n).astype(np.int32)
    c = np.minimum(nnbr, maxn)
    off = np.concatenate([[0], np.cumsum(c)])
    rows = np.concatenate([nbr[i // 64, :c[i], i % 64] for i in range(n)])
    for cap in (rows.size, rows.size // 2):
        out = torch.full((rows.size + 8,), -7, dtype=torch.int32, device=dev)
        o, _ = ops.list_to_csr(torch.as_tensor(nbr, device=dev).reshape(-1),
                               torch.as_tensor(nnbr, device=dev), maxn, cap=cap, csr=out)
        assert np.array_equal(o.cpu().numpy(), off)
        got = out.cpu().numpy()
        assert np.array_equal(got[:cap], rows[:cap]) and (got[cap:] == -7).all()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("ntypes", [1, 2])
@pytest.mark.parametrize("n", [1, 127, 129, 3001, 32768, 32769, 33001])
def test_half_list_block_shapes(dev, n, ntypes, prec):
    """Half-list forces, per-atom energies and sums against the full list's over block and
    group remainders and both sides of the small-grid line.  The two add the same pairs in
    other orders in FP64 (a mixed pair is the same number in both): each side is within (row
    length) rounding errors of a sum of terms whose magnitudes stay under the bound below."""
    import torch
    from paper_2109_09056_amd import md, ops
    L = np.full(3, max(1.1 * n ** (1.0 / 3.0), 8.5))
    x, types = _gas(n, L[0], n, ntypes)
    eps = np.array([1.0, 0.8, 1.3])[: ntypes * (ntypes + 1) // 2]
    sig = np.array([1.0, 0.95, 0.9])[: ntypes * (ntypes + 1) // 2]
    T = lambda a, d=torch.float64: torch.as_tensor(a, dtype=d, device=dev).contiguous()
    xs, _, ts, _, cs = ops.bin(L, 2.8, T(x), None, T(types, torch.int32))
    P = ops.FP64 if prec == "fp64" else ops.MIXED
    out = []
    for kind in (ops.FULL, ops.HALF):
        nl = md.NeighborList(L, 2.8, kind, device=dev).build(xs, cs)
        for energy in (True, False):
            out.append(ops.compute_forces(L, P, kind, 2.5, T(eps), T(sig), xs, ts, nl.nbr,
                                          nl.nnbr, nl.maxn, want_energy=energy))
    (F, e, ev), _, (Fh, eh, evh), (Fh0, _, _) = [
        tuple(t.cpu().numpy() if t is not None else None for t in o) for o in out]
    unit = 2.0 ** -52
    # 48 eps sigma^-1 (sigma/r)^13 at the closest 0.8 or more; fewer than 200 neighbours
    big = 48 * 1.3 * (1 / 0.8) ** 13 * 1.1
    assert np.abs(Fh - F).max() <= 200 * unit * big
    assert np.abs(Fh0 - F).max() <= 200 * unit * big
    assert np.abs(eh - e).max() <= 200 * unit * big
    assert np.abs(evh - ev).max() <= 200 * unit * big * max(n, 1)


@pytest.mark.parametrize("cells", [(3, 3, 3), (16, 16, 15), (16, 16, 16), (17, 16, 16),
                                   (32, 16, 16), (29, 29, 29)])
def test_bin_starts_over_scan_chunks(dev, cells):
    """Row starts of grids below, at and above one and several scan chunks."""
    import torch
    from paper_2109_09056_amd import ops
    L = 2.8 * 1.001 * np.array(cells, float)
    x = np.random.default_rng(cells[0]).uniform(0, 1, (5000, 3)) * L
    _, _, _, ids, cs = ops.bin(L, 2.8, torch.as_tensor(x, device=dev))
    assert tuple(ops.grid(L, 2.8)) == cells
    c = np.minimum(np.floor(x / (L / cells)).astype(int), np.array(cells) - 1)
    cell = (c[:, 2] * cells[1] + c[:, 1]) * cells[0] + c[:, 0]
    want = np.lexsort((np.arange(5000), cell))
    assert np.array_equal(ids.cpu().numpy(), want)
    assert np.array_equal(cs.cpu().numpy(),
                          np.searchsorted(cell[want], np.arange(np.prod(cells) + 1)))


@pytest.mark.parametrize("kind", ["full", "half"])
@pytest.mark.parametrize("per_cell", [1, 9, 17, 24, 29, 45])
@pytest.mark.parametrize("nc", [2, 3, 4])
def test_compressed_rows_with_and_without_hits(dev, kind, per_cell, nc):
    """Compressed rows with the full workspace (the filling pass reads the counting pass's
    hits) and with the smallest (it tests again): equal, also where cap cuts them; atoms
    outside the box and empty cells too (stencils that the integer test does not take)."""
    import torch
    from paper_2109_09056_amd import _lib, ops
    rl, k = 2.8, ops.FULL if kind == "full" else ops.HALF
    L = np.full(3, nc * rl * 1.01)
    n = per_cell * nc ** 3
    x = np.random.default_rng(per_cell).uniform(0, 1, (n, 3)) * L
    for outside in (False, True):
        xs, _, _, _, cs = ops.bin(L, rl, torch.as_tensor(x, device=dev))
        if outside:
            xs[n // 2] += torch.as_tensor(1.5 * L, device=dev)
        small = -(-4 * n // 256) * 256 + ops.workspace_bytes(ops.OP_CSR, n)
        full = ops.workspace_bytes(ops.OP_BUILD_CSR, n)
        assert small < full
        got = []
        for nbytes in (full, small):
            for part in (1, 2):
                off = torch.empty(n + 1, dtype=torch.int64, device=dev)
                csr = torch.full((n * n // part + 1,), -7, dtype=torch.int32, device=dev)
                cap = csr.numel() if part == 1 else int(got[0][0][-1]) // 2
                ws = torch.empty(nbytes, dtype=torch.uint8, device=dev)
                _lib.check(_lib.load().ljmd_build_neighbors_csr(
                    _lib.make_box(L), rl, k, n, xs.data_ptr(), cs.data_ptr(), off.data_ptr(),
                    csr.data_ptr(), cap, ws.data_ptr(), nbytes,
                    torch.cuda.current_stream(dev).cuda_stream), "build")
                got.append((off.cpu().numpy(), csr.cpu().numpy(), cap))
        for off, csr, cap in got:
            assert np.array_equal(off, got[0][0])
            m = min(cap, off[-1])
            assert np.array_equal(csr[:m], got[2][1][:m]) and (csr[m:] == -7).all()


@pytest.mark.parametrize("K", [(256, 256, 128), (256, 256, 256)])
def test_spme_tiles_of_large_grids(dev, K):
    """4,096 tiles (ordered in one launch) and 8,192 (scanned first)."""
    test_spme_tiles_against_direct_spreading(dev, 4, K, 3000)
