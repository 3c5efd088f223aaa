"""Both sides of rules that send a call to one of several kernels: against the oracle, or
against the general path on the same input."""
import numpy as np
import pytest

import lj_inputs as li
from helpers import gpu_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return gpu_device()


def _t(dev):
    import torch
    return lambda a, d=torch.float64: torch.as_tensor(np.ascontiguousarray(a), dtype=d, device=dev)


@pytest.mark.parametrize("far", [False, True])
@pytest.mark.parametrize("arc", [0.125, 1.5, 3.0, 3.4999, 3.5001, 6.0, 10.0])
def test_ewald_real_isolated_pairs(dev, orc, arc, far):
    """Real-space force of isolated pairs, each to the accuracy of its own value, with and
    without energies, and the energy; radii at the middle and both edges of every 128th of
    the cutoff (far: of those beyond 0.8 rc).  Bound: r^2 carries 2 roundings and x = alpha r
    half of them and 2 more, which enter the force 2 x^2 times over, the other factors 8, on
    either side; and the remainder of the polynomials of erfcx, (half an interval)^11 erfcx^(11)
    / 11! with erfcx^(11) / 11! at most 1 / Gamma(6.5), the largest at 0."""
    import torch
    from paper_2109_09056_amd import md, ops
    rc, m = 2.5, 8
    L = np.full(3, 8.0 * m)
    g = np.random.default_rng(int(100 * arc))
    frac = (np.arange(128)[:, None] + np.array([1e-9, 0.5, 1 - 1e-9])).reshape(-1)
    frac[0] = 0.02
    if far:
        frac = frac[frac > 0.8 * 128]
    r = rc * frac / 128.0
    sites = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)
    d = g.normal(size=(r.size, 3))
    d *= (r / np.linalg.norm(d, axis=1))[:, None]
    a = 8.0 * sites[: r.size] + 4.0
    x = np.concatenate([a, a + d])
    q = g.uniform(0.5, 1.5, 2 * r.size)
    T = _t(dev)
    xs, _, _, ids, cs = ops.bin(L, 2.8, T(x))
    qs = ops.gather_rows(ids, T(q))
    nl = md.NeighborList(L, 2.8, ops.FULL, device=dev).build(xs, cs)
    alpha = arc / rc
    F, E = ops.ewald_real(L, alpha, rc, xs, qs, nl.nbr, nl.nnbr, nl.maxn, want_energy=True)
    F2, _ = ops.ewald_real(L, alpha, rc, xs, qs, nl.nbr, nl.nnbr, nl.maxn)
    e_o, F_o = orc.ewald_direct(x, q, L, alpha, rc)
    near = np.linalg.norm(F_o, axis=1) > 0  # radii that round to the cutoff do not count
    assert near.sum() >= 2 * r.size - 2
    u = 2.0 ** -53
    xa = alpha * np.concatenate([r, r])
    rest = (arc / 64.0) ** 11 / 287.0
    tol = 2 * u * (8 + 2 * 3 * xa ** 2) + rest
    for f in (F, F2):
        err = np.linalg.norm(ops.scatter_rows(ids, f).cpu().numpy() - F_o, axis=1)
        assert (err <= tol * np.linalg.norm(F_o, axis=1)).all(), (err / tol)[near].max()
    assert abs(E.item() - e_o.sum()) <= tol.max() * e_o.sum()


def _recip(L, order, K, xt, qt, ws):
    """Reciprocal forces and energy through the C ABI with exactly this workspace."""
    import ctypes

    import torch
    from paper_2109_09056_amd import _lib
    F, e = torch.empty_like(xt), torch.empty(1, dtype=torch.float64, device=xt.device)
    _lib.check(_lib.load().ljmd_spme_recip(
        _lib.make_box(L), li.EWALD_ALPHA, order, (ctypes.c_int32 * 3)(*K), xt.shape[0],
        xt.data_ptr(), qt.data_ptr(), F.data_ptr(), e.data_ptr(), 0, ws.data_ptr(), ws.numel(),
        torch.cuda.current_stream(xt.device).cuda_stream), "spme")
    return F, e


def _spme_direct_bytes(n, npts):
    """The workspace without the tiles' part: charge is spread by atomics."""
    half = npts // 2 + npts // 8
    return npts * 8 + half * 16 + 3 * 256 * 8 + 8 * (-(-half // 512) + max(1, -(-n // 256))) + 256


@pytest.mark.parametrize("order,K,n", [(4, (32, 16, 64), 1025), (4, (64, 32, 64), 9000),
                                       (4, (128, 128, 64), 9000), (6, (128, 64, 128), 5000),
                                       (4, (256, 256, 256), 40000), (4, (8, 8, 8), 3000)])
def test_spme_crowded_tiles(dev, order, K, n):
    """Clumps in single tiles, over tile faces and box faces, next to sparse tiles, charges
    in random order: forces and energy with the tiles against those without, which differ in
    the order of at most n additions per grid point, as in the test of sparser tiles."""
    import torch
    from paper_2109_09056_amd import ops
    L = np.array([17.0, 16.0, 18.0])
    g = np.random.default_rng(n + order)
    h = L / K
    x = g.uniform(0, 1, (n, 3)) * L
    x[: n // 2] = L * 0.4 + 2.0 * h * g.uniform(0, 1, (n // 2, 3))  # inside a tile, or two
    x[n // 2: 3 * n // 4] = np.mod(3.0 * h * g.uniform(-1, 1, (n // 4 + n % 4, 3))[: 3 * n // 4 - n // 2], L)
    x = x[g.permutation(n)]
    q = g.uniform(-1.0, 1.0, n)
    T = _t(dev)
    xt, qt, npts = T(x), T(q), K[0] * K[1] * K[2]
    out = []
    for nbytes in (ops.workspace_bytes(ops.OP_SPME, n, ncells=npts), _spme_direct_bytes(n, npts)):
        ws = torch.full((nbytes,), 255, dtype=torch.uint8, device=dev)  # NaN everywhere
        F, e = _recip(L, order, K, xt, qt, ws)
        out.append((F.cpu().numpy(), e.item()))
    (Fa, ea), (Fb, eb) = out
    assert np.isfinite(Fa).all()
    scale = max(np.abs(Fb).max(), li.EWALD_ALPHA ** 2)
    assert np.abs(Fa - Fb).max() <= 1e-13 * scale * n / 100.0
    assert ea == pytest.approx(eb, rel=1e-12)


def _milliseconds(f, reps=5):
    import torch
    f()
    best = float("inf")
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


def test_spme_droplet_uses_the_chip(dev):
    """262,144 charges in an eighth of the edge of a 64^3 grid: with the tiles no more than
    twice as long as without them (a block per tile, whatever it holds, took 12 times)."""
    import torch
    from paper_2109_09056_amd import ops
    n, K, L = 262144, (64, 64, 64), np.full(3, 32.0)
    x = (0.1 + 0.125 * np.random.default_rng(3).uniform(0, 1, (n, 3))) * L
    x = x[np.lexsort(np.floor(x).T)]
    T = _t(dev)
    xt, qt, npts = T(x), T(np.where(np.arange(n) % 2, 1.0, -1.0)), 64 ** 3
    t = [_milliseconds(lambda: _recip(L, 4, K, xt, qt, ws)) for ws in
         (torch.empty(b, dtype=torch.uint8, device=dev)
          for b in (ops.workspace_bytes(ops.OP_SPME, n, ncells=npts), _spme_direct_bytes(n, npts)))]
    assert t[0] <= 2.0 * t[1], t


@pytest.mark.parametrize("cells", [(40, 40, 40), (41, 40, 40), (64, 64, 64), (101, 103, 107),
                                   (256, 256, 256)])
def test_bin_starts_of_sparse_grids(dev, cells):
    """Row starts and order on both sides of 65,536 cells, where the scan changes form,
    and over several chunks per thread of its middle pass."""
    import torch
    from paper_2109_09056_amd import ops
    L = 2.8 * 1.001 * np.array(cells, float)
    n = 7000
    x = np.random.default_rng(cells[0]).uniform(0, 1, (n, 3)) * L
    x[: n // 2] *= 0.01  # most of the first cells crowded, most cells empty
    _, _, _, ids, cs = ops.bin(L, 2.8, torch.as_tensor(x, device=dev))
    assert tuple(ops.grid(L, 2.8)) == cells
    c = np.minimum(np.floor(x / (L / cells)).astype(np.int64), np.array(cells) - 1)
    cell = (c[:, 2] * cells[1] + c[:, 1]) * cells[0] + c[:, 0]
    want = np.lexsort((np.arange(n), cell))
    assert np.array_equal(ids.cpu().numpy(), want)
    starts = np.concatenate([[0], np.cumsum(np.bincount(cell, minlength=int(np.prod(cells))))])
    assert np.array_equal(cs.cpu().numpy(), starts)


def test_bin_work_is_linear_in_the_cells(dev):
    """Eight times the cells may take at most sixteen times as long (a scan that sums all
    counts before each chunk took 37 times)."""
    import torch
    from paper_2109_09056_amd import ops
    t = []
    for m in (128, 256):
        L = np.full(3, 2.81 * m)
        x = torch.rand(1000, 3, dtype=torch.float64, device=dev) * L[0]
        out = ops.bin(L, 2.8, x)
        ws = torch.empty(ops.workspace_bytes(ops.OP_BIN, 1000, ncells=m ** 3), dtype=torch.uint8,
                         device=dev)
        t.append(_milliseconds(lambda: ops.bin(L, 2.8, x, out=out[:4], cell_start=out[4], ws=ws)))
    assert t[1] <= 16.0 * t[0], t


@pytest.mark.parametrize("kind", ["full", "half"])
@pytest.mark.parametrize("maxn", [128, 400])
@pytest.mark.parametrize("nc", [25, 26])
def test_lists_of_gases_on_large_grids(dev, orc, kind, maxn, nc):
    """Tiled and compressed lists on both sides of 16,384 cells (15,625 and 17,576), where
    the build has code for stencils of few slots: a gas of one or two, with clumps that bring
    every slot count up to the unstaged path, both build shapes; row by row against the
    oracle's lists, the compressed rows with and without the noted hits."""
    import torch
    from helpers import decode_rows
    from paper_2109_09056_amd import _lib, ops
    rl = 2.8
    L = np.full(3, nc * rl * 1.0005)
    g = np.random.default_rng(nc + maxn)
    clumps = [c + rl * g.uniform(-1.2, 1.2, (m, 3))
              for c, m in zip(g.uniform(0, 1, (16, 3)) * L, 60 * np.arange(1, 17))]
    x = np.mod(np.concatenate([g.uniform(0, 1, (12000, 3)) * L] + clumps), L)
    n, T = len(x), _t(dev)
    k = ops.FULL if kind == "full" else ops.HALF
    xs, _, _, ids, cs = ops.bin(L, rl, T(x))
    order = ids.cpu().numpy()
    off_o, nbr_o = orc.neighbor_lists(x[order], L, rl)
    want = [np.sort(nbr_o[a:b]) for a, b in zip(off_o[:-1], off_o[1:])]
    if kind == "half":
        want = [w[w > i] for i, w in enumerate(want)]
    nbr, nnbr, most = ops.build_neighbors(L, rl, k, xs, cs, maxn)
    assert int(most.item()) == max(map(len, want))
    rows = decode_rows(nbr.cpu().numpy(), nnbr.cpu().numpy(), maxn)
    for row, w in zip(rows, want):
        if len(w) <= maxn:
            assert np.array_equal(np.sort(row), w)
        else:
            assert len(row) == maxn and np.isin(row, w).all()
    for nbytes in (ops.workspace_bytes(ops.OP_BUILD_CSR, n),
                   -(-4 * n // 256) * 256 + ops.workspace_bytes(ops.OP_CSR, n)):
        off = torch.empty(n + 1, dtype=torch.int64, device=dev)
        csr = torch.full((sum(map(len, want)),), -7, dtype=torch.int32, device=dev)
        ws = torch.empty(nbytes, dtype=torch.uint8, device=dev)
        _lib.check(_lib.load().ljmd_build_neighbors_csr(
            _lib.make_box(L), rl, k, n, xs.data_ptr(), cs.data_ptr(), off.data_ptr(),
            csr.data_ptr(), csr.numel(), ws.data_ptr(), nbytes,
            torch.cuda.current_stream(dev).cuda_stream), "build")
        assert np.array_equal(np.diff(off.cpu().numpy()), [len(w) for w in want])
        c = np.split(csr.cpu().numpy(), off.cpu().numpy()[1:-1])
        assert all(np.array_equal(np.sort(a), w) for a, w in zip(c, want))


@pytest.mark.parametrize("ntypes", [1, 2])
@pytest.mark.parametrize("rows", ["short", "long"])
def test_csr_teams_over_ragged_rows(dev, ntypes, rows):
    """Every team size, with and without energies, over rows of every length (0 to about 20
    entries, and to 90): teams of two and four bitwise the tiled kernel's forces, the others
    the same pairs in another order, so within (row length) roundings of the largest term."""
    import torch
    from paper_2109_09056_amd import md, ops
    n = 3001
    L = np.full(3, 40.0 if rows == "short" else 19.0)
    g = np.random.default_rng(ntypes)
    m = int(np.ceil(n ** (1.0 / 3.0)))
    sites = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)
    x = (sites[g.permutation(m ** 3)[:n]] + 0.5 + g.uniform(-0.1, 0.1, (n, 3))) * (L / m)
    x[: n // 3] = 0.5 * x[: n // 3] + 0.25 * L  # denser in the middle
    T = _t(dev)
    xs, _, ts, _, cs = ops.bin(L, 2.8, T(x), None, T(g.integers(0, ntypes, n), torch.int32))
    nl = md.NeighborList(L, 2.8, ops.FULL, device=dev).build(xs, cs)
    off, csr = ops.list_to_csr(nl.nbr, nl.nnbr, nl.maxn)
    p = ntypes * (ntypes + 1) // 2
    for P in (ops.FP64, ops.MIXED):
        a = (L, P, 2.5, T([1.0, 0.9, 1.1][:p]), T([0.4, 0.38, 0.42][:p]), xs, ts)
        F, e, ev = (t.cpu().numpy() for t in ops.compute_forces(
            *a[:2], ops.FULL, *a[2:], nl.nbr, nl.nnbr, nl.maxn))
        big = np.abs(F).max()
        for team in (1, 2, 4, 8, 16):
            for want in (True, False):
                F2, e2, ev2 = ops.compute_forces_csr(*a, off, csr, team=team, want_energy=want)
                F2 = F2.cpu().numpy()
                tol = 0.0 if team in (2, 4) else 200 * 2.0 ** -53 * 100 * big
                assert np.abs(F2 - F).max() <= tol, (team, want)
                if want:
                    assert np.abs(e2.cpu().numpy() - e).max() <= tol * 2.5
                    assert np.abs(ev2.cpu().numpy() - ev).max() <= 1e-11 * np.abs(ev).max()


def _ragged(n, L, seed):
    """n atoms of a jittered lattice with sites taken out, the first third of them drawn in
    towards the middle: rows from empty to several times the mean."""
    g = np.random.default_rng(seed)
    m = int(np.ceil(n ** (1.0 / 3.0)))
    sites = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)
    x = (sites[g.permutation(m ** 3)[:n]] + 0.5 + g.uniform(-0.1, 0.1, (n, 3))) * (L / m)
    x[: n // 3] = 0.5 * x[: n // 3] + 0.25 * L
    return x


@pytest.mark.parametrize("edge", [20.0, 40.0])
@pytest.mark.parametrize("ntypes", [3, 8])
def test_vjp_of_many_types_over_ragged_rows(dev, orc, ntypes, edge):
    """VJP with three and eight types over rows of every remainder of a group of slots,
    against the oracle's (1e-12 of the largest)."""
    import torch
    from paper_2109_09056_amd import md, ops
    n, L = 1500, np.full(3, edge)
    x, g = _ragged(n, L, ntypes), np.random.default_rng(ntypes)
    ty = g.integers(0, ntypes, n)
    p = ntypes * (ntypes + 1) // 2
    eps, sig = np.linspace(0.8, 1.2, p), np.linspace(0.35, 0.45, p)
    T = _t(dev)
    xs, _, ts, ids, cs = ops.bin(L, 2.8, T(x), None, T(ty, torch.int32))
    nl = md.NeighborList(L, 2.8, ops.FULL, device=dev).build(xs, cs)
    c = g.normal(size=(n, 3))
    gx, ge, gs = ops.force_backward(L, ops.FP64, 2.5, T(eps), T(sig), xs, ts, nl.nbr, nl.nnbr,
                                    nl.maxn, ops.gather_rows(ids, T(c)))
    want = orc.force_vjp(x, L, 2.5, c, eps, sig, ty.astype(np.int32))
    for a, b in zip((ops.scatter_rows(ids, gx), ge, gs), want):
        assert np.abs(a.cpu().numpy() - b).max() <= 1e-12 * np.abs(b).max()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("ntypes", [1, 2])
def test_vjp_on_both_sides_of_the_short_row_line(dev, ntypes, prec):
    """The same rows in lists of capacity 64 (two lanes per atom beyond 65,536 atoms) and 65
    (four, which other tests hold against the oracle).  The terms are the same numbers in
    either: a row's sum of at most 64 differs by 64 roundings of its terms, a parameter's
    by as many as it has terms."""
    import torch
    from paper_2109_09056_amd import ops
    n, L = 66001, np.full(3, 110.0)
    x, g = _ragged(n, L, ntypes), np.random.default_rng(ntypes)
    p = ntypes * (ntypes + 1) // 2
    T = _t(dev)
    xs, _, ts, _, cs = ops.bin(L, 2.8, T(x), None, T(g.integers(0, ntypes, n), torch.int32))
    c = T(g.normal(size=(n, 3)))
    out = []
    for maxn in (64, 65):
        nbr, nnbr, most = ops.build_neighbors(L, 2.8, ops.FULL, xs, cs, maxn)
        assert int(most.item()) <= 64
        out.append([t.cpu().numpy() for t in ops.force_backward(
            L, ops.FP64 if prec == "fp64" else ops.MIXED, 2.5, T(np.linspace(0.8, 1.2, p)),
            T(np.linspace(0.35, 0.45, p)), xs, ts, nbr, nnbr, maxn, c)])
    (gx, ge, gs), (hx, he, hs) = out
    u = 2.0 ** -53
    assert np.abs(gx - hx).max() <= 2 * 64 * u * np.abs(hx).max()
    assert np.abs(ge - he).max() <= 2 * 64 * n * u * np.abs(he).max()
    assert np.abs(gs - hs).max() <= 2 * 64 * n * u * np.abs(hs).max()


@pytest.mark.parametrize("n", [1, 130, 3001])
def test_gas_rows_bitwise_the_general_path(dev, n):
    """Lists of small capacity leave out the gathers of absent slots (forces without energies
    up to 20 and, with two types or more, 28 entries; SPH densities up to 24, accelerations
    up to 28): bitwise the results over the same rows in a list of larger capacity."""
    import torch
    from paper_2109_09056_amd import ops
    L = np.full(3, 60.0)
    T, g = _t(dev), np.random.default_rng(n)
    xs, _, ts, _, cs = ops.bin(L, 2.8, T(_ragged(n, L, n)), None, T(g.integers(0, 2, n), torch.int32))
    lists = {}
    for maxn in (20, 24, 28, 40):
        nbr, nnbr, most = ops.build_neighbors(L, 2.8, ops.FULL, xs, cs, maxn)
        assert int(most.item()) <= 20
        lists[maxn] = (nbr, nnbr, maxn)
    rho = T(g.uniform(0.5, 1.5, n))

    def results(l):
        out = []
        for P in (ops.FP64, ops.MIXED):
            for eps, sig in (([1.0], [0.4]), ([1.0, 0.9, 1.1], [0.4, 0.38, 0.42])):
                out.append(ops.compute_forces(L, P, ops.FULL, 2.5, T(eps), T(sig), xs, ts, *l,
                                              want_energy=False)[0])
        out += ops.sph_density(L, 1.2, 1.0, 10.0, 1.0, xs, *l, want_energy=True)
        out.append(ops.sph_accel(L, 1.2, 1.0, 10.0, 1.0, xs, rho, *l))
        out += ops.sph_accel_step(L, 1.2, 1.0, 10.0, 1.0, xs.clone(), torch.ones_like(xs), rho, *l,
                                  1e-3)
        return out

    want = results(lists[40])
    for maxn in (20, 24, 28):
        assert all(torch.equal(a, b) for a, b in zip(results(lists[maxn]), want)), maxn


@pytest.mark.parametrize("order", [4, 8])
def test_smaller_workspaces_are_used_as_given(dev, order):
    """Workspaces of the smallest sizes (the full ones of earlier versions) passed to the
    Python calls: used, with nothing allocated in their place, to the same results; order 8,
    which never uses the tiles, allocates no more than that by itself."""
    import torch
    from paper_2109_09056_amd import ops
    n, L, K = 5000, np.full(3, 20.0), (32, 32, 32)
    T, g = _t(dev), np.random.default_rng(order)
    xs, _, ts, _, cs = ops.bin(L, 2.8, T(g.uniform(0, 1, (n, 3)) * L), None,
                               torch.zeros(n, dtype=torch.int32, device=dev))
    q = T(np.where(np.arange(n) % 2, 1.0, -1.0))
    empty = lambda op, **kw: torch.empty(ops.workspace_bytes(op, n, **kw), dtype=torch.uint8,
                                         device=dev)

    def grown(f):
        """f() and the bytes it had allocated at its peak beyond what it returns."""
        torch.cuda.synchronize()
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        out = f()
        return out, torch.cuda.max_memory_allocated() - max(before, torch.cuda.memory_allocated())

    F, e = torch.empty_like(xs), torch.empty(1, dtype=torch.float64, device=dev)
    least = empty(ops.OP_SPME_LEAST, ncells=32 ** 3)
    F0, _ = ops.spme_recip(L, 1.2, order, K, xs, q, want_energy=True)
    (_, extra) = grown(lambda: ops.spme_recip(L, 1.2, order, K, xs, q, F=F, e_total=e, ws=least))
    assert extra == 0
    assert (F - F0).abs().max().item() <= 1e-11 * F0.abs().max().item()
    (_, extra) = grown(lambda: ops.spme_recip(L, 1.2, order, K, xs, q, F=F, e_total=e))
    assert (extra < 1.1 * least.numel()) == (order == 8)

    off0, csr0 = ops.build_neighbors_csr(L, 2.8, ops.FULL, xs, cs)
    off, csr = torch.empty_like(off0), torch.full_like(csr0, -7)
    w = empty(ops.OP_BUILD_CSR_LEAST)
    (_, extra) = grown(lambda: ops.build_neighbors_csr(L, 2.8, ops.FULL, xs, cs, cap=csr.numel(),
                                                       offsets=off, csr=csr, ws=w))
    m = int(off0[n].item())
    assert extra == 0 and torch.equal(off, off0) and torch.equal(csr[:m], csr0[:m])

    one = T([1.0])
    nbr, nnbr, maxn = ops.build_neighbors(L, 2.8, ops.FULL, xs, cs, 200)[:2] + (200,)
    got = []
    for op in (ops.OP_MD_CHAIN, ops.OP_MD_CHAIN_LEAST):
        w, v = empty(op), torch.zeros_like(xs)
        x1 = ops.md_step_chained(L, ops.FP64, 2.5, one, T([0.3]), xs, ts, nbr, nnbr, maxn, 1e-4,
                                 1.0, v, 0, w)
        got.append((x1, v, ops.md_step_sums(n, 0, w)))
    assert all(torch.equal(a, b) for a, b in zip(*got))
    with pytest.raises(ValueError):
        ops.md_step_sums(n, 0, empty(ops.OP_MD_CHAIN_LEAST)[:-8])


def test_windows_of_any_cadence(dev, monkeypatch):
    """A negative cadence rebuilds as its absolute value does, and windows cut into pieces
    give bitwise the run in whole ones."""
    import torch
    from paper_2109_09056_amd import md
    w = li.Workload("t", 11, cells=4)
    s = li.make_system(w)
    out = []
    for every, most in ((7, 16384), (-7, 16384), (7, 3)):
        monkeypatch.setattr(md.LJSim, "MAX_WINDOW", most, raising=False)
        sim = md.LJSim(w.box, rebuild_every=every, device=dev)
        sim.load(s["x"], s["v"])
        sim.step(25)
        sim.step(4)
        out.append((sim.x, sim.v, sim.F, sim.ids, sim.ev, torch.tensor(sim.nl.builds),
                    torch.tensor(sim.step_count)))
    for other in out[1:]:
        assert all(torch.equal(a, b) for a, b in zip(out[0], other))


def test_more_than_2_to_the_30_particles(dev):
    """2^30 + 65 particles, whose four lanes each are more threads than one grid dimension
    takes: two close pairs, at the first and the last indices, everything else far from any
    list entry.  Forces over full and half lists, their adjoint, SPH densities and
    accelerations, Ewald real space: the pairs' values, and zeros (the kernel's own term for
    densities) in all others.  Needs 130 GB of device memory."""
    import torch
    from paper_2109_09056_amd import _lib
    if torch.cuda.mem_get_info(dev)[0] + torch.cuda.memory_reserved(dev) < 150e9:
        pytest.skip("not enough free device memory")
    torch.cuda.empty_cache()
    n, L = (1 << 30) + 65, np.full(3, 20.0)
    lib, p = _lib.load(), lambda t: None if t is None else t.data_ptr()
    box, st = _lib.make_box(L), torch.cuda.current_stream(dev).cuda_stream
    z = lambda *s, d=torch.float64: torch.zeros(*s, dtype=d, device=dev)
    pairs = torch.tensor([[0, 1], [n - 2, n - 1]], device=dev)
    tiles = (n + 63) // 64
    nbr, nnbr = z(tiles * 64, d=torch.int32), z(n, d=torch.int32)
    x = z(n, 3)
    x[pairs[:, 0]] = 5.0
    x[pairs[:, 1]] = 6.1
    one = torch.ones(1, dtype=torch.float64, device=dev)
    i, j = pairs[:, 0], pairs[:, 1]
    both = torch.cat([i, j])

    def lists(half):
        nnbr.zero_()
        nnbr[i] = 1
        nbr[i] = j.to(torch.int32)  # capacity 1: entry 0 of row r is nbr[r]
        nnbr[j] = 0 if half else 1
        nbr[j] = i.to(torch.int32)

    def only(t):
        """t's rows of the two pairs; the others must hold nothing."""
        rows = t[both].clone()
        t[both] = 0.0
        lo, hi = t.aminmax()
        assert lo.item() == 0.0 and hi.item() == 0.0
        return rows.cpu().numpy()

    d = np.array([[-1.1] * 3] * 2 + [[1.1] * 3] * 2)
    r2 = (d * d).sum(1, keepdims=True)
    lj = 24.0 / r2 * (2.0 / r2 ** 6 - 1.0 / r2 ** 3) * d
    out = torch.full((n, 3), -1.0, dtype=torch.float64, device=dev)
    for half in (False, True):
        lists(half)
        _lib.check(lib.ljmd_compute_forces(box, _lib.FP64, int(half), 2.5, 1, p(one), p(one), n, p(x),
                                           None, p(nbr), p(nnbr), 1, p(out), None, None, None, 0,
                                           st), "forces")
        assert np.abs(only(out) - lj).max() <= 1e-13 * np.abs(lj).max()
    lists(False)

    ws = torch.empty(36 << 30, dtype=torch.uint8, device=dev)
    g = z(n, 3)
    g[i] = 1.0
    ge, gs = z(1), z(1)
    _lib.check(lib.ljmd_force_backward(box, _lib.FP64, 2.5, 1, p(one), p(one), n, p(x), None, p(nbr),
                                       p(nnbr), 1, p(g), p(out), p(ge), p(gs), 0, p(ws), ws.numel(),
                                       st), "backward")
    gx = only(out)
    assert np.abs(gx[:2]).min() > 0 and np.abs(gx[:2] + gx[2:]).max() <= 1e-13 * np.abs(gx).max()
    assert ge.item() == pytest.approx(lj[:2].sum(), rel=1e-12)  # F is linear in eps = 1
    del g
    torch.cuda.empty_cache()

    rho = z(n)
    h, m = 1.2, 1.0
    _lib.check(lib.ljmd_sph_density(box, h, m, 1.0, 1.0, n, p(x), p(nbr), p(nnbr), 1, p(rho), None,
                                    None, 0, st), "density")
    alone = m / (np.pi * h ** 3)
    near = rho[both].cpu().numpy()
    assert (near > alone * 1.01).all() and np.ptp(near) <= 1e-13 * alone
    rho[both] = rho[2].item()
    lo, hi = rho.aminmax()
    assert lo.item() == hi.item() == pytest.approx(alone, rel=1e-14)
    rho.fill_(2.0)
    _lib.check(lib.ljmd_sph_accel(box, h, m, 1.0, 1.0, n, p(x), p(rho), p(nbr), p(nnbr), 1, p(out),
                                  p(ws), ws.numel(), st), "accel")
    acc = only(out)
    assert np.abs(acc[:2]).min() > 0 and np.abs(acc[:2] + acc[2:]).max() <= 1e-13 * np.abs(acc).max()
    q = rho  # charges of 2
    for e in (None, one):
        _lib.check(lib.ljmd_ewald_real(box, 1.0, 2.5, n, p(x), p(q), p(nbr), p(nnbr), 1, p(out),
                                       p(e), 0, p(ws), ws.numel(), st), "ewald")
        f = only(out)
        assert np.abs(f[:2]).min() > 0 and np.abs(f[:2] + f[2:]).max() <= 1e-13 * np.abs(f).max()
    del x, out, ws, rho, q, nbr, nnbr
    torch.cuda.empty_cache()
