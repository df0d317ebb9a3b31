"""Kernels at the sizes where their split of the work changes: tile and
batch remainders, the thresholds of a launch rule, the smallest inputs."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1611_00075_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1611_00075_amd import md
    md.lib()
    return md


# ---- reductions ---------------------------------------------------------------

@pytest.mark.parametrize("n", [1, 257, 2048 * 256, 2048 * 256 + 1, 70_000 * 16 + 3])
def test_kinetic_energy_either_side_of_the_one_block_sum(M, n):
    """One partial row per 256 atoms: up to 2,048 rows one block sums them,
    beyond that chunks of 64 rows are summed first.  n squares summed in FP64
    differ by at most n eps from another order (eps 1.1e-16)."""
    g = torch.Generator("cuda").manual_seed(n)
    v = torch.randn(3, n, dtype=torch.float64, device="cuda", generator=g)
    f = torch.randn(3, n, dtype=torch.float32, device="cuda", generator=g)
    grid = M.md_grid_init([100.0] * 3, 5.0)
    ws = torch.empty(M.md_workspace_bytes(grid, n), dtype=torch.uint8, device="cuda")
    M.md_workspace_init(grid, n, ws)
    ke = torch.full((1,), -1.0, dtype=torch.float64, device="cuda")
    want = 0.5 * 2.5 * float(((v + 0.5 * 0.01 * 3.0 * f.double()) ** 2).sum())
    M.md_integrate(M.MD_KICK, [100.0] * 3, n, v.clone(), v, f, 0.01, 3.0, 2.5, None, 0.0, None, 0, None, ke, 0, ws)
    assert ke.item() == pytest.approx(want, rel=max(1e-14, 3 * n * 1.2e-16))


@pytest.mark.parametrize("pot", ["lj", "eam"])
def test_energy_rows_either_side_of_the_one_block_sum(M, pot):
    """Energy and virial per atom of a perfect crystal do not depend on its
    size: 2,197 rows of 32 atoms (chunked) against 125 (one block).  The sums
    are FP64; LJ runs in FP64 throughout (n eps), the embedded-atom pair terms
    are FP32 (a few 2^-24 each, common to all pairs of a shell)."""
    from paper_1611_00075_amd.sim import Simulation
    ev = []
    for ncell in (10, 26):
        s = inputs.lj_fcc(ncell=ncell) if pot == "lj" else inputs.eam_cu(ncell=ncell)
        kw = dict(pair_fp64=True) if pot == "lj" else dict(potential="eam", fs=inputs.FS_CU, skin=1.0)
        sim = Simulation(s.L, s.x, np.zeros_like(s.x), **kw)
        sim.compute_forces(energy=True)
        ev.append(sim.ev.cpu().numpy() / s.n)
    scale = np.abs(ev[0]).max()
    assert np.abs(ev[1] - ev[0]).max() <= (1e-11 if pot == "lj" else 2e-6) * scale, ev


@pytest.mark.parametrize("pot", ["lj", "eam"])
@pytest.mark.parametrize("n", [2, 9, 63, 65, 257])
def test_energy_and_virial_of_partly_filled_wavefronts(orc, pot, n):
    """A cluster of n atoms (8 a wavefront, 32 a block).  Each pair's energy and
    force factor carries a few FP32 roundings (2^-24 each), at most 1e-5 of the
    summed magnitudes; the sums themselves are FP64."""
    from paper_1611_00075_amd.sim import Simulation
    s = inputs.jitter(inputs.lj_fcc(ncell=8) if pot == "lj" else inputs.eam_cu(ncell=8), 0.04, n)
    x = s.x[:n].copy()
    rc, skin = (2.5, 0.3) if pot == "lj" else (4.4, 1.0)
    kw = {} if pot == "lj" else dict(potential="eam", fs=inputs.FS_CU)
    sim = Simulation(s.L, x, np.zeros_like(x), skin=skin, **kw)
    sim.compute_forces(energy=True)
    got = sim.ev.cpu().numpy()
    xw = orc.wrap(x, s.L)
    off, idx = orc.neighbors_brute(xw, s.L, rc + skin)
    want = orc.forces_lj(xw, s.L, off, idx, rc=rc)[1] if pot == "lj" else orc.forces_eam(xw, s.L, off, idx, inputs.FS_CU)["ev"]
    # magnitudes of the virial terms: every pair's |g| |d|^2 is at most |F_ij| r
    i = np.repeat(np.arange(n), np.diff(off))
    d = xw[idx] - xw[i]
    d -= s.L * np.round(d / s.L)
    r = np.sqrt((d * d).sum(1))
    if pot == "lj":
        scale = np.abs(24 * (2 * r ** -12 - r ** -6))[r < rc].sum() + abs(want[0])
    else:
        scale = 20.0 * n      # eV: |psi' F'| r + |V'| r, about 1 eV for each of 12 neighbours
    assert np.abs(got - np.asarray(want)[: len(got)]).max() <= 1e-5 * scale, (got, want)


# ---- training -------------------------------------------------------------------

@pytest.mark.parametrize("batch,shift", [(1, 0), (17, 0), (32, 1), (33, 0), (4095, 1), (32 * 1024 + 5, 0)])
def test_gradient_at_group_edges(M, orc, batch, shift):
    """Batches around the 32-atom groups, one atom, more groups than partial
    rows (1,024), and parameters that start two bytes past a 16-byte boundary
    (shift): FP32 sums to 1e-5, plus what one activation rounded to the other
    bfloat16 neighbour (2^-8) can do to the batch's mean."""
    from oracle import mlp as om
    from paper_1611_00075_amd import mlp as P
    rng = np.random.default_rng(batch)
    rows = 600
    G = np.abs(rng.standard_normal((rows, 16)) * 3.0 + 4.0).astype(np.float32)
    target = (-3.5 + 0.05 * rng.standard_normal(rows)).astype(np.float32)
    sel = rng.integers(0, rows, batch).astype(np.int32)
    bits = P.bf16_bits(P.init_params(11, e_mean=-3.4, w3_scale=0.3))
    w = torch.zeros(M.MD_MLP_NPARAM + 8, dtype=torch.int16, device="cuda")[shift:shift + M.MD_MLP_NPARAM]
    w.copy_(bits)
    sp = P.spec(np.zeros(16), np.full(16, 0.25))
    grad = torch.full((M.MD_MLP_NPARAM,), np.nan, dtype=torch.float32, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    tws = torch.empty(M.md_mlp_workspace_bytes(batch), dtype=torch.uint8, device="cuda")
    M.md_mlp_grad(batch, torch.tensor(sel, device="cuda"), torch.tensor(G, device="cuda"),
                  torch.tensor(target, device="cuda"), sp, w, grad, loss, tws)
    g = grad.cpu().numpy().astype(np.float64)
    lo, go = om.loss_grad(G[sel].astype(np.float64), target[sel].astype(np.float64),
                          om.Spec(mean=np.zeros(16), inv_std=np.full(16, 0.25)), P.bf16_values(bits), bf16=True)
    tol = 1e-5 + 4 * 2.0 ** -8 / batch
    assert loss.item() == pytest.approx(lo, rel=tol)
    o = 0
    for name, shape in P.SHAPES:
        k = int(np.prod(shape)) if shape else 1
        rel = np.linalg.norm(g[o:o + k] - go[o:o + k]) / np.linalg.norm(go[o:o + k])
        assert rel < tol, (name, rel)
        o += k


# ---- FP64 Lennard-Jones ------------------------------------------------------------

def test_fp64_lj_rows_of_every_length(M, orc):
    """Rows of 0 to about 100 entries through the batched FP64 walk, to the
    1e-12 of the FP64 path."""
    from test_gpu_parity import _gpu_lists
    x, L = inputs.graded(14, inputs.fcc_lattice_constant(1.2), 0.03, seed=72)
    x = orc.wrap(x, L)
    n = len(x)
    _, st = _gpu_lists(M, x, L, 2.8)
    f = torch.full((3, n), np.nan, dtype=torch.float64, device="cuda")
    M.md_forces_lj(L, n, st["x"], None, st["cap"], st["idx"], st["cnt"], (1.0, 1.0, 2.5), f, None, M.MD_PAIR_FP64,
                   st["ws"])
    fg = np.empty((n, 3))
    fg[st["perm"].cpu().numpy()[:n]] = f.cpu().numpy().T
    oc, ic = orc.neighbors_cells(x, L, 2.8)
    fo, _ = orc.forces_lj(x, L, oc, ic, rc=2.5)
    assert np.linalg.norm(fg - fo) <= 1e-12 * np.linalg.norm(fo)


# ---- neighbour lists ----------------------------------------------------------------

def _ordered_rows(M, g, x, cell_start, want, atoms):
    """Rows of sorted atoms in the list's order: stencil cells x fastest,
    atoms of a cell in sorted order, kept where `want` (sets of sorted
    indices) says so."""
    nc, R = np.array(g.nc[:]), g.reach
    ranks = M.md_grid_cell_ranks(g)
    lin = np.empty(g.n_cells, np.int64)
    lin[ranks] = np.arange(g.n_cells)
    home = lin[np.searchsorted(cell_start, atoms, side="right") - 1]
    rows = []
    for i, l in zip(atoms, home):
        c = np.array([l % nc[0], (l // nc[0]) % nc[1], l // (nc[0] * nc[1])])
        row = []
        for dz in range(-R, R + 1):
            for dy in range(-R, R + 1):
                for dx in range(-R, R + 1):
                    v = (c + (dx, dy, dz)) % nc
                    r = ranks[v[0] + nc[0] * (v[1] + nc[1] * v[2])]
                    row += [j for j in range(cell_start[r], cell_start[r + 1]) if j in want[i]]
        rows.append(row)
    return rows


def _lists(M, orc, x, L, r_list, reach, row_cap):
    """(grid, cell_start, sorted positions, idx filled with -1 beforehand, counts, longest)"""
    n = len(x)
    g = M.md_grid_init(L, r_list, reach)
    ws = torch.empty(M.md_workspace_bytes(g, n), dtype=torch.uint8, device="cuda")
    M.md_workspace_init(g, n, ws)
    xd = torch.tensor(np.ascontiguousarray(x.T), dtype=torch.float64, device="cuda")
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device="cuda")   # noqa: E731
    cell, perm, cs, cnt, mx = i32(n), i32(n), i32(g.n_cells + 1), i32(n), i32(1)
    M.md_bin_cells(g, n, xd, cell, perm, cs, ws)
    xs = torch.empty_like(xd)
    M.md_permute(n, 3, perm, xd, xs, 8)
    idx = torch.full((M.ell_size(n, row_cap),), -1, dtype=torch.int32, device="cuda")
    M.md_build_neighbors(g, n, xs, cs, row_cap, idx, cnt, mx, ws)
    return g, cs.cpu().numpy(), xs.cpu().numpy().T.copy(), idx.cpu().numpy(), cnt.cpu().numpy(), int(mx[0])


def _row(idx, i, row_cap):
    return idx.reshape(-1, row_cap // 8, 8, 8)[i // 8, :, i % 8, :].reshape(-1)


LIST_CASES = [
    # box, r_list, reach, atoms: few homes per cell, about one and two matrix
    # tiles of 16, three batches of homes and more candidates than the table
    # of 1,024, 125-cell stencils, enough cells for one wavefront each
    ((11.3, 12.1, 13.0), 2.8, 1, 150),
    ((11.3, 12.1, 13.0), 2.8, 1, 1060),
    ((11.3, 12.1, 13.0), 2.8, 1, 2300),
    ((16.0, 16.5, 17.0), 3.9, 1, 9000),
    ((8.5, 9.0, 9.6), 2.8, 2, 700),
    ((36.5, 36.6, 37.0), 2.8, 1, 33000),
    # a box of three cells on one axis: the path without matrix cores
    ((9.0, 12.0, 12.5), 2.9, 1, 1500),
]


@pytest.mark.parametrize("L,r_list,reach,n", LIST_CASES)
def test_list_rows_in_order(M, orc, L, r_list, reach, n):
    L = np.array(L)
    x = orc.wrap(inputs.random_gas(n, L, n), L)
    cap = 640
    g, cs, xs, idx, cnt, longest = _lists(M, orc, x, L, r_list, reach, cap)
    off, ob = orc.neighbors_brute(xs, L, r_list) if n < 10_000 else orc.neighbors_cells(xs, L, r_list)
    assert np.array_equal(cnt, np.diff(off)) and longest == cnt.max() <= cap
    atoms = np.random.default_rng(n).choice(n, min(n, 250), replace=False)
    want = {i: set(ob[off[i]:off[i + 1]].tolist()) for i in atoms}
    for i, row in zip(atoms, _ordered_rows(M, g, xs, cs, want, atoms)):
        got = _row(idx, i, cap)
        assert got[:cnt[i]].tolist() == row, i
        assert (got[cnt[i]:] == -1).all()          # nothing is written past a row


@pytest.mark.parametrize("shell", [4, 6])
def test_list_cutoff_on_a_shell(M, orc, shell):
    """r_list equal to a shell radius of a perfect crystal: every pair of the
    shell is decided by the rounding of its own FP64 r^2."""
    s = inputs.lj_fcc(ncell=9)
    a = s.meta["a"]
    x = orc.wrap(s.x + np.array([0.1, 0.2, 0.3]), s.L)
    r_list = a * np.sqrt(shell / 2.0)
    g, cs, xs, idx, cnt, _ = _lists(M, orc, x, s.L, r_list, 1, 128)
    off, ob = orc.neighbors_brute(xs, s.L, r_list)
    assert np.array_equal(cnt, np.diff(off))
    for i in range(len(x)):
        assert np.array_equal(np.sort(_row(idx, i, 128)[:cnt[i]]), ob[off[i]:off[i + 1]])


def test_list_rows_past_the_capacity_are_cut(M, orc):
    L = np.array((11.3, 12.1, 13.0))
    n, cap = 1700, 24
    x = orc.wrap(inputs.random_gas(n, L, 5), L)
    full = _lists(M, orc, x, L, 2.8, 1, 400)
    cut = _lists(M, orc, x, L, 2.8, 1, cap)
    assert cut[5] == full[5] > cap and np.array_equal(cut[4], full[4])
    for i in range(n):
        k = min(cap, full[4][i])
        assert np.array_equal(_row(cut[3], i, cap)[:k], _row(full[3], i, 400)[:k])
        assert (_row(cut[3], i, cap)[k:] == -1).all()


def test_list_with_a_position_that_is_no_number(M, orc):
    """The atom has no neighbours and is nobody's; all other rows are those of
    the system without it."""
    L = np.array((11.3, 12.1, 13.0))
    x = orc.wrap(inputs.random_gas(900, L, 6), L)
    x[450] = np.nan
    _, _, xs, idx, cnt, _ = _lists(M, orc, x, L, 2.8, 1, 200)
    odd = np.flatnonzero(np.isnan(xs[:, 0]))
    assert len(odd) == 1 and cnt[odd[0]] == 0
    rest = np.flatnonzero(~np.isnan(xs[:, 0]))
    off, ob = orc.neighbors_brute(xs[rest], L, 2.8)
    for k, i in enumerate(rest):
        assert np.array_equal(np.sort(_row(idx, i, 200)[:cnt[i]]), rest[ob[off[k]:off[k + 1]]])


def _nan_systems():
    # few cells (batches of 4 homes), many cells (a batch is a cell), 125-cell
    # stencils, three cells on an axis (the path without matrix cores)
    return [((11.3, 12.1, 13.0), 2.8, 1, 900), ((36.5, 36.6, 37.0), 2.8, 1, 33000), ((8.5, 9.0, 9.6), 2.8, 2, 700),
            ((9.0, 12.0, 12.5), 2.9, 1, 800)]


@pytest.mark.parametrize("where,axes", [("first", (0, 1, 2)), ("first", (2,)), ("middle", (0, 1, 2)), ("last", (0, 1, 2)),
                                        ("two", (0, 1, 2))])
@pytest.mark.parametrize("L,r_list,reach,n", _nan_systems())
def test_list_with_no_number_anywhere_in_a_batch(M, orc, L, r_list, reach, n, where, axes):
    """Atoms whose position (or one component) is no number at the start, in the
    middle and at the end of their cell: they have no neighbours and are
    nobody's, and every other row is that of the system without them."""
    L = np.array(L)
    x = orc.wrap(inputs.random_gas(n, L, 6), L)
    for k in {"first": [0], "middle": [n // 2], "last": [n - 1], "two": [0, 1]}[where]:
        x[k, list(axes)] = np.nan
    cap = 400
    _, _, xs, idx, cnt, _ = _lists(M, orc, x, L, r_list, reach, cap)
    bad = np.isnan(xs).any(axis=1)
    assert (cnt[bad] == 0).all()
    rest = np.flatnonzero(~bad)
    off, ob = orc.neighbors_brute(xs[rest], L, r_list) if n < 10_000 else orc.neighbors_cells(xs[rest], L, r_list)
    assert np.array_equal(cnt[rest], np.diff(off))
    some = np.random.default_rng(n).choice(len(rest), min(len(rest), 900), replace=False)
    for k in np.union1d(some, np.arange(40)):
        i = rest[k]
        assert np.array_equal(np.sort(_row(idx, i, cap)[:cnt[i]]), rest[np.sort(ob[off[k]:off[k + 1]])])


@pytest.mark.parametrize("far", [1e19, 1e21, 1e25, 1e40, 1e200])
@pytest.mark.parametrize("L,r_list,reach,n", [((11.3, 12.1, 13.0), 2.8, 1, 900), ((36.5, 36.6, 37.0), 2.8, 1, 9000),
                                              ((8.5, 9.0, 9.6), 2.8, 2, 700)])
def test_list_with_positions_too_large_to_wrap(M, orc, L, r_list, reach, n, far):
    """Finite positions so large that FP64 has no digits left for the box, the first
    and the last atom among them: every row is that of the system without them."""
    L = np.array(L)
    x = orc.wrap(inputs.random_gas(n, L, 6), L)
    # most such numbers come out of the wrap as 0: take some that stay outside
    rng = np.random.default_rng(1)
    for k in (0, n - 1):
        while not (np.abs(orc.wrap(x[k:k + 1].copy(), L)) > 8 * L.max()).any():
            x[k] = far * rng.uniform(-1.0, 1.0, 3)
    cap = 400
    _, _, xs, idx, cnt, _ = _lists(M, orc, x, L, r_list, reach, cap)
    out = (np.abs(xs) > 8 * L.max()).any(axis=1)
    assert out.sum() == 2 and (cnt[out] == 0).all()
    rest = np.flatnonzero(~out)
    off, ob = orc.neighbors_brute(xs[rest], L, r_list)
    assert np.array_equal(cnt[rest], np.diff(off))
    for k, i in enumerate(rest):
        assert np.array_equal(np.sort(_row(idx, i, cap)[:cnt[i]]), rest[np.sort(ob[off[k]:off[k + 1]])])


@pytest.mark.parametrize("unit", [2.0 ** -75, 2.0 ** -41, 2.0 ** -40, 2.0 ** 38, 2.0 ** 39, 2.0 ** 75])
@pytest.mark.parametrize("reach", [1, 2])
def test_list_in_any_unit_of_length(M, orc, unit, reach):
    """The same system in units of length a power of two apart (every FP64
    operation of the definition scales exactly): the same rows in the same order,
    also where squares of lengths leave the FP32 range of the matrix cores."""
    L = np.array((14.2, 14.6, 15.0))
    n, cap = 900, 128
    x = orc.wrap(inputs.random_gas(n, L, 8), L)
    a = _lists(M, orc, x, L, 2.4, reach, cap)
    b = _lists(M, orc, x * unit, L * unit, 2.4 * unit, reach, cap)
    assert a[5] == b[5] <= cap and np.array_equal(a[4], b[4]) and np.array_equal(a[2] * unit, b[2])
    for i in range(n):
        assert np.array_equal(_row(a[3], i, cap), _row(b[3], i, cap))


# ---- learned potential ----------------------------------------------------------------

@pytest.mark.parametrize("dmu,width", [(0.2, 0.2), (0.3, 0.16)])
def test_learned_pair_pass_over_ragged_rows(M, orc, dmu, width):
    """Rows of every length (0 to 60 in range) in one slice, and Gaussian
    spacings on both sides of the rule that folds them into polynomials
    (exp(-32 (dmu / width)^2) above 1e-18: ratios 1 and 1.9).  FP32 pair
    terms from the same dE/dG: 1e-5 normwise."""
    from oracle import mlp as om
    from paper_1611_00075_amd import mlp as P
    from paper_1611_00075_amd.sim import Simulation
    x, L = inputs.graded(12, 3.5, 0.08, seed=31, n_gas=40, gas_sep=2.2)
    x = orc.wrap(x, L)
    n = len(x)
    spec = dict(rc=5.0, mu0=1.4, dmu=dmu, width=width)
    sim = Simulation(L, x, np.zeros_like(x), potential="mlp", mlp=M.mlp_spec(*spec.values()),
                     mlp_w=P.bf16_bits(P.init_params(5)).cuda(), skin=1.0, dt=1.0)
    ids = sim.ids.cpu().numpy()
    D = np.random.default_rng(3).standard_normal((n, 16)).astype(np.float32)
    sim.dEdG[:n] = torch.tensor(D[ids], device="cuda")
    f = torch.full((3, n), np.nan, dtype=torch.float32, device="cuda")
    M.md_forces_mlp(L, n, sim.xs, sim.row_cap, sim.idx, sim.count, sim.mlp, None, sim.dEdG, None, None, None, f, None,
                    M.MD_MLP_REUSE, sim.ws)
    off, idx = orc.neighbors_brute(x, L, 5.0)
    assert np.diff(off).min() <= 2 and np.diff(off).max() >= 45
    fo, _ = om.forces(x, L, off, idx, om.Spec(**spec), D.astype(np.float64))
    fg = np.empty((n, 3))
    fg[ids] = f.cpu().numpy().T
    assert np.linalg.norm(fg - fo) <= 1e-5 * np.linalg.norm(fo)


@pytest.mark.parametrize("r", [0.05, 0.4, 0.6, 0.9, 1.0, 1.2, 1.3, 2.0])
def test_learned_pair_pass_of_close_pairs(M, r):
    """Pairs so close that the Gaussian at the centre of the set underflows
    (3.6 - r above 2.64) or nearly does: the folded sums give what the Gaussians
    themselves give (the form with MD_ENERGY), finite and to the FP32 rounding of
    16 terms that cancel (1e-5 of the summed magnitudes)."""
    from paper_1611_00075_amd import mlp as P
    from paper_1611_00075_amd.sim import Simulation
    x = np.array([[5.0, 5.0, 5.0], [5.0 + 0.6 * r, 5.0 + 0.8 * r, 5.0], [9.0, 5.0, 5.5]])
    sim = Simulation(np.full(3, 20.0), x, np.zeros_like(x), potential="mlp", mlp=P.spec(),
                     mlp_w=P.bf16_bits(P.init_params(5)).cuda(), skin=1.0, dt=1.0)
    D = np.random.default_rng(3).uniform(0.5, 1.0, (3, 16)).astype(np.float32)
    out = []
    for energy in (0, M.MD_ENERGY):
        sim.dEdG[:3] = torch.tensor(D, device="cuda")
        f = torch.full((3, 3), np.nan, dtype=torch.float32, device="cuda")
        M.md_forces_mlp(sim.L, 3, sim.xs, sim.row_cap, sim.idx, sim.count, sim.mlp, None, sim.dEdG, None, None, None,
                        f, sim.ev, M.MD_MLP_REUSE | energy, sim.ws)
        out.append(f.cpu().numpy().astype(np.float64))
    assert np.isfinite(out[0]).all()
    t = r - (P.MU0 + P.DMU * np.arange(16))
    scale = (2 * np.exp(-t * t / (2 * P.WIDTH ** 2)) * (np.abs(t) / P.WIDTH ** 2 + 1)).sum()
    assert np.abs(out[0] - out[1]).max() <= 1e-5 * (scale + np.abs(out[1]).max()), out


@pytest.mark.parametrize("size", [1.0, 1e4, 1e7, 1e12, 1e20])
@pytest.mark.parametrize("dmu,r", [(0.2, 1.0), (0.2, 1.1), (0.2, 1.4), (0.2, 2.5), (0.225, 1.25), (0.225, 1.6), (0.1, 0.2),
                                   (0.1, 1.0)])
def test_learned_pair_pass_of_large_gradients(M, orc, dmu, r, size):
    """dE/dG of any size (inputs of small spread are scaled up by as much) for
    pairs down to where the central Gaussian leaves FP32 (13.2 widths of 0.2 below its
    centre): finite and right wherever the 16 terms are.  The exponents reach 127 and are
    rounded two or three times (2^-24 each, ln 2 of them relative), the ratio is
    taken to the eighth power: 1e-4 of the summed magnitudes."""
    from oracle import mlp as om
    from paper_1611_00075_amd import mlp as P
    from paper_1611_00075_amd.sim import Simulation
    x = np.array([[5.0, 5.0, 5.0], [5.0 + 0.6 * r, 5.0 + 0.8 * r, 5.0]])
    spec = dict(rc=P.RC, mu0=P.MU0, dmu=dmu, width=P.WIDTH)
    sim = Simulation(np.full(3, 20.0), x, np.zeros_like(x), potential="mlp", mlp=M.mlp_spec(*spec.values()),
                     mlp_w=P.bf16_bits(P.init_params(5)).cuda(), skin=1.0, dt=1.0)
    D = (size * np.random.default_rng(3).uniform(0.5, 1.0, (2, 16))).astype(np.float32)
    ids = sim.ids.cpu().numpy()
    off, idx = orc.neighbors_brute(x, np.full(3, 20.0), P.RC)
    want, _ = om.forces(x, np.full(3, 20.0), off, idx, om.Spec(**spec), D.astype(np.float64))
    t = r - (P.MU0 + dmu * np.arange(16))
    scale = (D.sum(0) * np.exp(-t * t / (2 * P.WIDTH ** 2)) * (np.abs(t) / P.WIDTH ** 2 + 1)).sum()
    for energy in (0, M.MD_ENERGY):
        sim.dEdG[:2] = torch.tensor(D[ids], device="cuda")
        f = torch.full((3, 2), np.nan, dtype=torch.float32, device="cuda")
        M.md_forces_mlp(sim.L, 2, sim.xs, sim.row_cap, sim.idx, sim.count, sim.mlp, None, sim.dEdG, None, None, None,
                        f, sim.ev, M.MD_MLP_REUSE | energy, sim.ws)
        got = np.empty((2, 3))
        got[ids] = f.cpu().numpy().T
        assert np.abs(got - want).max() <= 1e-4 * scale, (energy, got, want)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 64 * 512, 64 * 512 + 1])
@pytest.mark.parametrize("shift", [0, 1])
def test_network_at_block_edges(M, orc, n, shift):
    """Atoms around one 64-atom chunk, one chunk per block of the persistent
    grid and one more, with parameters at and off a 16-byte boundary, FP32
    activations: each atom within 2e-5 of the FP64 network."""
    from oracle import mlp as om
    from paper_1611_00075_amd import mlp as P
    rng = np.random.default_rng(n)
    G = np.abs(rng.standard_normal((n, 16)) * 2.0 + 3.0).astype(np.float32)
    bits = P.bf16_bits(P.init_params(12, e_mean=-3.4, w3_scale=0.3))
    w = torch.zeros(M.MD_MLP_NPARAM + 8, dtype=torch.int16, device="cuda")[shift:shift + M.MD_MLP_NPARAM]
    w.copy_(bits)
    e = torch.full((n,), np.nan, dtype=torch.float32, device="cuda")
    d = torch.full((n, 16), np.nan, dtype=torch.float32, device="cuda")
    M.md_mlp_eval(n, torch.tensor(G, device="cuda"), P.spec(np.zeros(16), np.full(16, 0.25), fp32_activations=True), w, e,
                  d)
    eo, do = om.energy(G.astype(np.float64), om.Spec(mean=np.zeros(16), inv_std=np.full(16, 0.25)), P.bf16_values(bits))
    assert np.abs(e.cpu().numpy() - eo).max() <= 2e-5 * np.abs(eo).max()
    assert np.abs(d.cpu().numpy() - do).max() <= 2e-5 * np.abs(do).max()


# ---- decomposed run ---------------------------------------------------------------------

@pytest.mark.parametrize("pot", ["lj", "eam"])
def test_decomposed_run_on_one_and_two_streams(M, pot):
    """The flag of a step is read beside the inner atoms' pass: with the
    exchange on its own stream and on the compute stream the run takes the
    same builds and gives the same bits, builds included."""
    from paper_1611_00075_amd.dd import DomainSimulation
    s = inputs.lj_fcc(ncell=12, T=1.4) if pot == "lj" else inputs.eam_cu(ncell=10, T=1500.0)
    kw = dict(skin=0.3, dt=0.005) if pot == "lj" else dict(
        potential="eam", fs=inputs.FS_CU, skin=0.4, dt=2.0, mass=inputs.CU_MASS_AMU,
        force_to_accel=1.0 / inputs.AMU_A2_FS2_IN_EV)
    out = []
    for one in (False, True):
        sim = DomainSimulation(s.L, s.x, s.v, p=(2, 2, 2) if pot == "eam" else (2, 1, 2), **kw)
        if one:
            sim.comm = torch.cuda.current_stream()
        sim.run(25)
        sim.run(15)
        out.append((sim.dd.builds, sim.positions(), sim.forces()))
        sim.close()
    assert out[0][0] == out[1][0] > 2
    assert np.array_equal(out[0][1], out[1][1]) and np.array_equal(out[0][2], out[1][2])


@pytest.mark.parametrize("pot", ["lj", "eam"])
@pytest.mark.parametrize("when", [0, 2])
def test_decomposed_run_keeps_its_forces_at_a_position_that_is_no_number(M, pot, when):
    """The run ends at the drift that met the position: no pass runs on the bad
    coordinates and f stays that of the last completed step."""
    from paper_1611_00075_amd.dd import DomainSimulation
    s = inputs.lj_fcc(ncell=12) if pot == "lj" else inputs.eam_cu(ncell=10)
    kw = dict(skin=0.3, dt=0.005) if pot == "lj" else dict(
        potential="eam", fs=inputs.FS_CU, skin=0.4, dt=2.0, mass=inputs.CU_MASS_AMU,
        force_to_accel=1.0 / inputs.AMU_A2_FS2_IN_EV)
    sim = DomainSimulation(s.L, s.x, s.v, p=(2, 2, 2) if pot == "eam" else (2, 1, 2), **kw)
    if when:
        sim.run(when)
    f = sim.f.clone()
    sim.v[1, 17] = float("nan")
    with pytest.raises(M.MDError) as e:
        sim.run(5)
    assert e.value.code == M.MD_ERR_NONFINITE and sim.dd.phase == 0 and sim.dd.steps == when
    torch.cuda.synchronize()
    assert torch.equal(sim.f, f)
    sim.close()


# ---- native driver ---------------------------------------------------------------------------

@pytest.mark.parametrize("polled", [True, False])
@pytest.mark.parametrize("pot,cells", [("lj", (5, 5, 5)), ("lj", (5, 6, 7)), ("lj64", (5, 5, 5)), ("eam", (4, 4, 4)),
                                       ("eam", (4, 5, 4)), ("tb", (4, 4, 4)), ("tbm", (5, 5, 5)), ("tbm", (5, 4, 5)),
                                       ("tab", (4, 4, 4)), ("tab", (4, 4, 5)), ("mlp", (4, 4, 4))])
def test_velocity_update_in_the_force_kernels(M, pot, cells, polled):
    """Runs of 1 to 7 steps, with builds at different places among them, against
    the same runs with a kick-drift launch per step (timing): all state bit for
    bit."""
    from paper_1611_00075_amd import mlp as P
    from paper_1611_00075_amd.sim import Simulation
    a = inputs.fcc_lattice_constant(0.8442) if pot.startswith("lj") else inputs.CU_A0 * (1.04 if pot == "tbm" else 1.0)
    x = _fcc(cells, a)
    n = len(x) - 3                      # not a whole number of wavefronts
    rng = np.random.default_rng(n)
    x = x[:n] + 0.02 * a * rng.standard_normal((n, 3))
    L = np.array(cells) * a
    if pot.startswith("lj"):
        kw = dict(skin=0.12, dt=0.005, pair_fp64=pot == "lj64")
        v = 1.5 * rng.standard_normal((n, 3))
    else:
        kw = dict(potential=pot, skin=0.2, dt=4.0, mass=inputs.CU_MASS_AMU,
                  force_to_accel=1.0 / inputs.AMU_A2_FS2_IN_EV)
        v = 0.004 * rng.standard_normal((n, 3))
        kw.update({"eam": dict(fs=inputs.FS_CU), "tb": dict(tb=inputs.TB_CU), "tab": dict(tab=inputs.fs_table(inputs.FS_CU)),
                   "tbm": dict(tbm=inputs.TB2_PAIRS, types=rng.integers(0, 2, n).astype(np.int32)),
                   "mlp": dict(mlp=P.spec(np.full(16, 4.0), np.full(16, 0.2)),
                               mlp_w=P.bf16_bits(P.init_params(5, e_mean=-3.5, w3_scale=0.3)).cuda())}[pot])
    sims = [Simulation(L, x, v, **kw) for _ in range(2)]
    if not polled:
        for sim in sims:
            sim._flag_host = None
    for steps in (1, 2, 3, 4, 7):
        sims[0].run(steps)
        sims[1].run(steps, timing=True)
        for name in ("x", "v", "f", "ids", "xref", "count") + (() if pot == "lj64" else ("xs",)):
            t, u = (getattr(sim, name) for sim in sims)
            if name == "xs":            # (after the rho pass the fourth word holds F')
                t, u = t[:, :3], u[:, :3]
            assert torch.equal(t, u), (steps, name)
        assert sims[0].builds == sims[1].builds
    assert sims[0].builds > 1


@pytest.mark.parametrize("pot", ["lj", "eam", "tb", "tbm", "tab"])
@pytest.mark.parametrize("timing", [False, True])
def test_lists_read_past_the_caches(M, pot, timing):
    """Rows of 24,576 entries' room make the lists of 3,500 atoms larger than the
    300 MB above which a run reads them past the caches: same trajectory, to the
    bit, as with rows of 104."""
    from paper_1611_00075_amd.sim import Simulation
    cells, a = (10, 10, 9), inputs.fcc_lattice_constant(0.8442) if pot == "lj" else inputs.CU_A0
    rng = np.random.default_rng(5)
    x = _fcc(cells, a)[:3500]
    x = x + 0.02 * a * rng.standard_normal(x.shape)
    kw = dict(skin=0.3, dt=0.005) if pot == "lj" else dict(
        potential=pot, skin=0.4, dt=2.0, mass=inputs.CU_MASS_AMU, force_to_accel=1.0 / inputs.AMU_A2_FS2_IN_EV,
        **{"eam": dict(fs=inputs.FS_CU), "tb": dict(tb=inputs.TB_CU), "tab": dict(tab=inputs.fs_table(inputs.FS_CU)),
           "tbm": dict(tbm=inputs.TB2_PAIRS, types=rng.integers(0, 2, 3500).astype(np.int32))}[pot])
    v = (0.8 if pot == "lj" else 0.003) * rng.standard_normal(x.shape)
    sims = [Simulation(np.array(cells) * a, x, v, row_cap=cap, **kw) for cap in (104, 24_576)]
    for sim in sims:
        sim.run(6, timing=timing)
    for name in ("x", "v", "f", "ids"):
        assert torch.equal(*(getattr(sim, name) for sim in sims)), name


def _fcc(cells, a):
    g = np.stack(np.meshgrid(*[np.arange(c) for c in cells], indexing="ij"), -1).reshape(-1, 1, 3)
    return ((g + np.array(inputs.FCC_BASIS)) * a).reshape(-1, 3)


@pytest.mark.parametrize("fp64", [False, True])
def test_run_ahead_of_the_flag(M, fp64):
    """With pinned memory the next step is queued before a step's flag is
    read, without it the flag is copied first: same bits, builds and capacity
    growth included, for runs of one, two and many steps."""
    from paper_1611_00075_amd.sim import Simulation
    s = inputs.lj_fcc(ncell=7, T=2.0)
    out = []
    for pinned in (True, False):
        sim = Simulation(s.L, s.x, s.v, pair_fp64=fp64, row_cap=72, list_slack=1.0)
        if not pinned:
            sim._flag_host = None
        for k in (1, 2, 1, 40, 7):
            sim.run(k)
        out.append((sim.builds, sim.row_cap, sim.positions(), sim.velocities(), sim.forces()))
    assert out[0][:2] == out[1][:2] and out[0][0] > 4
    assert all(np.array_equal(a, b) for a, b in zip(out[0][2:], out[1][2:]))


@pytest.mark.parametrize("when", [0, 3])
def test_run_ahead_stops_at_a_position_that_is_no_number(M, when):
    """A non-finite position ends the run at its own step: the state is that of
    the flow without pinned memory, not one step further."""
    from paper_1611_00075_amd.sim import Simulation
    s = inputs.lj_fcc(ncell=6)
    out = []
    for pinned in (True, False):
        sim = Simulation(s.L, s.x, s.v)
        if not pinned:
            sim._flag_host = None
        if when:
            sim.run(when)
        sim.v[1, 17] = float("inf")
        with pytest.raises(M.MDError) as e:
            sim.run(10)
        assert e.value.code == M.MD_ERR_NONFINITE
        assert sim._sys.step == when
        out.append((sim.x.cpu().numpy(), sim.v.cpu().numpy()))
    for a, b in zip(*out):
        assert np.array_equal(a, b, equal_nan=True)


@pytest.mark.parametrize("pot", ["lj", "tb"])
@pytest.mark.parametrize("when", [0, 3])
def test_nothing_is_left_on_the_stream_after_a_position_that_is_no_number(M, pot, when):
    """The steps queued ahead post their flags to the caller's host words, so a run
    that ends with an error waits for them: the stream is idle at the return."""
    import ctypes as C
    from paper_1611_00075_amd.sim import Simulation
    cells = (25, 25, 26)                # just below the largest system that queues two steps ahead
    a = inputs.fcc_lattice_constant(0.8442) if pot == "lj" else inputs.CU_A0
    x = _fcc(cells, a)
    kw = {} if pot == "lj" else dict(potential="tb", tb=inputs.TB_CU, skin=1.0, dt=1.0, mass=inputs.CU_MASS_AMU,
                                     force_to_accel=1.0 / inputs.AMU_A2_FS2_IN_EV)
    sim = Simulation(np.array(cells) * a, x, np.zeros_like(x), **kw)
    if when:
        sim.run(when)
    sim.v[2, 40000] = float("nan")
    S, stream = sim._system(), torch.cuda.current_stream()
    torch.cuda.synchronize()
    run, handle = M.lib().md_run, stream.cuda_stream
    rc = run(C.byref(S), 10, handle)
    idle = stream.query()
    assert rc == M.MD_ERR_NONFINITE and S.step == when
    assert idle


# ---- the energy flag ------------------------------------------------------------------------

def _small(M, pot, rng, cells=(6, 5, 7)):
    """(box, positions, keyword arguments): a displaced crystal of each form."""
    from paper_1611_00075_amd import mlp as P
    a = inputs.fcc_lattice_constant(0.8442) if pot.startswith("lj") else inputs.CU_A0 * (1.04 if pot == "tbm" else 1.0)
    x = _fcc(cells, a)[:-3]
    n = len(x)
    x = x + 0.02 * a * rng.standard_normal((n, 3))
    if pot.startswith("lj"):
        return np.array(cells) * a, x, dict(skin=0.3, dt=0.005, pair_fp64=pot == "lj64")
    kw = dict(potential=pot, skin=0.6, dt=2.0, mass=inputs.CU_MASS_AMU, force_to_accel=1.0 / inputs.AMU_A2_FS2_IN_EV)
    if pot.startswith("mlp"):
        # narrow Gaussians: exp(-32 (dmu / width)^2) below 1e-18, no folding
        width = P.WIDTH if pot == "mlp" else 0.13
        kw.update(potential="mlp", mlp=M.mlp_spec(P.RC, P.MU0, P.DMU, width, np.full(16, 4.0), np.full(16, 0.2)),
                  mlp_w=P.bf16_bits(P.init_params(5, e_mean=-3.5, w3_scale=0.3)).cuda())
    else:
        kw.update({"eam": dict(fs=inputs.FS_CU), "tb": dict(tb=inputs.TB_CU),
                   "tab": dict(tab=inputs.fs_table(inputs.FS_CU)),
                   "tbm": dict(tbm=inputs.TB2_PAIRS, types=rng.integers(0, 2, n).astype(np.int32))}[pot])
    return np.array(cells) * a, x, kw


FORMS = ["lj", "lj64", "eam", "tb", "tbm", "tab", "mlp", "mlp-narrow"]


@pytest.mark.parametrize("compensate", [True, False])
@pytest.mark.parametrize("pot", FORMS)
def test_forces_do_not_depend_on_the_energy_flag(M, pot, compensate):
    """MD_ENERGY also writes energy and virial: the forces are the same bits."""
    from paper_1611_00075_amd.sim import Simulation
    rng = np.random.default_rng(9)
    L, x, kw = _small(M, pot, rng)
    if pot == "lj64" and not compensate:
        pytest.skip("FP64 sums have no compensation")
    sim = Simulation(L, x, np.zeros_like(x), compensate=compensate, **kw)
    out = []
    for energy in (False, True):
        sim.f.fill_(float("nan"))
        sim.compute_forces(energy=energy)
        out.append(sim.f.clone())
    assert torch.isfinite(out[0]).all() and torch.equal(*out)


@pytest.mark.parametrize("pot", FORMS)
def test_reading_the_energy_does_not_change_a_trajectory(M, pot):
    from paper_1611_00075_amd.sim import Simulation
    rng = np.random.default_rng(9)
    L, x, kw = _small(M, pot, rng)
    v = (0.8 if pot.startswith("lj") else 0.003) * rng.standard_normal(x.shape)
    sims = [Simulation(L, x, v, **kw) for _ in range(2)]
    for look in (False, True):
        sims[look].run(5)
        if look:
            sims[look].energies()
        sims[look].run(5)
    for name in ("x", "v", "f", "ids"):
        assert torch.equal(*(getattr(s, name) for s in sims)), name


# ---- tabulated functions -------------------------------------------------------------

@pytest.mark.parametrize("cells", [(4, 4, 4), (13, 13, 13), (33, 32, 32), (51, 51, 51)])
def test_tabulated_forces_at_every_grid(M, cells):
    """Fewer slices than wavefronts, one round of blocks with one to a few
    slices a wavefront, two rounds: the table samples the Finnis-Sinclair set, so
    both forms give the same forces (each within 1e-5 normwise of the FP64 ones)."""
    from paper_1611_00075_amd.sim import Simulation
    x = _fcc(cells, inputs.CU_A0)
    x = x[: len(x) - 5]
    x = x + 0.1 * np.random.default_rng(len(x)).standard_normal(x.shape)
    out = []
    for kw in (dict(potential="tab", tab=inputs.fs_table(inputs.FS_CU)), dict(potential="eam", fs=inputs.FS_CU)):
        sim = Simulation(np.array(cells) * inputs.CU_A0, x, np.zeros_like(x), skin=1.0, dt=1.0, **kw)
        sim.f.fill_(float("nan"))
        sim.compute_forces()
        out.append(sim.f.double())
    assert (out[0] - out[1]).norm().item() <= 2e-5 * out[1].norm().item()


# ---- binning -------------------------------------------------------------------------

@pytest.mark.parametrize("n,nc", [(1, (3, 3, 3)), (1023, (16, 16, 16)), (1025, (5, 30, 7)), (4096, (17, 16, 16)),
                                  (8191, (4, 4, 4)), (8192, (16, 16, 16)), (8193, (16, 16, 16)), (8192, (25, 25, 26)),
                                  (9000, (26, 26, 26)), (9000, (162, 162, 162))])
def test_sort_at_the_sizes_of_its_launches(M, orc, n, nc):
    """One launch up to 8,192 atoms and 4,096 cells; scans of up to 16,384
    counts by one block, up to 2,048 tiles of 2,048 in two launches, three above:
    wrapped positions, cells, stable order and offsets are those of the
    definition, to the bit."""
    rng = np.random.default_rng(n + nc[0])
    L = np.array(nc) + 0.5
    x = rng.uniform(-0.3, 1.3, (n, 3)) * L
    x[rng.random(n) < 0.3] = 0.25 * L          # a crowded cell
    g = M.md_grid_init(L, 1.0)
    assert tuple(g.nc) == nc
    ws = torch.empty(M.md_workspace_bytes(g, n), dtype=torch.uint8, device="cuda")
    M.md_workspace_init(g, n, ws)
    xd = torch.tensor(x.T.copy(), device="cuda")
    cell, perm = (torch.full((n,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    start = torch.full((g.n_cells + 1,), -1, dtype=torch.int32, device="cuda")
    M.md_bin_cells(g, n, xd, cell, perm, start, ws)
    w = orc.wrap(x, L)
    c = orc.cell_coords(w, L, nc).astype(np.int64)
    rank = M.md_grid_cell_ranks(g)[c[:, 0] + nc[0] * (c[:, 1] + nc[1] * c[:, 2])]
    assert np.array_equal(xd.cpu().numpy().T, w)
    assert np.array_equal(cell.cpu().numpy(), rank)
    assert np.array_equal(perm.cpu().numpy(), np.argsort(rank, kind="stable"))
    assert np.array_equal(start.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(rank, minlength=g.n_cells))]))


@pytest.mark.parametrize("n,nc", [(8192, (5, 5, 5)), (8192, (4, 4, 4)), (8192, (2, 2, 2)), (4096, (3, 3, 3)),
                                  (4096, (3, 3, 2)), (1000, (2, 2, 2))])
def test_sort_of_crowded_cells(M, orc, n, nc):
    """Either side of the line from which crowded cells leave the one-launch sort."""
    test_sort_at_the_sizes_of_its_launches(M, orc, n, nc)


# ---- decomposed build ----------------------------------------------------------------

@pytest.mark.parametrize("p,L", [((2, 1, 1), (140.5, 70.5, 70.5)), ((2, 2, 1), (40.0, 40.0, 20.0)),
                                 ((3, 1, 2), (60.0, 20.0, 40.0))])
def test_decomposed_build_of_uneven_bricks(M, p, L):
    """A cluster of 4,000 atoms across brick faces and the box boundary, other
    bricks empty or nearly so; bricks of more than 16,384 cells (their scans go
    one by one) and of a few hundred (all in one launch).  Forces as without
    decomposition: FP32 sums in another order, 1e-5 normwise."""
    from paper_1611_00075_amd.dd import DomainSimulation
    from paper_1611_00075_amd.sim import Simulation
    L = np.array(L)
    rng = np.random.default_rng(7)
    x = _fcc((10, 10, 10), inputs.fcc_lattice_constant(0.8442)) + 0.04 * rng.standard_normal((4000, 3)) - 8.0
    v = 0.5 * rng.standard_normal(x.shape)
    dd = DomainSimulation(L, x, v, p=p, potential="lj", skin=0.3, dt=0.005)
    sim = Simulation(L, x, v, skin=0.3, dt=0.005)
    for _ in range(2):
        f, g = dd.forces(), sim.forces()
        assert np.linalg.norm(f - g) <= 1e-5 * np.linalg.norm(g)
        dd.run(7)
        sim.run(7)
        d = dd.positions() - sim.positions()
        assert np.abs(d - L * np.round(d / L)).max() < 1e-5
    assert sum(b[0] for b in dd.bricks()) == 4000
    dd.close()


def test_decomposed_build_of_more_cells_than_a_launch_takes(M):
    """Eight bricks of 8.9 M cells each (207 per axis): one launch with a wavefront
    per cell of all bricks would be 4.5e9 threads, past the 2^32 of a launch (which
    drops what is beyond, without an error).  A cluster around the corner that all
    bricks share; forces as without decomposition: FP32 sums in another order, 1e-5
    normwise."""
    from paper_1611_00075_amd.dd import DomainSimulation
    from paper_1611_00075_amd.sim import Simulation
    rng = np.random.default_rng(7)
    x = _fcc((5, 5, 5), inputs.fcc_lattice_constant(0.8442)) + 0.04 * rng.standard_normal((500, 3)) - 4.0
    L = np.full(3, 2 * 204.5 * 2.8)
    dd = DomainSimulation(L, x, np.zeros_like(x), p=(2, 2, 2), potential="lj", skin=0.3, dt=0.005)
    assert dd.dd.vgrid.n_cells * 8 * 64 >= 2 ** 32
    f = dd.forces()
    dd.close()
    g = Simulation(np.full(3, 60.0), x, np.zeros_like(x), skin=0.3, dt=0.005).forces()
    assert np.linalg.norm(f - g) <= 1e-5 * np.linalg.norm(g)
