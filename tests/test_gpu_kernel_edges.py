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
