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
