"""The work that programs have this library do, as cases whose time and
outputs can be measured: whole velocity-Verlet runs, single force
evaluations of every potential, list builds, the training-data loop and the
training steps of the learned potential, from a few hundred atoms to four
million.

A case is a dict of plain values: what is done ("do"), the potential
("pot"), the fcc cells per axis and the options.  `prepare` draws the
system and sets it up, `run` makes one pass through the public entry points
and returns what it computed, `work` counts the bytes and operations the
pass cannot do without, and `exact` gives the same outputs in plain FP64
torch from the definitions.
"""
import math

import numpy as np
import torch

from paper_1611_00075_amd import inputs
from paper_1611_00075_amd import md as M
from paper_1611_00075_amd import mlp as P
from paper_1611_00075_amd.dd import DomainSimulation
from paper_1611_00075_amd.sim import Simulation

LJ_A = inputs.fcc_lattice_constant(0.8442)
ALLOY_A = 0.75 * inputs.CU_A0 + 0.25 * inputs.AU_A0
FS, TB, TBM = inputs.FS_CU, inputs.TB_CU, inputs.TB2_PAIRS
RC = {"lj": 2.5, "eam": 4.4, "tb": 5.0, "tbm": 5.7, "tab": 4.4, "mlp": P.RC}


def _case(name, do, pot, nx, ny, nz, **opt):
    c = {"do": do, "pot": pot, "nx": nx, "ny": ny, "nz": nz, "voids": 0.0, "steps": 0, "energy": False,
         "fp64": False, "fp32act": False, "bricks": 0, "batch": 0}
    c.update(opt)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the 4,000-atom crystal in FP64: a short trajectory, bound by launches
        _case("lj-run-fp64-4k", "run", "lj", 10, 10, 10, steps=20, fp64=True),
        # production run of the porous system of 1.23 M atoms: forces, kicks and about two list builds
        _case("lj-run-voids-1.2M", "run", "lj", 80, 80, 80, voids=0.4, steps=16),
        # energy and virial of a porous sample with unequal box edges (thermodynamic output)
        _case("lj-energy-voids-80k", "forces", "lj", 31, 37, 29, voids=0.4, energy=True),
        # the 4 M-atom copper crystal: one embedded-atom force evaluation
        _case("eam-forces-4M", "forces", "eam", 100, 100, 100),
        # one snapshot of the 256-atom training trajectories: 20 steps, descriptors, site energies
        _case("eam-snapshot-256", "snapshot", "eam", 4, 4, 4, steps=20),
        # energy, virial and site energies of half a million copper atoms
        _case("eam-energy-500k", "forces", "eam", 50, 50, 50, energy=True),
        # sorting and list build of one million copper atoms after a drift
        _case("lists-eam-1M", "rebuild", "eam", 63, 63, 63),
        # two elements: forces of a random alloy
        _case("tbm-forces-500k", "forces", "tbm", 50, 50, 50),
        # tabulated functions on an odd-sized box
        _case("tab-forces-133k", "forces", "tab", 29, 31, 37),
        # the learned potential in its default form
        _case("mlp-forces-1M", "forces", "mlp", 63, 63, 63),
        # Adam steps of the learned potential at the default batch
        _case("mlp-train-4096", "train", "mlp", 4, 4, 4, steps=16, batch=4096),
        # the decomposed run: eight bricks with halo exchange
        _case("dd-run-500k", "run", "eam", 50, 50, 50, steps=8, bricks=2),
    ]


def draw(rng):
    """A case of the same ranges: sizes over their logarithm, each axis of
    its own length, every potential and option of the listed kinds."""
    kind = rng.choice(["run", "run", "forces", "forces", "forces", "energy", "energy", "rebuild", "snapshot",
                       "train", "dd"])
    if kind == "train":
        return _case(None, "train", "mlp", 4, 4, 4, steps=rng.randint(8, 16),
                     batch=int(math.exp(rng.uniform(math.log(500), math.log(8192)))))
    pot = {"run": ["lj", "lj", "eam", "tb", "tab", "mlp"], "forces": ["lj", "eam", "tb", "tbm", "tab", "mlp"],
           "energy": ["lj", "eam", "tb", "tbm", "tab", "mlp"], "rebuild": ["lj", "eam", "tb"],
           "snapshot": ["eam"], "dd": ["lj", "eam"]}[kind]
    pot = rng.choice(pot)
    lo, hi = {"run": (300, 500_000), "forces": (2_000, 2_000_000), "energy": (30_000, 1_000_000),
              "rebuild": (4_000, 1_000_000), "snapshot": (256, 6_000), "dd": (30_000, 500_000)}[kind]
    if pot == "mlp":
        hi = min(hi, 600_000)
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    least = {"dd": 11}.get(kind, 4)
    side = (n / 4.0) ** (1.0 / 3.0)
    w = [1.0, 1.0, 1.0] if rng.random() < 0.4 else [math.exp(rng.uniform(-0.2, 0.2)) for _ in range(3)]
    cells = [max(least, int(round(side * a))) for a in w]
    voids = round(rng.uniform(0.1, 0.45), 3) if pot == "lj" and min(cells) >= 8 and rng.random() < 0.6 else 0.0
    fp64 = kind == "run" and pot == "lj" and cells[0] * cells[1] * cells[2] < 5_000 and rng.random() < 0.6
    return _case(None, {"energy": "forces", "dd": "run"}.get(kind, kind), pot, *cells, voids=voids,
                 steps={"run": rng.randint(6, 20), "snapshot": 20, "dd": rng.randint(3, 8)}.get(kind, 0),
                 energy=kind == "energy", fp64=fp64, fp32act=pot == "mlp" and rng.random() < 0.4,
                 bricks=2 if kind == "dd" else 0)


# ---- the systems -------------------------------------------------------------

DEV = "cuda"


def _gen(seed, salt):
    return torch.Generator(DEV).manual_seed(1_000_003 * (salt + 1) + seed)


def _lattice(case):
    return {"lj": LJ_A, "tbm": ALLOY_A}.get(case["pot"], inputs.CU_A0)


def _units(pot):
    """(skin, dt, mass, force to acceleration, initial temperature in energy units, thermal displacement)"""
    if pot == "lj":
        return 0.3, 0.005, 1.0, 1.0, 0.72, 0.06
    return 1.0, 1.0, inputs.CU_MASS_AMU, 1.0 / inputs.AMU_A2_FS2_IN_EV, 600.0 * inputs.KB_EV, 0.1


def _positions(case, seed, width=1.0):
    """(box, positions (n, 3) FP64): a thermally displaced fcc crystal (`width`
    times the potential's usual displacement), with spherical voids of radius
    3 to 8 where the case asks for them."""
    a = _lattice(case)
    sigma = width * _units(case["pot"])[5]
    ax = [torch.arange(case[k], dtype=torch.float64, device=DEV) for k in ("nx", "ny", "nz")]
    cells = torch.stack(torch.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 1, 3)
    basis = torch.tensor(inputs.FCC_BASIS, dtype=torch.float64, device=DEV)
    x = ((cells + basis) * a).reshape(-1, 3)
    L = np.array([case["nx"], case["ny"], case["nz"]], dtype=np.float64) * a
    g = _gen(seed, 0)
    if case["voids"] > 0.0:
        # mean sphere volume of a radius uniform in [3, 8]: 4/3 pi (8^4 - 3^4) / (4 (8 - 3))
        mean = 4.0 / 3.0 * math.pi * (8.0 ** 4 - 3.0 ** 4) / 20.0
        count = max(1, round(-math.log(1.0 - case["voids"]) * float(np.prod(L)) / mean))
        Lt = torch.tensor(L, dtype=torch.float32, device=DEV)
        c = torch.rand(count, 3, device=DEV, generator=g) * Lt
        R = 3.0 + 5.0 * torch.rand(count, device=DEV, generator=g)
        # the sites deepest inside a void go, as many as the case says
        xf, depth = x.float(), torch.full((len(x),), 1e30, device=DEV)
        for k in range(0, count, 32):
            r2 = 0.0
            for b in range(3):
                d = (xf[:, b:b + 1] - c[k:k + 32, b]).abs()
                r2 = r2 + torch.minimum(d, Lt[b] - d) ** 2
            depth = torch.minimum(depth, (r2 / R[k:k + 32] ** 2).amin(1))
        x = x[torch.sort(torch.argsort(depth, stable=True)[round(case["voids"] * len(x)):])[0]]
    return L, x + sigma * torch.randn(x.shape, dtype=torch.float64, device=DEV, generator=g)


def _velocities(case, n, seed):
    _, _, mass, k, T, _ = _units(case["pot"])
    v = math.sqrt(T * k / mass) * torch.randn(n, 3, dtype=torch.float64, device=DEV, generator=_gen(seed, 1))
    return v - v.mean(0)


def _types(n, seed):
    return (torch.rand(n, device=DEV, generator=_gen(seed, 2)) < 0.25).to(torch.int32)


def _rows(seed, snaps):
    """Descriptor rows and site energies of `snaps` displaced 256-atom copper
    cells, FP64: what the training trajectories give."""
    c = _case(None, "train", "mlp", 4, 4, 4)
    G, E = [], []
    for s in range(snaps):
        L, x = _positions(c, 1000 * seed + s, width=0.5 + s / snaps)
        G.append(_descriptors(x, L)[0])
        E.append(_embedded(x, L, "eam", None)[3])
    return torch.cat(G), torch.cat(E)


def _network(seed):
    """(mean, inv_std, FP32 parameters) of an untrained network whose inputs
    are normalised over a displaced copper cell."""
    L, x = _positions(_case(None, "train", "mlp", 6, 6, 6), 77 + seed)
    G = _descriptors(x, L)[0]
    mean, std = G.mean(0), G.std(0, unbiased=False)
    inv = torch.where(std > 1e-6, 1.0 / std.clamp_min(1e-6), torch.ones_like(std))
    return (mean.float().cpu().numpy().astype(np.float64), inv.float().cpu().numpy().astype(np.float64),
            P.init_params(seed % 1000, e_mean=-3.5, w3_scale=0.3))


def prepare(case, seed):
    if case["do"] == "train":
        G, E = _rows(seed, 64)
        mean, inv, par = _network(seed)
        n, B = len(G), case["batch"]
        sel = torch.stack([torch.randint(0, n, (B,), dtype=torch.int32, device=DEV, generator=_gen(seed, 10 + k))
                           for k in range(case["steps"])])
        zero = lambda: torch.zeros(P.N_PARAM, dtype=torch.float32, device=DEV)   # noqa: E731
        return {"case": case, "G": G.float(), "E": E.float(), "sel": sel, "spec": P.spec(mean, inv),
                "adam": M.Adam(1e-3, 0.9, 0.999, 1e-8, 0), "master": torch.tensor(par, device=DEV), "m1": zero(),
                "m2": zero(), "w": P.bf16_bits(par).to(DEV),
                "losses": torch.zeros(case["steps"], dtype=torch.float64, device=DEV),
                "tws": torch.empty(M.md_mlp_workspace_bytes(B), dtype=torch.uint8, device=DEV)}
    L, x = _positions(case, seed)
    n = len(x)
    pot = case["pot"]
    skin, dt, mass, k, _, _ = _units(pot)
    moving = case["do"] in ("run", "snapshot")
    v = _velocities(case, n, seed) if moving else torch.zeros_like(x)
    kw = {"skin": skin, "dt": dt, "mass": mass, "force_to_accel": k}
    if case["bricks"]:
        b = case["bricks"]
        sim = DomainSimulation(L, x.cpu().numpy(), v.cpu().numpy(), p=(b, b, b), potential=pot, fs=FS, **kw)
        return {"case": case, "sim": sim}
    if pot == "eam":
        kw.update(fs=FS)
    elif pot == "tb":
        kw.update(tb=TB)
    elif pot == "tbm":
        kw.update(tbm=TBM, types=_types(n, seed).cpu().numpy())
    elif pot == "tab":
        kw.update(tab=inputs.fs_table(FS))
    elif pot == "mlp":
        mean, inv, par = _network(seed)
        kw.update(mlp=P.spec(mean, inv, case["fp32act"]), mlp_w=P.bf16_bits(par).to(DEV))
    sim = Simulation(L, x.cpu().numpy(), v.cpu().numpy(), potential=pot, pair_fp64=case["fp64"], **kw)
    state = {"case": case, "sim": sim}
    if case["do"] == "snapshot":
        state["spec"] = P.spec()
        state["G"] = torch.empty((n, M.MD_MLP_IN), dtype=torch.float32, device=DEV)
    if case["do"] == "rebuild":
        # the atoms in the order of an earlier build, some of them half a skin
        # away from there (entries past a row's end are whatever the buffer
        # held: zeros here)
        sim.x.add_(0.1 * skin * _drift(n, seed).T)
        sim.idx.zero_()
    return state


def _drift(n, seed):
    return torch.randn(n, 3, dtype=torch.float64, device=DEV, generator=_gen(seed, 3))


# ---- one pass ------------------------------------------------------------------

def run(state):
    case = state["case"]
    if case["do"] == "train":
        return _run_train(state)
    sim = state["sim"]
    if case["do"] == "rebuild":
        sim.rebuild()
        return {"x": sim.x, "ids": sim.ids, "cell_start": sim.cell_start, "count": sim.count, "idx": sim.idx}
    if case["do"] == "forces":
        sim.compute_forces(energy=case["energy"], site=case["energy"] and case["pot"] != "lj")
        return _forces_out(case, sim)
    sim.run(case["steps"])
    if case["do"] == "snapshot":
        sim.descriptors(state["spec"], out=state["G"])
        sim.compute_forces(site=True)
        return {"x": sim.x.float(), "ids": sim.ids, "f": sim.f, "e_atom": sim.e_atom, "G": state["G"]}
    # the frame of a trajectory: single precision where the forces are, as it is written out
    x, v = (sim.x, sim.v) if case["fp64"] else (sim.x.float(), sim.v.float())
    if case["bricks"]:
        ids = sim.ids.long()
        put = lambda t: torch.empty_like(t).index_copy_(1, ids, t)   # noqa: E731
        return {"x": put(x), "v": put(v), "f": put(sim.f)}
    return {"x": x, "v": v, "f": sim.f, "ids": sim.ids}


def _forces_out(case, sim):
    out = {"f": sim.f}
    if case["pot"] in ("eam", "tb", "tbm", "tab"):
        out.update(rho=sim.rho, fprime=sim.fprime)
    if case["pot"] == "mlp":
        out["dEdG"] = sim.dEdG
    if case["energy"]:
        out["ev"] = sim.ev
        if case["pot"] != "lj":
            out["e_atom"] = sim.e_atom
    return out


def _run_train(s):
    B = s["case"]["batch"]
    for k in range(s["case"]["steps"]):
        s["adam"].step += 1
        M.md_mlp_train_step(B, s["sel"][k], s["G"], s["E"], s["spec"], s["adam"], s["master"], s["m1"], s["m2"],
                            s["w"], s["losses"][k:k + 1], s["tws"])
    # losses in single precision: what a training log keeps
    return {"master": s["master"], "m1": s["m1"], "m2": s["m2"], "w": s["w"].view(torch.bfloat16),
            "losses": s["losses"].float()}


# ---- what a pass cannot do without ----------------------------------------------

def work(case):
    """Each list entry and each atom's state read once and written once per
    evaluation; operations of the pairs within the cutoff."""
    if case["do"] == "train":
        rows = case["batch"] * case["steps"]
        return {"bytes": rows * 68.0 + case["steps"] * P.N_PARAM * 28.0, "flops": rows * 6.0 * 5_200}
    a, pot = _lattice(case), case["pot"]
    n = 4.0 * case["nx"] * case["ny"] * case["nz"] * (1.0 - case["voids"])
    sphere = 4.0 / 3.0 * math.pi * 4.0 / a ** 3
    solid = 1.0 - 0.4 * case["voids"]            # neighbours lost at void surfaces
    rl = RC[pot] + _units(pot)[0]
    listed_pairs, inside = n * sphere * rl ** 3 * solid, n * sphere * RC[pot] ** 3 * solid
    per_pair = {"lj": 27, "eam": 40, "tb": 60, "tbm": 70, "tab": 50, "mlp": 280}[pot]
    passes = 2 if pot in ("eam", "tb", "tbm", "tab") else 1
    force = {"bytes": passes * 4.0 * listed_pairs + (76 if passes == 2 else 164 if pot == "mlp" else 36) * n,
             "flops": per_pair * inside + (20_480 * 2 * n if pot == "mlp" else 0)}
    if case["do"] == "rebuild":
        # positions and velocities in and out, the index, the list; one distance per pair of the list
        return {"bytes": 4.0 * listed_pairs + 112.0 * n, "flops": 9.0 * listed_pairs}
    if case["do"] == "forces":
        return force
    steps = case["steps"]
    w = {"bytes": steps * (force["bytes"] + 148.0 * n), "flops": steps * (force["flops"] + 20.0 * n)}
    if case["do"] == "snapshot":
        w = {"bytes": w["bytes"] + force["bytes"] + 100.0 * n, "flops": w["flops"] + force["flops"] + 60.0 * inside}
    return w


# ---- the same outputs in FP64 ----------------------------------------------------

def _wrap(x, L):
    w = x - L * torch.floor(x / L)
    w = torch.where(w >= L, w - L, w)
    return torch.where(w < 0, w + L, w)


def _sorted(x, L, r_list):
    """Order of the atoms (wrapped positions x) by the Morton code of their
    cell, input order within a cell."""
    nc = torch.floor(L / r_list)
    c = torch.minimum((x * (nc / L)).long(), (nc - 1).long())
    code = torch.zeros(len(x), dtype=torch.int64, device=x.device)
    for b in range(10):
        for ax in range(3):
            code |= ((c[:, ax] >> b) & 1) << (3 * b + ax)
    return torch.sort(code, stable=True)[1], code


def _pairs(x, L, rc):
    """All ordered pairs within rc, a chunk at a time: (i, j, d = r_j - r_i, r)."""
    n, L = len(x), torch.as_tensor(L, dtype=torch.float64, device=x.device)
    nc = torch.floor(L / rc).long()
    every = torch.arange(n, device=x.device)

    def near(i, j):
        d = x[j] - x[i]
        d = d - L * torch.round(d / L)
        r2 = (d * d).sum(-1)
        ok = (r2 < rc * rc) & (i != j)
        return i[ok], j[ok], d[ok], r2[ok].sqrt()

    if int(nc.min()) < 3:
        step = max(1, 8_000_000 // n)
        for k in range(0, n, step):
            i = every[k:k + step]
            yield near(i.repeat_interleave(n), every.repeat(len(i)))
        return
    c = torch.minimum((_wrap(x, L) * (nc / L)).long(), nc - 1)
    lin = c[:, 0] + nc[0] * (c[:, 1] + nc[1] * c[:, 2])
    order = torch.sort(lin)[1]
    size = torch.bincount(lin, minlength=int(nc.prod()))
    start = torch.cumsum(size, 0) - size
    offsets = [(p, q, r) for p in (-1, 0, 1) for q in (-1, 0, 1) for r in (-1, 0, 1)]
    for k in range(0, n, 1_000_000):
        i = every[k:k + 1_000_000]
        for o in offsets:
            m = (c[i] + torch.tensor(o, device=x.device)) % nc
            m = m[:, 0] + nc[0] * (m[:, 1] + nc[1] * m[:, 2])
            cnt = size[m]
            ii = i.repeat_interleave(cnt)
            first = (torch.cumsum(cnt, 0) - cnt).repeat_interleave(cnt)
            at = torch.arange(len(ii), device=x.device) - first
            yield near(ii, order[start[m].repeat_interleave(cnt) + at])


def _virial(W, g, d):
    """W += sum of g d_a d_b in the order xx, yy, zz, xy, xz, yz"""
    for k, (a, b) in enumerate(((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))):
        W[k] += (g * d[:, a] * d[:, b]).sum()


def _lj(x, L):
    f, ev = torch.zeros_like(x), torch.zeros(8, dtype=torch.float64, device=x.device)
    rc = RC["lj"]
    shift = 4.0 * (rc ** -12 - rc ** -6)
    for i, _, d, r in _pairs(x, L, rc):
        s6 = r ** -6
        g = 24.0 * s6 * (2.0 * s6 - 1.0) / (r * r)       # F_i = -g d
        f.index_add_(0, i, -g[:, None] * d)
        e = 4.0 * (s6 * s6 - s6)
        ev[0] += 0.5 * e.sum()
        ev[1] += 0.5 * (e - shift).sum()
        _virial(ev[2:], 0.5 * g, d)
    return f, ev


def _switch(r, t):
    u = ((r - t["rs"]) / (t["rc"] - t["rs"])).clamp(0.0, 1.0)
    return (1.0 - u ** 3 * (10.0 - 15.0 * u + 6.0 * u * u),
            -30.0 * u * u * (1.0 - u) ** 2 / (t["rc"] - t["rs"]))


def _tb_terms(r, t):
    """psi, psi', Phi, Phi' of the tight-binding form"""
    S, dS = _switch(r, t)
    q, p = -2.0 * t["q"] / t["r0"], -t["p"] / t["r0"]
    eq = t["xi"] ** 2 * torch.exp(q * (r - t["r0"]))
    ep = 2.0 * t["A"] * torch.exp(p * (r - t["r0"]))
    return eq * S, eq * (q * S + dS), ep * S, ep * (p * S + dS)


def _hermite(u, h, f, df):
    """Value and slope at u of the piecewise cubic through knots k h."""
    f, df = (torch.as_tensor(np.asarray(t), dtype=torch.float64, device=u.device) for t in (f, df))
    k = (u / h).long().clamp(0, len(f) - 2)
    s = u / h - k
    a1, a2, a3 = h * df[k], 3 * (f[k + 1] - f[k]) - h * (2 * df[k] + df[k + 1]), 2 * (f[k] - f[k + 1]) + h * (df[k] + df[k + 1])
    return f[k] + s * (a1 + s * (a2 + s * a3)), (a1 + s * (2 * a2 + 3 * a3 * s)) / h


def _pair_terms(pot, r, kind):
    if pot == "eam":
        psi, dpsi = (r - FS["d"]) ** 2, 2.0 * (r - FS["d"])
        q, dq = FS["c0"] + FS["c1"] * r + FS["c2"] * r * r, FS["c1"] + 2.0 * FS["c2"] * r
        t = torch.where(r < FS["c"], r - FS["c"], torch.zeros_like(r))
        return psi, dpsi, t * t * q, 2.0 * t * q + t * t * dq
    if pot == "tab":
        T = inputs.fs_table(FS)
        return (*_hermite(r, T["dr"], T["psi"], T["dpsi"]), *_hermite(r, T["dr"], T["phi"], T["dphi"]))
    if pot == "tb":
        return _tb_terms(r, TB)
    out = [torch.zeros_like(r) for _ in range(4)]
    for k in range(3):
        at = kind == k
        for o, v in zip(out, _tb_terms(r[at], TBM[k])):
            o[at] = v
    return out


def _embed(pot, rho):
    if pot == "tab":
        T = inputs.fs_table(FS)
        return _hermite(rho, T["drho"], T["F"], T["dF"])
    A = FS["A"] if pot == "eam" else 1.0
    s = rho.sqrt()
    zero = torch.zeros_like(rho)
    return -A * s, torch.where(rho > 0, -0.5 * A / s, zero)


def _embedded(x, L, pot, types):
    """(forces, ev, rho, site energies, F') of an embedded-atom form"""
    n, zero = len(x), torch.zeros(len(x), dtype=torch.float64, device=x.device)
    kind = lambda i, j: None if types is None else types[i] + types[j]   # noqa: E731
    rho, V = zero.clone(), zero.clone()
    for i, j, _, r in _pairs(x, L, RC[pot]):
        psi, _, phi, _ = _pair_terms(pot, r, kind(i, j))
        rho.index_add_(0, i, psi)
        V.index_add_(0, i, phi)
    F, Fp = _embed(pot, rho)
    f, W = torch.zeros_like(x), torch.zeros(6, dtype=torch.float64, device=x.device)
    for i, j, d, r in _pairs(x, L, RC[pot]):
        _, dpsi, _, dphi = _pair_terms(pot, r, kind(i, j))
        g = -((Fp[i] + Fp[j]) * dpsi + dphi) / r
        f.index_add_(0, i, -g[:, None] * d)
        _virial(W, 0.5 * g, d)
    ev = torch.cat([(F.sum() + 0.5 * V.sum())[None], F.sum()[None], W])
    return f, ev, rho, F + 0.5 * V, Fp


def _basis(r, k):
    """g_k and its derivative"""
    t = r - (P.MU0 + P.DMU * k)
    e = torch.exp(-t * t / (2.0 * P.WIDTH ** 2))
    fc, dfc = 0.5 * (torch.cos(math.pi * r / P.RC) + 1.0), -0.5 * math.pi / P.RC * torch.sin(math.pi * r / P.RC)
    return e * fc, e * (dfc - fc * t / P.WIDTH ** 2)


def _descriptors(x, L):
    G = torch.zeros(P.N_IN, len(x), dtype=torch.float64, device=x.device)
    n = len(x)
    for i, _, _, r in _pairs(x, L, P.RC):
        # sums in a fixed order: rows of equal i are consecutive
        i, order = torch.sort(i, stable=True)
        cnt = torch.bincount(i, minlength=n)
        end = torch.cumsum(cnt, 0)
        for k in range(P.N_IN):
            c = torch.cat([r.new_zeros(1), torch.cumsum(_basis(r[order], k)[0], 0)])
            G[k] += c[end] - c[end - cnt]
    return G.T.contiguous(), n


def _forward(G, par, mean, inv):
    """Per-atom energies of descriptor rows; par the flat parameter vector."""
    at, w = 0, []
    for _, shape in P.SHAPES:
        k = int(np.prod(shape)) if shape else 1
        w.append(par[at:at + k].reshape(shape))
        at += k
    W1, b1, W2, b2, w3, b3 = w
    silu = lambda a: a * torch.sigmoid(a)   # noqa: E731
    return silu(silu(((G - mean) * inv) @ W1.T + b1) @ W2.T + b2) @ w3 + b3


def _learned(x, L, seed):
    mean, inv, par = _network(seed)
    t = lambda a: torch.as_tensor(a, dtype=torch.float64, device=x.device)   # noqa: E731
    w = t(P.bf16_values(P.bf16_bits(par)))
    G = _descriptors(x, L)[0].requires_grad_(True)
    e = _forward(G, w, t(mean), t(inv))
    D = torch.autograd.grad(e.sum(), G)[0]
    e = e.detach()
    f, W = torch.zeros_like(x), torch.zeros(6, dtype=torch.float64, device=x.device)
    for i, j, d, r in _pairs(x, L, P.RC):
        s = torch.zeros_like(r)
        for k in range(P.N_IN):
            s += (D[i, k] + D[j, k]) * _basis(r, k)[1]
        f.index_add_(0, i, (s / r)[:, None] * d)
        _virial(W, -0.5 * s / r, d)
    return f, torch.cat([e.sum()[None], e.sum()[None], W]), D, e


def exact(case, seed):
    if case["do"] == "train":
        return _exact_train(case, seed)
    L, x = _positions(case, seed)
    Lt = torch.tensor(L, dtype=torch.float64, device=x.device)
    pot = case["pot"]
    skin, dt, mass, k, _, _ = _units(pot)
    if case["do"] in ("run", "snapshot"):
        return _exact_run(case, seed, L, Lt, x)
    x = _wrap(x, Lt)
    p = _sorted(x, Lt, RC[pot] + skin)[0]
    x = x[p]
    if case["do"] == "rebuild":
        y = _wrap(x + 0.1 * skin * _drift(len(x), seed), Lt)
        return {"x": y[_sorted(y, Lt, RC[pot] + skin)[0]].T, "ids": None, "cell_start": None, "count": None,
                "idx": None}
    out = {}
    if pot == "lj":
        f, ev = _lj(x, L)
    elif pot == "mlp":
        f, ev, out["dEdG"], e = _learned(x, L, seed)
    else:
        t = _types(len(x), seed).long()[p] if pot == "tbm" else None
        f, ev, out["rho"], e, out["fprime"] = _embedded(x, L, pot, t)
    out["f"] = f.T
    if case["energy"]:
        out["ev"] = ev
        if pot != "lj":
            out["e_atom"] = e
    return out


def _exact_run(case, seed, L, Lt, x):
    """Velocity Verlet with the rebuild rule, atoms in the order of the last
    build (input order for the decomposed run)."""
    pot = case["pot"]
    skin, dt, mass, k, _, _ = _units(pot)
    v = _velocities(case, len(x), seed)
    ids = torch.arange(len(x), device=x.device)
    learned = None

    def force(x):
        nonlocal learned
        if pot == "lj":
            return _lj(x, L)[0]
        if pot == "mlp":
            learned = _learned(x, L, seed)
            return learned[0]
        return _embedded(x, L, pot, None)[0]

    def build(x, v, ids):
        x = _wrap(x, Lt)
        if not case["bricks"]:
            p = _sorted(x, Lt, RC[pot] + skin)[0]
            x, v, ids = x[p], v[p], ids[p]
        return x, v, ids, x.clone()

    x, v, ids, ref = build(x, v, ids)
    f = force(x)
    h = 0.5 * dt * k / mass
    for _ in range(case["steps"]):
        v = v + h * f
        x = x + dt * v
        d = x - ref
        d = d - Lt * torch.round(d / Lt)
        if float((d * d).sum(1).max()) > 0.25 * skin * skin:
            x, v, ids, ref = build(x, v, ids)
        f = force(x)
        v = v + h * f
    if case["do"] == "snapshot":
        return {"x": x.T, "ids": None, "f": f.T, "e_atom": _embedded(x, L, pot, None)[3],
                "G": _descriptors(x, L)[0]}
    return {"x": x.T, "v": v.T, "f": f.T, "ids": None}


def _exact_train(case, seed):
    s = prepare(case, seed)
    G, E = s["G"].double(), s["E"].double()
    t = lambda a: torch.as_tensor(np.asarray(a[:]), dtype=torch.float64, device=G.device)   # noqa: E731
    mean, inv = t(s["spec"].mean), t(s["spec"].inv_std)
    master, m1, m2 = s["master"].double(), s["m1"].double(), s["m2"].double()
    lr, b1, b2, eps = s["adam"].lr, s["adam"].beta1, s["adam"].beta2, s["adam"].eps
    losses = []
    for k in range(case["steps"]):
        w = master.float().bfloat16().double().requires_grad_(True)
        at = s["sel"][k].long()
        loss = ((_forward(G[at], w, mean, inv) - E[at]) ** 2).mean()
        g = torch.autograd.grad(loss, w)[0]
        losses.append(loss.detach())
        m1, m2 = b1 * m1 + (1 - b1) * g, b2 * m2 + (1 - b2) * g * g
        master = master - lr * (m1 / (1 - b1 ** (k + 1))) / ((m2 / (1 - b2 ** (k + 1))).sqrt() + eps)
    return {"master": master, "m1": m1, "m2": m2, "w": master.float().bfloat16().double(),
            "losses": torch.stack(losses)}
