"""Performance cases: the work a user of this framework has it do, through `abi.AmrLbm` and `abi.AmrBatch`.

A pass is one turn of a user's main loop on a simulation that is already set up: some coarse time steps, then what that
loop reads or does between its steps (a field snapshot, the force on the cylinder, the refinement criterion and an
adaptation).  The kinds of loop:

  snapshot  steps on a mesh that stays, then rho and u of every output cell (monitoring, writing frames)
  restart   the same, then the populations of every output cell (checkpoints, offline analysis)
  force     steps, then the momentum exchange per level (drag and lift sampling)
  period    steps, the vorticity criterion or the ladder, an adaptation, the blocks' vorticity, a snapshot (the main
            loop of an AMR run)
  window    a refined region that moves away and back: two adaptations with the caller's own tags, steps after each
  whole     a short simulation from creation to its last snapshot (parameter studies)
  batch     steps of many simulations advanced together, then each member's mass and momentum and one member's snapshot

The set-ups are those of `workloads` (lid-driven cavity, flow past a square cylinder, uniform periodic level) at the
sizes of the benchmark and the tests, and between them.
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2308_08085_amd import abi, workloads as W

STORAGE_BYTES = {"f64": 8, "f32": 4, "f32s": 4, "f16s": 2, "bf16s": 2}
# block shapes of a batch: (dim, side in root cells, levels, Reynolds number); members take them in turn
BATCH_MEMBERS = ((2, 32, 2, 100.0), (2, 64, 3, 180.0), (2, 128, 4, 320.0), (2, 256, 3, 600.0),
                 (3, 32, 3, 120.0), (3, 48, 2, 250.0), (3, 64, 2, 400.0), (3, 32, 2, 160.0))


def listed():
    return [
        # the smallest call: a loop that watches a small 2-D run step by step (default eager launches)
        dict(name="watch_d2q9_cavity_f64", kind="snapshot", shape="cavity", q=9, nx=32, ny=32, nz=1, lmax=3,
             storage="f64", interp=0, re=100.0, graph=False, skip=False, steps=1),
        # a short run of the D2Q9 FP64 cavity set-up from creation to its fields, as a parameter study makes many
        dict(name="whole_d2q9_cavity_f64", kind="whole", shape="cavity", q=9, nx=64, ny=64, nz=1, lmax=3,
             storage="f64", interp=0, re=100.0, graph=True, skip=False, steps=300),
        # the paper's square cylinder: drag and lift sampled every 16 root steps
        dict(name="force_d2q9_fpsc_f64", kind="force", shape="fpsc", q=9, nx=256, ny=256, nz=1, lmax=3,
             storage="f64", interp=0, re=100.0, graph=True, skip=False, steps=16),
        # the same flow with cubic interpolation and the log2 ladder of the paper, single precision
        dict(name="period_d2q9_fpsc_cubic_f32", kind="period", shape="fpsc", q=9, nx=256, ny=256, nz=1, lmax=4,
             storage="f32", interp=1, re=100.0, graph=True, skip=False, steps=32),
        # the 1024 x 256 D2Q9 channel, four levels: one adaptation period
        dict(name="period_d2q9_cylinder_f32s", kind="period", shape="cylinder", q=9, nx=1024, ny=256, nz=1, lmax=4,
             storage="f32s", interp=0, re=100.0, graph=True, skip=True, steps=32),
        # the 64^3 D3Q19 cavity, three levels, stepped between snapshots
        dict(name="snapshot_d3q19_cavity_f32s", kind="snapshot", shape="cavity", q=19, nx=64, ny=64, nz=64, lmax=3,
             storage="f32s", interp=0, re=400.0, graph=True, skip=False, steps=50),
        # a refined region that follows something through a ragged cavity, 16-bit storage
        dict(name="window_d3q19_cavity_f16s", kind="window", shape="cavity", q=19, nx=52, ny=52, nz=52, lmax=3,
             storage="f16s", interp=0, re=250.0, graph=True, skip=False, steps=10),
        # populations for a restart from the half-size D3Q27 channel, FP64, default eager launches
        dict(name="restart_d3q27_cylinder_f64", kind="restart", shape="cylinder", q=27, nx=64, ny=32, nz=32, lmax=3,
             storage="f64", interp=0, re=50.0, graph=False, skip=False, steps=16),
        # one adaptation period of the half-size D3Q27 channel, 16-bit storage
        dict(name="period_d3q27_cylinder_f16s", kind="period", shape="cylinder", q=27, nx=128, ny=64, nz=64, lmax=3,
             storage="f16s", interp=0, re=100.0, graph=True, skip=True, steps=32),
        # a uniform periodic level (no refinement): the plain sweep
        dict(name="snapshot_d3q19_uniform_bf16s", kind="snapshot", shape="uniform", q=19, nx=160, ny=160, nz=160,
             lmax=1, storage="bf16s", interp=0, re=1000.0, graph=True, skip=False, steps=40),
        # a batch of 32 cavities of mixed size and lattice
        dict(name="batch_mixed_cavities_f16s", kind="batch", shape="cavity", q=0, nx=0, ny=0, nz=0, lmax=4,
             storage="f16s", interp=0, re=0.0, graph=True, skip=False, steps=50, members=32),
        # the largest: two adaptation periods' steps of the D3Q27 channel, 256 x 128 x 128 root cells, 9.3e5 blocks
        dict(name="period_d3q27_cylinder_f32s", kind="period", shape="cylinder", q=27, nx=256, ny=128, nz=128, lmax=3,
             storage="f32s", interp=0, re=200.0, graph=True, skip=True, steps=64),
    ]


def _log_int(rng, lo, hi, multiple):
    """an integer in [lo, hi], log-uniform, a multiple of `multiple`"""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return int(max(lo, min(hi, round(v / multiple) * multiple)))


def draw(rng):
    kind = rng.choice(("snapshot", "snapshot", "restart", "force", "period", "period", "window", "whole", "batch"))
    storage = rng.choice(("f64", "f32", "f32s", "f32s", "f16s", "bf16s"))
    c = dict(kind=kind, storage=storage, interp=0, graph=rng.random() < 0.75, skip=False,
             re=round(rng.uniform(100.0, 250.0), 1))
    if kind == "batch":
        c.update(shape="cavity", q=0, nx=0, ny=0, nz=0, lmax=4, re=0.0, storage=rng.choice(("f16s", "f32s", "f64")),
                 steps=rng.randint(10, 50), members=rng.randint(3, 32))
        return c
    two = rng.random() < 0.45
    c["q"] = 9 if two else rng.choice((19, 27))
    c["lmax"] = rng.randint(2, 4 if two else 3)
    if kind in ("force", "period"):
        c["shape"] = rng.choice(("cylinder", "fpsc")) if two else "cylinder"
        if c["shape"] == "fpsc":
            n = _log_int(rng, 128, 384, 128)
            c.update(nx=n, ny=n, nz=1, re=100.0)
        elif two:
            c.update(nx=_log_int(rng, 128, 1024, 16), ny=_log_int(rng, 64, 256, 8), nz=1)
        else:
            c.update(nx=_log_int(rng, 48, 144, 16), ny=_log_int(rng, 32, 80, 8), nz=_log_int(rng, 16, 80, 4))
        # the cylinder is 1/32 (2-D) or 1/16 of the length wide: a smaller one at a lower Reynolds number
        c["re"] = min(c["re"], 12.5 * max(4, c["nx"] // (32 if two else 16) // 4 * 4))
        c["steps"] = rng.randint(4, 40)
    elif kind in ("snapshot", "restart") and rng.random() < 0.3:
        side = (_log_int(rng, 64, 1024, 4), _log_int(rng, 64, 512, 4)) if two else \
            tuple(_log_int(rng, 32, 160, 4) for _ in range(3))
        c.update(shape="uniform", lmax=1, nx=side[0], ny=side[1], nz=1 if two else side[2], re=1000.0,
                 steps=rng.randint(1, 60))
    else:
        side = _log_int(rng, 32, 256, 4) if two else _log_int(rng, 32, 68, 4)
        c.update(shape="cavity", nx=side, ny=side, nz=1 if two else side, steps=rng.randint(1, 60))
    if kind == "window":
        c.update(lmax=max(2, c["lmax"]), steps=rng.randint(2, 20))
    if kind == "whole":
        c["steps"] = rng.randint(60, 300)
    c["interp"] = 1 if rng.random() < 0.25 and c["lmax"] > 1 else 0
    c["skip"] = c["interp"] == 0 and c["lmax"] > 1 and rng.random() < 0.5
    return c


# ------------------------------------------------------------------ set-ups
def _set_up(case, seed):
    """the `workloads.Case` of a case"""
    n = (case["nx"], case["ny"], case["nz"])
    dim = 2 if case["q"] == 9 else 3
    if case["shape"] == "fpsc":
        s = W.fpsc(case["nx"], case["lmax"], case["interp"], storage=case["storage"], seed=seed)
        return dataclasses.replace(s, noise=1e-6)
    if case["shape"] == "cylinder":
        side = max(4, n[0] // 32 // 4 * 4) if dim == 2 else max(4, n[0] // 16 // 4 * 4)
        s = W.cylinder(dim, case["q"], n[:dim], side, n[0] // 4 // 4 * 4, case["lmax"], case["re"],
                       storage=case["storage"], seed=seed, cap=int(np.prod(n[:dim])) // 4 ** dim * 24)
    else:
        s = W.cavity(dim, case["q"], n[0], case["lmax"], case["re"], storage=case["storage"], seed=seed)
        if case["shape"] == "uniform":
            root = tuple(v // 4 for v in n[:dim]) + (1,) * (3 - dim)
            # a viscosity of the benchmark's uniform level, whatever the size of this one
            s = dataclasses.replace(s, root=root, cap=int(np.prod(root)), periodic=(1, 1, 1 if dim == 3 else 0),
                                    nu0=0.0192, noise=1e-2)
    if case["kind"] in ("period", "whole"):
        # noise well below the criteria's thresholds, so that the flow and not the seed shapes the mesh
        s = dataclasses.replace(s, noise=1e-6)
    return dataclasses.replace(s, interp=case["interp"])


def _layer(s, level):
    """how far below the lid a cavity's blocks of `level` are refined, in finest cells"""
    return (4 << (s.lmax - 1)) * s.root[s.dim - 1] // (8 << level)


def _refine_lid(sim, s):
    """static refinement of a layer under the lid, by the caller's own tags"""
    for level in range(s.lmax - 1):
        m = sim.mesh()
        ax = s.dim - 1
        top = (4 << (s.lmax - 1)) * s.root[ax]
        width = 4 << (s.lmax - 1 - level)
        tags = np.zeros(sim.cap, np.int8)
        tags[(m["status"] == 0) & (m["level"] == level) & (m["X"][:, ax] + width > top - _layer(s, level))] = 2
        sim.tag(tags_in=tags)
        sim.adapt()


def _windows(s):
    """two regions of root blocks away from the lid's layer, one eighth to a quarter of the floor each"""
    b = np.arange(s.nroot)
    pos = np.stack((b % s.root[0], b // s.root[0] % s.root[1], b // (s.root[0] * s.root[1])), 1)[:, :s.dim]
    low = pos[:, -1] < max(1, s.root[s.dim - 1] // 3)
    left, right = pos[:, 0] < max(1, s.root[0] // 3), pos[:, 0] >= s.root[0] - max(1, s.root[0] // 3)
    return np.flatnonzero(low & left), np.flatnonzero(low & right)


def _simulation(case, s, stream=None):
    sim = abi.AmrLbm(s, stream=stream)
    sim.set_root_rho_u(s.initial_rho_u())
    if case["skip"]:
        sim.skip_parents(True)
    return sim


def _members(case, seed):
    for i in range(case["members"]):
        dim, side, lmax, re = BATCH_MEMBERS[i % len(BATCH_MEMBERS)]
        yield W.cavity(dim, 9 if dim == 2 else 19, side, lmax, re, storage=case["storage"], seed=seed + 1000 * i)


def prepare(case, seed):
    if case["kind"] == "batch":
        stream = torch.cuda.Stream()
        sims = []
        for s in _members(case, seed):
            sims.append(_simulation(case, s, stream))
            _refine_lid(sims[-1], s)
        return {"case": case, "sims": sims, "batch": abi.AmrBatch(sims)}
    s = _set_up(case, seed)
    if case["kind"] == "whole":  # a run's input: its set-up and its initial fields
        return {"case": case, "setup": s, "rho_u": s.initial_rho_u()}
    sim = _simulation(case, s)
    if case["shape"] == "cavity":
        _refine_lid(sim, s)
    for _ in range(s.dist_levels):  # near-wall refinement of the cylinder
        sim.tag(abi.TAG_DISTANCE, d_spec=s.d_spec, freeze=1)
        sim.adapt()
    state = {"case": case, "setup": s, "sim": sim}
    if case["kind"] == "period" and case["shape"] == "fpsc":
        for _ in range(24):  # the wake's refinement takes some periods to grow to its size
            sim.step(s.adapt_every, graph=True)
            _adapt_by_criterion(case, s, sim)
    if case["kind"] == "window":
        a, b = _windows(s)
        there, back = np.zeros(sim.cap, np.int8), np.zeros(sim.cap, np.int8)
        there[a], there[b] = -1, 1
        back[a], back[b] = 1, -1
        state["moves"] = (there, back)
        first = np.zeros(sim.cap, np.int8)
        first[a] = 1
        sim.tag(tags_in=first)
        sim.adapt()
    return state


def _adapt_by_criterion(case, s, sim):
    """the criterion's tags, and how many blocks were refined and coarsened"""
    if case["shape"] == "fpsc":
        tags = sim.tag(abi.TAG_LADDER, n_start=s.ladder[0], n_inc=s.ladder[1])
    else:
        tags = sim.tag(abi.TAG_VORTICITY_REL, theta=s.theta)
    try:
        st = sim.adapt()
    except abi.AmrError as e:  # no room for the refinement: the mesh stays as it is
        if e.code != abi.AMR_ERR_CAPACITY:
            raise
        return tags, np.array([-1, -1])
    return tags, np.array([st["n_refine"], st["n_coarsen"]])


def run(state):
    case = state["case"]
    kind, n, graph = case["kind"], case["steps"], case["graph"]
    if kind == "batch":
        state["batch"].step(n, graph=graph)
        return {"mass_mom": [g.mass_mom() for g in state["sims"]], "rho_u": state["sims"][-1].rho_u_out()}
    s = state["setup"]
    if kind == "whole":
        sim = abi.AmrLbm(s)
        sim.set_root_rho_u(state["rho_u"])
        if case["skip"]:
            sim.skip_parents(True)
        tags = []
        for _ in range(s.lmax):
            sim.step(n // s.lmax, graph=graph)
            tags.append(_adapt_by_criterion(case, s, sim)[0])
        out = {"tags": tags, "rho_u": sim.rho_u_out(), "mass_mom": sim.mass_mom()}
        sim.close()
        return out
    sim = state["sim"]
    if kind == "window":
        out = {}
        for key, tags in zip(("there", "back"), state["moves"]):
            out["tags_" + key] = sim.tag(tags_in=tags)
            st = sim.adapt()
            out["blocks_" + key] = np.array([st["n_refine"], st["n_coarsen"], st["n_reverted"], st["n_free"]])
            sim.step(n, graph=graph)
        out["rho_u"] = sim.rho_u_out()
        return out
    sim.step(n, graph=graph)
    if kind == "force":
        return {"force": sim.force(reset=True), "mass_mom": sim.mass_mom()}
    if kind == "restart":
        return sim.output()
    if kind == "period":
        tags, moved = _adapt_by_criterion(case, s, sim)
        out = {"tags": tags, "moved": moved, "vorticity": sim.crit(), "mass_mom": sim.mass_mom()}
        if case["shape"] != "fpsc":  # drag and lift runs look at the wake's vorticity, the channels write frames
            out["rho_u"] = sim.rho_u_out()
        return out
    return {"rho_u": sim.rho_u_out()}


# ------------------------------------------------------------------ what a pass cannot do without
def _level_blocks(s, shape):
    """blocks per level of the prepared mesh (the caller's or the near-wall refinement), from the geometry"""
    counts = [s.nroot - (int(s.solid.sum()) if s.solid is not None else 0)]
    if s.lmax == 1:
        return counts
    if shape == "cavity":
        ax = s.dim - 1
        for level in range(s.lmax - 1):
            layers = -(-_layer(s, level) // (4 << (s.lmax - 1 - level)))
            counts.append(int(np.prod(s.root[:ax])) * (2 ** level) ** ax * layers * 2 ** s.dim)
        return counts
    cells = s.root_cells
    sol = np.flatnonzero(s.solid)
    pos = np.stack((sol % s.root[0], sol // s.root[0] % s.root[1]), 1) * 4
    lo, hi = pos.min(0), pos.max(0) + 4
    for level in range(s.lmax - 1):
        w = 4.0 / 2 ** level
        x, y = (np.arange(cells[a] / w) * w for a in (0, 1))
        gx = np.maximum(np.maximum(lo[0] - (x + w), x - hi[0]), 0.0)[:, None]
        gy = np.maximum(np.maximum(lo[1] - (y + w), y - hi[1]), 0.0)[None, :]
        near = np.minimum(np.sqrt(gx ** 2 + gy ** 2), (cells[0] - (x + w))[:, None]) < s.d_spec / 2 ** level
        solid = ((x >= lo[0]) & (x < hi[0]))[:, None] & ((y >= lo[1]) & (y < hi[1]))[None, :]
        counts.append(int((near & ~solid).sum()) * (int(cells[2] / w) if s.dim == 3 else 1) * 2 ** s.dim)
    return counts


def _work_of(s, shape, steps, row_bytes):
    """updates of leaf cells, each population read and written once, and the rows read at the end"""
    blocks = _level_blocks(s, shape)
    updates = steps * W.mlups_updates(blocks, s.dim)
    leaf = sum((b - (blocks[L + 1] / 2 ** s.dim if L + 1 < len(blocks) else 0)) for L, b in enumerate(blocks)) * s.mb
    b = updates * 2 * s.q * STORAGE_BYTES[s.storage] + leaf * (row_bytes + s.q * STORAGE_BYTES[s.storage])
    return b, updates * 14.0 * s.q


def work(case):
    if case["kind"] == "batch":
        w = [_work_of(s, "cavity", case["steps"], 0) for s in _members(case, 0)]
        return {"bytes": sum(x[0] for x in w), "flops": sum(x[1] for x in w)}
    s = _set_up(case, 0)
    if case["kind"] == "whole":  # the first period is on the root level; what later ones refine follows from the flow
        s = dataclasses.replace(s, lmax=1)
        b, f = _work_of(s, case["shape"], case["steps"], 32)
        return {"bytes": b, "flops": f}
    row = {"restart": 8 * s.q + 40, "force": 0}.get(case["kind"], 32)
    b, f = _work_of(s, case["shape"], case["steps"] * (2 if case["kind"] == "window" else 1), row)
    return {"bytes": b, "flops": f}


# ------------------------------------------------------------------ 64-bit reference of the uniform level
def _velocity_set(q):
    """directions in the order of the populations, and weights"""
    if q == 9:
        c = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (-1, 0, 0), (0, -1, 0), (1, 1, 0), (-1, 1, 0), (-1, -1, 0), (1, -1, 0)]
        w = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4
        return c, w
    half = [(1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 0), (1, 0, 1), (0, 1, 1), (1, -1, 0), (1, 0, -1), (0, 1, -1),
            (1, 1, 1), (1, 1, -1), (1, -1, 1), (-1, 1, 1)]
    c = [(0, 0, 0)]
    for v in half:
        c += [v, tuple(-x for x in v)]
    by_speed = {19: (1 / 3, 1 / 18, 1 / 36), 27: (8 / 27, 2 / 27, 1 / 54, 1 / 216)}[q]
    return c[:q], [by_speed[sum(x * x for x in v)] for v in c[:q]]


def exact(case, seed):
    """BGK on the uniform periodic level in 64 bits.  Refined meshes give None: their result is that of the method's
    own rescaled interpolation and averaging between levels, which has no plain counterpart."""
    if case["shape"] != "uniform":
        return None
    s = _set_up(case, seed)
    device = "cuda" if torch.cuda.is_available() else "cpu"
    c, w = _velocity_set(s.q)
    bx, by, bz = s.root
    mz = 4 if s.dim == 3 else 1
    ru = torch.from_numpy(s.initial_rho_u()).to(device)
    ru = ru.view(bz, by, bx, mz, 4, 4, 4).permute(6, 0, 3, 1, 4, 2, 5).reshape(4, bz * mz, by * 4, bx * 4)

    def equilibrium(p, rho, u, uu):
        cu = sum(c[p][a] * u[a] for a in range(3))
        return w[p] * rho * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * uu)

    def moments(f):
        rho = sum(f)
        return rho, [sum(c[p][a] * f[p] for p in range(s.q) if c[p][a]) / rho if a < s.dim else torch.zeros_like(rho)
                     for a in range(3)]

    rho, u = ru[0], [ru[1], ru[2], ru[3]]
    f = [equilibrium(p, rho, u, sum(x * x for x in u)) for p in range(s.q)]
    omega = 1.0 / (0.5 + 3.0 * s.nu0)
    for _ in range(case["steps"]):
        rho, u = moments(f)
        uu = sum(x * x for x in u)
        for p in range(s.q):
            new = f[p] + omega * (equilibrium(p, rho, u, uu) - f[p])
            f[p] = torch.roll(new, (c[p][2], c[p][1], c[p][0]), (0, 1, 2))

    def rows(x):  # (..., z, y, x) of the grid to (block, cell) order
        x = x.view(-1, bz, mz, by, 4, bx, 4).permute(1, 3, 5, 2, 4, 6, 0)
        return x.reshape(s.nroot * s.mb, -1).cpu().numpy()

    rho, u = moments(f)
    if case["kind"] == "restart":
        return {"blk": None, "cell": None, "rho": rows(rho)[:, 0], "u": rows(torch.stack(u[:s.dim])),
                "f": rows(torch.stack(f))}
    return {"rho_u": rows(torch.stack([rho] + u))}
