"""The work that users of the framework have it do, as timed cases.

A case is a dict of plain values.  ``kind`` says which public entry points
it goes through:

  lattice   one ``Stefan`` handle: ``step`` and the queries after it
  batch     ``StefanBatch``: many uneven lattices advanced together
  gradient  ``HotWallFront``: forward tape and reverse sweep (a training
            step: front out, gradients back)
  noalloc   ``step_noalloc``: one step from a caller's state to a caller's
            buffer (a serving loop's call)

``heat`` names the physical set-up: "melt" (x = 0 at +1, x = nx - 1 at
-0.5, the remaining walls periodic or bounce-back: the 1D bar, the planar
front, the cavity and the cube) or "freeze" (the quarter cavity or octant
cooled to -2 on its low faces with symmetry on its high ones).  Lattices
start from a developed front a few cells from the hot (cold) wall, with a
seeded wiggle and noise of 1e-3, which is where a run spends its steps.

``exact`` is the method of arXiv 2505.13097 (Algorithms 1 to 3 with the
closures of Section 4.2) in plain torch, 64 bits, sharing no code with the
framework.
"""
import math
import types

import numpy as np
import torch

import synth
from paper_2505_13097_amd import (HotWallFront, Stefan, StefanBatch,
                                  step_noalloc, variant_names)

DEVICE = "cuda"


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # the 1D melting bar (FP64, 256 nodes): hundreds of steps between
        # two looks at temperature and front; pure latency
        dict(name="bar1d_256", kind="lattice", heat="melt", q=3, nx=256,
             ny=1, nz=1, storage="f64", scheme="irebm", side="periodic",
             tau=0.8, ste=0.1, cells=5.1, steps=500, variant="", again=True,
             out="fields"),
        # the paper's 2D freezing case at its smallest tabulated size, FP64,
        # symmetry walls
        dict(name="freeze2d_q5_201", kind="lattice", heat="freeze", q=5,
             nx=201, ny=201, nz=1, storage="f64", scheme="irebm", side="",
             tau=0.84, ste=0.0521, cells=1.0, steps=100, variant="",
             again=True, out="fields"),
        # the explicit scheme on the largest 2D freezing lattice
        dict(name="freeze2d_q9_801_eebm", kind="lattice", heat="freeze",
             q=9, nx=801, ny=801, nz=1, storage="f64", scheme="eebm",
             side="", tau=0.84, ste=0.0521, cells=4.0, steps=60, variant="",
             again=True, out="fields"),
        # the inner-loop scheme on the 2D freezing lattice
        dict(name="freeze2d_q9_201_ilfbm", kind="lattice", heat="freeze",
             q=9, nx=201, ny=201, nz=1, storage="f64", scheme="ilfbm",
             side="", tau=0.84, ste=0.0521, cells=1.0, steps=3, variant="",
             again=False, out="fields"),
        # a ragged cavity in FP64 with its statistics, default settings: an
        # ordinary desktop-size study
        dict(name="cavity_q9_1001x777_f64", kind="lattice", heat="melt",
             q=9, nx=1001, ny=777, nz=1, storage="f64", scheme="irebm",
             side="bounceback", tau=0.6, ste=0.3, cells=1.5, steps=50,
             variant="", again=True, out="stats"),
        # the planar front of 2048 x 2048, FP32 populations, default settings
        dict(name="planar_q5_2048_f32", kind="lattice", heat="melt", q=5,
             nx=2048, ny=2048, nz=1, storage="f32", scheme="irebm",
             side="periodic", tau=0.7, ste=0.05, cells=1.0, steps=50,
             variant="", again=False, out="state"),
        # the headline cavity, 8192 x 8192, in the benchmark's variant
        dict(name="cavity_q9_8192_f32", kind="lattice", heat="melt", q=9,
             nx=8192, ny=8192, nz=1, storage="f32", scheme="irebm",
             side="bounceback", tau=0.6, ste=0.144197, cells=1.5, steps=10,
             variant="128x4/t2/r32/nt", again=False, out="state"),
        # uneven lattices advanced together, the benchmark's schedule, their
        # statistics and fronts read after a stretch of steps
        dict(name="batch48_q5_f32", kind="batch", count=48, q=5, lo=64,
             hi=1024, by=64, storage="f32", scheme="irebm", steps=60,
             variant="128x2/t2s/r96/nt", graph=20),
        # the cube of 512 nodes a side on D3Q19, the benchmark's variant
        dict(name="cube_q19_512_f32", kind="lattice", heat="melt", q=19,
             nx=512, ny=512, nz=512, storage="f32", scheme="irebm",
             side="bounceback", tau=0.6, ste=0.144197, cells=1.5, steps=4,
             variant="256x1/npt2/z4/nt", again=False, out="state"),
        # the freezing octant at its tabulated size, FP64, default settings
        dict(name="octant_q7_101_f64", kind="lattice", heat="freeze", q=7,
             nx=101, ny=101, nz=101, storage="f64", scheme="irebm", side="",
             tau=0.84, ste=0.0521, cells=0.5, steps=20, variant="",
             again=True, out="state"),
        # one training step of the hot-wall profile
        dict(name="gradient_q5_512_f32", kind="gradient", q=5, nx=512,
             ny=512, storage="f32", tau=0.8, ste=0.2, cells=1.5, steps=64,
             interval=8),
        # one step of a small lattice with no handle
        dict(name="noalloc_q5_96x64_f32", kind="noalloc", heat="melt", q=5,
             nx=96, ny=64, nz=1, storage="f32", scheme="irebm",
             side="bounceback", tau=0.7, ste=0.2, cells=1.0, steps=1,
             variant=""),
    ]


def draw(rng):
    """One more case of the same ranges."""
    def log_int(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    def log_real(a, b):
        return round(math.exp(rng.uniform(math.log(a), math.log(b))), 5)

    what = rng.choice(("bar", "freeze", "freeze", "planar", "cavity",
                       "cavity", "ilfbm", "batch", "cube", "octant",
                       "gradient", "noalloc"))
    f = rng.choice(("f32", "f64"))
    if what == "bar":
        n = log_int(65, 2048)
        return dict(kind="lattice", heat="melt", q=3, nx=n, ny=1, nz=1,
                    storage="f64", scheme=rng.choice(("irebm", "irebm",
                                                      "eebm")),
                    side="periodic", tau=round(rng.uniform(0.55, 1.0), 3),
                    ste=log_real(0.05, 1.0),
                    cells=round(rng.uniform(1.0, 6.0), 2),
                    steps=rng.randrange(100, 600), variant="", again=True,
                    out="fields")
    if what == "freeze":
        n = log_int(101, 801)
        return dict(kind="lattice", heat="freeze", q=rng.choice((5, 9)),
                    nx=n, ny=n, nz=1, storage="f64",
                    scheme=rng.choice(("irebm", "irebm", "eebm")), side="",
                    tau=0.84, ste=0.0521,
                    cells=round(0.02 * (n - 1) / 4.0, 3),
                    steps=rng.randrange(30, 120), variant="", again=True,
                    out="fields")
    if what == "ilfbm":
        if rng.random() < 0.5:
            return dict(kind="lattice", heat="melt", q=3,
                        nx=log_int(101, 801), ny=1, nz=1, storage="f64",
                        scheme="ilfbm", side="periodic", tau=0.62,
                        ste=log_real(0.1, 0.5), cells=1.0,
                        steps=rng.randrange(10, 60), variant="", again=False,
                        out="fields")
        n = log_int(81, 401)
        return dict(kind="lattice", heat="freeze", q=9, nx=n, ny=n, nz=1,
                    storage="f64", scheme="ilfbm", side="", tau=0.84,
                    ste=0.0521, cells=1.0, steps=rng.randrange(2, 5),
                    variant="", again=False, out="fields")
    if what in ("planar", "cavity"):
        nx, ny = log_int(150, 4096), log_int(150, 4096)
        q = 5 if what == "planar" else 9
        return dict(kind="lattice", heat="melt", q=q, nx=nx, ny=ny, nz=1,
                    storage=f, scheme=rng.choice(("irebm", "irebm", "eebm")),
                    side="periodic" if what == "planar" else "bounceback",
                    tau=round(rng.uniform(0.55, 1.0), 3),
                    ste=log_real(0.03, 1.0),
                    cells=round(rng.uniform(0.75, 2.0), 2),
                    steps=rng.randrange(11, 41),
                    variant=rng.choice(("", "", "128x4/t2/r32/nt")),
                    again=False, out="state")
    if what == "batch":
        return dict(kind="batch", count=rng.randrange(9, 48), q=5, lo=64,
                    hi=rng.choice((320, 640, 1024)), by=rng.choice((64, 37)),
                    storage="f32", scheme=rng.choice(("irebm", "irebm",
                                                      "eebm")),
                    steps=rng.randrange(40, 61),
                    variant=rng.choice(("", "128x2/t2s/r96/nt")),
                    graph=rng.choice((0, 20)))
    if what == "cube":
        return dict(kind="lattice", heat="melt", q=rng.choice((7, 19)),
                    nx=log_int(120, 400), ny=log_int(60, 300),
                    nz=log_int(60, 300), storage=f,
                    scheme=rng.choice(("irebm", "irebm", "eebm")),
                    side="bounceback", tau=0.6, ste=log_real(0.03, 1.0),
                    cells=round(rng.uniform(0.75, 2.0), 2),
                    steps=rng.randrange(3, 9), variant="", again=False,
                    out="state")
    if what == "octant":
        n = log_int(61, 161)
        return dict(kind="lattice", heat="freeze", q=rng.choice((7, 19)),
                    nx=n, ny=n, nz=n, storage="f64",
                    scheme=rng.choice(("irebm", "irebm", "eebm")), side="",
                    tau=0.84, ste=0.0521,
                    cells=round(0.02 * (n - 1) / 4.0, 3),
                    steps=rng.randrange(8, 24), variant="", again=True,
                    out="state")
    if what == "gradient":
        return dict(kind="gradient", q=rng.choice((5, 5, 9)),
                    nx=log_int(100, 600), ny=log_int(100, 600), storage=f,
                    tau=round(rng.uniform(0.6, 0.9), 3),
                    ste=log_real(0.1, 0.5),
                    cells=round(rng.uniform(1.5, 3.0), 2),
                    steps=rng.randrange(30, 81),
                    interval=rng.choice((1, 6, 8)))
    q = rng.choice((5, 9))
    return dict(kind="noalloc", heat="melt", q=q, nx=log_int(64, 512),
                ny=log_int(64, 512), nz=1, storage=f,
                scheme=rng.choice(("irebm", "irebm", "eebm")),
                side="bounceback", tau=round(rng.uniform(0.55, 1.0), 3),
                ste=log_real(0.05, 1.0),
                cells=round(rng.uniform(0.75, 2.0), 2), steps=1, variant="")


# ------------------------------------------------- lattices and their inputs

def _dim(q):
    return {3: 1, 5: 2, 9: 2, 7: 3, 19: 3}[q]


def _spec(c):
    """Walls, spacing and melting width of a lattice, as plain values."""
    dim = _dim(c["q"])
    if c["heat"] == "freeze":
        dx = 4.0 / (c["nx"] - 1)
        bc = ["dirichlet", "neumann"] * 3
        wall = [-2.0, 0.0] * 3
    else:
        dx = 1.0 / (c["nx"] - 1)
        bc = ["dirichlet", "dirichlet"] + [c["side"]] * 4
        wall = [1.0, -0.5, 0.0, 0.0, 0.0, 0.0]
    if dim < 3:
        bc[4:] = ["periodic"] * 2
    if dim < 2:
        bc[2:4] = ["periodic"] * 2
    # one cell of temperature is the spacing of the melting set-ups and of
    # the freezing ones alike (the paper's caption: 2e-2 is about dx at 201)
    return types.SimpleNamespace(
        q=c["q"], nx=c["nx"], ny=c["ny"], nz=c["nz"], dx=dx, bc=bc,
        wall=wall, tau=c["tau"], ste=c["ste"], delta=c["cells"] * dx,
        scheme=c["scheme"], tol=1e-12, max_it=200 if c["scheme"] == "ilfbm"
        else 32, profile=None)


def _problem(c, s, T0=None):
    p = synth.Problem(
        dim=_dim(s.q), q=s.q, nx=s.nx, ny=s.ny, nz=s.nz, tau=s.tau,
        ste=s.ste, delta=s.delta, bc=tuple(s.bc[:4]),
        wall_T=tuple(s.wall[:4]), bc_z=tuple(s.bc[4:]),
        wall_T_z=tuple(s.wall[4:]), tol=s.tol, max_it=s.max_it,
        storage=c["storage"], scheme=s.scheme, dx=s.dx, T0=T0)
    return p


def _temperature(c, s, seed, dev=None):
    """A developed front: (nz, ny, nx) temperatures, walls at theirs."""
    dev = dev or DEVICE
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    f64 = dict(dtype=torch.float64, device=dev)
    x = torch.arange(s.nx, **f64).view(1, 1, -1)
    y = torch.arange(s.ny, **f64).view(1, -1, 1)
    z = torch.arange(s.nz, **f64).view(-1, 1, 1)
    r = torch.rand(4, generator=g, **f64)
    at = 4.0 + 6.0 * r[0]       # cells from the wall to the front
    at = at * (1.0 + 0.15 * torch.sin(
        2 * math.pi * (2 * y / max(s.ny, 2) + z / max(s.nz, 2) + r[1])))
    if c["heat"] == "freeze":
        d = x
        if _dim(s.q) > 1:
            d = torch.minimum(d, y)
        if _dim(s.q) > 2:
            d = torch.minimum(d, z)
        T = torch.where(d < at, -2.0 * (1 - d / at),
                        1 - torch.exp(-(d - at) / (2 * at)))
    else:
        T = torch.where(x < at, 1 - x / at,
                        -0.5 * (1 - torch.exp(-(x - at) / (2 * at))))
    T = T.expand(s.nz, s.ny, s.nx).contiguous()
    T += 1e-3 * (2 * torch.rand(T.shape, generator=g, **f64) - 1)
    for k in reversed(range(2 * _dim(s.q))):
        if s.bc[k] == "dirichlet":
            T.select(2 - k // 2, -(k % 2)).fill_(s.wall[k])
    return T


def _weights(q):
    if q == 3:
        return [2 / 3] + [1 / 6] * 2
    if q == 5:
        return [1 / 3] + [1 / 6] * 4
    if q == 9:
        return [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4
    if q == 7:
        return [0.0] + [1 / 6] * 6
    return [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12


def _velocities(q):
    if q == 3:
        return [(0, 0, 0), (1, 0, 0), (-1, 0, 0)]
    if q in (5, 9):
        v = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (-1, 0, 0), (0, -1, 0),
             (1, 1, 0), (-1, 1, 0), (-1, -1, 0), (1, -1, 0)]
        return v[:q]
    v = [(1, 0, 0), (0, 1, 0), (0, 0, 1)]
    e = [(1, 1, 0), (1, -1, 0), (1, 0, 1), (1, 0, -1), (0, 1, 1), (0, 1, -1)]

    def neg(a):
        return [tuple(-b for b in t) for t in a]
    return ([(0, 0, 0)] + v + neg(v) + e + neg(e))[:q]


def _planes(s, T, dtype):
    """Equilibrium post-collision populations of a temperature field."""
    w = _weights(s.q)
    om = torch.empty((s.q,) + tuple(T.shape), dtype=dtype, device=T.device)
    if s.scheme == "eebm":
        om[0] = T + (T > 0) / s.ste - (1 - w[0]) * T
    else:
        om[0] = w[0] * T
    for i in range(1, s.q):
        om[i] = w[i] * T
    return om


def _torch_type(storage):
    return torch.float64 if storage == "f64" else torch.float32


def _shape(s):
    return ((s.nz,) if _dim(s.q) == 3 else ()) + (s.ny, s.nx)


# ------------------------------------------------------------ prepare and run

def prepare(case, seed):
    c = dict(case)
    st = types.SimpleNamespace(c=c)
    if c["kind"] == "batch":
        st.specs, fields = _batch_inputs(c, seed)
        st.b = StefanBatch([_problem(dict(c, heat="melt"), s, T0)
                            for s, T0 in zip(st.specs, fields)])
        if c["variant"] or c["graph"]:
            v = (variant_names(c["q"], c["storage"]).index(c["variant"])
                 if c["variant"] else -1)
            st.b.set_schedule(v, 0, c["graph"])
        return st
    if c["kind"] == "gradient":
        s, wall, target = _gradient_inputs(c, seed)
        st.prob = _problem(c, s, np.full((s.ny, s.nx), -0.5))
        t = _torch_type(c["storage"])
        st.wall = wall.to(t).requires_grad_()
        st.ste = torch.tensor(s.ste, dtype=torch.float64, requires_grad=True)
        st.delta = torch.tensor(s.delta, dtype=torch.float64,
                                requires_grad=True)
        st.target = target
        return st
    s = _spec(c)
    T = _temperature(c, s, seed)
    if c["kind"] == "noalloc":
        st.prob = _problem(c, s)
        st.src = _planes(s, T, _torch_type(c["storage"]))
        st.dst = torch.empty_like(st.src)
        return st
    v = -1
    if c["variant"]:
        v = variant_names(c["q"], c["storage"]).index(c["variant"])
    if c["scheme"] == "ilfbm":
        # its state holds the liquid fraction too: built from the field
        st.handle = Stefan(_problem(c, s, T.view(_shape(s)).cpu().numpy()), v)
    else:
        st.handle = Stefan(_problem(c, s), v)
        om = _planes(s, T, _torch_type(c["storage"])).view(
            (s.q,) + _shape(s))
        st.handle.set_state(om)
        if c["again"]:
            st.start = om
    torch.cuda.synchronize()
    return st


def run(st):
    c = st.c
    if c["kind"] == "batch":
        st.b.step(c["steps"])
        stats = st.b.stats()
        fronts = [st.b.front(k) for k in range(len(st.b))]
        return {"front": np.concatenate(fronts).astype(np.float32),
                "energy": np.array([x["energy"] for x in stats], np.float32),
                "nonconverged": np.array([x["nonconverged"] for x in stats])}
    if c["kind"] == "gradient":
        st.wall.grad = st.ste.grad = st.delta.grad = None
        xf = HotWallFront.apply(st.wall, st.ste, st.delta, st.prob,
                                c["steps"], c["interval"])
        loss = 0.5 * ((xf - st.target) ** 2).sum()
        loss.backward()
        t = _torch_type(c["storage"])
        return {"front": xf.detach().to(t), "wall": st.wall.grad,
                "ste": st.ste.grad.to(t), "delta": st.delta.grad.to(t)}
    if c["kind"] == "noalloc":
        step_noalloc(st.prob, st.src, st.dst)
        return st.dst
    h = st.handle
    if c["again"]:
        h.set_state(st.start)       # from the same start in every pass
    if c["out"] == "stats":
        h.reset_stats()
        r = h.step(c["steps"], stats=True)
        return {"state": _state_of(h), "energy": r["energy"],
                "flux": np.array([r["flux_in"], r["flux_out"]]),
                "nonconverged": r["nonconverged"]}
    h.step(c["steps"])
    if c["out"] == "state":
        return _state_of(h)
    r = {"T": h.temperature(), "front": h.front()}
    if c["scheme"] == "ilfbm":
        r["liquid"] = h.liquid()
    return r


def _state_of(h):
    """The handle's current planes, where they lie in its workspace."""
    t = _torch_type(h.prob.storage)
    at = h.state_ptr() - h.workspace.data_ptr()
    n = h.prob.q * h.prob.nodes * t.itemsize
    return h.workspace[at:at + n].view(t).view((h.prob.q,)
                                               + h.prob.field_shape)


def _batch_inputs(c, seed):
    """Sizes from the case (the same for every seed); Stefan number, width
    and relaxation time of each lattice, and its field, from the seed."""
    size = np.random.Generator(np.random.PCG64(c["count"] * 1000 + c["by"]))
    rng = np.random.Generator(np.random.PCG64(seed))
    choice = np.arange(c["lo"], c["hi"] + 1, c["by"])
    specs, fields = [], []
    for _ in range(c["count"]):
        n = int(size.choice(choice))
        d = dict(c, heat="melt", side="periodic", nx=n, ny=n, nz=1,
                 tau=float(rng.uniform(0.55, 1.0)),
                 ste=float(math.exp(rng.uniform(math.log(0.01), 0.0))),
                 cells=float(rng.uniform(0.5, 2.0)))
        s = _spec(d)
        specs.append(s)
        fields.append(_temperature(d, s, int(rng.integers(1 << 30)))[0]
                      .cpu().numpy())
    return specs, fields


def _gradient_inputs(c, seed):
    s = _spec(dict(c, heat="melt", side="periodic", nz=1, scheme="irebm"))
    rng = np.random.Generator(np.random.PCG64(seed))
    y = np.arange(s.ny) / s.ny
    w = 1.0 + sum(0.05 * rng.uniform(-1, 1)
                  * np.sin(2 * np.pi * (k * y + rng.uniform()))
                  for k in range(1, 5))
    s.profile = torch.from_numpy(w).to(_torch_type(c["storage"])).double()
    target = torch.from_numpy(s.dx * (3 + rng.uniform(0, 2, s.ny)))
    return s, torch.from_numpy(w), target


# ------------------------------------------------------------------- the work

def work(case):
    """Each state (or field) read once and written once, however many steps
    lie between, and the arithmetic of the node updates: a population sum
    for the temperature and one for the zeroth moment, and a multiply-add
    per population (a Newton solve, rare, is not counted)."""
    c = case
    b = 8 if c.get("storage") == "f64" else 4
    per_node = 4 * c["q"] + 10
    if c["kind"] == "batch":
        n = sum(s.nx * s.ny for s in _batch_sizes(c))
        return {"bytes": 2 * n * c["q"] * b, "flops": n * per_node
                * c["steps"]}
    n = c["nx"] * c["ny"] * c.get("nz", 1)
    flops = n * per_node * c["steps"]
    if c["kind"] == "gradient":
        # forward, and the reverse step's own arithmetic with its forward
        # values; the tape is not part of the least traffic
        return {"bytes": n * c["q"] * (b + 8), "flops": 4 * flops}
    return {"bytes": 2 * n * c["q"] * b, "flops": flops}


def _batch_sizes(c):
    size = np.random.Generator(np.random.PCG64(c["count"] * 1000 + c["by"]))
    choice = np.arange(c["lo"], c["hi"] + 1, c["by"])
    for _ in range(c["count"]):
        n = int(size.choice(choice))
        yield types.SimpleNamespace(nx=n, ny=n)


# --------------------------------------------------- the method, in 64 bits

def exact(case, seed):
    c = case
    if c["kind"] == "batch":
        if c["count"] * c["steps"] > 3000:      # one lattice after another
            return None
        specs, fields = _batch_inputs(c, seed)
        front, energy = [], []
        for s, T0 in zip(specs, fields):
            T = torch.from_numpy(T0).to(DEVICE)[None]
            om = _planes(s, T, torch.float64)
            for _ in range(c["steps"]):
                om = _step(s, om)
            front.append(_front(s, om).cpu().numpy().reshape(-1))
            energy.append(_energy(s, om))
        return {"front": np.concatenate(front), "energy": np.array(energy),
                "nonconverged": None}
    if c["kind"] == "gradient":
        return _exact_gradient(c, seed)
    s = _spec(c)
    if s.nx * s.ny * s.nz * s.q > 3 << 30:
        return None
    T = _temperature(c, s, seed)
    if s.scheme == "ilfbm":
        om, lf = _planes(s, T, torch.float64), (T > 0).double()
        del T
        for _ in range(c["steps"]):
            om, lf = _step_ilfbm(s, om, lf)
        T = om.sum(0)
        return {"T": T.view(_shape(s)).cpu(),
                "front": (s.dx * _trapezoid(lf)).cpu().reshape(-1),
                "liquid": lf.view(_shape(s)).cpu()}
    om = _planes(s, T, _torch_type(c["storage"])).double()
    del T
    for _ in range(c["steps"]):
        om = _step(s, om)
    if c["kind"] == "noalloc":
        return om
    state = om.view((s.q,) + _shape(s))
    if c["out"] == "state":
        return state
    if c["out"] == "stats":
        return {"state": state, "energy": _energy(s, om), "flux": None,
                "nonconverged": None}
    m0 = om.sum(0)
    T = _theta(s, m0) if s.scheme == "eebm" else m0
    return {"T": T.view(_shape(s)).cpu(),
            "front": _front(s, om).cpu().reshape(_shape(s)[:-1])}


def _phi(s, T):
    return torch.sigmoid(2.0 * T / s.delta)


def _theta(s, H):
    return torch.where(H < 0, H, (H - 1.0 / s.ste).clamp_min(0.0))


def _trapezoid(v):
    return v.sum(-1) - 0.5 * (v[..., 0] + v[..., -1])


def _front(s, om):
    m0 = om.sum(0)
    if s.scheme == "eebm":
        return s.dx * _trapezoid((s.ste * m0).clamp(0.0, 1.0))
    return s.dx * _trapezoid(_phi(s, m0))


def _energy(s, om):
    m0 = om.sum(0)
    if s.scheme == "eebm":
        return float(m0.sum())
    return float((m0 + _phi(s, m0) / s.ste).sum())


def _root(s, T, m0):
    """t + phi(t)/Ste = m0 + phi(T)/Ste at every node, by bisection and
    Newton steps."""
    c = m0 + _phi(s, T) / s.ste
    t = m0.clone()
    band = 45.0 * s.delta
    act = ~(((T < -band) & (m0 < -band)) | ((T > band) & (m0 > band)))
    ca = c[act]
    lo, hi = ca - 1.0 / s.ste, ca.clone()
    for _ in range(46):
        mid = 0.5 * (lo + hi)
        up = mid + _phi(s, mid) / s.ste > ca
        hi = torch.where(up, mid, hi)
        lo = torch.where(up, lo, mid)
    ta = 0.5 * (lo + hi)
    for _ in range(3):
        p = _phi(s, ta)
        ta = ta - (ta + p / s.ste - ca) / (
            1.0 + 2.0 * p * (1 - p) / (s.delta * s.ste))
    t[act] = ta
    return t


def _close(s, q, pulled, T, target):
    """The closures of Section 4.2 on the list q of streamed populations
    (changed in place); pulled(i) is the node's own collision."""
    dim = _dim(s.q)
    e, w = _velocities(s.q), _weights(s.q)
    n = (s.nx, s.ny, s.nz)
    shape, dev = q[0].shape, q[0].device
    opp = [e.index(tuple(-a for a in v)) for v in e]

    def edge(k):
        """nodes on wall k as a broadcastable mask"""
        a = k // 2
        m = torch.zeros(n[a], dtype=torch.bool, device=dev)
        m[-(k % 2)] = True
        return m.view([-1 if 2 - d == a else 1 for d in range(3)])

    walls = [k for k in range(2 * dim) if s.bc[k] != "periodic"]
    if not walls:
        return
    no = torch.zeros((1, 1, 1), dtype=torch.bool, device=dev)
    known, bounce = [], []
    for v in e:
        miss, other = no, no
        for k in walls:
            if v[k // 2] == (1 if k % 2 == 0 else -1):
                miss = miss | edge(k)
                if s.bc[k] != "bounceback":
                    other = other | edge(k)
        known.append(~miss)
        bounce.append(miss & ~other)
    done = list(known)
    streamed = list(q)
    for i in range(1, s.q):
        m = bounce[i] & known[opp[i]]
        if s.bc.count("bounceback"):
            q[i] = torch.where(m, streamed[opp[i]], q[i])
        done[i] = known[i] | m
    on = [edge(k) if k in walls and s.bc[k] == "dirichlet" else no
          for k in range(6)]
    share, D = no, None
    for k in reversed(range(2 * dim)):
        if k in walls and s.bc[k] == "dirichlet":
            TD = torch.full((1, 1, 1), s.wall[k], dtype=torch.float64,
                            device=dev)
            if k == 0 and s.profile is not None:
                TD = s.profile.to(dev).view(1, -1, 1)
            val = target(TD)
            D = val if D is None else torch.where(on[k], val, D)
            share = share | on[k]
    if "neumann" in s.bc:
        ix = [torch.arange(m, device=dev) for m in n]
        mirror = no
        for k in walls:
            if s.bc[k] == "neumann":
                ix[k // 2][-(k % 2)] = 1 if k % 2 == 0 else n[k // 2] - 2
                mirror = mirror | edge(k)
        M = sum(streamed)[ix[2]][:, ix[1]][:, :, ix[0]]
        D = M if D is None else torch.where(share, D, M)
        share = share | mirror
    if D is not None:
        D = D.expand(shape)
        wu = torch.zeros((1, 1, 1), dtype=torch.float64, device=dev)
        for i in range(s.q):
            D = D - torch.where(done[i], q[i], 0.0)
            wu = wu + (~done[i]).double() * w[i]
        wu = torch.where(wu > 0, wu, 1.0)
        for i in range(1, s.q):
            q[i] = torch.where(share & ~done[i], D * (w[i] / wu), q[i])
            done[i] = done[i] | share
    for i in range(1, s.q):
        if bool((~done[i]).any()):
            q[i] = torch.where(done[i], q[i], pulled(opp[i]))


def _streamed(s, om):
    return [torch.roll(om[i], (v[2], v[1], v[0]), (0, 1, 2)) if any(v)
            else om[i] for i, v in enumerate(_velocities(s.q))]


def _step(s, om):
    """One step of Algorithm 3 (or 2) on the post-collision planes."""
    w, a = _weights(s.q), 1.0 - 1.0 / s.tau
    T = sum(om[i] for i in range(s.q))
    q = _streamed(s, om)
    if s.scheme == "eebm":
        _close(s, q, lambda i: om[i], T,
               lambda TD: TD + (TD > 0).double() / s.ste)
        H = sum(q)
        th = _theta(s, H)
        f = [a * q[i] + (w[i] / s.tau) * th for i in range(s.q)]
        f[0] = a * q[0] + (H - (1 - w[0]) * th) / s.tau
        return torch.stack(f)
    _close(s, q, lambda i: om[i], T,
           lambda TD: TD + (_phi(s, TD) - _phi(s, T)) / s.ste)
    m0 = sum(q)
    with torch.no_grad():
        t = _root(s, T, m0)
        p = _phi(s, t)
        J = 1.0 + 2.0 * p * (1 - p) / (float(s.delta) * float(s.ste))
    if om.requires_grad:
        # a Newton step from the root: its derivative is the root's
        t = t - (t + _phi(s, t) / s.ste - m0 - _phi(s, T) / s.ste) / J
        p = _phi(s, t)
    src = (_phi(s, T) - p) / s.ste
    f = [q[i] + w[i] * src for i in range(s.q)]
    M = sum(f)
    if om.requires_grad:
        return torch.stack([a * f[i] + (w[i] / s.tau) * M
                            for i in range(s.q)])
    out = torch.empty_like(om)
    for i in range(s.q):
        out[i] = a * f[i] + (w[i] / s.tau) * M
    return out


def _step_ilfbm(s, om, lf):
    """One step of Algorithm 1: the inner loop on the liquid fraction."""
    w, a = _weights(s.q), 1.0 - 1.0 / s.tau
    lp = lf
    for _ in range(s.max_it):
        src = (lf - lp) / s.ste
        col = torch.stack([om[i] + w[i] * src for i in range(s.q)])
        q = _streamed(s, col)
        _close(s, q, lambda i: col[i], None, lambda TD: TD)
        m0 = sum(q)
        ln = (s.ste * (m0 + lp / s.ste)).clamp(0.0, 1.0)
        change = float((ln - lp).abs().max())
        lp = ln
        if change <= s.tol:
            break
    return torch.stack([a * q[i] + (w[i] / s.tau) * m0
                        for i in range(s.q)]), lp


def _exact_gradient(c, seed):
    s, wall, target = _gradient_inputs(c, seed)
    if s.nx * s.ny * s.q * c["steps"] > 1 << 28:
        return None
    wall = s.profile.clone().to(DEVICE).requires_grad_()
    ste = torch.tensor(s.ste, dtype=torch.float64, device=DEVICE,
                       requires_grad=True)
    delta = torch.tensor(s.delta, dtype=torch.float64, device=DEVICE,
                         requires_grad=True)
    s.profile, s.ste, s.delta = wall, ste, delta
    T = torch.full((1, s.ny, s.nx), -0.5, dtype=torch.float64, device=DEVICE)
    T = torch.cat([wall.view(1, -1, 1), T[:, :, 1:]], dim=2)
    om = torch.stack([v * T for v in _weights(s.q)])
    for _ in range(c["steps"]):
        om = _step(s, om)
    xf = _front(s, om).view(-1)
    loss = 0.5 * ((xf - target.to(DEVICE)) ** 2).sum()
    loss.backward()
    return {"front": xf.detach().cpu(), "wall": wall.grad.cpu(),
            "ste": ste.grad.cpu(), "delta": delta.grad.cpu()}
