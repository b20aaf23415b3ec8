"""The framework's working set as measurable cases.

listed()             what users of the framework have it do, from the smallest call to the largest
draw(rng)            one more case from the same ranges
prepare(case, seed)  what a user's program holds before the call (contexts and inputs, on the GPU)
run(state)           one pass through the public entry points
work(case)           bytes and operations a pass cannot do without
exact(case, seed)    the same outputs in 64-bit torch, without the framework's code

Kinds of cases:
  mpm      Simulator.step from a given state: the environment step of a control loop
  grad     MpmRollout and BlobLoss forward and backward: one iteration of a policy optimisation
  gas      GasSim.step: one control frame of the gas environment, episode after episode
  gasgrad  GasRollout with the sensor loss, forward and backward
  closure  MLP.init, train and predict: the learned cone return fitted to logged records
"""
import ctypes
import math

import numpy as np
import torch

from paper_2303_02346_amd import closure, gas, scenes, sim

KINDS = {"elastic": scenes.ELASTIC, "liquid": scenes.LIQUID, "sand": scenes.SAND, "vonmises": scenes.VONMISES,
         "box": scenes.BOX, "rigid": scenes.RIGID}
SIGMA = 0.05            # width of the blob loss
LR = 1e-3               # closure training rate


def listed():
    def mpm(name, particles, grid, materials, steps, ppc, n_scenes=1, graph=False):
        return {"name": name, "kind": "mpm", "particles": particles, "grid": grid, "materials": materials,
                "steps": steps, "ppc": ppc, "scenes": n_scenes, "graph": graph}

    def grad(name, particles, grid, materials, steps, ppc, ckpt, graph=False):
        return {"name": name, "kind": "grad", "particles": particles, "grid": grid, "materials": materials,
                "steps": steps, "ppc": ppc, "scenes": 1, "ckpt": ckpt, "graph": graph}

    return [
        # one substep of a test-sized scene of every basic material: a unit test or an interactive probe
        mpm("mpm_probe_step", 1500, 32, "elastic,liquid,sand", 1, 8.0),
        # one frame of a Gym-style loop at the paper's operating point: 1e5 particles, 64^3, 10 substeps
        mpm("mpm_env_frame", 100_000, 64, "liquid,liquid,elastic", 10, 16.0),
        # a whole 200-step episode in one captured call: the benchmark's water and sand on 128^3
        mpm("mpm_episode", 250_000, 128, "liquid,sand", 200, 7.5, graph=True),
        # the other plastic materials, with a count and a grid that fill neither blocks nor wavefronts
        mpm("mpm_plastic_ragged", 77_777, 101, "vonmises,box,elastic", 25, 5.0),
        # many independent scenes of ragged sizes stepped together (data generation): the largest work
        mpm("mpm_batch", 3_800_000, 64, "elastic,liquid,sand", 20, 12.0, n_scenes=64, graph=True),
        # one large scene on a fine grid: 1M sand particles hitting the floor
        mpm("mpm_sand_impact", 1_000_000, 256, "sand", 20, 5.0),
        # one iteration of policy optimisation with checkpoints: the gradient benchmark's 100k particles on 96^3
        grad("mpm_policy_grad", 100_000, 96, "liquid,sand", 64, 7.0, 16),
        # the same at 250k particles with every step's record kept in HBM, captured
        grad("mpm_policy_grad_records", 250_000, 128, "liquid,sand", 64, 7.5, 0, graph=True),
        # water pushing a rigid body, forward and backward
        grad("rigid_policy_grad", 250_000, 128, "liquid,rigid", 32, 7.5, 16),
        # one control frame of the air-circulation room at the paper's gas resolution
        {"name": "gas_env_frame", "kind": "gas", "nx": 128, "ny": 128, "nz": 128, "scalars": 2, "steps": 10},
        # one policy iteration on the same room
        {"name": "gas_policy_grad", "kind": "gasgrad", "nx": 128, "ny": 128, "nz": 128, "scalars": 2, "steps": 8,
         "ckpt": 16},
        # fitting the learned closure to logged records and evaluating it on held-out ones
        {"name": "closure_fit", "kind": "closure", "records": 131_072, "batch": 4096, "heldout": 100_000},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["mpm", "mpm", "mpm", "grad", "grad", "gas", "gasgrad", "closure"])
    if kind == "closure":
        n = int(_log(rng, 5_000, 250_000))
        return {"kind": kind, "records": n, "batch": int(_log(rng, max(256, n // 64), min(n, 8192))),
                "heldout": int(_log(rng, 100, 300_000))}
    if kind in ("gas", "gasgrad"):
        dims = [4 * int(_log(rng, 4, 36)) for _ in range(3)]
        case = {"kind": kind, "nx": dims[0], "ny": dims[1], "nz": dims[2], "scalars": rng.randint(1, 3),
                "steps": rng.randint(1, 10)}
        if kind == "gasgrad":
            case["ckpt"] = rng.choice([3, 8, 16])
        return case
    if kind == "mpm":
        n = int(_log(rng, 200, 1_000_000)) | 1
        names = rng.sample(["elastic", "liquid", "sand", "vonmises", "box"], rng.randint(1, 3))
        n_scenes = rng.choice([1, 1, 1, rng.randint(2, 24)])
        steps = max(1, min(int(_log(rng, 1, 100)), 20_000_000 // n))
    else:
        n = int(_log(rng, 500, 250_000)) | 1
        names = ["liquid"] + rng.sample(["elastic", "sand", "vonmises", "box"], rng.randint(0, 2))
        n_scenes = 1
        steps = max(2, min(int(_log(rng, 2, 64)), 8_000_000 // n))
    # particles per cell from sparse to dense, and the grid on which the boxes then have a common size
    ppc = _log(rng, 4.0, 16.0)
    side = rng.uniform(0.12, 0.2)
    per_box = max(1.0, n / (len(names) * n_scenes))
    most = 96 if n_scenes > 1 else (128 if kind == "grad" else 256)
    grid = int(min(most, max(16, (per_box / ppc) ** (1.0 / 3.0) / side)))
    case = {"kind": kind, "particles": n, "grid": grid, "materials": ",".join(names), "steps": steps,
            "ppc": round(ppc, 2), "scenes": n_scenes, "graph": rng.random() < 0.5}
    if kind == "grad":
        case["ckpt"] = rng.choice([0, 8, 16])
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _f32(a):
    """The nearest FP32 values, held in FP64: what the framework and the 64-bit reference both start from."""
    return np.asarray(a, np.float32).astype(np.float64)


def _material(name, vol, count):
    mu, lam = scenes.SOLID_MU, scenes.SOLID_LAMBDA
    m = {"elastic": lambda: scenes.Material(scenes.ELASTIC, mu, lam, 1.0),
         "liquid": lambda: scenes.Material(scenes.LIQUID, 0.0, scenes.WATER_LAMBDA, 1.0, viscosity=0.1),
         "sand": lambda: scenes.Material(scenes.SAND, mu, lam, 1.0, friction_deg=30.0),
         "vonmises": scenes.ice_cream, "box": scenes.plasticine, "rigid": scenes.rigid_object}[name]()
    m.p_vol = vol / count
    m.p_mass = m.rho * m.p_vol
    return m


def _scene(rng, count, grid, names, steps, ppc):
    """Boxes of the materials side by side just above the floor band, falling and stirred by a smooth
    velocity field, and the cylinder moving into the first box; dt keeps the elastic CFL number at 0.21."""
    k, dx, dt = len(names), 1.0 / grid, 6.4e-3 / grid
    margin = max(0.08, 4.0 * dx)
    slot = (1.0 - 2.0 * margin) / k
    per = [count // k] * k
    per[0] += count - sum(per)
    xs, vs, mats, materials = [], [], [], []
    first = None
    for b, name in enumerate(names):
        if per[b] == 0:
            continue
        side = min((per[b] / ppc) ** (1.0 / 3.0) * dx, 0.92 * slot)
        height = min(per[b] / ppc * dx ** 3 / side ** 2, 1.0 - 2.0 * margin)
        lo = np.array([margin + slot * b + rng.uniform(0.0, 0.5) * (slot - side), 3.0 * dx,
                       rng.uniform(margin, 1.0 - margin - side)])
        ext = np.array([side, height, side])
        x = lo + ext * rng.random((per[b], 3))
        if first is None:
            first = (lo, side)
        if name == "rigid":
            v = np.tile(rng.uniform(-0.2, 0.2, 3), (per[b], 1))
        else:
            v = np.empty_like(x)
            for a in range(3):
                d = rng.normal(size=3)
                wave = 2.0 * math.pi / max(side, 8.0 * dx) * d / np.linalg.norm(d)
                v[:, a] = 0.3 * np.sin(x @ wave + rng.uniform(0.0, 2.0 * math.pi))
        v[:, 1] -= 0.4
        xs.append(x)
        vs.append(v)
        mats.append(np.full(per[b], len(materials), np.int32))
        materials.append(_material(name, float(np.prod(ext)), per[b]))
    x = np.concatenate(xs)
    n = x.shape[0]
    radius = 0.05
    sc = scenes.Scene(
        n_grid=grid, dt=dt, x=_f32(x), v=_f32(np.concatenate(vs)), C=np.zeros((n, 3, 3)),
        F=np.tile(np.eye(3), (n, 1, 1)), J=np.ones(n), mat=np.concatenate(mats), materials=materials,
        actions=_f32(scenes.smooth_actions(rng, steps, dt, u_mean=(0.5, 0.0, 0.0))), cyl_radius=radius,
        cyl_pos0=_f32(first[0] + np.array([-radius - dx, 0.0, 0.5 * first[1]])))
    sc.target_mu = _f32(rng.uniform([0.3, 0.1, 0.3], [0.7, 0.3, 0.7]))
    sc.target_sigma = SIGMA
    return sc


def _scenes(case, seed):
    rng = np.random.default_rng([int(seed) & 0x7FFFFFFF, 1])
    names = case["materials"].split(",")
    s = case["scenes"]
    if s == 1:
        return [_scene(rng, case["particles"], case["grid"], names, case["steps"], case["ppc"])]
    # ragged scenes: counts over a factor of 20 that add up to the total, one to all of the materials in each
    share = np.exp(rng.uniform(0.0, math.log(20.0), s))
    counts = np.maximum(8, (case["particles"] * share / share.sum()).astype(int))
    counts[counts.argmax()] += case["particles"] - counts.sum()
    out = []
    for c in counts:
        k = int(rng.integers(1, len(names) + 1))
        pick = [names[i] for i in rng.permutation(len(names))[:k]]
        out.append(_scene(rng, int(c), case["grid"], pick, case["steps"], case["ppc"]))
    return out


def _gas_scene(case, seed):
    sc = scenes.gas_room((case["nx"], case["ny"], case["nz"]), steps=max(case["steps"], 1), seed=int(seed) & 0x7FFFFFFF,
                         n_scalars=case["scalars"], translate=True)
    for f in ("u", "v", "w", "s", "actions"):
        setattr(sc, f, _f32(getattr(sc, f)))
    return sc


def _records(n, seed):
    """Cone-case returns as the simulator logs them: log singular values of the trial deformation (descending),
    the cone's slope, cohesion and stiffness ratio, and the exact projection."""
    g = torch.Generator(device="cuda").manual_seed(int(seed) & 0x7FFFFFFF)

    def uni(lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(*shape, device="cuda", dtype=torch.float64, generator=g)

    s = torch.sin(uni(20.0, 40.0, n) * math.pi / 180.0)
    alpha = math.sqrt(2.0 / 3.0) * 2.0 * s / (3.0 - s)
    nu = uni(0.2, 0.35, n)
    kappa = (3.0 * nu / (1.0 - 2.0 * nu) + 1.0)
    coh = torch.where(uni(0.0, 1.0, n) < 0.5, torch.zeros_like(nu), uni(0.0, 0.01, n))
    trace = -0.03 * uni(0.02, 1.0, n) ** 2
    d = torch.randn(n, 3, device="cuda", dtype=torch.float64, generator=g)
    d = d - d.mean(1, keepdim=True)
    d = torch.sort(d / d.norm(dim=1, keepdim=True), dim=1, descending=True).values
    limit = -kappa * alpha * trace                           # deviatoric radius of the cone
    e = trace[:, None] / 3.0 + coh[:, None] + d * (limit * (1.0 + uni(0.0, 0.3, n)))[:, None]
    p = trace[:, None] / 3.0 + coh[:, None] + d * limit[:, None]
    return torch.cat([e, alpha[:, None], coh[:, None], kappa[:, None], p], 1).float().contiguous()


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "mpm":
        s = sim.Simulator(_scenes(case, seed), horizon=case["steps"], graph=case["graph"])
        st.update(sim=s, start=s.buf.clone(), actions=s.actions.clone())
    elif kind == "grad":
        sc = _scenes(case, seed)[0]
        s = sim.Simulator(sc, requires_grad=True, ckpt_every=case["ckpt"], graph=case["graph"])
        st.update(sim=s, actions=s.actions.clone(), target=sc.target_mu)
    elif kind == "gas":
        # the episode is 200 control frames long
        s = gas.GasSim(_gas_scene(case, seed), horizon=200 * case["steps"])
        st.update(sim=s, actions=s.actions[: case["steps"]].clone())
    elif kind == "gasgrad":
        s = gas.GasSim(_gas_scene(case, seed), requires_grad=True, ckpt_every=case["ckpt"])
        st.update(sim=s, actions=s.actions.clone())
    else:
        st.update(mlp=closure.MLP(), records=_records(case["records"], seed),
                  heldout=_records(case["heldout"], int(seed) + 7919), seed=int(seed) & 0x7FFFFFFF)
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "mpm":
        # set the environment to a state, then step it
        s = st["sim"]
        s.buf.copy_(st["start"])
        s.set_state()
        s.set_actions(st["actions"])
        s.step(case["steps"])
        return {"x": s.x, "v": s.v, "C": s.C, "F": s.F, "J": s.J}
    if kind == "grad":
        s = st["sim"]
        a = st["actions"].detach().requires_grad_()
        x, v = sim.MpmRollout.apply(a, s)
        loss = sim.BlobLoss.apply(x, s, st["target"], SIGMA)
        loss.backward()
        return {"loss": loss.detach(), "x": x.detach(), "v": v.detach(), "actions_grad": a.grad}
    if kind == "gas":
        s = st["sim"]
        if s.clock() + case["steps"] > s.horizon:
            s.reset()                                      # the episode is over
        s.set_actions(st["actions"], s.clock())
        s.step(case["steps"])
        u, v, w, q = s.split(s.buf)
        return {"u": u, "v": v, "w": w, "s": q}
    if kind == "gasgrad":
        s = st["sim"]
        a = st["actions"].detach().requires_grad_()
        out = gas.GasRollout.apply(a, s)
        loss, g = s.sensor_loss()
        out.backward(g)
        u, v, w, q = s.split(out.detach())
        return {"loss": loss, "u": u, "v": v, "w": w, "s": q, "actions_grad": a.grad}
    m = st["mlp"]
    m.init(st["records"], seed=st["seed"])
    hist = m.train(st["records"], epochs=1, batch=case["batch"], lr=LR, seed=st["seed"])
    params, _, _ = m.params()
    return {"loss": hist, "params": params, "prediction": m.predict(st["heldout"])}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind == "closure":
        # per record: 9 floats read; forward, input and weight gradients of the 6-64-64-3 network
        macs = 6 * 64 + 64 * 64 + 64 * 3
        return {"bytes": 36.0 * case["records"] + 48.0 * case["heldout"],
                "flops": 6.0 * macs * case["records"] + 2.0 * macs * case["heldout"]}
    if kind in ("gas", "gasgrad"):
        n = [case["nx"], case["ny"], case["nz"]]
        cells = float(n[0] * n[1] * n[2])
        values = cells * (3 + case["scalars"])
        # a step: the state read and written; about 60 operations a value for the advection, and forward and
        # inverse fast transforms along the three axes for the projection
        flops = 60.0 * values + 2.0 * sum(2.5 * math.log2(m) for m in n) * cells
        steps = case["steps"]
        if kind == "gas":
            return {"bytes": 8.0 * values * steps, "flops": flops * steps}
        # the adjoint step reads the state and the adjoint and writes the adjoint
        return {"bytes": (8.0 + 12.0) * values * steps, "flops": 3.0 * flops * steps}
    names = case["materials"].split(",")
    n = case["particles"] / len(names)
    # a particle's state read and written, 56 B a grid node (about one node a cell, plus the boxes' rims);
    # about 27 x 45 operations for the transfers and 800 for the decomposition of a solid
    per = sum(129.0 if m == "liquid" else 193.0 for m in names) * n
    ops = sum(1300.0 if m == "liquid" else 2100.0 for m in names) * n
    nodes = 1.5 * case["particles"] / case["ppc"]
    b, f = (per + 56.0 * nodes) * case["steps"], ops * case["steps"]
    if kind == "mpm":
        return {"bytes": b, "flops": f}
    return {"bytes": 2.5 * b, "flops": 3.0 * f}             # the adjoint reads the state and the adjoint


# ---------------------------------------------------------------------------
# the same in 64 bits: plain torch, differentiated by autograd
# ---------------------------------------------------------------------------
def _c32(v):
    return ctypes.c_float(v).value


def _svd3(F):
    """F = U diag(s) V^T for batches of 3 x 3 matrices of positive determinant: cyclic Jacobi on F^T F."""
    A = F.transpose(1, 2) @ F
    a = {(i, j): A[:, i, j].clone() for i in range(3) for j in range(i, 3)}
    V = [[torch.full_like(A[:, 0, 0], float(i == j)) for j in range(3)] for i in range(3)]
    for _ in range(6):
        for p, q in ((0, 1), (0, 2), (1, 2)):
            r = 3 - p - q
            apq = a[p, q]
            small = apq.abs() < 1e-300
            th = (a[q, q] - a[p, p]) / torch.where(small, torch.ones_like(apq), 2.0 * apq)
            t = torch.where(th >= 0, 1.0, -1.0) / (th.abs() + torch.sqrt(th * th + 1.0))
            t = torch.where(small, torch.zeros_like(t), t)
            c = 1.0 / torch.sqrt(t * t + 1.0)
            s = t * c
            a[p, p], a[q, q] = a[p, p] - t * apq, a[q, q] + t * apq
            a[p, q] = torch.zeros_like(apq)
            kp, kq = (min(p, r), max(p, r)), (min(q, r), max(q, r))
            a[kp], a[kq] = c * a[kp] - s * a[kq], s * a[kp] + c * a[kq]
            for i in range(3):
                V[i][p], V[i][q] = c * V[i][p] - s * V[i][q], s * V[i][p] + c * V[i][q]
    V = torch.stack([torch.stack(r, -1) for r in V], 1)
    B = F @ V
    s = B.norm(dim=1)
    return B / s[:, None, :], s, V


class _Iso(torch.autograd.Function):
    """U diag(g(s)) V^T of F = U diag(s) V^T, with the derivative of an isotropic matrix function."""

    @staticmethod
    def forward(ctx, F, g):
        U, s, V = _svd3(F)
        with torch.enable_grad():
            sv = s.detach().requires_grad_()
            gv = g(sv)
            dg = [torch.autograd.grad(gv[:, i].sum(), sv, retain_graph=True)[0] if gv.requires_grad
                  else torch.zeros_like(s) for i in range(3)]
        gv = gv.detach()
        ctx.save_for_backward(U, s, V, gv, torch.stack(dg, 1))
        return (U * gv[:, None, :]) @ V.transpose(1, 2)

    @staticmethod
    def backward(ctx, bar):
        U, s, V, g, dg = ctx.saved_tensors
        M = U.transpose(1, 2) @ bar @ V
        diag = torch.diagonal(M, dim1=1, dim2=2)
        si, sj, gi, gj = s[:, :, None], s[:, None, :], g[:, :, None], g[:, None, :]
        near = (si - sj).abs() < 1e-6
        dd = torch.diagonal(dg, dim1=1, dim2=2)[:, :, None]
        sym = torch.where(near, dd - dg, (gi - gj) / torch.where(near, torch.ones_like(si - sj), si - sj))
        anti = (gi + gj) / (si + sj)
        Mt = M.transpose(1, 2)
        A = sym * 0.5 * (M + Mt) + anti * 0.5 * (M - Mt)
        eye = torch.eye(3, dtype=s.dtype, device=s.device)
        A = A * (1.0 - eye) + torch.diag_embed((diag[:, :, None] * dg).sum(1))
        return U @ A @ V.transpose(1, 2), None


def _skew(w):
    z = torch.zeros_like(w[..., 0])
    return torch.stack([torch.stack([z, -w[..., 2], w[..., 1]], -1), torch.stack([w[..., 2], z, -w[..., 0]], -1),
                        torch.stack([-w[..., 1], w[..., 0], z], -1)], -2)


class _Mpm:
    """MLS-MPM over one or more independent scenes, in FP64."""

    def __init__(self, scs):
        dev = "cuda"
        t = lambda a: torch.as_tensor(np.asarray(a), dtype=torch.float64, device=dev)  # noqa: E731
        self.n, self.S = scs[0].n_grid, len(scs)
        self.dx, self.dt = 1.0 / self.n, _c32(scs[0].dt)
        self.g = t([_c32(v) for v in scs[0].gravity])
        self.band, self.fric, self.bound = _c32(scs[0].contact_band), _c32(scs[0].contact_friction), scs[0].bound
        self.radius = [_c32(sc.cyl_radius) for sc in scs]
        self.c0 = [t(_f32(sc.cyl_pos0)) for sc in scs]
        self.scene = torch.cat([torch.full((sc.n,), i, dtype=torch.int64, device=dev) for i, sc in enumerate(scs)])
        cat = lambda f: t(np.concatenate([getattr(sc, f) for sc in scs]))  # noqa: E731
        self.state = {k: cat(k) for k in ("x", "v", "C", "F", "J")}

        def per(f):
            return torch.cat([t([f(m) for m in sc.materials])[torch.as_tensor(sc.mat, device=dev).long()] for sc in scs])

        self.kind = per(lambda m: m.kind).long()
        self.mu, self.lam = per(lambda m: _c32(m.mu)), per(lambda m: _c32(m.lam))
        self.eta, self.vol, self.mass = per(lambda m: _c32(m.viscosity)), per(lambda m: _c32(m.p_vol)), per(lambda m: _c32(m.p_mass))
        sp = per(lambda m: math.sin(math.radians(m.friction_deg)))
        self.alpha = math.sqrt(2.0 / 3.0) * 2.0 * sp / (3.0 - sp)
        self.coh, self.ys = per(lambda m: m.cohesion), per(lambda m: m.yield_stress)
        self.lo, self.hi = 1.0 - per(lambda m: m.theta_c), 1.0 + per(lambda m: m.theta_s)
        at = lambda *ks: torch.nonzero(sum(self.kind == k for k in ks))[:, 0]  # noqa: E731
        self.liq, self.cor, self.hen = at(KINDS["liquid"]), at(KINDS["elastic"], KINDS["box"], KINDS["rigid"]), at(KINDS["sand"], KINDS["vonmises"])
        self.sand, self.vm, self.boxes = at(KINDS["sand"]), at(KINDS["vonmises"]), at(KINDS["box"])
        self.rigid = at(KINDS["rigid"])
        if self.rigid.numel():
            m, X = self.mass[self.rigid, None], self.state["x"][self.rigid]
            r = X - (m * X).sum(0) / m.sum()
            eye = torch.eye(3, dtype=torch.float64, device=dev)
            inertia = (m[:, :, None] * ((r * r).sum(1)[:, None, None] * eye - r[:, :, None] * r[:, None, :])).sum(0)
            self.rest, self.inv_inertia = r, torch.linalg.inv(inertia)
        self.offs = [(i, j, k) for i in range(3) for j in range(3) for k in range(3)]

    def stencil(self, x):
        X = x / self.dx
        base = torch.floor(X.detach() - 0.5)
        f = X - base
        w = [0.5 * (1.5 - f) ** 2, 0.75 - (f - 1.0) ** 2, 0.5 * (f - 0.5) ** 2]
        b = base.long()
        node = ((self.scene * self.n + b[:, 0]) * self.n + b[:, 1]) * self.n + b[:, 2]
        return f, w, node

    def corner(self, f, w, node, o):
        d = (torch.tensor(o, dtype=f.dtype, device=f.device) - f) * self.dx
        return w[o[0]][:, 0] * w[o[1]][:, 1] * w[o[2]][:, 2], d, node + (o[0] * self.n + o[1]) * self.n + o[2]

    def stress(self, s):
        eye = torch.eye(3, dtype=torch.float64, device="cuda")
        tau = torch.zeros_like(s["F"])
        if self.liq.numel():
            i = self.liq
            J, C = s["J"][i], s["C"][i]
            t = (self.lam[i] * J * (J - 1.0))[:, None, None] * eye + (self.eta[i] * J)[:, None, None] * (C + C.transpose(1, 2))
            tau = tau.index_put((i,), t)
        if self.cor.numel():
            i = self.cor
            F = s["F"][i]
            J = torch.linalg.det(F)
            R = _Iso.apply(F, lambda v: torch.ones_like(v))
            t = 2.0 * self.mu[i][:, None, None] * (F - R) @ F.transpose(1, 2) + (self.lam[i] * J * (J - 1.0))[:, None, None] * eye
            tau = tau.index_put((i,), t)
        if self.hen.numel():
            i = self.hen
            F, mu, lam = s["F"][i], self.mu[i][:, None], self.lam[i][:, None]

            def pk1(v):
                e = torch.log(v)
                return (2.0 * mu * e + lam * e.sum(1, keepdim=True)) / v

            tau = tau.index_put((i,), _Iso.apply(F, pk1) @ F.transpose(1, 2))
        return tau

    def project(self, F):
        if self.sand.numel():
            i = self.sand
            c, al, ka = self.coh[i][:, None], self.alpha[i][:, None], ((3 * self.lam[i] + 2 * self.mu[i]) / (2 * self.mu[i]))[:, None]

            def cone(v):
                e = torch.log(v) - c
                t = e.sum(1, keepdim=True)
                dev = e - t / 3.0
                nd = dev.norm(dim=1, keepdim=True)
                dg = nd + ka * al * t
                out = torch.where(dg <= 0, e, e - dg * dev / torch.where(nd > 0, nd, torch.ones_like(nd)))
                return torch.exp(torch.where(t > 0, 0.0 * e, out) + c)

            F = F.index_put((i,), _Iso.apply(F[i], cone))
        if self.vm.numel():
            i = self.vm
            rho = (self.ys[i] / (2.0 * self.mu[i]))[:, None]

            def ball(v):
                e = torch.log(v)
                t = e.sum(1, keepdim=True) / 3.0
                dev = e - t
                nd = dev.norm(dim=1, keepdim=True)
                return torch.exp(torch.where(nd > rho, t + rho * dev / torch.where(nd > 0, nd, torch.ones_like(nd)), e))

            F = F.index_put((i,), _Iso.apply(F[i], ball))
        if self.boxes.numel():
            i = self.boxes
            lo, hi = self.lo[i][:, None], self.hi[i][:, None]
            F = F.index_put((i,), _Iso.apply(F[i], lambda v: torch.minimum(torch.maximum(v, lo), hi)))
        return F

    def contact(self, x, v, c, R, u, w, radius):
        a, r = R[:, 1], x - c
        rp = r - (r @ a)[:, None] * a
        dist = rp.norm(dim=1)
        d = dist - radius
        nrm = rp / dist[:, None]
        vco = u + torch.cross(w.expand_as(r), r, dim=1)
        rel = v - vco
        vn = (rel * nrm).sum(1)
        vt = rel - vn[:, None] * nrm
        sq = (vt * vt).sum(1)
        vtn = torch.sqrt(torch.where(sq > 0, sq, torch.ones_like(sq))) * (sq > 0)
        stick = vtn <= -self.fric * vn
        slide = vt + (self.fric * vn / torch.where(stick, torch.ones_like(vtn), vtn))[:, None] * vt
        vc = torch.where((vn < 0)[:, None], torch.where(stick[:, None], torch.zeros_like(vt), slide) + vco, v)
        al = torch.clamp(torch.exp(-d / self.dx), max=1.0)[:, None]
        return torch.where((d < self.band * self.dx)[:, None], al * vc + (1.0 - al) * v, v)

    def step(self, s, poses, acts):
        n, dx, dt = self.n, self.dx, self.dt
        nodes = self.S * n ** 3
        f, w, node = self.stencil(s["x"])
        A = -(dt * self.vol * 4.0 / dx ** 2)[:, None, None] * self.stress(s) + self.mass[:, None, None] * s["C"]
        m = torch.zeros(nodes, dtype=torch.float64, device="cuda")
        mv = torch.zeros(nodes, 3, dtype=torch.float64, device="cuda")
        for o in self.offs:
            ww, d, q = self.corner(f, w, node, o)
            m = m.index_add(0, q, ww * self.mass)
            mv = mv.index_add(0, q, ww[:, None] * (self.mass[:, None] * s["v"] + (A * d[:, None, :]).sum(2)))
        act = torch.nonzero(m.detach() > 0)[:, 0]
        v = mv[act] / m[act][:, None] + dt * self.g
        ijk = torch.stack([(act // (n * n)) % n, (act // n) % n, act % n], 1)
        xi = ijk.double() * dx
        sc = act // n ** 3
        for k in range(self.S):
            if self.radius[k] > 0:
                if self.S == 1:
                    v = self.contact(xi, v, poses[k][0], poses[k][1], acts[k][:3], acts[k][3:], self.radius[k])
                else:
                    i = torch.nonzero(sc == k)[:, 0]
                    v = v.index_put((i,), self.contact(xi[i], v[i], poses[k][0], poses[k][1], acts[k][:3], acts[k][3:], self.radius[k]))
        out = ((ijk < self.bound) & (v < 0)) | ((ijk > n - 1 - self.bound) & (v > 0))
        vg = torch.zeros_like(mv).index_put((act,), torch.where(out, torch.zeros_like(v), v))
        vn = torch.zeros_like(s["v"])
        B = torch.zeros_like(s["C"])
        for o in self.offs:
            ww, d, q = self.corner(f, w, node, o)
            wv = ww[:, None] * vg[q]
            vn = vn + wv
            B = B + wv[:, :, None] * d[:, None, :]
        C = 4.0 / dx ** 2 * B
        M = torch.eye(3, dtype=torch.float64, device="cuda") + dt * C
        F = self.project(M @ s["F"])
        J = s["J"]
        if self.liq.numel():
            F = F.index_put((self.liq,), s["F"][self.liq])
            J = J.index_put((self.liq,), J[self.liq] * torch.linalg.det(M[self.liq]))
        s = {"x": s["x"] + dt * vn, "v": vn, "C": C, "F": F, "J": J}
        if self.rigid.numel():
            i = self.rigid
            m = self.mass[i, None]
            x, v = s["x"][i], s["v"][i]
            c, vc = (m * x).sum(0) / m.sum(), (m * v).sum(0) / m.sum()
            R = _Iso.apply((m[:, :, None] * (x - c)[:, :, None] * self.rest[:, None, :]).sum(0)[None], lambda q: torch.ones_like(q))[0]
            L = (m * torch.cross(x - c, v - vc, dim=1)).sum(0)
            om = R @ (self.inv_inertia @ (R.T @ L))
            q = self.rest @ R.T
            s["x"] = s["x"].index_put((i,), c + q)
            s["v"] = s["v"].index_put((i,), vc + torch.cross(om.expand_as(q), q, dim=1))
            s["C"] = s["C"].index_put((i,), _skew(om).expand(i.numel(), 3, 3))
            s["F"] = s["F"].index_put((i,), R.expand(i.numel(), 3, 3))
        return s

    def rollout(self, actions):
        """actions: (steps, scenes, 6)"""
        s = self.state
        eye = torch.eye(3, dtype=torch.float64, device="cuda")
        poses = [(self.c0[k], eye) for k in range(self.S)]
        for t in range(actions.shape[0]):
            s = self.step(s, poses, actions[t])
            poses = [(c + self.dt * actions[t, k, :3], torch.linalg.matrix_exp(self.dt * _skew(actions[t, k, 3:])) @ R)
                     for k, (c, R) in enumerate(poses)]
        return s


class _Gas:
    """Stam's advection and exact projection on a staggered grid with closed walls, in FP64."""

    def __init__(self, sc):
        t = lambda a: torch.as_tensor(np.asarray(a), dtype=torch.float64, device="cuda")  # noqa: E731
        self.sc, self.n = sc, tuple(sc.n)
        self.h, self.dt, self.beta, self.tamb = (_c32(v) for v in (sc.h, sc.dt, sc.buoyancy, sc.t_amb))
        self.sig, self.kap, self.spd = (_c32(v) for v in (sc.emit_sigma, sc.emit_kappa, sc.emit_speed))
        self.grids = [t(sc.u), t(sc.v), t(sc.w)] + [t(q) for q in sc.s]
        self.src = [_c32(v) for v in sc.src]
        self.c0, self.R0 = t(_f32(sc.emit_pos0)), t(_f32(sc.emit_rot0)).reshape(3, 3)
        self.dct, lam = [], []
        for m in self.n:
            k = torch.arange(m, dtype=torch.float64, device="cuda")
            self.dct.append(torch.cos(math.pi / m * (k[:, None] + 0.5) * k[None, :]))
            lam.append(-4.0 * torch.sin(math.pi * k / (2.0 * m)) ** 2)
        self.lam = lam[0][:, None, None] + lam[1][None, :, None] + lam[2][None, None, :]

    def origin(self, q):
        return [0.0 if a == q else 0.5 for a in range(3)]

    def sample(self, F, q, x):
        """F, values of grid q (3 and up: cells), at the points x (..., 3), clamped to the grid"""
        o = self.origin(q)
        base, frac = [], []
        for a in range(3):
            g = torch.clamp(x[a] / self.h - o[a], 0.0, F.shape[a] - 1.0)
            b = torch.clamp(torch.floor(g.detach()), max=F.shape[a] - 2)
            base.append(b.long())
            frac.append(g - b)
        out = 0.0
        flat = F.reshape(-1)
        for i in (0, 1):
            for j in (0, 1):
                for k in (0, 1):
                    w = ((frac[0] if i else 1 - frac[0]) * (frac[1] if j else 1 - frac[1]) * (frac[2] if k else 1 - frac[2]))
                    out = out + w * flat[((base[0] + i) * F.shape[1] + base[1] + j) * F.shape[2] + base[2] + k]
        return out

    def solve(self, f):
        def along(x, a, M):
            return torch.movedim(torch.movedim(x, a, -1) @ M, -1, a)
        for a in range(3):
            f = along(f, a, self.dct[a])
        lam = torch.where(self.lam != 0, self.lam, torch.ones_like(self.lam))
        f = torch.where(self.lam != 0, f / lam, torch.zeros_like(f))
        for a in range(3):
            m = self.n[a]
            wt = torch.full((m, 1), 2.0 / m, dtype=torch.float64, device="cuda")
            wt[0] = 1.0 / m
            f = along(f, a, wt * self.dct[a].T)
        return f

    def step(self, G, c, R):
        new = []
        for q, F in enumerate(G):
            o = self.origin(q)
            pos = torch.meshgrid(*[(torch.arange(F.shape[a], dtype=torch.float64, device="cuda") + o[a]) * self.h for a in range(3)], indexing="ij")
            U = [self.sample(G[a], a, pos) for a in range(3)]
            val = self.sample(F, q, [pos[a] - self.dt * U[a] for a in range(3)])
            chi = self.kap * torch.exp(-sum((pos[a] - c[a]) ** 2 for a in range(3)) / (2.0 * self.sig ** 2))
            new.append(val + chi * ((self.spd * R[q, 1] if q < 3 else self.src[q - 3]) - val))
        T = new[3]
        v = new[1].clone()
        v[:, 1:-1] = new[1][:, 1:-1] + self.dt * self.beta * (0.5 * (T[:, :-1] + T[:, 1:]) - self.tamb)
        vel = [new[0], v, new[2]]
        inner = [vel[a].narrow(a, 1, self.n[a] - 1) for a in range(3)]

        def closed(x, a):
            z = torch.zeros_like(x.narrow(a, 0, 1))
            return torch.cat([z, x, z], a)

        psi = self.solve(sum(torch.diff(closed(inner[a], a), dim=a) for a in range(3)))
        out = [closed(inner[a] - torch.diff(psi, dim=a), a) for a in range(3)]
        return out + new[3:]

    def rollout(self, actions):
        G, c, R = self.grids, self.c0, self.R0
        for t in range(actions.shape[0]):
            G = self.step(G, c, R)
            c, R = c + self.dt * actions[t, :3], torch.linalg.matrix_exp(self.dt * _skew(actions[t, 3:])) @ R
        return G


def exact(case, seed):
    kind = case["kind"]
    if kind == "closure":
        # the fitted weights follow from updates through BF16 roundings: there is no 64-bit value to be near to
        return None
    if kind in ("gas", "gasgrad"):
        sc = _gas_scene(case, seed)
        a = torch.as_tensor(sc.actions[: case["steps"]], dtype=torch.float64, device="cuda")
        if kind == "gas":
            with torch.no_grad():
                G = _Gas(sc).rollout(a)
            return {"u": G[0], "v": G[1], "w": G[2], "s": torch.stack(G[3:])}
        a.requires_grad_()
        G = _Gas(sc).rollout(a)
        e = G[3].reshape(-1)[torch.as_tensor(sc.sensors, device="cuda").long()] - torch.as_tensor(sc.targets, dtype=torch.float64, device="cuda")
        loss = e.abs().sum()
        loss.backward()
        return {"loss": loss.detach().reshape(1), "u": G[0].detach(), "v": G[1].detach(), "w": G[2].detach(),
                "s": torch.stack(G[3:]).detach(), "actions_grad": a.grad}
    scs = _scenes(case, seed)
    m = _Mpm(scs)
    acts = torch.stack([torch.as_tensor(sc.actions, dtype=torch.float64, device="cuda") for sc in scs], 1)
    if kind == "mpm":
        with torch.no_grad():
            s = m.rollout(acts)
        n = s["x"].shape[0]
        return {"x": s["x"].T, "v": s["v"].T, "C": s["C"].reshape(n, 9).T, "F": s["F"].reshape(n, 9).T, "J": s["J"]}
    acts.requires_grad_()
    s = m.rollout(acts)
    xl = s["x"][m.liq]
    mu = torch.as_tensor(scs[0].target_mu, dtype=torch.float64, device="cuda")
    loss = ((xl - mu) ** 2).sum(1).mean() + 3.0 * _c32(SIGMA) ** 2
    loss.backward()
    return {"loss": loss.detach(), "x": s["x"].detach().T, "v": s["v"].detach().T, "actions_grad": acts.grad}
