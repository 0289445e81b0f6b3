"""What a program does with this framework, as cases that can be timed and compared.

A case is a dict of plain values.  These calls are covered:

  "march"    Solver.step on a flow problem, then the fields that such a program reads back.  `problem` and its
             sizes name a generator of `workloads`; `levels` says how the velocity spaces are chosen:
             "uniform" (the base grid everywhere), "criterion" (one adaptation on the initial state, kept while
             the steps run) or "adaptive" (an adaptation every `interval` steps inside the steps).
  "snapshot" Solver.features and Solver.labels: one training snapshot of the learned level selector (the labels
             run the criterion on every cell).
  "network"  mlp_eval_noalloc: forward and backward of the selector network on device buffers.
  "predict"  mlp_predict: inference of the selector network on host arrays, as a program outside a solver does.

The flow fields are smooth seeded modes on top of a developed state of each problem (a plume for the jet, a
boundary layer around the cylinder, a thin front between the two cavities), so that the limiter, the levels and
the cross-level faces meet what they meet in a run, and no cell starts near vacuum.  Marching outputs are the whole fields per cell
(density, velocity, temperature, heat flux); FP64 problems also return the stress, as the cavity and cylinder
results read it, and a problem small enough to be read back after a call returns its whole distributions.  With
FP32 storage the fields are returned in FP32.
"""
import dataclasses
import math

import numpy as np
import torch

import paper_2609_35258_amd as mlvs
import workloads

# Thresholds of the adaptation, as the benchmark runs them (the cavity's are its own).
ADAPT = dict(C_split=0.01, C_merge=0.005, eps_merge=2e-5, tau_clust=0.05, flux_test=True, interval=0)
CAVITY_ADAPT = dict(C_split=5e-3, C_merge=2.5e-3, eps_merge=5e-5, tau_clust=0.05, flux_test=True, interval=0)
# Velocity points per cell that the criterion keeps on these fields, over the base grid's (for work() only).
KEPT = {"cavity": 0.31, "cylinder": 0.12, "jet": 0.10, "two_cavity": 0.15}
# A problem with at most this many distribution values per array returns them whole.
WHOLE_STATE = 1 << 16
# Most distribution values of one array in a drawn case: the largest listed case's.
MOST_POINTS = 256 * 128 * 161 * 161


def listed():
    return [
        # the smallest call: a 1-D shock tube, eight steps between two looks at the state; launches and latency
        dict(name="sod_uvs_fp64", kind="march", problem="sod", ni=200, nj=1, nv=101, precision=64, levels="uniform",
             steps=8),
        # the lid-driven cavity on its Gauss-Hermite grid, FP64, one uniform velocity space
        dict(name="cavity_uvs_fp64", kind="march", problem="cavity", ni=64, nj=64, nv=28, precision=64,
             levels="uniform", steps=20),
        # the same cavity multi-level with adaptation inside the steps, FP64: grouping and level switches count
        dict(name="cavity_adaptive_fp64", kind="march", problem="cavity", ni=64, nj=64, nv=28, precision=64,
             levels="adaptive", interval=10, steps=20),
        # the Mach 3 cylinder on its body-fitted O-grid, FP32 storage: the ordinary production step
        dict(name="cylinder_uvs_fp32", kind="march", problem="cylinder", ni=256, nj=128, nv=101, precision=32,
             levels="uniform", steps=4),
        dict(name="cylinder_mlvs_fp32", kind="march", problem="cylinder", ni=256, nj=128, nv=101, precision=32,
             levels="criterion", steps=10),
        # an odd-sized cylinder with the higher-order corrections (eight-moment targets, nine-moment mapping), FP64
        dict(name="cylinder_mlvs_8_9_fp64", kind="march", problem="cylinder", ni=95, nj=45, nv=61, precision=64,
             levels="criterion", steps=5, compat=8, map_moments=9),
        # the slot jet at its full velocity grid: the largest distributions, rows of 25921 points
        dict(name="jet_uvs_fp32", kind="march", problem="jet", ni=256, nj=128, nv=161, precision=32,
             levels="uniform", steps=2),
        # the slot jet multi-level: the benchmark's headline kind of step
        dict(name="jet_mlvs_fp32", kind="march", problem="jet", ni=256, nj=128, nv=161, precision=32,
             levels="criterion", steps=10),
        # the two-cavity expansion on triangles and quadrilaterals
        dict(name="two_cavity_uvs_fp32", kind="march", problem="two_cavity", ni=48, nj=48, nv=101, precision=32,
             levels="uniform", steps=10),
        # the same multi-level with adaptation every 5 steps, as the expansion is run; FP64, on a coarser mesh
        dict(name="two_cavity_adaptive_fp64", kind="march", problem="two_cavity", ni=32, nj=32, nv=61, precision=64,
             levels="adaptive", interval=5, steps=10),
        # one training snapshot of the learned selector on the cylinder: features, and the criterion on every cell
        dict(name="cylinder_snapshot_fp32", kind="snapshot", problem="cylinder", ni=256, nj=128, nv=101,
             precision=32, levels="criterion"),
        # forward and backward of the selector network on a training batch held on the device
        dict(name="network_batch", kind="network", batch=1024, classes=6),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["march"] * 8 + ["snapshot", "network", "predict"])
    if kind == "network":
        return dict(kind=kind, batch=log(16, 4096), classes=rng.randint(2, 16))
    if kind == "predict":
        return dict(kind=kind, batch=log(1000, 100000), classes=rng.randint(2, 16))
    problem = rng.choice(["cavity", "cylinder", "jet", "two_cavity"] + (["sod"] if kind == "march" else []))
    precision = 64 if problem == "sod" else rng.choice([32, 64])
    while True:
        if problem == "sod":
            ni, nj, nv = log(20, 4000), 1, rng.choice([65, 101, 201])
        elif problem == "cavity":
            ni = log(12, 128)
            nj, nv = ni, rng.choice([20, 28, 40])
        elif problem == "two_cavity":
            ni = rng.choice([16, 32, 48])
            nj, nv = ni, rng.choice([41, 61, 80, 101])
        elif problem == "cylinder":
            ni, nj, nv = log(33, 256), log(17, 128), rng.choice([60, 61, 81, 101])
        else:
            nj = log(20, 128)
            ni, nv = 2 * nj - rng.randint(0, 1), rng.choice([80, 101, 121, 161])
        points = _cells(problem, ni, nj) * nv ** (1 if problem == "sod" else 2)
        if points * precision // 32 <= MOST_POINTS // 2:
            break
    case = dict(kind=kind, problem=problem, ni=ni, nj=nj, nv=nv, precision=precision)
    if kind == "snapshot":
        return dict(case, levels="criterion")
    levels = "uniform" if problem == "sod" else rng.choice(["uniform", "criterion"] + ["adaptive"] * (precision == 64))
    case.update(levels=levels, steps=max(2, min(40, int(4e8 / points))))
    if levels == "adaptive":
        case["interval"] = rng.choice([5, 10])
    if problem != "sod" and rng.random() < 0.3:
        case.update(compat=rng.choice([0, 4, 8]), map_moments=rng.choice([4, 9]))
    return case


def _cells(problem, ni, nj):
    # two_cavity: 2 n^2 squares cut into two triangles each, and n (2 n // 16) channel quadrilaterals
    return 4 * ni * ni + ni * (2 * (ni // 16)) if problem == "two_cavity" else ni * nj


# ---------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------
def _modes(x, y, lx, ly, rng):
    """A smooth seeded field of rms about one: six random plane waves of up to three periods over lx, ly."""
    f = np.zeros_like(x)
    for _ in range(6):
        kx, ky, ph = rng.uniform(0.5, 3.0), rng.uniform(0.5, 3.0) * rng.choice([-1.0, 1.0]), rng.uniform(0, 2 * math.pi)
        f += np.sin(2 * math.pi * (kx * x / lx + ky * y / ly) + ph)
    return f / math.sqrt(3.0)


def _problem(case, seed):
    """The problem of a case with a seeded smooth initial state."""
    rng = np.random.default_rng(seed)
    ni, nj, nv, name = case["ni"], case["nj"], case["nv"], case["problem"]
    if name == "sod":
        p = workloads.sod_1d(ni, nv=nv)
    elif name == "cavity":
        p = workloads.cavity(ni, nv=nv)
    elif name == "cylinder":
        p = workloads.cylinder(ni, nj, nv=nv)
    elif name == "jet":
        p = workloads.jet(ni, nj, nv=nv)
    else:
        p = workloads.two_cavity(ni, nv=nv, seed=3)
    if name == "two_cavity":
        ends = p.cell_ptr
        cell = np.repeat(np.arange(p.n_cells), np.diff(ends))
        n = np.bincount(cell)
        x = np.bincount(cell, p.nodes[p.cell_node, 0]) / n
        y = np.bincount(cell, p.nodes[p.cell_node, 1]) / n
        lx, ly = 3.0, 1.0
    else:
        X, Y = p.X, p.Y
        x = 0.25 * (X[:-1, :-1] + X[1:, :-1] + X[:-1, 1:] + X[1:, 1:])
        y = 0.25 * (Y[:-1, :-1] + Y[1:, :-1] + Y[:-1, 1:] + Y[1:, 1:])
        lx, ly = float(np.ptp(X)), float(np.ptp(Y))
    rho, u, v, T = p.rho0.copy(), p.u0.copy(), p.v0.copy(), p.T0.copy()
    amp = 0.05
    if name == "cavity":
        v_lid = p.bcs[1].u
        turn = np.sin(math.pi * x) * np.sin(math.pi * y)
        u, v = v_lid * turn * (2 * y - 1), -v_lid * turn * (2 * x - 1)
    elif name == "cylinder":
        r = np.hypot(x, y)
        layer = 1.0 - np.exp(-(r - 1.0) / 0.6)
        U = p.u0.ravel()[0]
        u = U * layer * (1.0 - 0.3 * np.exp(-(r - 1.0)))
        T = 1.0 + 1.2 * np.exp(-((r - 1.8) / 0.9) ** 2) * (0.6 - 0.4 * x / r)
        rho = 1.0 + 0.8 * np.exp(-((r - 1.6) / 0.6) ** 2) * (0.5 - 0.5 * x / r)
    elif name == "jet":
        plume = np.exp(-(y / (0.6 + 0.12 * x)) ** 2) * np.exp(-x / 14.0)
        rho = rho + (1.0 - rho) * plume
        u = p.bcs[1].u * plume ** 0.5
        T = 1.0 - 0.25 * plume * np.tanh(x / 4.0)
    elif name == "two_cavity":
        front = 0.5 * (1.0 - np.tanh(x / 0.15))
        rho = 1e-3 + (1.0 - 1e-3) * front
    rho = rho * (1.0 + amp * _modes(x, y, lx, ly, rng))
    T = T * (1.0 + 0.5 * amp * _modes(x, y, lx, ly, rng))
    u = u + 0.5 * amp * _modes(x, y, lx, ly, rng)
    if p.dim == 2:
        v = v + 0.5 * amp * _modes(x, y, lx, ly, rng)
    return dataclasses.replace(p, rho0=rho, u0=u, v0=v, T0=T)


def _network(case, seed):
    """Seeded parameters in the layout of mlp_nparams, features and labels of a batch."""
    rng = np.random.default_rng(seed)
    K, B = case["classes"], case["batch"]
    P = workloads.mlp_init_params(K, seed)
    P[-20:-10] = 0.1 * rng.normal(size=10)
    P[-10:] = rng.uniform(0.5, 2.0, size=10)
    return P.astype(np.float32), rng.normal(size=(B, 10)).astype(np.float32), rng.integers(0, K, B).astype(np.int32)


def prepare(case, seed):
    if case["kind"] in ("network", "predict"):
        P, X, y = _network(case, seed)
        state = dict(case=case, P=P, X=X)
        if case["kind"] == "network":
            dev = torch.device("cuda", torch.cuda.current_device())
            state.update(P=torch.from_numpy(P).to(dev), X=torch.from_numpy(X).to(dev), y=torch.from_numpy(y).to(dev))
        return state
    p = _problem(case, seed)
    adapt = None
    if case["levels"] != "uniform":
        adapt = dict(CAVITY_ADAPT if case["problem"] == "cavity" else ADAPT, interval=case.get("interval", 0))
    solver = mlvs.Solver.from_problem(p, precision=case["precision"], compat=case.get("compat", 4),
                                      map_moments=case.get("map_moments", 4), adapt=adapt, graph=True)
    if case["levels"] == "criterion":
        solver.adapt()
    return dict(case=case, solver=solver)


# ---------------------------------------------------------------------------------------------------------------
# the call
# ---------------------------------------------------------------------------------------------------------------
def run(state):
    case = state["case"]
    if case["kind"] == "network":
        P, X, y, K = state["P"], state["X"], state["y"], case["classes"]
        probs = torch.empty((len(X), K), dtype=torch.float32, device=X.device)
        grad = torch.empty_like(P)
        loss = torch.empty(1, dtype=torch.float64, device=X.device)
        mlvs.mlp_eval_noalloc(P.data_ptr(), K, X.data_ptr(), y.data_ptr(), len(X), probs.data_ptr(), grad.data_ptr(),
                              loss.data_ptr(), torch.cuda.current_stream(X.device).cuda_stream)
        return dict(probs=probs, grad=grad, loss=loss)
    if case["kind"] == "predict":
        classes, probs = mlvs.mlp_predict(state["P"], case["classes"], state["X"], bf16=False)
        return dict(classes=classes, probs=probs)
    s = state["solver"]
    if case["kind"] == "snapshot":
        return dict(features=s.features(), labels=s.labels())
    real = np.float32 if case["precision"] == 32 else np.float64
    s.step(case["steps"])
    out = dict(fields=s.moments().astype(real, copy=False))
    if case["precision"] == 64 and s.dim == 2:
        out["stress"] = s.stress()
    if case["levels"] == "adaptive":
        out["cell_levels"] = s.cell_levels()
    if case["levels"] == "uniform" and s.n_cells * s.n_base <= WHOLE_STATE:
        state_now = s.get_state()
        out["g"] = np.concatenate([g for g, _ in state_now]).astype(real, copy=False)
        out["h"] = np.concatenate([h for _, h in state_now]).astype(real, copy=False)
    return out


def work(case):
    if case["kind"] in ("network", "predict"):
        B, K = case["batch"], case["classes"]
        weights = 64 * 10 + 64 * 64 + 64 * K
        back = case["kind"] == "network"
        return {"bytes": 4 * (10 * B + K * B + (weights + 148 + K) * (2 if back else 1) + B),
                "flops": 2 * weights * B * (3 if back else 1)}
    points = _cells(case["problem"], case["ni"], case["nj"]) * case["nv"] ** (1 if case["problem"] == "sod" else 2)
    if case["levels"] != "uniform":
        points *= KEPT[case["problem"]]
    cells = _cells(case["problem"], case["ni"], case["nj"])
    size = case["precision"] // 8
    if case["kind"] == "snapshot":
        # both distributions read once, the features and labels written once; per point its mass and energy sums
        return {"bytes": 2 * size * points + 44 * cells, "flops": 8 * points}
    # Per step and velocity point: both distributions read once and written once.  Arithmetic: two Maxwellian
    # targets (cell and face, about 40 each), two limited slopes and two extrapolations (60), the cell and face
    # moments (2 x 40) and the update (20).
    return {"bytes": case["steps"] * points * 4 * size + 8 * 6 * cells, "flops": case["steps"] * points * 240}


# ---------------------------------------------------------------------------------------------------------------
# the same in 64 bits, in plain torch
# ---------------------------------------------------------------------------------------------------------------
def exact(case, seed):
    if case["kind"] in ("network", "predict"):
        return _network_64(case, seed)
    # Multi-level spaces and unstructured meshes have no short closed form here; their kernels are the same
    # reconstruction, targets and updates as the uniform cases check, and they are compared with the start's.
    if case["kind"] != "march" or case["levels"] != "uniform" or case["problem"] == "two_cavity":
        return None
    if case.get("compat", 4) == 8:
        return None
    return _march_64(case, seed)


def _network_64(case, seed):
    P, X, y = _network(case, seed)
    K = case["classes"]
    shapes = ((64, 10), (64,), (64, 64), (64,), (K, 64), (K,), (10,), (10,))
    parts, at = [], 0
    for sh in shapes:
        n = int(np.prod(sh))
        parts.append(torch.tensor(P[at:at + n], dtype=torch.float64).reshape(sh).requires_grad_(True))
        at += n
    W1, b1, W2, b2, W3, b3, mean, std = parts
    x = (torch.tensor(X, dtype=torch.float64) - mean.detach()) / std.detach()
    z = torch.relu(torch.relu(x @ W1.T + b1) @ W2.T + b2) @ W3.T + b3
    probs = torch.softmax(z, 1)
    if case["kind"] == "predict":
        return dict(classes=None, probs=probs.detach())
    losses = torch.nn.functional.cross_entropy(z, torch.tensor(y, dtype=torch.int64), reduction="none")
    losses.mean().backward()
    grad = torch.cat([(q.grad if k < 6 else torch.zeros_like(q)).reshape(-1) for k, q in enumerate(parts)])
    return dict(probs=probs.detach(), grad=grad, loss=losses.sum().reshape(1).detach())


def _axis(p):
    """Nodes and weights of one velocity axis: Gauss-Hermite, or composite Boole, Simpson or midpoint."""
    n, a = p.nv, p.vmax
    if p.vel_kind == "gh":
        x, w = np.polynomial.hermite.hermgauss(n)
        c = math.sqrt(2 * p.R * p.gh_scale_T)
        return c * x, c * w * np.exp(x * x)
    if n % 2 == 0:
        return (np.arange(n) + 0.5) * (2 * a / n) - a, np.full(n, 2 * a / n)
    h, w = 2 * a / (n - 1), np.zeros(n)
    rule, k = ((np.array([7.0, 32, 12, 32, 7]) * 2 / 45, 4) if (n - 1) % 4 == 0 else (np.array([1.0, 4, 1]) / 3, 2))
    for q in range(0, n - 1, k):
        w[q:q + k + 1] += rule * h
    return a * (2.0 * np.arange(n) - (n - 1)) / (n - 1), w


class _Geometry:
    """Cells and faces of a structured mesh.  Faces: left and right cell (right = -1 - boundary id on a boundary,
    with the normal pointing out), unit normal, length, and the face centre seen from both cell centres."""

    def __init__(self, p, dev):
        X, Y, ni, nj = p.X, p.Y, p.ni, p.nj
        N = np.stack([X, Y], -1)
        quad = [N[:-1, :-1], N[:-1, 1:], N[1:, 1:], N[1:, :-1]]
        area, cen = 0.0, 0.0
        for k in range(4):
            a, b = quad[k], quad[(k + 1) % 4]
            cross = a[..., 0] * b[..., 1] - b[..., 0] * a[..., 1]
            area = area + 0.5 * cross
            cen = cen + (a + b) * cross[..., None]
        cen = cen / (6 * area[..., None])
        cells = np.arange(ni * nj).reshape(nj, ni)
        L, R, n, A, xf, xL, xR = [], [], [], [], [], [], []
        end = np.zeros((nj, ni, 4, 2))            # face centres W, E, S, N
        nbr = -np.ones((nj, ni, 4), np.int64)
        dist = np.ones((nj, ni, 4))

        def add(l, r, nn, aa, ff, cl, cr):
            L.append(l); R.append(r); n.append(nn); A.append(aa); xf.append(ff); xL.append(cl); xR.append(cr)

        for d in ([0] if p.dim == 1 else [0, 1]):
            t = N[1:, :] - N[:-1, :] if d == 0 else N[:, 1:] - N[:, :-1]
            mid = 0.5 * (N[1:, :] + N[:-1, :] if d == 0 else N[:, 1:] + N[:, :-1])
            ln = np.hypot(t[..., 0], t[..., 1])
            nor = np.stack([t[..., 1], -t[..., 0]] if d == 0 else [-t[..., 1], t[..., 0]], -1) / ln[..., None]
            m = ni if d == 0 else nj
            take = (lambda a, k: a[:, k]) if d == 0 else (lambda a, k: a[k])
            put = (lambda a, k, s, v: a.__setitem__((slice(None), k, s), v)) if d == 0 else (
                lambda a, k, s, v: a.__setitem__((k, slice(None), s), v))
            wrap = p.periodic_i if d == 0 else p.periodic_j
            shift = (N[0, ni] - N[0, 0] if d == 0 else N[nj, 0] - N[0, 0]) if wrap else 0.0
            for k in range(m + (0 if wrap else 1)):
                f, a, nn = take(mid, k), take(ln, k), take(nor, k)
                if 0 < k < m or wrap:
                    l, r = (k - 1) % m, k
                    cl, cr = take(cen, l) - (shift if k == 0 else 0.0), take(cen, r)
                    add(take(cells, l), take(cells, r), nn, a, f, cl, cr)
                    put(end, l, 2 * d + 1, f + (shift if k == 0 else 0.0)); put(end, r, 2 * d, f)
                    gap = np.hypot(*(cr - cl).T)
                    put(nbr, l, 2 * d + 1, take(cells, r)); put(dist, l, 2 * d + 1, gap)
                    put(nbr, r, 2 * d, take(cells, l)); put(dist, r, 2 * d, gap)
                else:
                    c, low = (0, True) if k == 0 else (m - 1, False)
                    ids = (p.bc_imin if low else p.bc_imax) if d == 0 else (p.bc_jmin if low else p.bc_jmax)
                    cc = take(cen, c)
                    add(take(cells, c), -1 - np.asarray(ids, np.int64), -nn if low else nn, a, f, cc, cc)
                    put(end, c, 2 * d + (0 if low else 1), f)
        unit = lambda a: a / np.hypot(a[..., 0], a[..., 1])[..., None]  # noqa: E731
        ti = unit(end[:, :, 1] - end[:, :, 0])
        tj = unit(end[:, :, 3] - end[:, :, 2]) if p.dim == 2 else np.broadcast_to([0.0, 1.0], ti.shape)
        G = np.linalg.inv(np.stack([ti, tj], -2))
        used = 4 if p.dim == 2 else 2
        gaps = np.hypot(*(end - cen[:, :, None]).transpose(3, 0, 1, 2))[:, :, :used]
        self.hmin = 2.0 * float(gaps.min())
        up = lambda a: torch.as_tensor(np.ascontiguousarray(a), device=dev)  # noqa: E731
        cat = lambda a: up(np.concatenate([np.asarray(q) for q in a]))  # noqa: E731
        self.vol, self.nbr, self.dist = up(area.ravel()), up(nbr.reshape(-1, 4)), up(dist.reshape(-1, 4))
        self.G = up(G.reshape(-1, 2, 2))
        self.L, self.R, self.n, self.A = cat(L), cat(R), cat(n), cat(A)
        self.dL, self.dR = cat(xf) - cat(xL), cat(xf) - cat(xR)


class _Gas:
    """States, collision targets and their moment corrections for rows of (rho, u, v, T, qx, qy)."""

    def __init__(self, p, compat, x, y, w):
        self.D, self.K, self.R, self.Pr = p.dim, p.K, p.R, p.Pr
        self.omega, self.T_ref, self.compat = p.omega, p.T_ref, compat
        self.mu_ref = (15 * math.sqrt(math.pi) / (2 * (5 - 2 * p.omega) * (7 - 2 * p.omega)) * p.Kn * p.rho_ref
                       * math.sqrt(2 * p.R * p.T_ref) * p.L_ref)
        self.x, self.y, self.w = x, y, w
        self.chunk = 1024

    def chunks(self):
        n = len(self.x)
        return [slice(a, min(n, a + self.chunk)) for a in range(0, n, self.chunk)]

    def tau(self, s):
        return self.mu_ref * (s[:, 3] / self.T_ref) ** self.omega / (s[:, 0] * self.R * s[:, 3])

    def sums(self, cl, g, h):
        """Raw moments of a chunk: 1, x, y, xx, xy, yy, x|xi|^2, y|xi|^2 of g, and 1, x, y of h."""
        x, y, w = self.x[cl], self.y[cl], self.w[cl]
        q = x * x + y * y
        B = torch.stack([w, w * x, w * y, w * x * x, w * x * y, w * y * y, w * x * q, w * y * q], 1)
        return torch.cat([g @ B, h @ B[:, :3]], 1)

    def state(self, m, damp):
        """(rho, u, v, T, qx, qy); q = 2 tau q~ / (2 tau + damp Pr)."""
        rho, u, v = m[:, 0], m[:, 1] / m[:, 0], m[:, 2] / m[:, 0]
        T = ((m[:, 3] + m[:, 5] + m[:, 8]) / rho - (u * u + v * v)) / ((3.0 + self.K) * self.R)
        uu = u * u + v * v
        tr = m[:, 3] + m[:, 5]
        cx = m[:, 6] - 2 * (u * m[:, 3] + v * m[:, 4]) + uu * m[:, 1] - u * tr + 2 * u * (u * m[:, 1] + v * m[:, 2]) - u * uu * rho
        cy = m[:, 7] - 2 * (u * m[:, 4] + v * m[:, 5]) + uu * m[:, 2] - v * tr + 2 * v * (u * m[:, 1] + v * m[:, 2]) - v * uu * rho
        s = torch.stack([rho, u, v, T, 0.5 * (cx + m[:, 9] - u * m[:, 8]), 0.5 * (cy + m[:, 10] - v * m[:, 8])], 1)
        t = self.tau(s)
        s[:, 4:] *= (2 * t / (2 * t + damp * self.Pr))[:, None]
        return s

    def target(self, s, cl, a=None):
        """The reduced Shakhov pair of each row on a chunk, with the correction's coefficients a."""
        rho, u, v, T, qx, qy = (s[:, k, None] for k in range(6))
        x, y = self.x[cl][None], self.y[cl][None]
        cx, cy = x - u, y - v if self.D == 2 else torch.zeros_like(x - u)
        c2, RT = cx * cx + cy * cy, self.R * T
        ge = rho / (2 * math.pi * RT) ** (0.5 * self.D) * torch.exp(-c2 / (2 * RT))
        X = (1 - self.Pr) * (cx * qx + cy * qy) / (5 * rho * RT * RT)
        kD = self.K + 3.0 - self.D
        g = ge * (1 + X * (c2 / RT - self.D - 2))
        h = ge * RT * (kD + X * ((c2 / RT - self.D) * kD - 2 * self.K))
        if a is not None:
            f = 1 + a[:, 0, None] + a[:, 1, None] * x + a[:, 2, None] * y + a[:, 3, None] * 0.5 * (kD * RT + x * x + y * y)
            g, h = g * f, h * f
        return g, h

    def correction(self, s):
        """Coefficients on (1, xi, (kD R T + |xi|^2)/2) that give the target its mass, momentum and energy."""
        if not self.compat:
            return None
        rho, u, v, T = (s[:, k] for k in range(4))
        M = torch.zeros((len(s), 4, 4), dtype=s.dtype, device=s.device)
        kD = self.K + 3.0 - self.D
        for cl in self.chunks():
            g, h = self.target(s, cl)
            x, y, w = self.x[cl], self.y[cl], self.w[cl]
            q = x * x + y * y
            base = [torch.ones_like(x), x, y, 0.5 * q]
            for i in range(4):
                # sums of psi_i times the basis without its constant energy part, which is added below
                pair = torch.stack([w * base[i] * base[j] for j in range(4)], 1)
                M[:, i] += g @ pair
                if i == 3:
                    M[:, i] += h @ torch.stack([0.5 * w * base[j] for j in range(4)], 1)
        low = M[:, :, 0].clone()
        M[:, :, 3] += 0.5 * kD * self.R * T[:, None] * low
        want = torch.stack([rho, rho * u, rho * v, 0.5 * rho * (u * u + v * v) + 0.5 * (3 + self.K) * rho * self.R * T], 1)
        keep = [0, 1, 2, 3] if self.D == 2 else [0, 1, 3]
        a = torch.zeros((len(s), 4), dtype=s.dtype, device=s.device)
        a[:, keep] = torch.linalg.solve(M[:, keep][:, :, keep], (want - low)[:, keep])
        return a


def _march_64(case, seed):
    """The uniform-space scheme step by step in FP64 torch, a chunk of velocities at a time."""
    dev = torch.device("cuda", torch.cuda.current_device()) if torch.cuda.is_available() else torch.device("cpu")
    p = _problem(case, seed)
    x1, w1 = _axis(p)
    if p.dim == 2:
        x, y, w = np.tile(x1, p.nv), np.repeat(x1, p.nv), np.outer(w1, w1).ravel()
    else:
        x, y, w = x1, np.zeros_like(x1), w1
    up = lambda a: torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device=dev)  # noqa: E731
    gas = _Gas(p, case.get("compat", 4), up(x), up(y), up(w))
    geo = _Geometry(p, dev)
    dt = p.cfl * geo.hmin / float(np.sqrt(x * x + y * y).max())
    s = 0.5 * dt
    nc = p.n_cells
    zero = np.zeros(nc)
    start = up(np.stack([p.rho0.ravel(), p.u0.ravel(), p.v0.ravel() if p.dim == 2 else zero, p.T0.ravel(), zero, zero], 1))
    a0 = gas.correction(start)
    g = torch.empty((nc, len(x)), dtype=torch.float64, device=dev)
    h = torch.empty_like(g)
    for cl in gas.chunks():
        g[:, cl], h[:, cl] = gas.target(start, cl, a0)
    inner = geo.R >= 0
    Li, Ri = geo.L[inner], geo.R[inner]
    walls = {}
    for b in range(len(p.bcs)):
        walls[b] = torch.nonzero(geo.R == -1 - b)[:, 0]

    def moments():
        return sum(gas.sums(cl, g[:, cl], h[:, cl]) for cl in gas.chunks())

    def limited(f):
        nb, have = geo.nbr.clamp(min=0), (geo.nbr >= 0)[:, :, None]
        d = [torch.where(have[:, k], (f - f[nb[:, k]]) / geo.dist[:, k, None], torch.zeros_like(f)) for k in range(4)]
        out = []
        for lo, hi in ((d[0], -d[1]), (d[2], -d[3])):
            pr = lo * hi
            out.append(torch.where(pr > 0, 2 * pr / torch.where(pr > 0, lo + hi, torch.ones_like(pr)), torch.zeros_like(pr)))
        G = geo.G
        return (G[:, 0, 0, None] * out[0] + G[:, 0, 1, None] * out[1], G[:, 1, 0, None] * out[0] + G[:, 1, 1, None] * out[1])

    def faces(cl, cell, al, be, a_cell):
        """phi_bar+ of every cell and phi_bar of every face on a chunk."""
        gs, hs = gas.target(cell, cl, a_cell)
        bar = (al * g[:, cl] + be * gs, al * h[:, cl] + be * hs)
        dn = geo.n[:, 0, None] * gas.x[cl] + geo.n[:, 1, None] * gas.y[cl]
        at = []
        for f in bar:
            sx, sy = limited(f)

            def reach(c, d):
                return f[c] + (d[:, 0, None] - gas.x[cl] * s) * sx[c] + (d[:, 1, None] - gas.y[cl] * s) * sy[c]

            left = reach(geo.L, geo.dL)
            right = reach(geo.R.clamp(min=0), geo.dR)
            up_ = torch.where(dn > 0, left, torch.where(dn < 0, right, 0.5 * (left + right)))
            at.append(torch.where(inner[:, None], up_, left))
        return bar, at, dn

    for _ in range(case["steps"]):
        cell = gas.state(moments(), dt)
        a_cell = gas.correction(cell)
        t = gas.tau(cell)
        al, be = ((2 * t - s) / (2 * t + dt))[:, None], (3 * s / (2 * t + dt))[:, None]
        fm = torch.zeros((int(inner.sum()), 11), dtype=torch.float64, device=dev)
        out_flux = torch.zeros(len(geo.L), dtype=torch.float64, device=dev)
        for cl in gas.chunks():
            _, at, dn = faces(cl, cell, al, be, a_cell)
            fm += gas.sums(cl, at[0][inner], at[1][inner])
            out_flux += (torch.where(dn > 0, dn * at[0], torch.zeros_like(dn)) * gas.w[cl]).sum(1)
        face = gas.state(fm, s)
        a_face = gas.correction(face)
        tf = gas.tau(face)
        k1, k2 = (2 * tf / (2 * tf + s))[:, None], (s / (2 * tf + s))[:, None]
        given = {}
        for b, at_b in walls.items():
            if not len(at_b) or p.bcs[b].kind == workloads.OUTFLOW:
                continue
            bc = p.bcs[b]
            wall = bc.kind == workloads.WALL
            row = up([[1.0 if wall else bc.rho, bc.u, bc.v, bc.T, 0.0, 0.0]])
            scale = torch.ones(len(at_b), dtype=torch.float64, device=dev)
            if wall:
                into = torch.zeros(len(at_b), dtype=torch.float64, device=dev)
                for cl in gas.chunks():
                    dn = geo.n[at_b, 0, None] * gas.x[cl] + geo.n[at_b, 1, None] * gas.y[cl]
                    into += (torch.where(dn < 0, dn * gas.target(row, cl)[0], torch.zeros_like(dn)) * gas.w[cl]).sum(1)
                scale = -out_flux[at_b] / into
            given[b] = (row, scale)
        for cl in gas.chunks():
            bar, at, dn = faces(cl, cell, al, be, a_cell)
            full = gas.target(face, cl, a_face)
            for comp, keep in ((0, g), (1, h)):
                phi = at[comp]
                phi[inner] = k1 * phi[inner] + k2 * full[comp]
                for b, at_b in walls.items():
                    if not len(at_b):
                        continue
                    if b in given:
                        row, scale = given[b]
                        come = scale[:, None] * gas.target(row, cl)[comp]
                    else:
                        come = bar[comp][geo.L[at_b]]
                    phi[at_b] = torch.where(dn[at_b] > 0, phi[at_b], come)
                flux = geo.A[:, None] * dn * phi
                total = torch.zeros_like(bar[comp]).index_add_(0, geo.L, flux).index_add_(0, Ri, -flux[inner])
                keep[:, cl] = 4 / 3 * bar[comp] - keep[:, cl] / 3 - (dt / geo.vol)[:, None] * total
    m = moments()
    end = gas.state(m, dt)
    out = dict(fields=end)
    if case["precision"] == 64 and p.dim == 2:
        press = end[:, 0] * p.R * end[:, 3]
        out["stress"] = torch.stack([m[:, 3] - m[:, 1] ** 2 / m[:, 0] - press, m[:, 4] - m[:, 1] * m[:, 2] / m[:, 0],
                                     m[:, 5] - m[:, 2] ** 2 / m[:, 0] - press], 1)
    if nc * len(x) <= WHOLE_STATE:
        out["g"], out["h"] = g.reshape(-1), h.reshape(-1)
    return out
