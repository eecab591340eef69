"""The work a user has this library do, as cases to be timed and compared.

A pass advances a simulation by `steps` S2O4 steps and reads the state back to the host, as a program
does that writes a snapshot every so many steps; the training case fits the indicator network for
one epoch and fetches its parameters.  The mesh is the plan a program keeps: it is built once per
mesh and shared by every state on it, while the initial data of a state come from the seed.
Sizes are those of the named configurations, the tests and the benchmark (`workloads.CONFIGS`,
bench.py) where these have one, smaller ones of the same generators otherwise.

The snapshot of a mixed-precision state is kept in single precision, the precision its momenta and
gradients are held in.
"""
import functools
import io
import math

import numpy as np

import paper_2306_04467_amd as gks
from workloads import meshes

G, EPS, EPS_NUM, CFL = 9.81, 0.05, 5.0, 0.3
H_DRY = 1e-6
MLP_IN, MLP_H = 44, 64

# flow -> (density ratio, boundary)
FLOWS = {
    "periodic": (0.98, "periodic"),  # smooth plane waves on right triangles of [0, 2]^2
    "lake": (0.98, "wall"),          # lake at rest over a bump with a perturbed interface in a disk
    "dam": (0.95, "wall"),           # two-layer dam break over a sinusoidal bottom
    "smooth": (0.95, "wall"),        # both layers varying smoothly over a low bump
    "dry": (1.0, "wall"),            # the paper's two-layer dam break onto a dry upper bed
}


def listed():
    return [
        # the smallest configuration: 800 right triangles, where a step is launches and latency
        _case("periodic_800_fp64", "periodic", 20, "fp64", 50),
        # the well-balance test's size with walls, monitored: device diagnostics every 10 steps
        _case("lake_3200_logged_fp64", "lake", 40, "fp64", 40, log_every=10),
        # a test-sized dam break with nonlinear weights along its front, 10,082 triangles
        _case("dam_10k_fp64", "dam", 71, "fp64", 20),
        # the mixed path at an ordinary size: smooth flow over a bump, 20,000 triangles
        _case("smooth_20k_fp32", "smooth", 100, "fp32", 15),
        # the higher-order layer coupling on a dam break, 180,000 triangles
        _case("dam_180k_src4_fp64", "dam", 300, "fp64", 40, src_order=4),
        # discontinuous interface values in the gradient update, mixed path, 180,000 triangles
        _case("smooth_180k_disc_fp32", "smooth", 300, "fp32", 60, grad_mode="discontinuous"),
        # wet/dry layers: the paper's dam break at its fine cell size, 160,000 triangles
        _case("dry_160k_fp64", "dry", 400, "fp64", 40),
        # the headline workload, both precisions: 520,200 triangles, perturbed lake at rest
        _case("lake_520k_fp64", "lake", 510, "fp64", 100),
        _case("lake_520k_fp32", "lake", 510, "fp32", 100),
        # the million-triangle dam break
        _case("dam_1M_fp64", "dam", 707, "fp64", 50),
        # an ensemble of uneven scenarios replayed from one graph, FP32 with the learned indicator
        _case("ensemble_12_ind_fp32", "lake", 50, "fp32", 50, scenarios=12, n_max=158, indicator=True),
        # one epoch of the indicator's training on 32,768 samples
        {"name": "train_32k", "flow": "train", "samples": 32768, "batch": 2048},
    ]


def _case(name, flow, n, precision, steps, **options):
    c = {"name": name, "flow": flow, "n": n, "precision": precision, "steps": steps, "log_every": 0, "graph": False,
         "src_order": 2, "grad_mode": "continuous", "alpha_mode": "reading", "indicator": False, "scenarios": 1,
         "n_max": n}
    c.update(options)
    return c


def draw(rng):
    """One more case: log-uniform sizes from 200 to a million triangles, both precisions, eager steps or
    graph replay, now and then an ensemble, a training epoch, or one of the scheme's options."""

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.random()
    if kind < 0.08:
        return {"flow": "train", "samples": log_int(4000, 60000), "batch": rng.choice([256, 512, 1024, 2048])}
    precision = rng.choice(["fp64", "fp32"])
    if kind < 0.25:
        n = log_int(20, 60)
        return _unnamed("lake", n, precision, rng.randint(20, 40), scenarios=rng.randint(2, 16),
                        n_max=rng.randint(n + 10, 170), indicator=rng.random() < 0.5)
    if kind < 0.55:
        # the options, at the sizes they are benchmarked at
        n, option = log_int(260, 510), rng.randrange(5)
        steps = rng.randint(20, 40)
        if option == 0:
            return _unnamed("dam", n, precision, steps, src_order=4)
        if option == 1:
            return _unnamed("smooth", n, precision, steps, grad_mode="discontinuous")
        if option == 2:
            return _unnamed("lake", n, precision, steps, alpha_mode="paper")
        if option == 3:
            return _unnamed("dam", n, precision, steps, indicator=True)
        return _unnamed("dry", n + 120, precision, steps)
    flow = rng.choice(["periodic", "lake", "dam", "smooth"])
    n = log_int(10, 600)
    steps = rng.randint(5, 60) if n < 300 else rng.randint(10, 50)
    return _unnamed(flow, n, precision, steps, graph=rng.random() < 0.3, log_every=rng.choice([0, 0, 0, 5, 10]))


def _unnamed(*args, **options):
    c = _case("", *args, **options)
    del c["name"]
    return c


# ---------------------------------------------------------------------------------------------
# inputs


@functools.lru_cache(maxsize=64)
def _grid(flow, n, mesh_seed):
    """(node_xy, tri, node_B, periodic_L) of a flow's mesh."""
    if flow == "periodic":
        xy, tri, L = meshes.periodic_square(n, 2.0)
        return xy, tri, np.zeros(len(xy)), L
    if flow == "dry":
        xy, tri = meshes.jittered_rect(n, max(n // 2, 2), 1.0, 0.5, mesh_seed)
        return xy, tri, np.zeros(len(xy)), None
    xy, tri = meshes.jittered_square(n, mesh_seed)
    if flow == "dam":
        B = 0.1 * np.sin(2 * np.pi * xy[:, 0]) * np.sin(2 * np.pi * xy[:, 1])
    else:
        amp, k = (0.5, 50.0) if flow == "lake" else (0.1, 30.0)
        B = amp * np.exp(-k * ((xy[:, 0] - 0.5) ** 2 + (xy[:, 1] - 0.5) ** 2))
    return xy, tri, B, None


@functools.lru_cache(maxsize=64)
def _mesh(flow, n, mesh_seed):
    xy, tri, B, L = _grid(flow, n, mesh_seed)
    return gks.Mesh(xy, tri, B, L, boundary=FLOWS[flow][1])


def _members(case):
    """(flow, n, mesh seed) of each scenario; sizes of an ensemble spread over their logarithm."""
    s = case["scenarios"]
    if s == 1:
        return [(case["flow"], case["n"], 20230604)]
    lo, hi = math.log(case["n"]), math.log(case["n_max"])
    return [(case["flow"], int(round(math.exp(lo + (hi - lo) * ((7 * i) % s) / (s - 1)))), 20230607 + i)
            for i in range(s)]


@functools.lru_cache(maxsize=8)
def _batch(members):
    return gks.Mesh.batch([_mesh(*m) for m in members])


# degree-5 rule of 7 points on the triangle (barycentric orbits and weights), 3-point Gauss on [0, 1]
_TRI = [(1 / 3, 1 / 3, 1 / 3, 0.225)]
for _a, _b, _w in ((0.101286507323456, 0.797426985353087, 0.125939180544827),
                   (0.470142064105115, 0.059715871789770, 0.132394152788506)):
    _TRI += [(_b, _a, _a, _w), (_a, _b, _a, _w), (_a, _a, _b, _w)]
_GL3 = [(0.5 - math.sqrt(0.15), 5 / 18), (0.5, 8 / 18), (0.5 + math.sqrt(0.15), 5 / 18)]


def _averages(xy, tri, fn):
    """Cell averages [6, T] and cell-averaged gradients [6, 2, T] of fn(x, y) -> [6, T]."""
    p = [xy[tri[:, k]] for k in range(3)]
    W = 0.0
    for a, b, c, w in _TRI:
        q = a * p[0] + b * p[1] + c * p[2]
        W = W + w * fn(q[:, 0], q[:, 1])
    area = 0.5 * ((p[1] - p[0])[:, 0] * (p[2] - p[0])[:, 1] - (p[2] - p[0])[:, 0] * (p[1] - p[0])[:, 1])
    g = 0.0
    for k in range(3):
        e = p[(k + 1) % 3] - p[k]
        for s, w in _GL3:
            q = p[k] + s * e
            v = w * fn(q[:, 0], q[:, 1]) / area
            g = g + np.stack([v * e[:, 1], -v * e[:, 0]], axis=1)
    return W, g


def _bottom(xy, tri, B):
    """Cell mean and gradient of the piecewise linear bottom."""
    p = [xy[tri[:, k]] for k in range(3)]
    b = [B[tri[:, k]] for k in range(3)]
    e1, e2 = p[1] - p[0], p[2] - p[0]
    r1, r2 = b[1] - b[0], b[2] - b[0]
    det = e1[:, 0] * e2[:, 1] - e1[:, 1] * e2[:, 0]
    grad = np.stack([(r1 * e2[:, 1] - e1[:, 1] * r2) / det, (e1[:, 0] * r2 - r1 * e2[:, 0]) / det])
    return (b[0] + b[1] + b[2]) / 3.0, grad


def _initial(member, rng):
    """Cell averages and gradients of (h2, h2U2, h2V2, h1, h1U1, h1V1) at t = 0."""
    flow = member[0]
    xy, tri, B, _ = _grid(*member)
    T = len(tri)
    a, b, ph = rng.uniform(0.5, 1.0), rng.uniform(0.5, 1.0), rng.uniform(0.0, 2 * np.pi)
    if flow == "periodic":
        def cons(x, y):
            s = np.sin(np.pi * (x + y) + ph)
            h1, h2 = 1 + 0.2 * a * s, 1 - 0.1 * b * s
            return np.stack([h2, 0.5 * h2, 0.5 * h2, h1, 0.5 * h1, 0.5 * h1])
        return _averages(xy, tri, cons)
    Bm, gB = _bottom(xy, tri, B)
    if flow == "smooth":
        tp = 2 * np.pi

        def cons(x, y):
            eta = 1 + 0.05 * a * np.sin(tp * x + ph) * np.cos(tp * y)
            h2 = 0.5 + 0.04 * b * np.cos(tp * x + 0.4) * np.sin(tp * y + ph)
            return np.stack([h2, 0.1 * h2 * np.cos(tp * (x + y)), 0.15 * h2,
                             eta, eta * (0.2 + 0.1 * np.sin(tp * y)), -0.1 * eta * np.cos(tp * x)])
        W, g = _averages(xy, tri, cons)
        U, V = W[4] / W[3], W[5] / W[3]
        W[3] -= Bm
        W[4], W[5] = U * W[3], V * W[3]
        g[3] -= gB
        g[4] -= U * gB
        g[5] -= V * gB
        return W, g
    c = xy[tri].mean(axis=1)
    W, g = np.zeros((6, T)), np.zeros((6, 2, T))
    if flow == "lake":
        eta, h2 = np.full(T, 0.8), np.full(T, 0.2)
        x0, y0 = rng.uniform(0.25, 0.75, 2)
        inside = (c[:, 0] - x0) ** 2 + (c[:, 1] - y0) ** 2 < 0.1 ** 2
        eta[inside] += 2e-3 * a
        h2[inside] -= 2e-3 * a
    elif flow == "dam":
        left = c[:, 0] < 0.4 + 0.2 * (a - 0.5)
        eta, h2 = np.where(left, 0.9 + 0.1 * a, 0.5), np.where(left, 0.5, 0.9 + 0.1 * b)
    else:  # dry
        left = c[:, 0] < 0.4 + 0.2 * (a - 0.5)
        eta, h2 = np.full(T, 0.3 + 0.1 * b), np.where(left, 1.0, 0.0)
    W[0], W[3] = h2, eta - Bm
    g[3] = -gB
    return W, g


def _quiescence_network():
    """Parameters of an indicator that skips the nonlinear weights where both levels vary by less than
    about 1e-7 of their thickness: the decision a trained one comes to, without the training.  The other
    weights are small, so that the whole network takes part."""
    rng = np.random.default_rng(7)
    W1 = rng.normal(0, 1e-3, (MLP_IN, MLP_H))
    W2 = rng.normal(0, 1e-3, (MLP_H, MLP_H))
    w3 = rng.normal(0, 1e-3, MLP_H)
    b1, b2 = np.zeros(MLP_H), np.zeros(MLP_H)
    for k in range(2):  # features 34 and 35: log10(variation / thickness) / 4
        W1[34 + k, k] = 4.0
        b1[k] = 7.0
        W2[k, k] = 1.0
        w3[k] = -8.0
    p = [W1.ravel(), b1, W2.ravel(), b2, w3, np.array([2.0])]
    return np.concatenate(p).astype(np.float32)


def _training_set(case, seed):
    """Feature rows of the shapes a state gives (scaled differences and gradients, sizes of the
    variation, geometry), labels 1 where the variation is small, and initial parameters."""
    rng = np.random.default_rng(seed)
    n = case["samples"]
    X = np.empty((n, MLP_IN), dtype=np.float32)
    X[:, :34] = rng.normal(0, 0.4, (n, 34)).clip(-1, 1)
    X[:, 34:38] = rng.uniform(-2.0, 0.0, (n, 4))
    X[:, 38:] = rng.uniform(0.5, 2.0, (n, 6))
    y = (X[:, 34] + X[:, 35] + 0.2 * X[:, 0] * X[:, 17] + rng.normal(0, 0.1, n) < -2.0).astype(np.uint8)
    P = [rng.normal(0, math.sqrt(2 / MLP_IN), MLP_IN * MLP_H), np.zeros(MLP_H),
         rng.normal(0, math.sqrt(2 / MLP_H), MLP_H * MLP_H), np.zeros(MLP_H),
         rng.normal(0, math.sqrt(1 / MLP_H), MLP_H), np.zeros(1)]
    return X, y, np.concatenate(P).astype(np.float32)


def _chi(case, i):
    return FLOWS[case["flow"]][0] - 0.005 * i  # the scenarios of an ensemble differ in their density ratio


def prepare(case, seed):
    if case["flow"] == "train":
        X, y, P = _training_set(case, seed)
        trainer = gks.Trainer(len(y), P, max_batch=case["batch"])
        trainer.add(X, y)
        return {"case": case, "trainer": trainer, "seed": seed % 1000}
    rng = np.random.default_rng(seed)
    members = _members(case)
    data = [_initial(m, rng) for m in members]
    mesh = _mesh(*members[0]) if len(members) == 1 else _batch(tuple(members))
    params = [gks.make_params(G=G, chi=_chi(case, i), cfl=CFL, eps=EPS, eps_num=EPS_NUM, precision=case["precision"],
                              alpha_mode=case["alpha_mode"], src_order=case["src_order"],
                              grad_mode=case["grad_mode"], h_dry=H_DRY if case["flow"] == "dry" else 0.0)
              for i in range(len(members))]
    st = gks.State(mesh, np.concatenate([d[0] for d in data], axis=1), np.concatenate([d[1] for d in data], axis=2),
                   params=params)
    if case["indicator"]:
        st.indicator(_quiescence_network(), 0.0)
    return {"case": case, "state": st}


def run(state):
    case = state["case"]
    if case["flow"] == "train":
        losses = state["trainer"].fit(1, batch=case["batch"], lr=2e-3, seed=state["seed"])
        return {"loss": losses, "params": state["trainer"].params()}
    st = state["state"]
    out = {}
    if case["log_every"]:
        last = st.run_logged(case["steps"], io.StringIO(), every=case["log_every"])
        out["log"] = np.array([last[k] for k in st.DIAGNOSTICS])
    elif case["scenarios"] > 1 or case["graph"]:
        st.batch_step(case["steps"])
    else:
        st.step(case["steps"])
    W, grad, t = st.read()
    out.update(W=W, grad=grad, t=np.float64(t))
    if case["precision"] == "fp32":
        out = {k: v.astype(np.float32) for k, v in out.items()}
    return out


def work(case):
    """Per stage and cell: the least-squares operator, geometry and stencil once, the state in and out
    and the stage carry once, the edges' normals and bottom; then the snapshot.  Arithmetic as counted
    from the scheme (12 kFLOP per cell and stage).  Training: features once, 2 + 4 FLOPs per weight and
    sample."""
    if case["flow"] == "train":
        weights = MLP_IN * MLP_H + MLP_H * MLP_H + MLP_H
        return {"bytes": 4.0 * case["samples"] * (MLP_IN + 1), "flops": 6.0 * weights * case["samples"]}
    T = sum(_cells(m) for m in _members(case))
    r = 8 if case["precision"] == "fp64" else 4
    cell = 153 * r + 13 * r + 9 * 4 + 5 * 8 + 9 * 8 + 2 * (2 * 8 + 16 * r) + (6 * 8 + 12 * r)
    edge = 4 * r + 2 * 8 + 3 * 4
    stages = 2 * case["steps"]
    return {"bytes": float(stages * T * (cell + 1.5 * edge) + 18 * 8 * T), "flops": 12e3 * stages * T}


def _cells(member):
    flow, n, _ = member
    return 2 * n * max(n // 2, 2) if flow == "dry" else 2 * n * n


# ---------------------------------------------------------------------------------------------
# the same in plain numpy, 64 bits


def exact(case, seed):
    if case["flow"] == "train":
        return _exact_training(case, seed)
    members = _members(case)
    if 2 * case["steps"] * sum(_cells(m) for m in members) > 6e5:
        return None  # over about 20 seconds
    if case["indicator"]:
        return None  # the network decides in bfloat16 which cells take the linear weights
    rng = np.random.default_rng(seed)
    floor = 1e-18 if case["precision"] == "fp64" else 1e-10  # of the smoothness indicators, per precision
    runs = []
    for i, m in enumerate(members):
        s = _Scheme(m, _chi(case, i), floor)
        runs.append((s, s.advance(*_initial(m, rng), case["steps"])))
    out = {"W": np.concatenate([r[1][0] for r in runs], axis=1),
           "grad": np.concatenate([r[1][1] for r in runs], axis=2), "t": np.float64(runs[0][1][2])}
    if case["log_every"]:
        s, (W, _, t, dt) = runs[0]
        eta1 = W[3] + s.Bm
        speed = [(np.hypot(W[k + 1], W[k + 2]) / W[k]).max() for k in (0, 3)]
        out["log"] = np.array([t, dt, (s.area * W[0]).sum(), (s.area * W[3]).sum(), speed[0], speed[1],
                               np.ptp(eta1), np.ptp(eta1 + W[0])])
    return out


def _exact_training(case, seed):
    X, y, P = (a.astype(np.float64) for a in _training_set(case, seed))
    n, batch, lr = len(y), case["batch"], float(np.float32(2e-3))
    # the sample order: Fisher-Yates on splitmix64 from the seed
    order, x, mask = list(range(n)), seed % 1000, (1 << 64) - 1
    for i in range(n - 1, 0, -1):
        x = (x + 0x9E3779B97F4A7C15) & mask
        z = ((x ^ (x >> 30)) * 0xBF58476D1CE4E5B9) & mask
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & mask
        j = (z ^ (z >> 31)) % (i + 1)
        order[i], order[j] = order[j], order[i]
    cut = np.cumsum([MLP_IN * MLP_H, MLP_H, MLP_H * MLP_H, MLP_H, MLP_H])
    m, v, losses = np.zeros_like(P), np.zeros_like(P), []
    b1, b2 = float(np.float32(0.9)), float(np.float32(0.999))
    for k, off in enumerate(range(0, n, batch)):
        idx = order[off:off + batch]
        W1, c1, W2, c2, w3, c3 = np.split(P, cut)
        W1, W2 = W1.reshape(MLP_IN, MLP_H), W2.reshape(MLP_H, MLP_H)
        h1 = np.maximum(X[idx] @ W1 + c1, 0)
        h2 = np.maximum(h1 @ W2 + c2, 0)
        z = h2 @ w3 + c3
        losses.append((np.maximum(z, 0) + np.log1p(np.exp(-np.abs(z))) - y[idx] * z).mean())
        dz = (1 / (1 + np.exp(-z)) - y[idx]) / len(idx)
        d2 = np.where(h2 > 0, dz[:, None] * w3, 0)
        d1 = np.where(h1 > 0, d2 @ W2.T, 0)
        g = np.concatenate([(X[idx].T @ d1).ravel(), d1.sum(0), (h1.T @ d2).ravel(), d2.sum(0), dz @ h2, [dz.sum()]])
        m = b1 * m + (1 - b1) * g
        v = b2 * v + (1 - b2) * g * g
        P = P - lr * (m / (1 - b1 ** (k + 1))) / (np.sqrt(v / (1 - b2 ** (k + 1))) + 1e-8)
    return {"loss": np.array([np.mean(losses)]), "params": P}


class _Scheme:
    """The compact gas-kinetic scheme with its default options on one mesh."""

    def __init__(self, member, chi, floor):
        xy, tri, B, L = _grid(*member)
        self.chi, self.floor, T = chi, floor, len(tri)
        P = xy[tri]                                             # [T, 3, 2]
        self.Bm, self.gB = _bottom(xy, tri, B)
        e1, e2 = P[:, 1] - P[:, 0], P[:, 2] - P[:, 0]
        self.area = 0.5 * (e1[:, 0] * e2[:, 1] - e1[:, 1] * e2[:, 0])
        self.hs = np.sqrt(2 * self.area)
        cen = P.mean(axis=1)
        side = np.roll(P, -1, axis=1) - P                       # edge k: vertex k to k + 1
        length = np.hypot(side[..., 0], side[..., 1])           # [T, 3]
        self.dx = (2 * self.area / length.max(axis=1)).min()
        # edges: pairs of (cell, local edge) with the same end points (modulo the periods)
        node = np.arange(len(xy))
        if L is not None:
            q = np.round(np.mod(xy / np.array(L), 1.0) * 2 ** 30).astype(np.int64) % 2 ** 30
            node = np.unique(q, axis=0, return_inverse=True)[1].reshape(-1)
        ends = np.sort(np.stack([node[tri], node[np.roll(tri, -1, axis=1)]], axis=-1).reshape(-1, 2), axis=1)
        eid = np.unique(ends, axis=0, return_inverse=True)[1].reshape(-1)
        E = eid.max() + 1
        first = np.full(E, 3 * T)
        np.minimum.at(first, eid, np.arange(3 * T))
        last = np.full(E, -1)
        np.maximum.at(last, eid, np.arange(3 * T))
        self.eL, self.kL, self.eR, self.kR = first // 3, first % 3, last // 3, last % 3
        self.wall = first == last
        self.edge = eid.reshape(T, 3)
        self.left = first[self.edge] == np.arange(3 * T).reshape(T, 3)
        s = side[self.eL, self.kL]
        self.n = np.stack([s[:, 1], -s[:, 0]]) / length[self.eL, self.kL]   # [2, E]
        sign = np.where(self.left, 1.0, -1.0)
        self.fl = sign * length / self.area[:, None]            # [T, 3]
        self.gg = self.fl[:, None, :] * np.moveaxis(self.n[:, self.edge], 0, 1)   # [T, 2, 3]
        gp = 0.5 - math.sqrt(3) / 6, 0.5 + math.sqrt(3) / 6
        self.gp = gp
        Bp, Bq = B[tri[self.eL, self.kL]], B[tri[self.eL, (self.kL + 1) % 3]]
        self.Bg = np.stack([(1 - g) * Bp + g * Bq for g in gp])             # [2, E]
        gBL, gBR = self.gB[:, self.eL], self.gB[:, self.eR]
        mirrored = gBL - 2 * (gBL * self.n).sum(0) * self.n
        self.egB = 0.5 * (gBL + np.where(self.wall, mirrored, gBR))         # [2, E]
        # images of the neighbours: cell, linear part (reflection across a wall) and offset
        other = np.where(self.left, self.eR[self.edge], self.eL[self.edge])
        back = np.where(self.left, self.kR[self.edge], self.kL[self.edge])
        u = side / length[..., None]
        R = np.where(self.wall[self.edge][..., None, None],
                     2 * u[..., :, None] * u[..., None, :] - np.eye(2), np.eye(2))       # [T, 3, 2, 2]
        there = P[other, (back + 1) % 3]
        there = np.where(self.wall[self.edge][..., None], P, there)  # the image of this edge's first vertex
        off = P - np.einsum("tkij,tkj->tki", R, there)
        cells, maps, offs = [other], [R], [off]
        for k in range(3):
            for q in (1, 2):
                b = (back[:, k] + q) % 3
                f = other[:, k]
                cells.append(other[f, b][:, None])
                maps.append(np.einsum("tij,tjk->tik", R[:, k], R[f, b])[:, None])
                offs.append((np.einsum("tij,tj->ti", R[:, k], off[f, b]) + off[:, k])[:, None])
        self.sten, self.map = np.concatenate(cells, axis=1), np.concatenate(maps, axis=1)     # [T, 9], [T, 9, 2, 2]
        offs = np.concatenate(offs, axis=1)
        img = np.einsum("tsij,tsvj->tsvi", self.map, P[self.sten]) + offs[:, :, None]
        img = (np.concatenate([P[:, None], img], axis=1) - cen[:, None, None]) / self.hs[:, None, None, None]
        # least squares: averages over the nine neighbours, mean gradients of the cell and its face neighbours
        mean, mx, my = self._means(img)
        self.mean0 = mean[:, 0]
        A = np.concatenate([mean[:, 1:] - mean[:, :1], np.stack([mx[:, :4], my[:, :4]], axis=2).reshape(T, 8, 9)], axis=1)
        Q, Rt = np.linalg.qr(A)
        self.M = np.linalg.solve(Rt, np.swapaxes(Q, 1, 2))      # [T, 9, 17]
        c1 = img[:, 1:4].mean(axis=2)                           # face neighbours' centroids
        c2 = np.roll(c1, -1, axis=1)
        self.cross = c1[..., 0] * c2[..., 1] - c1[..., 1] * c2[..., 0]
        size = np.hypot(c1[..., 0], c1[..., 1]) * np.hypot(c2[..., 0], c2[..., 1])
        self.cand = np.concatenate([np.abs(self.cross) >= 0.2 * size, np.ones((T, 1), bool)], axis=1)
        self.c1, self.c2 = c1, c2
        v = img[:, 0]                                           # [T, 3, 2] scaled vertices
        self.pts = np.stack([v[:, k] + g * (v[:, (k + 1) % 3] - v[:, k]) for k in range(3) for g in gp], axis=1)
        self.v = v

    @staticmethod
    def _basis(x, y):
        one, nul = np.ones_like(x), np.zeros_like(x)
        f = np.stack([x, y, x * x, x * y, y * y, x ** 3, x * x * y, x * y * y, y ** 3], axis=-1)
        fx = np.stack([one, nul, 2 * x, y, nul, 3 * x * x, 2 * x * y, y * y, nul], axis=-1)
        fy = np.stack([nul, one, nul, x, 2 * y, nul, x * x, 2 * x * y, 3 * y * y], axis=-1)
        return f, fx, fy

    def _means(self, img):
        """Means over triangles img[..., 3, 2] of the basis and its derivatives (a degree-5 rule)."""
        f = fx = fy = 0.0
        s15 = math.sqrt(15.0)
        rule = [((1 / 3, 1 / 3, 1 / 3), 0.225)]
        for sg in (1, -1):
            a, w = (6 - sg * s15) / 21, (155 - sg * s15) / 1200
            rule += [(tuple(1 - 2 * a if i == j else a for i in range(3)), w) for j in range(3)]
        for lam, w in rule:
            p = sum(l * img[..., i, :] for i, l in enumerate(lam))
            b, bx, by = self._basis(p[..., 0], p[..., 1])
            f, fx, fy = f + w * b, fx + w * bx, fy + w * by
        return f, fx, fy

    def advance(self, W, g, steps):
        W, g, t, dt = W.copy(), g.copy(), 0.0, 0.0
        for _ in range(steps):
            speed = max((np.hypot(W[k + 1], W[k + 2]) / W[k] + np.sqrt(G * W[k])).max() for k in (0, 3))
            dt = CFL * self.dx / speed
            L, Lt, GG, GGt = self._rates(W, g, dt)
            Wh, gh = W + 0.5 * dt * L + dt * dt / 8 * Lt, GG + 0.5 * dt * GGt
            _, Lt2, _, GGt2 = self._rates(Wh, gh, dt)
            W, g = W + dt * L + dt * dt * (Lt / 6 + Lt2 / 3), GG + dt * GGt2
            t += dt
        return W, g, t, dt

    def _rates(self, W, g, dt):
        vals, grads, ratio = self._reconstruct(W, g)
        return self._evolve(W, vals, grads, ratio, dt)

    def _reconstruct(self, W, g):
        """Values [6, T, 6] and gradients [6, 2, T, 6] at the Gauss points (eta1 in place of h1), and
        the weight ratios omega0 / d0 of eta1 and h2."""
        Q, gq = W.copy(), g.copy()
        Q[3] += self.Bm
        gq[3] += self.gB
        S, A, T = self.sten, self.map, len(self.area)
        F, Af = S[:, :3], A[:, :3]
        vals, grads, ratios = np.empty((6, T, 6)), np.empty((6, 2, T, 6)), {}
        f, fx, fy = self._basis(self.pts[..., 0], self.pts[..., 1])     # [T, 6, 9]
        f = f - self.mean0[:, None]
        cand, d = self.cand, 0.05 * self.cand
        d0 = 1 - d.sum(axis=1)
        for v in range(6):
            if v % 3 == 0:
                q = Q[v][S]
                ng = np.einsum("tsij,jts->tsi", Af, gq[v][:, F])
            else:
                m = 3 * (v // 3) + 1
                i = v - m
                q = A[..., i, 0] * Q[m][S] + A[..., i, 1] * Q[m + 1][S]
                jac = Af[..., i, 0][..., None] * np.moveaxis(gq[m][:, F], 0, -1) + \
                    Af[..., i, 1][..., None] * np.moveaxis(gq[m + 1][:, F], 0, -1)
                ng = np.einsum("tsij,tsj->tsi", Af, jac)
            own = gq[v].T
            diff = q - Q[v][:, None]
            rhs = np.concatenate([diff, self.hs[:, None] * np.concatenate([own, ng.reshape(T, 6)], axis=1)], axis=1)
            a = np.einsum("tij,tj->ti", self.M, rhs)
            ra, rb = diff[:, :3], np.roll(diff[:, :3], -1, axis=1)
            with np.errstate(divide="ignore", invalid="ignore"):
                bx = np.where(cand[:, :3], (ra * self.c2[..., 1] - self.c1[..., 1] * rb) / self.cross, 0)
                by = np.where(cand[:, :3], (self.c1[..., 0] * rb - ra * self.c2[..., 0]) / self.cross, 0)
            bx = np.concatenate([bx, rhs[:, 9:10]], axis=1)
            by = np.concatenate([by, rhs[:, 10:11]], axis=1)
            beta0, bm = self._smoothness(a), 0.5 * (bx * bx + by * by)
            tau = np.where(cand, np.abs(beta0[:, None] - bm), 0).sum(axis=1) / cand.sum(axis=1)
            hl = W[3 * (v // 3)]
            floor = self.floor * np.maximum(Q[v] ** 2, 1e-20 if v % 3 == 0 else 1e-16 * G * hl ** 3)
            t0 = d0 * (1 + tau / (beta0 + floor))
            tm = d * (1 + tau[:, None] / (bm + floor[:, None]))
            tot = t0 + tm.sum(axis=1)
            ratio = t0 / tot / d0
            cm = tm / tot[:, None] - ratio[:, None] * d
            sx, sy = (cm * bx).sum(axis=1)[:, None], (cm * by).sum(axis=1)[:, None]
            px, py = self.pts[..., 0], self.pts[..., 1]
            dev = ratio[:, None] * np.einsum("tgk,tk->tg", f, a) + sx * px + sy * py
            gx = (ratio[:, None] * np.einsum("tgk,tk->tg", fx, a) + sx) / self.hs[:, None]
            gy = (ratio[:, None] * np.einsum("tgk,tk->tg", fy, a) + sy) / self.hs[:, None]
            if v % 3 == 0:
                ratios[v] = ratio
                hbar = W[v][:, None]
                slope = self.gB if v == 3 else np.zeros((2, T))
                bdev = self.hs[:, None] * (slope[0][:, None] * px + slope[1][:, None] * py)
                with np.errstate(divide="ignore", invalid="ignore"):
                    th = np.where(dev < 0, np.maximum(0, (0.9 * hbar - bdev) / -dev), 1).min(axis=1)
                th = np.minimum(1, th)[:, None]
                dev, gx, gy = th * dev, th * gx, th * gy
            vals[v], grads[v, 0], grads[v, 1] = Q[v][:, None] + dev, gx, gy
        return vals, grads, ratios

    def _smoothness(self, a):
        """1/2 mean |grad P|^2 + 1/4 mean |second derivatives|^2 + 1/8 |third derivatives|^2."""
        x, y = self.v[..., 0], self.v[..., 1]
        s1 = 0.0
        for q, w in ((0.445948490915964886, 0.223381589678011466), (0.091576213509770743, 1 / 3 - 0.223381589678011466)):
            for j in range(3):
                lam = [1 - 2 * q if i == j else q for i in range(3)]
                px, py = (sum(l * c[:, i] for i, l in enumerate(lam)) for c in (x, y))
                _, fx, fy = self._basis(px, py)
                s1 = s1 + w * ((fx * a).sum(-1) ** 2 + (fy * a).sum(-1) ** 2)
        s2 = 0.0
        for j in range(3):
            px, py = (0.5 * (c[:, j] + c[:, (j + 1) % 3]) for c in (x, y))
            pxx = 2 * a[:, 2] + 6 * a[:, 5] * px + 2 * a[:, 6] * py
            pxy = a[:, 3] + 2 * a[:, 6] * px + 2 * a[:, 7] * py
            pyy = 2 * a[:, 4] + 2 * a[:, 7] * px + 6 * a[:, 8] * py
            s2 = s2 + (pxx ** 2 + pxy ** 2 + pyy ** 2) / 3
        s3 = 36 * a[:, 5] ** 2 + 4 * a[:, 6] ** 2 + 4 * a[:, 7] ** 2 + 36 * a[:, 8] ** 2
        return 0.5 * s1 + 0.25 * s2 + 0.125 * s3

    def _evolve(self, W, vals, grads, ratio, dt):
        n, wall, E = self.n, self.wall, len(self.eL)
        tang = np.stack([-n[1], n[0]])
        slots = [[(self.eL, 2 * self.kL + g), (self.eR, np.where(wall, 2 * self.kL + g, 2 * self.kR + 1 - g))]
                 for g in (0, 1)]
        plane = self._plane(vals, slots)
        out = {"F": np.zeros((6, E)), "Ft": np.zeros((6, E)), "Wb": np.zeros((6, E)), "Wbt": np.zeros((6, E)),
               "H": np.zeros((2, E)), "Ht": np.zeros((2, E))}
        for layer in (0, 1):                       # 0 upper (h2), 1 lower (h1)
            o = 3 * layer
            fv = 3 - o                             # the other layer's height drives the force
            rt = ratio[fv]
            w = np.minimum(1, np.minimum(rt[self.eL], np.where(wall, rt[self.eL], rt[self.eR])))
            w = np.where(w < 1 - 1e-12, w, 1.0)
            gB = self.egB if layer == 1 else np.zeros((2, E))
            for g in (0, 1):
                sides = []
                for s, (cell, slot) in enumerate(slots[g]):
                    h = vals[o, cell, slot] - (self.Bg[g] if layer == 1 else 0)
                    dl = grads[o, :, cell, slot].T                       # slope of the level
                    m = vals[o + 1:o + 3, cell, slot]
                    J = np.stack([grads[o + 1, :, cell, slot].T, grads[o + 2, :, cell, slot].T])   # [comp, dir, E]
                    f = w * grads[fv, :, cell, slot].T + (1 - w) * plane[fv][:, cell]
                    acc = -G * (self.chi if layer == 1 else 1.0) * f - G * gB
                    rot = np.stack([n, tang])                            # local axes
                    loc = {"h": h, "U": (m * n).sum(0) / h, "V": (m * tang).sum(0) / h,
                           "dh": np.einsum("aie,ie->ae", rot, dl - gB), "phi": np.einsum("aie,ie->ae", rot, acc),
                           "J": np.einsum("aie,bje,ije->abe", rot, rot, J)}
                    sides.append(loc)
                # the wall's mirror image of the left side
                mir = {k: v.copy() for k, v in sides[0].items()}
                mir["U"] = -mir["U"]
                # normal derivatives of even quantities and tangential ones of odd quantities change sign;
                # the single-valued bottom slope has no normal part at a wall
                for k in ("dh", "phi"):
                    mir[k][0] = -mir[k][0]
                mir["J"][0, 1] = -mir["J"][0, 1]
                mir["J"][1, 0] = -mir["J"][1, 0]
                R = {k: np.where(wall, mir[k], sides[1][k]) for k in mir}
                F, Ft, Wb, Wbt = self._gas_kinetic(sides[0], R, dt)
                F[0], Ft[0] = np.where(wall, 0, F[0]), np.where(wall, 0, Ft[0])
                for name, q in (("F", F), ("Ft", Ft), ("Wb", Wb), ("Wbt", Wbt)):
                    out[name][o] += 0.5 * q[0]
                    out[name][o + 1:o + 3] += 0.5 * (q[1] * n + q[2] * tang)
                out["H"][layer] += 0.25 * (sides[0]["h"] + R["h"])
                out["Ht"][layer] -= 0.25 * sum(q["J"][0, 0] + q["J"][1, 1] for q in (sides[0], R))
        ed = self.edge
        L, Lt = (-(self.fl * out[k][:, ed]).sum(-1) for k in ("F", "Ft"))
        GG, GGt = (np.einsum("tdk,vtk->vdt", self.gg, out[k][:, ed]) for k in ("Wb", "Wbt"))
        gH, gHt = (np.einsum("tdk,vtk->vdt", self.gg, out[k][:, ed]) for k in ("H", "Ht"))
        H, Ht = out["H"][:, ed].mean(-1), out["Ht"][:, ed].mean(-1)
        rate = L[[0, 3]].copy()                    # thickness rates of the two layers
        for layer in (0, 1):
            o, c = 3 * layer, self.chi if layer == 1 else 1.0
            L[o + 1:o + 3] += -G * W[o] * self.gB - c * G * H[layer] * gH[1 - layer]
            Lt[o + 1:o + 3] += -G * rate[layer] * self.gB - c * G * (Ht[layer] * gH[1 - layer] + H[layer] * gHt[1 - layer])
        return L, Lt, GG, GGt

    def _plane(self, vals, slots):
        """Gradients of the planes through the edge heights of eta1 (carried by the lower layer's
        velocity) and h2 (the upper layer's), per driving field."""
        hm = {0: 0.0, 3: 0.0}
        for g in (0, 1):
            for field, vel in ((3, 3), (0, 0)):
                z, h, un = [], [], []
                for cell, slot in slots[g]:
                    zz = vals[field, cell, slot]
                    hh = zz - (self.Bg[g] if field == 3 else 0)
                    z.append(zz)
                    h.append(hh)
                    un.append((vals[vel + 1:vel + 3, cell, slot] * self.n).sum(0) / hh)
                un[1] = np.where(self.wall, -un[0], un[1])
                lam = 2 / (G * (h[0] + h[1]))
                xi = 0.5 * _erfc(-np.sqrt(lam) * 0.5 * (un[0] + un[1]))
                hm[field] = hm[field] + 0.5 * (xi * z[0] + (1 - xi) * z[1])
        return {f: np.einsum("tdk,tk->dt", self.gg, hm[f][self.edge]) for f in hm}

    @staticmethod
    def _half(U, th, sign):
        """u-moments 0..5 of the Gaussian with mean U and variance th over sign * u > 0 (None: all u)."""
        if sign is None:
            M = [np.ones_like(U), U]
        else:
            m0 = 0.5 * _erfc(-sign * U / np.sqrt(2 * th))
            M = [m0, U * m0 + sign * np.sqrt(th / (2 * np.pi)) * np.exp(-U * U / (2 * th))]
        for k in range(2, 6):
            M.append(U * M[-1] + (k - 1) * th * M[-2])
        return M

    @staticmethod
    def _moments(q, h, U, V, M, e):
        """<u^e psi (a_n u + a_t v - 2 lam phi . c)> for psi = (1, u, v) over a (half) Maxwellian of
        thickness h, means U, V and u-moments M, the slopes from the data q."""
        lam, th = 1 / (G * h), 0.5 * G * h

        def N(k, j):  # <u^k (u - U)^j>
            return M[k] if j == 0 else N(k + 1, j - 1) - U * N(k, j - 1)

        al = [lam * q["dh"][d] / h for d in (0, 1)]
        be = [2 * lam * (q["J"][0, d] - U * q["dh"][d]) / h for d in (0, 1)]
        ga = [2 * lam * (q["J"][1, d] - V * q["dh"][d]) / h for d in (0, 1)]
        pn, pt = 2 * lam * q["phi"][0], 2 * lam * q["phi"][1]

        def plain(k):
            quad = N(k, 2) + th * N(k, 0)
            return (al[0] * (N(k + 1, 2) + th * N(k + 1, 0)) + be[0] * N(k + 1, 1) +
                    V * (al[1] * quad + be[1] * N(k, 1)) + ga[1] * th * N(k, 0) - pn * N(k, 1))

        cv = (th * (ga[0] * N(e + 1, 0) + V * ga[1] * N(e, 0) - pt * N(e, 0)) +
              al[1] * (th * N(e, 2) + 3 * th * th * N(e, 0)) + be[1] * th * N(e, 1))
        p = plain(e)
        return np.stack([h * p, h * plain(e + 1), h * (V * p + cv)])

    def _gas_kinetic(self, a, b, dt):
        half = self._half
        th = [0.5 * G * q["h"] for q in (a, b)]
        ML, MR = half(a["U"], th[0], 1), half(b["U"], th[1], -1)
        wb = [a["h"] * ML[k] + b["h"] * MR[k] for k in range(3)]
        hb = wb[0]
        U = wb[1] / hb
        V = (a["h"] * ML[0] * a["V"] + b["h"] * MR[0] * b["V"]) / hb
        B4 = np.stack([wb[1], wb[2], a["h"] * ML[1] * a["V"] + b["h"] * MR[1] * b["V"]])
        B5 = self._moments(a, a["h"], a["U"], a["V"], ML, 1) + self._moments(b, b["h"], b["U"], b["V"], MR, 1)
        t = 0.5 * G * hb
        Mp, Mm = half(U, t, 1), half(U, t, -1)
        wt = -(self._moments(a, hb, U, V, Mp, 0) + self._moments(b, hb, U, V, Mm, 0))
        pa, pb = a["phi"], b["phi"]
        c1 = [[M[k + 1] - U * M[k] for M in (Mp, Mm)] for k in range(3)]
        wt[0] -= 0.5 / G * (pa[0] * c1[0][0] + pb[0] * c1[0][1])
        B1 = np.stack([hb * U, hb * U * U + 0.5 * G * hb * hb, hb * U * V])
        B2 = self._moments(a, hb, U, V, Mp, 1) + self._moments(b, hb, U, V, Mm, 1)
        sn, stt = pa[0] + pb[0], pa[1] + pb[1]
        B2[1] -= 0.5 / G * (pa[0] * c1[2][0] + pb[0] * c1[2][1] - sn * U * t)
        B2[2] -= 0.5 / G * (V * (pa[0] * c1[1][0] + pb[0] * c1[1][1]) + t * (pa[1] * Mp[1] + pb[1] * Mm[1]) -
                            0.5 * t * (sn * V + stt * U))
        lam = 1 / (G * hb)
        aA, bA, gA = lam * wt[0] / hb, 2 * lam * (wt[1] - U * wt[0]) / hb, 2 * lam * (wt[2] - V * wt[0]) / hb
        mA = 2 * aA * t
        B3 = np.stack([hb * (U * mA + bA * t), hb * (U * U * mA + 2 * U * bA * t + 4 * aA * t * t),
                       hb * (U * V * mA + U * gA * t + V * bA * t)])
        pl, pr = a["h"] ** 2, b["h"] ** 2
        r = EPS + EPS_NUM * np.abs((pl - pr) / (pl + pr))   # collision time / dt

        def coefficients(s):  # the flux integrated over [0, s dt], per dt
            E = np.exp(-s / r)
            return np.stack([s - r * (1 - E), dt * (-r * s + 2 * r * r * (1 - E) - r * s * E),
                             dt * (0.5 * s * s - r * s + r * r * (1 - E)), r * (1 - E),
                             dt * (r * s * E - r * r * (1 - E))])

        full, part = coefficients(1.0), coefficients(0.5)
        B = [B1, B2, B3, B4, B5]
        I1, I2 = (sum(c[i] * B[i] for i in range(5)) for c in (full, part))
        return 4 * I2 - I1, 4 * (I1 - 2 * I2) / dt, np.stack([hb, wb[1], hb * V]), wt


def _erfc(x):
    """Complementary error function in 64 bits."""
    return _ERFC(x).astype(np.float64)


_ERFC = np.frompyfunc(math.erfc, 1, 1)
