"""Cases for timing the framework through its public entry points.

They cover what a program does with it, in the order in which it does it:
stencils of a point cloud, a shape parameter per stencil (network proposal,
its training, bisection) and the weights, the sparse operator, and time
stepping (explicit and implicit), each at the sizes of the repository's own
workloads: the 2500-node sphere with a fixed shape parameter up to the
1e6-node point cloud with n = 50, stencil sizes from the paper's n = 11 to
n = 101, FP64 and FP32 state.

Node sets are made from the seed on the GPU: Fibonacci spheres and
ellipsoids (rotated at random and jittered a little) and jittered parametric
tori, in an order that has nothing to do with space, as point clouds come.
Operators for the stepping cases hold a point-cloud Laplacian with Gaussian
weights, whose rows sum to zero and whose spectrum is bounded, so that every
seed gives a stable run.
"""
import math

import torch

import paper_1404_0812_amd as rb

SCHNAK = (0.1, 0.9, 50.0)                             # a, b, gamma
TURING_SPOTS = (0.899, -0.91, -0.899, 0.02, 0.2)      # alpha, beta, gamma, tau1, tau2


# ------------------------------------------------------------------ cases ----

def listed():
    return [
        # the smallest build: the 2500-node sphere, multiquadric, degree-2
        # border, one shape parameter for all stencils; stencils included
        dict(name="weights sphere 2500", kind="weights", surface="sphere", N=2500, n=31, kernel="mq", degree=2,
             mode="fixed", kappa=0.0),
        # the paper's own local system (inverse multiquadric, constant
        # border, n = 31) with bisection, on one of its sphere sizes
        dict(name="weights paper bisection", kind="weights", surface="sphere", N=10242, n=31, kernel="imq", degree=0,
             mode="bisect", kappa=1e12),
        # the point-cloud workload: proposals checked against the band, a few
        # fall back to bisection
        dict(name="weights cloud learned", kind="weights", surface="torus", N=250000, n=50, kernel="mq", degree=2,
             mode="learned", kappa=1e10),
        # many surfaces of uneven size and n (31, 50, 70, 101) in one call
        dict(name="weights batch", kind="batch", surfaces=16, nmax=101, low=400, high=4000, kappa=1e12),
        # extended precision for the convergence studies' high targets
        dict(name="weights double-double", kind="dd", N=2562, n=31, kernel="imq", mode="bisect", kappa=1e18),
        # stencils and spatial order of the large point cloud
        dict(name="knn cloud 1e6", kind="knn", surface="torus", N=1000000, n=50),
        # the network's shape parameters for the large point cloud
        dict(name="predict cloud 1e6", kind="predict", surface="torus", N=1000000, n=50),
        # training steps of the network on labelled stencils
        dict(name="train", kind="train", count=200000, n=50, batch=4096, steps=50),
        # operator of new stencils and weights, and its first application
        dict(name="operator 2e5", kind="operator", surface="torus", N=200000, n=50, prec="f64", applies=2),
        # reaction-diffusion of the large point cloud, FP32 state
        dict(name="rk4 cloud 1e6 f32", kind="rk4", surface="torus", N=1000000, n=50, prec="f32",
             reaction="schnakenberg", forced=False, steps=50),
        # heat on the small sphere to t = 0.1, FP64 state: launches count
        dict(name="rk4 sphere 2500 f64", kind="rk4", surface="sphere", N=2500, n=31, prec="f64", reaction="none",
             forced=False, steps=1000),
        # semi-implicit steps of a reaction-diffusion system, dt 100 times RK4's
        dict(name="imex sphere 10242", kind="imex", surface="sphere", N=10242, n=31, order=2, reaction="schnakenberg",
             dt_factor=100.0, steps=10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["weights", "weights", "weights", "batch", "dd", "knn", "predict", "train", "operator", "rk4",
                       "rk4", "imex"])
    surface = rng.choice(["sphere", "torus", "ellipsoid"])
    if kind == "weights":
        mode = rng.choice(["fixed", "bisect", "learned"])
        if mode == "fixed":
            n, N = rng.randint(11, 70), _log_int(rng, 2000, 20000)
            return dict(kind=kind, surface="sphere", N=N, n=n, kernel=rng.choice(["mq", "imq", "ga"]),
                        degree=rng.choice([0, 1, 2]) if n >= 20 else 0, mode=mode, kappa=0.0)
        if mode == "bisect":
            degree = rng.choice([0, 2])
            n = rng.randint(11, 31) if degree == 0 else rng.randint(25, 64)
            return dict(kind=kind, surface=surface, N=_log_int(rng, 600, 20000), n=n,
                        kernel="imq" if degree == 0 else "mq", degree=degree, mode=mode,
                        kappa=rng.choice([1e10, 1e12]))
        return dict(kind=kind, surface=surface, N=_log_int(rng, 5000, 250000), n=rng.randint(28, 54), kernel="mq",
                    degree=2, mode=mode, kappa=rng.choice([1e10, 1e12]))
    if kind == "batch":
        return dict(kind=kind, surfaces=rng.randint(3, 16), nmax=rng.choice([50, 70, 101]), low=_log_int(rng, 250, 500),
                    high=_log_int(rng, 1000, 4000), kappa=rng.choice([1e10, 1e12]))
    if kind == "dd":
        return dict(kind=kind, N=_log_int(rng, 642, 2562), n=rng.choice([11, 17, 31]),
                    kernel=rng.choice(["imq", "mq"]), mode=rng.choice(["bisect", "bisect", "given"]),
                    kappa=rng.choice([1e16, 1e18, 1e20]))
    if kind == "knn":
        return dict(kind=kind, surface=surface, N=_log_int(rng, 2000, 1000000), n=rng.choice([11, 17, 31, 50, 70]))
    if kind == "predict":
        return dict(kind=kind, surface=surface, N=_log_int(rng, 5000, 1000000), n=rng.randint(17, 50))
    if kind == "train":
        return dict(kind=kind, count=_log_int(rng, 20000, 200000), n=rng.randint(31, 50),
                    batch=64 * rng.choice([8, 15, 32, 64]), steps=rng.randint(10, 50))
    if kind == "operator":
        return dict(kind=kind, surface=surface, N=_log_int(rng, 2000, 200000), n=rng.randint(17, 101),
                    prec=rng.choice(["f64", "f32"]), applies=rng.randint(1, 3))
    if kind == "rk4":
        N = _log_int(rng, 642, 500000)
        return dict(kind=kind, surface=surface, N=N, n=rng.choice([17, 31, 50, 70]) if N < 200000 else rng.randint(31, 50),
                    prec=rng.choice(["f64", "f32"]), reaction=rng.choice(["none", "schnakenberg", "turing"]),
                    forced=rng.random() < 0.25, steps=_log_int(rng, 100, 1000) if N < 20000 else rng.randint(20, 50))
    N = _log_int(rng, 2000, 100000)
    return dict(kind=kind, surface=surface, N=N, n=rng.choice([17, 31, 50]), order=rng.choice([1, 2, 4]),
                reaction=rng.choice(["none", "schnakenberg", "turing"]), dt_factor=rng.choice([10.0, 100.0]),
                steps=rng.randint(5, 10))


# ------------------------------------------------------------------ nodes ----

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _nodes(surface, N, seed):
    """(xyz, normals), N x 3 FP64 each, in random order; everything from the seed."""
    g = _gen(seed)
    kw = dict(dtype=torch.float64, device="cuda")
    jit = (torch.rand(N, 2, generator=g, **kw) - 0.5) * 0.5
    if surface == "torus":  # R = 1, r = 1/3
        n_phi = max(3, round(math.sqrt(N / 3.0)))
        n_lam = -(-N // n_phi)
        i = torch.arange(N, **kw)
        phi = (torch.floor(i / n_lam) + 0.5 + jit[:, 0]) * (2 * math.pi / n_phi)
        lam = (i - torch.floor(i / n_lam) * n_lam + 0.5 + jit[:, 1]) * (2 * math.pi / n_lam)
        ring = 1.0 + torch.cos(phi) / 3.0
        x = torch.stack([ring * torch.cos(lam), ring * torch.sin(lam), torch.sin(phi) / 3.0], 1)
        nrm = torch.stack([torch.cos(phi) * torch.cos(lam), torch.cos(phi) * torch.sin(lam), torch.sin(phi)], 1)
    else:
        i = torch.arange(N, **kw)
        z = 1.0 - (2.0 * i + 1.0) / N
        lon = i * (math.pi * (3.0 - math.sqrt(5.0)))
        s = torch.sqrt(torch.clamp(1.0 - z * z, min=0.0))
        u = torch.stack([s * torch.cos(lon), s * torch.sin(lon), z], 1)
        h = math.sqrt(4 * math.pi / N)  # spacing: jitter a small part of it
        u = u + 0.4 * h * torch.cat([jit, jit.sum(1, keepdim=True)], 1)
        u = u / u.norm(dim=1, keepdim=True)
        q, _ = torch.linalg.qr(torch.randn(3, 3, generator=g, **kw).cpu())
        axes = torch.ones(3, **kw)
        if surface == "ellipsoid":
            axes = 0.7 + 0.8 * torch.rand(3, generator=g, **kw)
        x = u * axes
        nrm = x / (axes * axes)
        nrm = nrm / nrm.norm(dim=1, keepdim=True)
        q = q.cuda()
        x, nrm = x @ q, nrm @ q
    order = torch.randperm(N, generator=g, device="cuda")
    return x[order].contiguous(), nrm[order].contiguous()


def _offsets(xyz, idx, rows):
    """|x_j - x_i| for the stencil entries of some rows (N x n)."""
    return (xyz[idx[rows].long()] - xyz[rows].unsqueeze(1)).norm(dim=2)


def _cloud_laplacian(xyz, idx):
    """Gaussian point-cloud Laplacian on the stencils: weights (N x n, rows
    summing to zero) and a bound on its spectral radius."""
    N, n = idx.shape
    r2 = torch.empty(N, n, dtype=torch.float64, device="cuda")
    for a in range(0, N, 200000):
        rows = torch.arange(a, min(N, a + 200000), device="cuda")
        r2[a:a + 200000] = _offsets(xyz, idx, rows) ** 2
    s2 = 0.4 * r2[:, -1:].clone()
    w = torch.exp(-r2 / s2)
    w[:, 0] = 0.0
    w = w / w.sum(1, keepdim=True) * (4.0 / s2)
    w[:, 0] = -w[:, 1:].sum(1)
    return w.contiguous(), 2.0 * float((4.0 / s2).max())


def _opts(c):
    kw = dict(kernel=c["kernel"], degree=c["degree"], eps_mode=c["mode"])
    if c["mode"] == "fixed":  # eps grows with the resolution, as in the sphere sweep; wider stencils need more
        kw["eps"] = 2.0 * math.sqrt(c["N"] / 2500.0) * max(1.0, math.sqrt(c["n"] / 31.0)) * (1.5 if c["degree"] == 0 else 1.0)
    else:
        kw.update(kappa_target=c["kappa"], band=(c["kappa"] / 10, c["kappa"] * 10))
    return kw


def _network(n, seed):
    """Parameters of a trained network's size and scale (FP32 numpy)."""
    return rb.mlp_init(seed=seed % 1000003, n_in=2 * (n - 1), bias_out=-0.285)


def _state(c, N, seed):
    g = _gen(seed + 77)
    noise = torch.rand(2, N, generator=g, dtype=torch.float64, device="cuda") * 0.02 - 0.01
    if c["reaction"] == "none":
        return (1.0 + 10.0 * noise[:1]).contiguous()
    if c["reaction"] == "schnakenberg":  # steady state (a + b, b / (a + b)^2) plus noise
        return (noise + torch.tensor([[1.0], [0.9]], dtype=torch.float64, device="cuda")).contiguous()
    return (20.0 * noise).contiguous()


# ------------------------------------------------------- prepare and run ----

def prepare(case, seed):
    c, k = case, case["kind"]
    s = dict(case=c)
    if k == "weights":
        s["xyz"], s["nrm"] = _nodes(c["surface"], c["N"], seed)
        s["opts"] = _opts(c)
        if c["mode"] == "learned":
            # proposals as far from the root as a trained network's (0.037 in log eps)
            s["idx"], _ = rb.knn(s["xyz"], c["n"])
            kw = dict(s["opts"], eps_mode="bisect")
            label = rb.build_weights(s["xyz"], s["nrm"], c["n"], idx=s["idx"], **kw).eps
            z = torch.randn(c["N"], generator=_gen(seed + 5), dtype=torch.float64, device="cuda")
            s["eps"] = label * torch.exp(0.037 * z)
    elif k == "batch":
        sizes = [n for n in (31, 50, 70, 101) if n <= c["nmax"]]
        kinds = ("sphere", "torus", "ellipsoid")
        s["surfaces"] = []
        for i in range(c["surfaces"]):
            f = ((i * 7) % c["surfaces"] + 0.5) / c["surfaces"]  # N log-spaced over the range, in mixed order
            N = int(c["low"] * (c["high"] / c["low"]) ** f)
            x, nrm = _nodes(kinds[i % 3], N, seed * 131 + i)
            s["surfaces"].append((x, nrm, sizes[i % len(sizes)]))
    elif k == "dd":
        s["xyz"], s["nrm"] = _nodes("sphere", c["N"], seed)
        s["opts"] = dict(kernel=c["kernel"], degree=0, eps_mode=c["mode"], kappa_target=c["kappa"])
        s["eps"] = None
        if c["mode"] == "given":
            s["eps"] = torch.full((c["N"],), 1.2 * math.sqrt(c["N"] / 642.0), dtype=torch.float64, device="cuda")
    elif k == "knn":
        s["xyz"], _ = _nodes(c["surface"], c["N"], seed)
    elif k == "predict":
        s["xyz"], s["nrm"] = _nodes(c["surface"], c["N"], seed)
        s["idx"], _ = rb.knn(s["xyz"], c["n"])
        s["params"] = _network(c["n"], seed)
        s["net"] = rb.MLP(s["params"])
    elif k == "train":
        x, nrm = _nodes("torus", c["count"], seed)
        idx, _ = rb.knn(x, c["n"])
        s["feats"], _ = rb.mlp_features(x, nrm, idx)
        g = _gen(seed + 3)
        f = s["feats"].view(torch.bfloat16).to(torch.float32)
        s["target"] = (-0.285 + 0.05 * torch.tanh(f[:, :2 * (c["n"] - 1)].square().mean(1) * 4 - 1)
                       + 0.02 * torch.randn(c["count"], generator=g, device="cuda"))
        s["params"] = _network(c["n"], seed)
        s["seed"] = 1 + seed % 1000003
    else:
        x, _ = _nodes(c["surface"], c["N"], seed)
        idx, perm = rb.knn(x, c["n"])
        w, rho = _cloud_laplacian(x, idx)
        s.update(idx=idx, perm=perm, w=w)
        if k == "operator":
            s["u"] = torch.randn(c["N"], generator=_gen(seed + 9), dtype=torch.float64, device="cuda")
        else:
            D = {"none": (1.0,), "schnakenberg": (1.0, 10.0), "turing": (0.516 * 2.87e-4, 2.87e-4)}[c["reaction"]]
            params = {"none": (), "schnakenberg": SCHNAK, "turing": TURING_SPOTS}[c["reaction"]]
            dt = min(0.5 * 2.785 / (rho * max(D)), 0.01)
            s["op"] = rb.Operator(idx, w, perm)
            s["state"] = _state(c, c["N"], seed)
            s["kw"] = dict(D=D, reaction=c["reaction"], params=params)
            if k == "imex":
                s["dt"] = min(dt * c["dt_factor"], 0.01)
            else:
                s["dt"] = dt
                if c["forced"]:
                    s["kw"].update(forcing=0.1 * torch.roll(s["state"], 1, 1), t0=0.1, lam=-0.5)
    return s


def _weights(r):
    return dict(idx=r.idx, w=r.w, eps=r.eps, kappa=r.kappa, status=r.status, nevals=r.nevals)


def run(s):
    c, k = s["case"], s["case"]["kind"]
    if k == "weights":
        return _weights(rb.build_weights(s["xyz"], s["nrm"], c["n"], idx=s.get("idx"), eps_in=s.get("eps"),
                                         **s["opts"]))
    if k == "batch":
        out = rb.build_weights_batched(s["surfaces"], eps_mode="bisect", kappa_target=c["kappa"])
        return [[r.idx, r.w, r.eps] for r in out]
    if k == "dd":
        return _weights(rb.build_weights_dd(s["xyz"], s["nrm"], c["n"], eps_in=s["eps"], **s["opts"]))
    if k == "knn":
        return rb.knn(s["xyz"], c["n"])
    if k == "predict":
        return s["net"].predict_eps(s["xyz"], s["nrm"], s["idx"])
    if k == "train":
        net = rb.MLP(s["params"])
        losses = net.train(s["feats"], s["target"], steps=c["steps"], batch=c["batch"], lr=1e-3, seed=s["seed"])
        return dict(params=net.params, losses=losses)
    if k == "operator":
        op = rb.Operator(s["idx"], s["w"], s["perm"])
        v = s["u"]
        out = []
        for _ in range(c["applies"]):
            v = op.apply(v, c["prec"])
            out.append(v)
        return out
    if k == "rk4":
        return s["op"].step(s["state"], s["dt"], c["steps"], prec=c["prec"], **s["kw"])
    # the state alone: the iteration count and the last residual sit at the
    # rounding level of the solve and are not something a program computes with
    return s["op"].step_imex(s["state"], s["dt"], c["steps"], order=c["order"], maxit=3000, **s["kw"])[0]


# ------------------------------------------------------------------- work ----

def _evals(c, n, N):
    """kappa_2 evaluations of a bisection from the default bracket to 1e-4."""
    radius = math.sqrt(max(n, 8) * 4.0 / N)
    return 3 + max(0, math.ceil(math.log2(20.0 / radius / 1e-4)))


def _weights_work(N, n, degree, evals, stencils):
    m = n + {0: 1, 1: 4, 2: 10}[degree]
    flops = N * (evals * (4.0 / 3.0 * m ** 3 + 10.0 * n * n) + 30.0 * m * m + 40.0 * n * n)
    return N * (n * 4 + 48 + n * 8 + 24 + 8) + (N * n * 4 if not stencils else 0), flops


def work(case):
    c, k = case, case["kind"]
    if k == "weights":
        ev = {"fixed": 1, "learned": 1, "bisect": _evals(c, c["n"], c["N"])}[c["mode"]]
        b, f = _weights_work(c["N"], c["n"], c["degree"], ev, c["mode"] != "learned")
        return dict(bytes=b, flops=f)
    if k == "batch":
        sizes = [n for n in (31, 50, 70, 101) if n <= c["nmax"]]
        b = f = 0.0
        for i in range(c["surfaces"]):
            x = ((i * 7) % c["surfaces"] + 0.5) / c["surfaces"]
            N, n = int(c["low"] * (c["high"] / c["low"]) ** x), sizes[i % len(sizes)]
            bb, ff = _weights_work(N, n, 2, _evals(c, n, N), True)
            b, f = b + bb, f + ff
        return dict(bytes=b, flops=f)
    if k == "dd":  # one double-double multiply-add is about 20 FP64 operations
        ev = _evals(c, c["n"], c["N"]) if c["mode"] == "bisect" else 1
        b, f = _weights_work(c["N"], c["n"], 0, ev, True)
        return dict(bytes=b, flops=20.0 * f)
    if k == "knn":
        return dict(bytes=c["N"] * (24.0 + 4 * c["n"] + 4), flops=0.0)
    if k == "predict":
        return dict(bytes=c["N"] * (48.0 + 4 * c["n"] + 8), flops=c["N"] * 2.0 * 2 * 128 * 128)
    if k == "train":
        return dict(bytes=c["steps"] * (c["batch"] * 260.0 + 28 * 33153), flops=c["steps"] * c["batch"] * 6.0 * 2 * 128 * 128)
    N, n = c["N"], c["n"]
    if k == "operator":
        e = 8 if c["prec"] == "f64" else 4
        return dict(bytes=N * (12.0 * n + 4) + c["applies"] * (N * (n - 1) * (e + 2.0) + 16 * N),
                    flops=c["applies"] * 2.0 * N * n)
    S = 1 if c["reaction"] == "none" else 2
    if k == "rk4":
        e = 8 if c["prec"] == "f64" else 4
        per = 4 * N * ((n - 1) * (e + 2.0)) + N * S * e * 17
        return dict(bytes=c["steps"] * per, flops=c["steps"] * 8.0 * N * n * S)
    # implicit: at least one operator application per step, with the vectors of one BiCGSTAB iteration
    return dict(bytes=c["steps"] * (2 * N * (n - 1) * 10.0 + S * 16 * 8 * N), flops=c["steps"] * S * 4.0 * N * n)


# ------------------------------------------------------------------ exact ----

def _apply64(w, idx, u):
    """L u in plain FP64 (S x N)."""
    out = torch.empty_like(u)
    N = idx.shape[0]
    for a in range(0, N, 250000):
        j = idx[a:a + 250000].long()
        for s in range(u.shape[0]):
            out[s, a:a + 250000] = (w[a:a + 250000] * (u[s][j] - u[s, a:a + 250000].unsqueeze(1))).sum(1)
    return out


def _react64(y, reaction, p):
    if reaction == "none":
        return torch.zeros_like(y)
    u, v = y[0], y[1]
    if reaction == "schnakenberg":
        a, b, g = p
        return torch.stack([g * (a - u + u * u * v), g * (b - u * u * v)])
    al, be, ga, t1, t2 = p
    return torch.stack([al * u * (1 - t1 * v * v) + v * (1 - t2 * u),
                        be * v * (1 + al * t1 / be * u * v) + u * (ga + t2 * v)])


def _exact_fixed_weights(c, s):
    """First rows of sum_d G^d G^d by batched dense solves, one eps."""
    xyz, nrm, n, deg, eps = s["xyz"], s["nrm"], c["n"], c["degree"], s["opts"]["eps"]
    idx, _ = rb.knn(xyz, n)
    P = xyz[idx.long()]
    nu = nrm[idx.long()]
    nu = nu / nu.norm(dim=2, keepdim=True)
    d = P.unsqueeze(2) - P.unsqueeze(1)                       # x_i - x_j
    r2 = (d * d).sum(3)
    t = 1.0 + eps * eps * r2
    if c["kernel"] == "mq":
        phi, psi = t.sqrt(), eps * eps / t.sqrt()
    elif c["kernel"] == "imq":
        phi, psi = 1 / t.sqrt(), -eps * eps / (t.sqrt() * t)
    else:
        phi = torch.exp(-eps * eps * r2)
        psi = -2 * eps * eps * phi
    rho = r2[:, 0].max(1).values.sqrt()
    X = (P - P[:, :1]) / rho[:, None, None]
    one, zero = torch.ones_like(X[..., 0]), torch.zeros_like(X[..., 0])
    x, y, z = X[..., 0], X[..., 1], X[..., 2]
    M = {0: 1, 1: 4, 2: 10}[deg]
    U = torch.stack([one, x, y, z, x * x, y * y, z * z, x * y, x * z, y * z][:M], 2)
    G = torch.stack([
        torch.stack([zero, one, zero, zero, 2 * x, zero, zero, y, z, zero][:M], 2),
        torch.stack([zero, zero, one, zero, zero, 2 * y, zero, x, zero, z][:M], 2),
        torch.stack([zero, zero, zero, one, zero, zero, 2 * z, zero, x, y][:M], 2)], 2) / rho[:, None, None, None]
    out = []
    drop = 1 if deg == 2 else 0                               # on the sphere one quadratic combination vanishes
    u_, s_, vh = torch.linalg.svd(U, full_matrices=False)
    keep = M - drop
    C = vh.transpose(1, 2)[:, :, :keep] / s_[:, None, :keep]   # orthonormal border columns
    U, G = U @ C, torch.matmul(G, C.unsqueeze(1))
    m = n + keep
    A = torch.zeros(P.shape[0], m, m, dtype=torch.float64, device=P.device)
    A[:, :n, :n] = phi
    if deg == 0:
        U, G = torch.ones_like(U), torch.zeros_like(G)
    A[:, :n, n:] = U
    A[:, n:, :n] = U.transpose(1, 2)
    grad = torch.cat([psi.unsqueeze(2) * d.transpose(2, 3), G], 3)          # rows i, components, columns
    B = grad - nu.unsqueeze(3) * (nu.unsqueeze(3) * grad).sum(2, keepdim=True)
    g = torch.linalg.solve(A, B[:, 0].transpose(1, 2))                       # m x 3
    r = (B * g[:, :n].unsqueeze(3)).sum((1, 2))
    w = torch.linalg.solve(A, r.unsqueeze(2))[:, :n, 0]
    lam = torch.linalg.eigvalsh(A.cpu()).abs()
    return dict(idx=None, w=w, eps=torch.full_like(w[:, 0], eps), kappa=(lam.max(1).values / lam.min(1).values).cuda(),
                status=None, nevals=None)


def exact(case, seed):
    c, k = case, case["kind"]
    if k in ("batch", "dd", "knn", "train"):
        return None
    if k == "weights":
        if c["mode"] != "fixed" or c["N"] > 5000:
            return None
        return _exact_fixed_weights(c, prepare(case, seed))
    s = prepare(case, seed)
    if k == "predict":
        x, nrm, idx, n = s["xyz"], s["nrm"], s["idx"], c["n"]
        p = torch.as_tensor(s["params"]).cuda().double()
        W1, b1, W2, b2 = p[:16384].view(128, 128), p[16384:16512], p[16512:32896].view(128, 128), p[32896:33024]
        w3, b3 = p[33024:33152], p[33152]
        out = torch.empty(c["N"], dtype=torch.float64, device="cuda")
        for a in range(0, c["N"], 250000):
            d = x[idx[a:a + 250000].long()] - x[a:a + 250000].unsqueeze(1)
            rho = d.norm(dim=2).max(1).values
            nu = nrm[a:a + 250000] / nrm[a:a + 250000].norm(dim=1, keepdim=True)
            t1 = d[:, 1] - (d[:, 1] * nu).sum(1, keepdim=True) * nu
            t1 = t1 / t1.norm(dim=1, keepdim=True)
            t2 = torch.linalg.cross(nu, t1)
            f = torch.zeros(d.shape[0], 128, dtype=torch.float64, device="cuda")
            f[:, 0:2 * (n - 1):2] = (d[:, 1:] * t1.unsqueeze(1)).sum(2) / rho.unsqueeze(1)
            f[:, 1:2 * (n - 1):2] = (d[:, 1:] * t2.unsqueeze(1)).sum(2) / rho.unsqueeze(1)
            h = torch.relu(torch.relu(f @ W1.T + b1) @ W2.T + b2)
            out[a:a + 250000] = torch.exp(h @ w3 + b3) / rho
        return out
    w, idx = s["w"], s["idx"]
    if k == "operator":
        v, out = s["u"].unsqueeze(0), []
        for _ in range(c["applies"]):
            v = _apply64(w, idx, v)
            out.append(v[0])
        return out
    y, dt, kw = s["state"], s["dt"], s["kw"]
    D = torch.tensor(kw["D"], dtype=torch.float64, device="cuda").unsqueeze(1)
    if k == "rk4":
        F, t0, lam = kw.get("forcing"), kw.get("t0", 0.0), kw.get("lam", 0.0)

        def f(t, v):
            r = D * _apply64(w, idx, v) + _react64(v, c["reaction"], kw["params"])
            return r if F is None else r + math.exp(lam * t) * F
        for i in range(c["steps"]):
            t = t0 + i * dt
            k1 = f(t, y)
            k2 = f(t + dt / 2, y + dt / 2 * k1)
            k3 = f(t + dt / 2, y + dt / 2 * k2)
            k4 = f(t + dt, y + dt * k3)
            y = y + dt / 6 * (k1 + 2 * k2 + 2 * k3 + k4)
        return y
    if c["N"] > 12000:
        return None
    L = torch.zeros(c["N"], c["N"], dtype=torch.float64, device="cuda")
    L.scatter_(1, idx.long(), w)
    rows = {1: ([1.0, -1.0], [1.0]), 2: ([1.5, -2.0, 0.5], [2.0, -1.0]),
            3: ([11 / 6, -3.0, 1.5, -1 / 3], [3.0, -3.0, 1.0]),
            4: ([25 / 12, -4.0, 3.0, -4 / 3, 0.25], [4.0, -6.0, 4.0, -1.0])}
    hist, lus = [y], {}
    for _ in range(c["steps"]):
        q = min(c["order"], len(hist))
        a, b = rows[q]
        rhs = torch.zeros_like(y)
        for j in range(1, q + 1):
            rhs = rhs - a[j] * hist[-j] + dt * b[j - 1] * _react64(hist[-j], c["reaction"], kw["params"])
        new = torch.empty_like(y)
        for sp in range(y.shape[0]):
            if (q, sp) not in lus:
                eye = torch.eye(c["N"], dtype=torch.float64, device="cuda")
                lus[(q, sp)] = torch.linalg.lu_factor(a[0] * eye - dt * kw["D"][sp] * L)
            new[sp] = torch.linalg.lu_solve(*lus[(q, sp)], rhs[sp].unsqueeze(1))[:, 0]
        hist = (hist + [new])[-4:]
    return hist[-1]
