"""Weights at the edges of the register tilings (m = n + border at and around
32, 48 and 64, multiples of 8 and 16, the smallest systems), for odd numbers
of stencils, against the oracle."""
import numpy as np
import pytest

from oracle.knn import knn as oracle_knn
from oracle.shape import stencil_kappa
from oracle.weights import build_weights as oracle_weights
from synth import fibonacci_sphere, jittered_torus

U = 2.0 ** -53


def _check(rb, X, nrm, n, degree, kernel, rows):
    import torch

    Xd, Nd = torch.as_tensor(X).cuda(), torch.as_tensor(nrm).cuda()
    idx = oracle_knn(X, n)
    eps = 2.5 * np.sqrt(len(X) / 2500.0) * np.sqrt(n / 31.0)
    r = rb.build_weights(Xd, Nd, n, kernel=kernel, degree=degree, eps_mode="fixed", eps=float(eps))
    assert np.array_equal(r.idx.cpu().numpy(), idx)
    assert (r.status.cpu().numpy() == 0).all() and (r.nevals.cpu().numpy() == 1).all()
    w, kap = r.w.cpu().numpy(), r.kappa.cpu().numpy()
    wo = oracle_weights(X, nrm, idx, np.full(len(X), eps), rows=rows, kernel=kernel, degree=degree)
    for t, i in enumerate(rows):
        k = stencil_kappa(X[idx[i]], eps, kernel=kernel, degree=degree)
        # 20 kappa u, and the search's own end: log(1e30) / 33^7 / 2 on log min |lambda|
        assert abs(kap[i] - k) <= max(1e-9, 20 * k * U) * k, ("kappa", n, degree, i, kap[i], k)
        err = np.linalg.norm(w[i] - wo[t]) / np.linalg.norm(wo[t])
        assert err <= max(1e-9, 0.5 * k * U), ("weights", n, degree, i, err, k)
    return r


@pytest.mark.gpu
@pytest.mark.parametrize("n,degree", [(6, 0), (7, 0), (8, 0), (15, 0), (16, 0), (30, 0), (31, 0), (32, 0), (47, 0),
                                      (48, 0), (63, 0), (64, 0), (12, 1), (28, 1), (29, 1), (44, 1), (45, 1),
                                      (22, 2), (23, 2), (30, 2), (38, 2), (39, 2), (54, 2), (55, 2), (63, 2),
                                      (70, 2), (86, 2), (87, 2), (118, 2), (127, 0)])
def test_tiling_edges(lib, n, degree):
    X, nrm = jittered_torus(13, 39)  # 507 stencils: odd
    _check(lib, X, nrm, n, degree, "mq", [0, 1, 255, 506])


@pytest.mark.gpu
def test_two_stencils_per_wave_match_single_rows(lib):
    """n = 22, degree 2 (m <= 32): a sphere stencil next to torus stencils
    drops a border column, so the two halves of a wavefront differ in m."""
    import torch

    S, sn = fibonacci_sphere(301)
    T, tn = jittered_torus(11, 27)
    X, nrm = np.concatenate([S, T + np.array([5.0, 0.0, 0.0])]), np.concatenate([sn, tn])
    idx = np.concatenate([oracle_knn(S, 22), oracle_knn(T, 22) + len(S)]).astype(np.int32)
    # alternate rows of the two surfaces: neighbours in a wavefront
    mix = np.empty(2 * len(T), dtype=np.int64)
    mix[0::2], mix[1::2] = np.arange(len(T)), len(S) + np.arange(len(T))
    N = len(X)
    full = np.concatenate([mix, np.setdiff1d(np.arange(N), mix)])
    Xd, Nd = torch.as_tensor(X).cuda(), torch.as_tensor(nrm).cuda()
    kw = dict(degree=2, eps_mode="bisect", kappa_target=1e9)
    a = lib.build_weights(Xd, Nd, 22, idx=torch.as_tensor(idx).cuda(), **kw)
    b = lib.build_weights(Xd, Nd, 22, idx=torch.as_tensor(idx[full]).cuda(), **kw)
    p = torch.as_tensor(full).cuda()
    for f in ("w", "eps", "kappa", "status", "nevals"):
        assert torch.equal(getattr(a, f)[p], getattr(b, f)), f
    assert (a.status == 0).all()


@pytest.mark.gpu
@pytest.mark.parametrize("kernel", ["mq", "imq"])
@pytest.mark.parametrize("n", [2, 3, 9, 16, 17, 30, 31, 32, 33, 46, 47])
def test_double_double_tiling_edges(lib, n, kernel):
    """m = n + 1 around the rows of a lane (multiples of 4 and 16) and at both
    sides of 32; well conditioned, so the FP64 oracle holds to its own error."""
    import torch

    X, nrm = jittered_torus(9, 27)
    idx = oracle_knn(X, n)
    eps = 6.0
    r = lib.build_weights_dd(torch.as_tensor(X).cuda(), torch.as_tensor(nrm).cuda(), n, kernel=kernel, degree=0,
                             eps_mode="fixed", eps=eps)
    assert (r.status.cpu().numpy() == 0).all()
    rows = [0, 121, 242]
    wo = oracle_weights(X, nrm, idx, np.full(len(X), eps), rows=rows, kernel=kernel, degree=0)
    w, kap = r.w.cpu().numpy(), r.kappa.cpu().numpy()
    for t, i in enumerate(rows):
        k = stencil_kappa(X[idx[i]], eps, kernel=kernel, degree=0)
        assert abs(kap[i] - k) <= max(1e-12, 20 * k * U) * k, (i, kap[i], k)
        err = np.linalg.norm(w[i] - wo[t]) / np.linalg.norm(wo[t])
        assert err <= max(1e-12, 0.5 * k * U), (i, err, k)
