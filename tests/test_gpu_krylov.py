"""The fused BiCGSTAB kernels of the implicit steps where they can go wrong:
part-filled slices, more block partials than a kernel sums by itself, an
operator too large for the kernels that form p and s as they gather, slices
whose neighbours do not fit the staged list, and a workspace that an earlier
call with another layout has left behind.

One first-order step without reaction solves (I - dt L) u1 = u0.  The solver
stops at a relative residual of tol by its own recursion; the residual that
NumPy computes in FP64 may differ from it by the rounding of the iterations
(some 1e-14 each), so the bar is 2 tol at tol = 1e-11.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def graph_operator(lib, N, n, far, seed):
    """L = weighted graph Laplacian (rows sum to zero) on near or random neighbours."""
    rng = np.random.default_rng(seed)
    idx = np.empty((N, n), np.int32)
    idx[:, 0] = np.arange(N)
    steps = rng.choice(np.arange(1, N), n - 1, replace=False) if far else np.arange(1, n)
    idx[:, 1:] = (np.arange(N)[:, None] + steps * (rng.integers(0, 2, N)[:, None] * 2 - 1)) % N
    if far:
        idx[:, 1:] = (idx[:, 1:] * 7919 + rng.integers(0, N, N)[:, None]) % N
        idx[:, 1:] += (idx[:, 1:] == idx[:, :1])
        idx[:, 1:] %= N
    w = np.empty((N, n))
    w[:, 1:] = rng.uniform(0.5, 2.0, (N, n - 1))
    w[:, 0] = -w[:, 1:].sum(1)
    op = lib.Operator(torch.as_tensor(idx).cuda(), torch.as_tensor(w).cuda(),
                      perm=torch.arange(N, dtype=torch.int32, device="cuda"))
    return idx, w, op


@pytest.mark.parametrize("N,n,far", [(65, 11, False), (257, 12, False), (2049, 19, False), (20000, 64, True),
                                     (131072, 11, False), (131073, 11, False), (140001, 14, False),
                                     (640001, 66, False), (840001, 66, False)])
def test_first_order_step_solves_its_system(lib, N, n, far):
    idx, w, op = graph_operator(lib, N, n, far, N)
    u0 = np.random.default_rng(1).standard_normal(N)
    dt, tol = 0.05, 1e-11
    got, its, res = op.step_imex(torch.as_tensor(u0).cuda(), dt, 1, order=1, tol=tol, maxit=100)
    u1 = got.cpu().numpy().reshape(-1)
    r = u0 - (u1 - dt * np.einsum("ij,ij->i", w, u1[idx]))
    true = np.linalg.norm(r) / np.linalg.norm(u0)
    print(f"[krylov] N={N} n={n} far={far}: {its} iterations, residual {res:.1e}, true {true:.1e}", flush=True)
    assert its > 2 and res <= tol and true <= 2 * tol


def test_workspace_of_another_layout_leaves_nothing_behind(lib):
    """A fourth-order two-species call lays its vectors out differently and
    fills padding rows of its reaction terms; the same bits must come out of
    the next, smaller call as out of a new operator."""
    u0 = torch.as_tensor(np.random.default_rng(2).standard_normal((2, 1000))).cuda()
    _, _, fresh = graph_operator(lib, 1000, 15, False, 5)
    want, _, _ = fresh.step_imex(u0[:1], 0.02, 4, order=2)
    _, _, op = graph_operator(lib, 1000, 15, False, 5)
    op.step_imex(0.1 * u0, 1e-3, 6, order=4, D=(1.0, 10.0), reaction="schnakenberg", params=(0.1, 0.9, 5.0))
    got, _, _ = op.step_imex(u0[:1], 0.02, 4, order=2)
    assert torch.equal(got, want)


@pytest.mark.parametrize("N,n", [(1000, 3), (1000, 30), (4097, 66), (840001, 50), (840001, 66)])
def test_apply_in_every_slot_mode(lib, N, n):
    """L u where the slots stay in the caches, where they stream, and where
    they stream without reading ahead (FP32 above 256 MB and n = 64, FP64 above
    512 MB).  Per row, FP64 and FP32 rounding of n terms: (n + 2) u sum |w| (|u_j| + |u_i|)."""
    idx, w, op = graph_operator(lib, N, n, False, N + n)
    u = np.random.default_rng(4).standard_normal(N)
    du = u[idx] - u[:, None]
    want = np.einsum("ij,ij->i", w, du)
    scale = np.einsum("ij,ij->i", np.abs(w), np.abs(u[idx]) + np.abs(u)[:, None])
    for prec, eps in (("f64", 2.0 ** -53), ("f32", 2.0 ** -24)):
        got = op.apply(torch.as_tensor(u).cuda(), prec=prec).cpu().numpy().reshape(-1)
        worst = np.max(np.abs(got - want) / scale)
        print(f"[apply] N={N} n={n} {prec}: {worst:.1e}", flush=True)
        assert worst <= (n + 2) * eps
