"""Operator build at the edges of its slices and halos: rows past a slice, slot
counts around the groups of four, halos at and beyond the staged limit, many
surfaces; applied against a plain dense/sparse sum."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _random(N, n, spread, seed):
    """Stencils of n distinct rows, centre first, within `spread` rows of the centre (wrapping)."""
    rng = np.random.default_rng(seed)
    off = np.stack([1 + rng.choice(spread, n - 1, replace=False) for _ in range(N)])
    idx = np.concatenate([np.arange(N)[:, None], (np.arange(N)[:, None] + off) % N], axis=1).astype(np.int32)
    w = rng.standard_normal((N, n))
    w[:, 0] = -w[:, 1:].sum(1)
    return idx, w, rng.permutation(N).astype(np.int32)


@pytest.mark.parametrize("N,n,spread", [(2, 2, 1), (64, 5, 40), (65, 6, 60), (127, 7, 100), (130, 50, 120),
                                        (300, 128, 290), (640, 9, 575), (641, 64, 640), (1300, 64, 1200),
                                        (2000, 33, 576), (2000, 33, 577), (2000, 127, 700)])
def test_build_and_apply(lib, N, n, spread):
    idx, w, perm = _random(N, n, spread, N + n)
    u = np.random.default_rng(1).standard_normal(N)
    ref = (w * u[idx]).sum(1)
    scale = (np.abs(w) * np.abs(u[idx])).sum(1)
    c = lambda a: torch.as_tensor(a).cuda()
    for p in (None, perm):
        op = lib.Operator(c(idx), c(w), c(p) if p is not None else None)
        got = op.apply(c(u), "f64").cpu().numpy()
        assert np.all(np.abs(got - ref) <= 2 * n * 2.0 ** -53 * scale)
        # FP32 weights, values and sums of differences: n terms of |w| (|u_j| + |u_i|)
        g32 = op.apply(c(u), "f32").cpu().numpy()
        s32 = (np.abs(w[:, 1:]) * (np.abs(u[idx[:, 1:]]) + np.abs(u)[:, None])).sum(1)
        assert np.all(np.abs(g32 - ref) <= (n + 4) * 2.0 ** -24 * s32)
        # the halos: distinct rows of every slice, in internal order
        inv = np.empty(N, dtype=np.int64)
        inv[p if p is not None else np.arange(N)] = np.arange(N)
        rows = idx[p if p is not None else np.arange(N)][:, 1:]
        sizes = [len(np.unique(inv[rows[a:a + 64]])) for a in range(0, N, 64)]
        ns, hs, hr, he = op.stats()
        keep = [(h, min(64, N - 64 * q)) for q, h in enumerate(sizes) if h <= 640]
        assert (ns, hs, hr, he) == (len(sizes), len(keep), sum(r for _, r in keep), sum(h for h, _ in keep))


def test_many_surfaces_bitwise(lib):
    parts, us = [], []
    for t, (N, n) in enumerate([(65, 9), (64, 33), (1000, 50), (3, 3)]):
        idx, w, perm = _random(N, n, min(N - 1, 200), t)
        parts.append(tuple(torch.as_tensor(a).cuda() for a in (idx, w, perm)))
        us.append(torch.randn(N, dtype=torch.float64, device="cuda"))
    out = lib.Operator.batched(parts).apply(torch.cat(us))
    one = torch.cat([lib.Operator(*p).apply(u) for p, u in zip(parts, us)])
    assert torch.equal(out, one)


def test_bad_entries_still_refused(lib):
    idx, w, perm = _random(200, 9, 150, 3)
    c = lambda a: torch.as_tensor(a).cuda()
    for where, val in (((5, 3), 200), ((199, 8), -1), ((7, 0), 8)):
        bad = idx.copy()
        bad[where] = val
        with pytest.raises(lib.RbffdError):
            lib.Operator(c(bad), c(w), c(perm))
    twice = perm.copy()
    twice[0] = twice[1]
    with pytest.raises(lib.RbffdError):
        lib.Operator(c(idx), c(w), c(twice))
    lib.Operator(c(idx), c(w), c(perm))
