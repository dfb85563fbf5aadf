"""The neighbour search where its branches meet, against the oracle's exact
answer (distance, then index): stencils around the sizes at which another
kernel is chosen, lattices full of equal distances, coincident nodes, clusters
with more candidates than are held in registers, and strays that need shells
far from their cell.
"""
import numpy as np
import pytest
import torch

from oracle.knn import knn as oracle_knn

pytestmark = pytest.mark.gpu


def cloud(kind, N, seed=1):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((N, 3))
    X /= np.linalg.norm(X, axis=1)[:, None]
    if kind == "lattice":
        m = int(np.ceil(np.sqrt(N)))
        g = np.stack(np.meshgrid(np.arange(m), np.arange(m), [0.0]), -1).reshape(-1, 3)[:N].astype(float)
        return g[rng.permutation(N)]
    if kind == "duplicates":
        return X[rng.integers(0, N // 3, N)]
    if kind == "clusters":
        c = rng.integers(0, 5, N)
        X = X[:5][c] + 1e-3 * rng.standard_normal((N, 3))
        X[: N // 50] = 3.0 * rng.standard_normal((N // 50, 3))
        return X
    if kind == "strays":
        X[: N // 20] *= 1.0 + rng.random((N // 20, 1))
        return X
    if kind == "offset":
        return 1e-3 * X + np.array([1e3, -2e3, 5.0])
    return X


@pytest.mark.parametrize("n", [1, 2, 3, 31, 55, 56, 57, 64, 65, 66, 84, 85, 127, 128])
@pytest.mark.parametrize("kind", ["sphere", "lattice", "duplicates", "clusters", "strays", "offset"])
def test_neighbours_are_exact(lib, kind, n):
    X = cloud(kind, 1500)
    idx, _ = lib.knn(torch.as_tensor(X).cuda(), n)
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), oracle_knn(X, n))


@pytest.mark.parametrize("N", [1, 2, 9, 64, 65, 130])
def test_every_node_of_a_small_cloud(lib, N):
    """n = N: nothing may be left out, whatever the shells hold."""
    X = cloud("sphere", N)
    n = min(N, 128)
    idx, _ = lib.knn(torch.as_tensor(X).cuda(), n)
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), oracle_knn(X, n))


@pytest.mark.parametrize("N,n,nans", [(12, 11, (3,)), (40, 11, (0, 39)), (70, 31, (5, 6, 7)), (200, 31, range(0, 200, 3)),
                                      (64, 64, (1,)), (1500, 50, (0, 700, 1499)), (130, 128, range(60))])
def test_nan_coordinates_are_nobodys_neighbours(lib, N, n, nans):
    """Whole blocks of candidates at or below the search's limit, some of them
    at no distance: the others' neighbours are exact, a node without
    coordinates has none, and where too few nodes are left the row ends in -1."""
    X = cloud("sphere", N)
    nans = np.array(list(nans))
    for t, i in enumerate(nans):
        X[i, t % 3] = np.nan
    good = np.setdiff1d(np.arange(N), nans)
    idx, _ = lib.knn(torch.as_tensor(X).cuda(), n)
    torch.cuda.synchronize()
    idx = idx.cpu().numpy()
    assert np.array_equal(idx[:, 0], np.arange(N))
    assert (idx[nans, 1:] == -1).all()
    k = min(n, len(good))
    want = good[oracle_knn(X[good], k)]
    if k == n:
        assert np.array_equal(idx[good], want)
    else:
        assert np.array_equal(np.sort(idx[good][:, 1:k]), np.sort(want[:, 1:])) and (idx[good][:, k:] == -1).all()
