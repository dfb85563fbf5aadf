"""m <= 32 runs two stencils per wavefront.  Every kind of stencil next to every
other -- border columns kept or dropped (another m), an index out of range, a
zero normal, coincident nodes, proposals that are kept, missed or not numbers --
gives the bits that it gives next to itself."""
import numpy as np
import pytest
import torch

from oracle.knn import knn as oracle_knn
from synth import fibonacci_sphere, jittered_torus

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,kw", [("fixed", dict(eps=2.0)), ("bisect", dict(kappa_target=1e9)),
                                     ("bisect", dict(kappa_target=1e9, band_stop=True, band=(1e8, 1e10))),
                                     ("bisect", dict(kappa_target=1e30, max_expand=2)), ("given", {}),
                                     ("learned", dict(kappa_target=1e9, band=(1e8, 1e10)))])
@pytest.mark.parametrize("kernel", ["mq", "imq", "ga"])
@pytest.mark.parametrize("n,degree", [(22, 2), (13, 2), (28, 1), (31, 0), (3, 0)])
def test_any_neighbour_in_the_wavefront(lib, n, degree, kernel, mode, kw):
    S, sn = fibonacci_sphere(60)
    T, tn = jittered_torus(5, 9)
    X, nrm = np.concatenate([S, T + np.array([5.0, 0.0, 0.0])]), np.concatenate([sn, tn])
    N = len(X)
    idx = np.concatenate([oracle_knn(S, n), oracle_knn(T, n) + len(S)]).astype(np.int32)
    kinds = idx[[0, 7, 62, 70, 80, 33, 90, 17]].copy()
    kinds[4, n // 2] = N + 5      # out of range
    kinds[5, 1] = kinds[5, 0]     # coincident
    nrm[kinds[6, 1]] = 0.0        # no normal
    eps = np.array([1.5, np.nan, 0.4, 3.0, -1.0, 0.9, np.inf, 2.2])
    a, b = np.divmod(np.arange(64), 8)
    rows = np.stack([a, b], 1).ravel()           # every pair of kinds
    c = lambda x: torch.as_tensor(x).cuda()
    e = lambda r: c(np.resize(eps[r], N)) if mode in ("given", "learned") else None

    def run(r):
        r = np.resize(r, N) if len(r) < N else r[:N - N % 2]
        full = np.concatenate([r, r[:N - len(r)]])
        return lib.build_weights(c(X), c(nrm), n, idx=c(kinds[full]), eps_in=e(full), kernel=kernel, degree=degree,
                                 eps_mode=mode, **kw)

    own = run(np.repeat(np.arange(8), 2))        # each next to itself
    for first in range(0, len(rows), N - N % 2):
        part = rows[first:first + N - N % 2]
        got = run(part)
        pick = torch.as_tensor(2 * part).cuda()
        for f in ("w", "eps", "kappa", "status", "nevals"):
            x, y = getattr(got, f)[:len(part)], getattr(own, f)[pick]
            assert torch.equal(torch.nan_to_num(x.double(), 7.0, 8.0, 9.0), torch.nan_to_num(y.double(), 7.0, 8.0, 9.0)), f
