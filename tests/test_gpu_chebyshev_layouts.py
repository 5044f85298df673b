"""GPU tests of the Chebyshev recurrence on every layout of its product: widths
of one strip (40), of several 64-wide strips (128), without a lane shuffle
(80, 112), of eight doubles a lane (272), and rows of more than 256 entries,
which a workgroup of its own sums.  The start block comes by columns in the
first application and as a dense block in the second of the squared method, and
each step writes over the block before the last.  Against the float64 oracle at
the tolerances of the two precisions."""
import numpy as np
import pytest

from oracle import cheb
from paper_2301_06384_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)
gk = pytest.importorskip("paper_2301_06384_amd.gk")


def with_hubs(n, seed):
    """A sparse weighted random graph, two of its nodes joined to 300 and 700 others."""
    rng = np.random.default_rng(seed)
    ij = np.concatenate([rng.integers(0, n, (4 * n, 2)),
                         np.stack([np.full(300, 5), rng.choice(n, 300, replace=False)], 1),
                         np.stack([np.full(700, n - 2), rng.choice(n, 700, replace=False)], 1)])
    ij = np.sort(ij[ij[:, 0] != ij[:, 1]], 1)
    key = np.unique(ij[:, 0].astype(np.int64) * n + ij[:, 1])
    return I.laplacian_from_edges(n, key // n, key % n, rng.uniform(0.5, 1.5, key.size))


_G = {}


def graph(kind):
    if kind not in _G:
        L = with_hubs(1501, 3) if kind == "hubs" else I.rgg_knn(1403, 8, seed=1403)
        _G[kind] = (L, gk.Graph.from_laplacian(L, flags=gk.REORDER))
    return _G[kind]


@pytest.mark.parametrize("s", [3, 40, 70, 100, 128, 260])
@pytest.mark.parametrize("kind", ["rgg", "hubs"])
def test_layouts(kind, s):
    L, g = graph(kind)
    assert (L.max_degree() > 256) == (kind == "hubs")
    W = I.samples(L.n, s, s)
    if kind == "hubs":   # a hub among the samples, and a node next to it
        W = np.unique(np.append(W[2:], [5, L.n - 2]))
    phi = dict(kind="diffusion", t=0.02 if kind == "hubs" else 0.6)
    for variant, f in (("cheb", cheb.cheb), ("cheb2", cheb.cheb2)):
        for m in (7, 12):
            ref = f(L.to_scipy(), W, phi, m)
            for prec, tol in (("fp64", 1e-10), ("mixed", 1e-5)):
                P, K, _ = gk.krylov_kernel_columns(g, W, phi, m, variant, prec)
                e = (np.linalg.norm(P - ref["P"]) / np.linalg.norm(ref["P"]),
                     np.linalg.norm(K - ref["Kww_gathered"]) / np.linalg.norm(ref["Kww_gathered"]))
                assert max(e) < tol, (variant, m, prec, e)
