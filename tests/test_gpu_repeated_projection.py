"""GPU tests of the float64 steps that repeat their projection against the basis.

Copies of 4 + 6 nodes joined by one edge of weight 2e-9, a sample among the
four: the fourth step leaves a block of norm 2e-9, on which the coefficients of
the first projection (rounding of the product, 1e-16) are above the 1e-8 that a
single projection is kept at, and far above the deflation threshold (1e-12 of
the spectral bound).  Everything the columns hold on the six nodes comes from
the steps behind that one, and after ten steps the columns are exact, so both
halves are compared with the dense phi(L).  Tolerances: near half, 1e-12 for
entries of order one; far half, rounding of the small block 2.2e-16 * 6 / 2e-9 =
7e-7 a step, over ten steps 1e-5 of its own norm, and on top the rounding of
the coefficients phi(H_m) F_1, whose eigenvectors are good to ten steps of
2.2e-16 of the whole column: 2e-15."""
import numpy as np
import pytest

from oracle import krylov
from paper_2301_06384_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)
gk = pytest.importorskip("paper_2301_06384_amd.gk")

WEAK = 2e-9
NEAR = [(0, 1), (1, 2), (2, 3), (0, 2)]
FAR = [(4, 5), (5, 6), (6, 7), (7, 8), (8, 9), (4, 7), (5, 9)]


def copies(count):
    rng = np.random.default_rng(1)
    e = np.array(NEAR + FAR + [(3, 4)])
    w = np.append(rng.uniform(0.5, 1.5, len(NEAR) + len(FAR)), WEAK)
    off = 10 * np.arange(count)[:, None]
    return I.laplacian_from_edges(10 * count, (e[:, 0] + off).ravel(), (e[:, 1] + off).ravel(), np.tile(w, count))


# gbl: the same node of every copy, so that the blocks of all copies run out
# together; widths of the narrow and wide float64 products and of the dots
@pytest.mark.parametrize("variant,s", [("sbl", 1), ("sbl", 9), ("sbl", 48), ("sbl", 260), ("gbl", 1), ("gbl", 9),
                                       ("gbl", 48), ("gbl", 260), ("cbl", 1), ("cbl", 9), ("cbl", 20), ("cbl", 40),
                                       ("cbl", 64), ("cbl", 70), ("cbl", 130)])
@pytest.mark.parametrize("m", [10, 12])
def test_repeated_projection(variant, s, m):
    L = copies(s + 3)
    g = gk.Graph.from_laplacian(L)
    try:
        W = 10 * np.arange(s) + (0 if variant == "gbl" else np.arange(s) % 4)
        w, V = np.linalg.eigh(L.to_scipy().toarray()[:10, :10])   # a copy
        E = (V * np.exp(-0.3 * w)) @ V.T
        P, K, _ = gk.krylov_kernel_columns(g, W, dict(kind="diffusion", t=0.3), m, variant, "fp64")
        ref = np.zeros_like(P)
        for j, i in enumerate(W):
            ref[i // 10 * 10:i // 10 * 10 + 10, j] = E[:, i % 10]
        far = np.arange(L.n) % 10 >= 4
        assert np.linalg.norm(P - ref) < 1e-12 * np.linalg.norm(ref)
        assert np.linalg.norm((P - ref)[far]) < 1e-5 * np.linalg.norm(ref[far]) + 2e-15 * np.linalg.norm(ref)
        assert np.linalg.norm(K - ref[W]) < 1e-12 * np.linalg.norm(ref[W])
    finally:
        g.release()


# the sampled block of gbl and sbl beside their columns
@pytest.mark.parametrize("s", [1, 30, 48, 260])
@pytest.mark.parametrize("variant", ["gbl", "sbl"])
def test_sampled_block(variant, s):
    L = I.rgg_knn(1403, 8, seed=1403)
    g = gk.Graph.from_laplacian(L, flags=gk.REORDER)
    try:
        W, phi = I.samples(L.n, s, s), dict(kind="diffusion", t=0.6)
        for m in (2, 7):
            ref = getattr(krylov, variant)(L.to_scipy(), W, phi, m)["Kww_gathered"]
            for prec, tol in (("fp64", 1e-10), ("mixed", 1e-5)):
                _, K, _ = gk.krylov_kernel_columns(g, W, phi, m, variant, prec)
                assert np.linalg.norm(K - ref) < tol * np.linalg.norm(ref), (m, prec)
    finally:
        g.release()


# elsewhere a step projects once, early and late in the call: the work of the
# launches that were not skipped is that of one projection a step
@pytest.mark.parametrize("m", [12, 30, 45])
def test_one_projection_a_step(m):
    n, s = 12_000, 64
    L = I.rgg_knn(n, 8, seed=7)
    g = gk.Graph.from_laplacian(L, flags=gk.REORDER)
    try:
        W, phi = I.samples(n, s, 2), dict(kind="diffusion", t=0.6)
        gk.krylov_kernel_columns(g, W, phi, m, "cbl", "fp64", flags=gk.TIMING)
        work = {r["name"]: r["alg_flops"] for r in gk.kernel_timings()}
        # the first Gram pass of step k reads k + 1 blocks, and its X^T X one triangle
        assert work["tsgemm"] == sum(2.0 * n * s * s * (k + 1) for k in range(1, m))
        assert work["gram"] == sum(2.0 * n * s * s * (k + 1) + n * s * (s + 1.0) for k in range(1, m))
    finally:
        g.release()
