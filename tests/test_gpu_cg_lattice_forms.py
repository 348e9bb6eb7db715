"""CG with its vectors on the lattice in every form that a lattice has: one-chain
blurs, the wider stencil, the Matern kernel, tiles of fewer than 256 points,
chains of graph replays. Iterates against the oracle's point-space CG.

Bar, derived before the first run: both sides run the same recurrence in fp64
with the same fp32 weights; after 6 iterations the iterates differ by the fp32
rounding of x and of the weights (6e-8 each, the latter amplified by the
iteration's polynomial, below 1e-6 in point space at this count): 1e-5."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

BLURS = ("symmetric", "forward", "reverse")

# seed, n, d, kind, lengthscale range, kernel, order, blur, columns, solve_rows
CASES = [
    (203, 30000, 9, "mixture", (0.5, 2.0), "rbf", 1, "forward", 3, 0),          # m = 4,979
    (203, 30000, 9, "mixture", (0.5, 2.0), "rbf", 1, "reverse", 16, 29000),
    (212, 40000, 6, "mixture", (0.3, 0.8), "rbf", 2, "symmetric", 4, 0),        # 6,671
    (212, 40000, 6, "mixture", (0.3, 0.8), "rbf", 2, "forward", 1, 39001),
    (211, 30000, 7, "mixture", (0.5, 1.4), "matern32", 1, "symmetric", 5, 0),   # 5,562
    (210, 30000, 7, "mixture", (0.5, 1.4), "matern32", 2, "reverse", 8, 0),     # 5,930
    (213, 40000, 16, "mixture", (1.2, 3.0), "rbf", 1, "symmetric", 8, 0),       # 5,752; tiles of 240
    (214, 30011, 20, "mixture", (2.0, 5.0), "rbf", 1, "forward", 2, 30000),     # 19,868; tiles of 192
]


def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2106_06695_amd as sgp
    return sgp, lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


@pytest.mark.parametrize("seed,n,d,kind,ell,kernel,order,blur,C,rows", CASES)
def test_lattice_cg_forms(seed, n, d, kind, ell, kernel, order, blur, C, rows):
    import oracle
    sgp, cuda = _gpu()
    w = workloads.small_case(seed, n, d, channels=C, kind=kind, ell_range=ell)
    lat = sgp.lattice_build(cuda(w.X), w.lengthscales, order=order, kernel=kernel, blur=blur, outputscale=1.7,
                            solve_rows=rows)
    print(f"lattice cg {kernel} order={order} {blur} d={d} m={lat.m} C={C} rows={rows}", flush=True)
    assert lat.m >= 4096 and 3 * lat.m <= 2 * n
    x, iters, rel = sgp.cg_solve(lat, cuda(w.values), 0.1, 0.0, max_iter=6)
    olat = oracle.Lattice(w.X, w.lengthscales, r=order, kernel=int(kernel == "matern32"))
    xo, _, relo, _ = olat.cg(w.values.astype(np.float64), 0.1, 0.0, max_iter=6, mode=BLURS.index(blur),
                             outputscale=1.7, **({"rows": rows} if rows else {}))
    x = x.cpu().numpy().astype(np.float64)
    assert np.all(iters == 6)
    if rows:
        assert np.all(x[rows:] == 0.0)
    err = np.linalg.norm(x - xo, axis=0) / np.linalg.norm(xo, axis=0)
    assert err.max() <= 1e-5, err
    assert np.all(np.abs(rel - relo) <= 1e-5 * np.asarray(relo)), (rel, relo)
    lat.free()


@pytest.mark.parametrize("tol,max_iter", [(0.0, 45), (1e-5, 300)])
def test_lattice_cg_graph_replay(tol, max_iter):
    """Replayed blocks of iterations give the bits of single launches, over
    several solves with other work on the lattice in between."""
    sgp, cuda = _gpu()
    w = workloads.small_case(203, 30000, 9, channels=5, kind="mixture")
    lat = sgp.lattice_build(cuda(w.X), w.lengthscales)
    assert lat.m >= 4096 and 3 * lat.m <= 2 * lat.n
    print(f"lattice cg graph m={lat.m} tol={tol}", flush=True)
    B = cuda(w.values)

    def solve():
        x, it, rel = sgp.cg_solve(lat, B, 0.05, tol, max_iter=max_iter)
        return [x.cpu().numpy(), np.asarray(it), np.asarray(rel)]

    prev = sgp.cg_graph_enable(False)
    try:
        ref = solve()
        sgp.cg_graph_enable(True)
        for _ in range(3):
            sgp.lattice_mvm(lat, B)
            for a, b in zip(solve(), ref):
                np.testing.assert_array_equal(a, b)
    finally:
        sgp.cg_graph_enable(prev)
        lat.free()
    assert tol == 0.0 or np.all(ref[1] > 13)  # blocks were replayed
