"""CG with its vectors on the lattice (taken where 4096 <= m <= 2n/3): iterates
against the oracle's point-space CG, at the edges of its tiles and chunks.

Bars, derived before the first run: both sides run the same recurrence in fp64
with the same fp32 weights, so after 6 iterations the iterates differ by the
fp32 rounding of x (6e-8 relative) and of the weights (the oracle's are fp64;
6e-8 per weight, amplified by at most the iteration's polynomial, observed
below 1e-6 in point space at this count); 1e-5 leaves a factor of ten. To a
tolerance, x must satisfy the oracle's fp64 operator to 1.05 tol.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sgp():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2106_06695_amd as sgp
    sgp._lib.load()
    return sgp


def _cuda(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def _on_lattice(lat):
    return lat.m >= 4096 and 3 * lat.m <= 2 * lat.n


# seed, n (odd tile remainders), d, kind, lengthscale range, columns, solve_rows (0: all)
CASES = [
    (201, 20011, 7, "mixture", (0.3, 0.8), 1, 0),
    (201, 20011, 7, "mixture", (0.3, 0.8), 2, 19000),
    (203, 30000, 9, "mixture", (0.5, 2.0), 3, 0),
    (203, 30000, 9, "mixture", (0.5, 2.0), 4, 29999),
    (205, 16001, 11, "mixture", (0.7, 2.0), 5, 0),
    (205, 16001, 11, "mixture", (0.7, 2.0), 8, 15001),
    (206, 40000, 3, "uniform", (0.05, 0.06), 16, 0),   # tiles with more runs than one staged chunk
    (206, 40000, 3, "uniform", (0.05, 0.06), 20, 39000),  # two chunks, the second partly filled
]


@pytest.mark.parametrize("seed,n,d,kind,ell,C,rows", CASES)
def test_lattice_cg_iterates(sgp, seed, n, d, kind, ell, C, rows):
    import oracle
    print(f"lattice cg seed={seed} n={n} d={d} C={C} rows={rows}", flush=True)
    w = workloads.small_case(seed, n, d, channels=C, kind=kind, ell_range=ell)
    lat = sgp.lattice_build(_cuda(w.X), w.lengthscales, solve_rows=rows, outputscale=1.3)
    assert _on_lattice(lat)
    olat = oracle.Lattice(w.X, w.lengthscales)
    x, iters, rel = sgp.cg_solve(lat, _cuda(w.values), 0.1, 0.0, max_iter=6)
    xo, _, relo, _ = olat.cg(w.values.astype(np.float64), 0.1, 0.0, max_iter=6, outputscale=1.3,
                             **({"rows": rows} if rows else {}))
    x = x.cpu().numpy().astype(np.float64)
    assert np.all(iters == 6)
    if rows:
        assert np.all(x[rows:] == 0.0)
    err = np.linalg.norm(x - xo, axis=0) / np.linalg.norm(xo, axis=0)
    assert err.max() <= 1e-5, err
    assert np.all(np.abs(rel - relo) <= 1e-5 * np.asarray(relo))
    # a rhs and an x that are not 16-byte aligned give the same bits
    import torch
    flat = torch.empty(n * C + 1, device="cuda")
    b1 = flat[1:].view(n, C)
    b1.copy_(_cuda(w.values))
    x1 = torch.empty(n * C + 1, device="cuda")[1:].view(n, C)
    sgp.cg_solve(lat, b1, 0.1, 0.0, max_iter=6, x=x1)
    np.testing.assert_array_equal(x1.cpu().numpy(), x.astype(np.float32))
    # a column alone gives the same bits as in the batch
    c = C - 1
    xc, _, _ = sgp.cg_solve(lat, _cuda(w.values[:, c:]), 0.1, 0.0, max_iter=6)
    np.testing.assert_array_equal(xc.cpu().numpy()[:, 0], x.astype(np.float32)[:, c])
    lat.free()


def test_lattice_cg_tolerance_and_zero_and_nan_columns(sgp):
    """Columns stop on their own; a zero column takes no iterations and a NaN
    one leaves the others alone; the answer meets a tight tolerance."""
    import oracle
    w = workloads.small_case(203, 30000, 9, channels=3, kind="mixture", ell_range=(0.5, 2.0))
    V = w.values.copy()
    V[:, 1] = 0.0
    lat = sgp.lattice_build(_cuda(w.X), w.lengthscales)
    assert _on_lattice(lat)
    x, iters, rel = sgp.cg_solve(lat, _cuda(V), 1.0, 1e-6, max_iter=2000)
    x = x.cpu().numpy()
    assert iters[1] == 0 and np.all(x[:, 1] == 0.0) and rel[0] <= 1e-6 and rel[2] <= 1e-6
    olat = oracle.Lattice(w.X, w.lengthscales)
    b = V[:, [0, 2]].astype(np.float64)
    xg = x[:, [0, 2]].astype(np.float64)
    res = b - (olat.mvm(xg) + xg)
    # x is fp32: its rounding alone leaves a residual of 6e-8 |A| |x| / |b|
    floor = 6e-8 * np.linalg.norm(olat.mvm(np.abs(xg)) + np.abs(xg), axis=0) / np.linalg.norm(b, axis=0)
    assert np.all(np.linalg.norm(res, axis=0) / np.linalg.norm(b, axis=0) <= 1.05e-6 + floor)
    V[5, 1] = np.nan
    xn, itn, _ = sgp.cg_solve(lat, _cuda(V), 1.0, 1e-6, max_iter=2000)
    np.testing.assert_array_equal(xn.cpu().numpy()[:, [0, 2]], x[:, [0, 2]])
    assert itn[0] == iters[0] and itn[2] == iters[2]
    lat.free()
