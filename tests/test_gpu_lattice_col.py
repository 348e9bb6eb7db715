"""The lattice part of an MVM as one block per column (three-tap lattices of up
to 2,048 points): bitwise the same MVM and CG iterates as separate launches, in
every blur order, at the smallest lattice, one row a thread and one more, the
largest that takes the path and one more point, with lattice points whose
partial rows span many gather ranges."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _points(cells, copies, d):
    """`copies` points at each of `cells` places that share no lattice point
    ((d + 1) vertices each): m = cells * (d + 1)."""
    X = np.zeros((cells, d))
    X[:, 0] = 50.0 * (np.arange(cells) - cells // 2)
    X[:, 1:] = 0.3
    return np.repeat(X, copies, axis=0), cells * (d + 1)


# (cells, copies, d, random points): m = 4, 1024, 1026, 2048, 2050; then
# neighbours that are present: d = 3, n = 40,000 (m of some 200: hundreds of
# tiles on each point) and d = 6, n = 8,000 (m of some 1,500)
CASES = [(1, 1, 3), (1, 20000, 3), (256, 3, 3), (171, 90, 5), (512, 40, 3), (410, 3, 4), (0, 40000, 3), (0, 8000, 6)]


@pytest.mark.parametrize("blur", ["symmetric", "forward", "reverse"])
@pytest.mark.parametrize("cells,copies,d", CASES)
def test_one_block_per_column_matches_separate_launches(cells, copies, d, blur):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2106_06695_amd as sgp
    if cells:
        X, m = _points(cells, copies, d)
    else:
        X, m = np.random.default_rng(7).standard_normal((copies, d)) / (1.6 if d > 3 else 1.0), None
    lat = sgp.lattice_build(torch.from_numpy(X.astype(np.float32)).cuda(), np.ones(d), blur=blur)
    try:
        assert m is None or lat.m == m
        assert m is not None or 100 < lat.m <= 2048
        for C in (1, 3, 16, 40):
            print(f"column blocks {blur} d={d} n={len(X)} m={lat.m} C={C}", flush=True)
            V = torch.from_numpy(np.random.default_rng(C).standard_normal((len(X), C)).astype(np.float32)).cuda()

            def run():
                x, iters, rel = sgp.cg_solve(lat, V[:, :16].contiguous(), 0.1, 1e-6, max_iter=6)
                return [t.cpu().numpy() if hasattr(t, "cpu") else np.asarray(t)
                        for t in (sgp.lattice_mvm(lat, V), x, iters, rel)]

            prev = sgp.blur_fuse_enable(False)
            try:
                ref = run()
            finally:
                sgp.blur_fuse_enable(prev)
            for got, want in zip(run(), ref):
                np.testing.assert_array_equal(got, want)
    finally:
        lat.free()
