"""The blur by groups of directions: bitwise the same MVM and CG iterates as
separate launches, with groups of four, three, two and one direction (parts
that outgrow a tile divide their group), a part of exactly a tile's 255 points,
a lattice that keeps no groups, whole and broken vectors of columns, every blur
order, both chains together or one after the other, and stencils of order 2."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (d, n, data, lengthscale, groups). The groups follow from the largest parts
# (computed on the CPU from the lattice's neighbours): d = 5, n = 4,000: 357
# over three directions, 57 over two; d = 6: 2,003 over four, 355 over three,
# 62 over two; d = 7: 615 over four, 158 over three; d = 9: 285 in the first
# group of four alone; d = 11 and 20: 184 and 5 over four; "flat": 281 over two
# in the first group, 10 over three in the other; d = 5, n = 200,000: 255 over
# two. d = 5, n = 400,000 at a shorter lengthscale has more than that
# throughout, and room for four groups only: none (three launches a blur).
CASES = [
    (5, 4000, "normal", 0.35, 3),
    (6, 60000, "normal", 0.6, 4),
    (7, 20000, "normal", 0.8, 3),
    (9, 20000, "normal", 1.0, 4),
    (11, 17000, "normal", 1.0, 3),
    (20, 3000, "normal", 1.0, 6),
    (5, 100000, "flat", 1.0, 4),
    (5, 200000, "normal", 0.2, 3),
    (5, 400000, "normal", 0.18, 0),
]


def _points(d, n, data):
    X = np.random.default_rng(d + n).standard_normal((n, d))
    if data == "flat":
        X *= 0.1
        X[:, :2] = np.random.default_rng(1).uniform(-60, 60, (n, 2))
    return X.astype(np.float32)


def _run(sgp, lat, X, C, fp64):
    import torch
    V = torch.from_numpy(np.random.default_rng(C).standard_normal((len(X), C)).astype(np.float32)).cuda()

    def run():
        if fp64:
            return sgp.cg_solve(lat, V, 0.1, 0.0, max_iter=2)[0].cpu().numpy()
        return sgp.lattice_mvm(lat, V).cpu().numpy()

    prev = sgp.blur_fuse_enable(False)
    try:
        ref = run()
    finally:
        sgp.blur_fuse_enable(prev)
    np.testing.assert_array_equal(run(), ref)


@pytest.mark.parametrize("d,n,data,ell,groups", CASES)
def test_groups_match_single_steps(d, n, data, ell, groups):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2106_06695_amd as sgp
    X = _points(d, n, data)
    lat = sgp.lattice_build(torch.from_numpy(X).cuda(), np.full(d, ell))
    try:
        print(f"blur groups d={d} n={n} {data} m={lat.m}", flush=True)
        V = torch.ones((n, 3), device="cuda")
        sgp.lattice_mvm(lat, V)
        with sgp.profile() as prof:
            sgp.lattice_mvm(lat, V)
            torch.cuda.synchronize()
        assert prof.results["blur"][0] == (groups + 1 if groups else (d + 2) // 2)
        for C, fp64 in ((1, False), (3, False), (33, False), (1, True), (7, True), (16, True)):
            _run(sgp, lat, X, C, fp64)
    finally:
        lat.free()


@pytest.mark.parametrize("blur", ["forward", "reverse"])
def test_one_chain(blur):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2106_06695_amd as sgp
    X = _points(9, 20000, "normal")
    lat = sgp.lattice_build(torch.from_numpy(X).cuda(), np.full(9, 1.0), blur=blur)
    try:
        for C, fp64 in ((5, False), (16, False), (4, True)):
            print(f"blur groups {blur} C={C} fp64={fp64}", flush=True)
            _run(sgp, lat, X, C, fp64)
    finally:
        lat.free()


def test_chains_one_after_the_other():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2106_06695_amd as sgp
    X = _points(5, 200000, "normal")
    lat = sgp.lattice_build(torch.from_numpy(X).cuda(), np.full(5, 0.2))
    try:
        C = 96
        assert 2 * lat.m * C * 4 > 384 << 20  # bytes of the two chains' arrays
        print(f"blur groups in sequence m={lat.m} C={C}", flush=True)
        _run(sgp, lat, X, C, False)
    finally:
        lat.free()


@pytest.mark.parametrize("d,n,ell,blur", [(5, 60000, 0.6, "symmetric"), (9, 60000, 1.0, "forward"),
                                          (11, 17000, 1.0, "symmetric"), (20, 3000, 1.0, "reverse")])
def test_order_2(d, n, ell, blur):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2106_06695_amd as sgp
    X = _points(d, n, "normal")
    lat = sgp.lattice_build(torch.from_numpy(X).cuda(), np.full(d, ell), order=2, blur=blur)
    try:
        print(f"blur groups, order 2, d={d} n={n} m={lat.m}", flush=True)
        V = torch.ones((n, 3), device="cuda")
        sgp.lattice_mvm(lat, V)
        with sgp.profile() as prof:
            sgp.lattice_mvm(lat, V)
            torch.cuda.synchronize()
        assert prof.results["blur"][0] <= (d + 1) // 2 + 1  # groups, not a launch per direction
        for C, fp64 in ((1, False), (5, False), (16, False), (1, True), (7, True), (16, True)):
            _run(sgp, lat, X, C, fp64)
    finally:
        lat.free()
