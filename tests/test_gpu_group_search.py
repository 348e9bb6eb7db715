"""The search for blur groups: what it keeps where sampled parts tell that a
group outgrows a tile, where no sample does and the counts tell, and where a new
cut holds a range that is known not to fit; and, where the groups are no fewer
passes than the fused pairs, which of the two each width of rows takes. Bitwise
the same MVM and CG iterates as one launch per step."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# d, n, lengthscale, order, groups, fp32 widths that take them, widths that take
# pairs. The groups follow from the lattice's neighbours (computed on the CPU).
# d = 5: parts of 264 points over two directions in one of three groups, which
# leaves 2, 1, 1, 2, a pass more than pairs; 78% of the points lie in parts that
# outgrow the first cut. d = 6, m = 61,289: 2, 1, 2, 2, as many passes as pairs;
# rows from 32 bytes on take groups when the lattice has 8 MiB of them. d = 8,
# m = 539,083: all of three groups of three outgrow a tile by up to ten points,
# 0.05% of the points; the next cut starts with the first of them again, which
# leaves 2, 1, 2, 2, 2. Order 2: 258 points in one group of three, 0.06%.
CASES = [
    (5, 204000, 0.2, 1, 4, (5, 16, 32), (1, 3, 8, 12)),
    (6, 60000, 0.6, 1, 4, (3, 32), (1, 4, 8, 16, 20)),
    (8, 200000, 0.65, 1, 5, (3, 8, 16), (1, 4)),
    (8, 200000, 0.9, 2, 4, (1, 8), ()),
]


@pytest.mark.parametrize("d,n,ell,order,groups,by_groups,by_pairs", CASES)
def test_group_search(d, n, ell, order, groups, by_groups, by_pairs):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2106_06695_amd as sgp
    X = np.random.default_rng(d + n).standard_normal((n, d)).astype(np.float32)
    lat = sgp.lattice_build(torch.from_numpy(X).cuda(), np.full(d, ell), order=order)
    try:
        for C in by_groups + by_pairs:
            print(f"group search d={d} n={n} order={order} m={lat.m} C={C}", flush=True)
            V = torch.from_numpy(np.random.default_rng(C).standard_normal((n, C)).astype(np.float32)).cuda()

            def run():
                with sgp.profile() as prof:
                    y = sgp.lattice_mvm(lat, V)
                    torch.cuda.synchronize()
                x = sgp.cg_solve(lat, V, 0.1, 0.0, max_iter=2)[0]
                return y, x, prof.results["blur"][0]

            y, x, launches = run()
            assert launches == (groups + 1 if C in by_groups else (d + 2) // 2)
            prev = sgp.blur_fuse_enable(False)
            try:
                yr, xr, _ = run()
            finally:
                sgp.blur_fuse_enable(prev)
            assert torch.equal(y, yr) and torch.equal(x, xr)
    finally:
        lat.free()
