"""The search for blur groups: what it keeps where sampled parts tell that a
group outgrows a tile, where no sample does and the counts tell, where a new cut
holds a range that is known not to fit, and where the groups would be more
passes than the fused pairs. Bitwise the same MVM as one launch per step."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# d, n, lengthscale, order, groups (from the lattice's neighbours, on the CPU).
# d = 5: parts of 264 and 271 points over two directions in one of three groups,
# which leaves 2, 1, 1, 2 and 2, 2, 1, 1: no groups, as there are three pairs;
# with 78% of the points in the parts that outgrow the first cut. d = 8: all of
# three groups of three outgrow a tile by up to ten points, 0.05% of the points;
# the next cut starts with the first of them again. Order 2: 258 points in one
# group of three, 0.06%, against a launch per direction.
CASES = [(5, 204000, 0.2, 1, 0), (5, 210300, 0.2, 1, 0), (8, 200000, 0.65, 1, 5), (8, 200000, 0.9, 2, 4)]


@pytest.mark.parametrize("d,n,ell,order,groups", CASES)
def test_group_search(d, n, ell, order, groups):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2106_06695_amd as sgp
    X = np.random.default_rng(d + n).standard_normal((n, d)).astype(np.float32)
    lat = sgp.lattice_build(torch.from_numpy(X).cuda(), np.full(d, ell), order=order)
    try:
        for C in (1, 8):
            print(f"group search d={d} n={n} order={order} m={lat.m} C={C}", flush=True)
            V = torch.from_numpy(np.random.default_rng(C).standard_normal((n, C)).astype(np.float32)).cuda()
            with sgp.profile() as prof:
                got = sgp.lattice_mvm(lat, V)
                torch.cuda.synchronize()
            assert prof.results["blur"][0] == (groups + 1 if groups else (d + 2) // 2)
            prev = sgp.blur_fuse_enable(False)
            try:
                ref = sgp.lattice_mvm(lat, V)
            finally:
                sgp.blur_fuse_enable(prev)
            assert torch.equal(got, ref)
    finally:
        lat.free()
