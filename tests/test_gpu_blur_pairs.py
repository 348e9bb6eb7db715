"""The blur's fused pairs of steps on lattices without groups of directions and
too large for the one-block-per-column path, and its chains one after the other,
there and with groups: bitwise the same MVM and CG iterates as one launch per
step, in every blur order, with an even and an odd number of directions. Launch
counts show that the intended kernels ran."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# n, d, lengthscale: m = 5,897 and 6,130 (d < 5 keeps no groups), 6,008 and
# 5,897 (below 8,192 points); half of the neighbours are present or more
CASES = [(9000, 3, 0.2), (30000, 4, 0.5), (9000, 6, 1.0), (5000, 7, 1.2)]


def _lattice(n, d, ell, **kw):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2106_06695_amd as sgp
    X = np.random.default_rng(n + d).standard_normal((n, d)).astype(np.float32)
    return sgp, sgp.lattice_build(torch.from_numpy(X).cuda(), np.full(d, ell), **kw)


def _run(sgp, lat, C):
    """An MVM's and two CG iterations' results, and the launches of the MVM's blur."""
    import torch
    V = torch.from_numpy(np.random.default_rng(C).standard_normal((lat.n, C)).astype(np.float32)).cuda()
    with sgp.profile() as prof:
        y = sgp.lattice_mvm(lat, V)
        torch.cuda.synchronize()
    x, _, rel = sgp.cg_solve(lat, V, 0.1, 0.0, max_iter=2)
    return [y.cpu().numpy(), x.cpu().numpy(), np.asarray(rel)], prof.results["blur"][0]


@pytest.mark.parametrize("blur", ["symmetric", "forward", "reverse"])
@pytest.mark.parametrize("n,d,ell", CASES)
def test_pairs_match_single_steps(n, d, ell, blur):
    sgp, lat = _lattice(n, d, ell, blur=blur)
    D = d + 1
    try:
        assert lat.m > 2048 and (d < 5 or lat.m < 8192)
        for C in (1, 3, 8, 16, 20):
            print(f"blur pairs {blur} d={d} m={lat.m} C={C}", flush=True)
            prev = sgp.blur_fuse_enable(False)
            try:
                ref, steps = _run(sgp, lat, C)
            finally:
                sgp.blur_fuse_enable(prev)
            assert steps == D
            # both chains of a launch together; all pairs of one, then of the other
            for limit, launches in ((-1, (D + 1) // 2), (0, 2 * ((D - 1) // 2) + 1 if blur == "symmetric" else (D + 1) // 2)):
                prev = sgp.blur_seq_bytes(limit)
                try:
                    got, count = _run(sgp, lat, C)
                finally:
                    sgp.blur_seq_bytes(prev)
                assert count == launches
                for a, b in zip(got, ref):
                    np.testing.assert_array_equal(a, b)
    finally:
        lat.free()


@pytest.mark.parametrize("order", [1, 2])
def test_groups_chains_in_sequence(order):
    """The threshold of the sequential chains holds for groups of directions."""
    sgp, lat = _lattice(20000, 9, 1.0, order=order)
    try:
        for C in (3, 16):
            print(f"blur groups in sequence order={order} m={lat.m} C={C}", flush=True)
            prev = sgp.blur_seq_bytes(-1)
            try:
                ref, together = _run(sgp, lat, C)
                sgp.blur_seq_bytes(0)
                got, apart = _run(sgp, lat, C)
            finally:
                sgp.blur_seq_bytes(prev)
            assert 3 <= together - 1 < 10 and apart == 2 * (together - 1)
            assert _run(sgp, lat, C)[1] == together  # the default: far from 768 MiB
            for a, b in zip(got, ref):
                np.testing.assert_array_equal(a, b)
    finally:
        lat.free()
