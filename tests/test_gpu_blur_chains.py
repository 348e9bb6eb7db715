"""The blur in place over chains of neighbours (large three-tap lattices whose
value arrays outgrow the L2s): bitwise the same MVM and CG iterates as one
launch per direction step, in every blur order, with an even and an odd number
of directions, chains of 2 to 9 points, whole and broken vectors of columns,
and both chains together or one after the other."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _cuda(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


# d = 9: m = 302,649, one chain in 24 longer than 4 points; d = 16: m ~ 0.29M
CASES = [(305, 60000, 9, "mixture", (0.2, 0.6)), (306, 20000, 16, "uniform", (0.3, 3.0))]


@pytest.mark.parametrize("blur", ["symmetric", "forward", "reverse"])
@pytest.mark.parametrize("seed,n,d,kind,ell", CASES)
def test_blur_chains_match_single_steps(seed, n, d, kind, ell, blur):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2106_06695_amd as sgp
    w = workloads.small_case(seed, n, d, channels=64, kind=kind, ell_range=ell)
    lat = sgp.lattice_build(_cuda(w.X), w.lengthscales, blur=blur)
    assert lat.m >= 131072 and lat.m * 32 * 4 > 32 << 20  # 32 fp32 columns take the chains
    try:
        for C, fp64 in ((32, False), (33, False), (64, False), (18, True)):
            print(f"blur chains {blur} d={d} m={lat.m} C={C} fp64={fp64}", flush=True)
            V = _cuda(w.values[:, :C])

            def run():
                if fp64:
                    return sgp.cg_solve(lat, V, 0.1, 0.0, max_iter=3)[0].cpu().numpy()
                return sgp.lattice_mvm(lat, V).cpu().numpy()

            prev = sgp.blur_fuse_enable(False)
            try:
                ref = run()
            finally:
                sgp.blur_fuse_enable(prev)
            np.testing.assert_array_equal(run(), ref)
            seq = sgp.blur_seq_bytes(-1)
            try:
                np.testing.assert_array_equal(run(), ref)
            finally:
                sgp.blur_seq_bytes(seq)
    finally:
        lat.free()
