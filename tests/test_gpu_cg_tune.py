"""Autotuned launch shapes of CG, with its vectors on the lattice and per point:
the iteration itself is timed, and no choice changes a bit."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _cuda(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


# seed, n, d: m = 4,979 (vectors on the lattice); m = 16,474 of 17,000 points (per point)
@pytest.mark.parametrize("seed,n,d,on_lattice", [(203, 30000, 9, True), (500, 17000, 11, False)])
@pytest.mark.parametrize("C", [1, 3, 16, 20])
def test_autotune_times_the_iteration(seed, n, d, on_lattice, C):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2106_06695_amd as sgp
    w = workloads.small_case(seed, n, d, channels=C, kind="mixture")
    lat = sgp.lattice_build(_cuda(w.X), w.lengthscales)
    print(f"autotune cg m={lat.m} C={C}", flush=True)
    assert (lat.m >= 4096 and 3 * lat.m <= 2 * lat.n) == on_lattice
    B = _cuda(w.values)

    def solve():
        return [np.asarray(t.cpu() if hasattr(t, "cpu") else t) for t in sgp.cg_solve(lat, B, 0.1, 0.0, max_iter=21)]

    sgp.autotune_reset()
    try:
        ref = solve()
        with sgp.profile() as prof:
            ch = sgp.autotune(lat, C, fp64=True, reps=3)
        runs = prof.results
        widths = {1: 1, 3: 3, 16: 3, 20: 3}[C]  # times one or many blocks per CU of the splat (and slice)
        if on_lattice:  # five iterations a candidate, and no slice
            assert runs["slice"][0] == 0 and runs["cg_dir"][0] == 2 * widths * 5
        else:
            assert runs["slice"][0] == 4 * widths * 5 == runs["cg_alpha"][0]
        assert ch["chunk"] in (1, 2, 4, 8, 16) and ch["ms_per_mvm"] > 0
        assert ch["splat_blocks_per_cu"] in (0, 1) and ch["slice_blocks_per_cu"] in ((0,) if on_lattice else (0, 1))
        for _ in range(2):
            for a, b in zip(solve(), ref):
                np.testing.assert_array_equal(a, b)
    finally:
        sgp.autotune_reset()
        lat.free()
