"""The splat's gather with lattice points requested in the batch and ahead of it
(one lane a range from 2^18 partial rows, more lanes from 3 * 2^19): a column
alone, in a narrow and in a wide call gives the same bits, on either side of both
lines, and the products meet the oracle's (fp32 sums of some ten terms per step:
1e-5 of the result's norm)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# n, d, lengthscale: about 0.14M, 0.66M and 2.3M partial rows
CASES = [(200000, 3, 0.1), (200000, 6, 0.45), (1300000, 6, 0.45)]


@pytest.mark.parametrize("n,d,ell", CASES)
def test_gather_widths_agree(n, d, ell):
    import oracle
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2106_06695_amd as sgp
    X = np.random.default_rng(n + d).standard_normal((n, d)).astype(np.float32)
    lat = sgp.lattice_build(torch.from_numpy(X).cuda(), np.full(d, ell))
    V = np.random.default_rng(1).standard_normal((n, 16)).astype(np.float32)
    Vc = torch.from_numpy(V).cuda()
    base = sgp.lattice_info(lat)["device_bytes"]
    wide = sgp.lattice_mvm(lat, Vc)
    rows = (sgp.lattice_info(lat)["device_bytes"] - base) / 64 - 4 * lat.m
    print(f"gather n={n} d={d} m={lat.m} rows at most {rows:.0f}", flush=True)
    for c, C in ((3, 1), (8, 2), (4, 3), (12, 4), (0, 8)):
        part = sgp.lattice_mvm(lat, Vc[:, c:c + C].contiguous())
        assert torch.equal(part, wide[:, c:c + C]), C
    x = sgp.cg_solve(lat, Vc, 0.1, 0.0, max_iter=2)[0]
    for c, C in ((3, 1), (8, 2), (4, 3), (0, 8)):
        assert torch.equal(sgp.cg_solve(lat, Vc[:, c:c + C].contiguous(), 0.1, 0.0, max_iter=2)[0], x[:, c:c + C]), C
    if n <= 200000:
        ref = oracle.Lattice(X, np.full(d, ell)).mvm(V[:, :2].astype(np.float64))
        err = np.linalg.norm(wide[:, :2].cpu().numpy() - ref) / np.linalg.norm(ref)
        assert err <= 1e-5, err
    lat.free()
