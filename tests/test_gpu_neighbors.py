"""The neighbour table where a thread of the look-up takes four directions
(2^20 table rows and more) and just below: equal to the oracle's."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _cells(cells):
    """One point in each of `cells` simplices that share no vertex (d = 3): 16
    table rows each."""
    X = np.zeros((cells, 3), np.float32)
    X[:, 0] = 50.0 * (np.arange(cells) - cells // 2)
    X[:, 1:] = 0.3
    return X


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("case", ["2^20 - 16", "2^20", "d = 16", "d = 9"])
def test_neighbours_match_oracle(case, order):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2106_06695_amd as sgp
    if case.startswith("2^20"):
        X = _cells((1 << 16) - (1 if "-" in case else 0))
    else:
        d = int(case.split()[-1])
        X = np.random.default_rng(d).standard_normal((15000, d)).astype(np.float32)
    ell = np.ones(X.shape[1])
    print(f"neighbours {case} order {order}", flush=True)
    keys, idx, w, nbr = oracle.Lattice(X, ell, r=order).export()
    lat = sgp.lattice_build(torch.from_numpy(X).cuda(), ell, order=order)
    try:
        ex = sgp.lattice_export(lat)
    finally:
        lat.free()
    np.testing.assert_array_equal(ex[0], keys)
    np.testing.assert_array_equal(ex[3], nbr)
