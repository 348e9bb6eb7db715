"""The server's bound on a build's memory counts blur groups exactly where a
lattice can have them."""
import pytest

from paper_2106_06695_amd.serve import build_peak_bytes


@pytest.mark.parametrize("N,d,order,groups", [
    (200000, 3, 1, False), (200000, 4, 2, False),   # fewer than five dimensions
    (1365, 5, 1, False), (1366, 5, 1, True),        # 8,190 and 8,196 vertices
    (30000, 20, 3, False), (30000, 20, 2, True), (30000, 20, 1, True),
])
def test_groups_counted_where_they_can_be(N, d, order, groups):
    D, L = d + 1, N * (d + 1)
    without = (136 + 4 * d + 8 * order * D) * L + 8 * N * d + (64 << 20)
    # a record of 4 + 8 order bytes per row and group; at most a quarter of a
    # tile's rows are empty and 2 (d+1) / 3 groups kept
    extra = (4 + 8 * order) * 1.25 * (2 * D // 3) * L
    got = build_peak_bytes(N, d, order)
    assert got == without if not groups else without + extra <= got
