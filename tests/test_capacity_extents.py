"""Row capacities (longest and total local rows) against the boxes counted axis by axis, up to hundreds of distinct extents."""
import numpy as np
import pytest

from paper_2602_04361_amd import sparvar as sv


def extents(n, n_prev, b, radius, dil, below):
    e, ep = min(b, n), min(b, n_prev)
    T, Tp = -(-n // e), -(-n_prev // ep)
    a = np.arange(T)
    lo = np.maximum(a * e * n_prev // n // ep - dil, 0)
    hi = np.minimum((-(-np.minimum(a * e + e, n) * n_prev // n) - 1) // ep + dil, Tp - 1)
    win = np.minimum(a + radius, T - 1) - np.maximum(a - radius, 0) + 1
    return (hi - lo + 1 if below else np.zeros(T, int)), win


@pytest.mark.parametrize("h,w,b,ns,radius,dil", [
    ([1, 4, 16, 40], [1, 4, 16, 40], 8, 2, 1, 0), ([2, 5, 9], [3, 4, 7], 2, 0, 2, 1), ([3, 7], [3, 7], 2, 1, 1, 0),
    ([4, 500, 600], [1, 2, 2], 1, 1, 300, 2), ([4, 2, 2], [1, 450, 700], 1, 0, 350, 0), ([1, 33, 47], [1, 20, 31], 4, 1, 3, 2)])
def test_local_row_capacities(h, w, b, ns, radius, dil):
    g = sv.Geometry(h, w, b, ns)
    k = len(h)
    info = [g.scale_info(l) for l in range(1, k + 1)]
    n_sink = info[ns - 1]["n_blocks_le"] if ns else 0
    fr, wr = extents(h[-1], h[-2], b, radius, dil, k - 1 > ns)
    fc, wc = extents(w[-1], w[-2], b, radius, dil, k - 1 > ns)
    rows = n_sink + np.outer(fr, fc) + np.outer(wr, wc)
    assert sv.sparvar_local_blocks_capacity(g, k, radius, dil) == rows.sum()
    per_row = rows.max() + 2
    assert sv.sparvar_map_index_capacity(g, k - 1, k, 3, 5, 2, radius, dil) == 15 * rows.size * (per_row + 1)
