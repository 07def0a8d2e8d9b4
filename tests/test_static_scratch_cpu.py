"""Where the partials of an allocation-free decode call stand in the library's static buffer, without a GPU: every region inside the
buffer and apart from the others, up to the last call that is not refused."""
import numpy as np
import pytest

import paper_2510_08525_amd as rl

ROWS, D = 16384, 128


def layout(n_wg, n_pairs, group, gated):
    at = np.full(4, -7, np.int64)
    end = rl.load_library().rlkv_plan_static_scratch(n_wg, n_pairs, group, gated, at.ctypes.data)
    return end, at.tolist()


@pytest.mark.parametrize("gated", [0, 1], ids=["plain", "blending"])
@pytest.mark.parametrize("n_wg,n_pairs,group", [
    (256, 1, 1), (256, 8, 4), (256, 256, 16), (256, 257, 16), (256, 258, 16), (256, 300, 16), (256, 767, 16), (256, 768, 16),
    (256, 769, 16), (256, 16128, 1), (256, 16129, 1), (2048, 2048, 4), (2048, 2049, 4), (2048, 6144, 2)])
def test_regions(n_wg, n_pairs, group, gated):
    rows = (n_wg + n_pairs) * group
    end, (m, l, set_o, set_ml) = layout(n_wg, n_pairs, group, gated)
    assert (end < 0) == (rows * (2 if gated else 1) > ROWS)          # what is refused stays what it was
    if end < 0:
        return
    assert end <= ROWS * (D + 2)
    regions = []
    for s in range(2 if gated else 1):
        regions += [(s * set_o, rows * D), (m + s * set_ml, rows), (l + s * set_ml, rows)]
    regions.sort()
    assert regions[0][0] == 0 and sum(regions[-1]) <= end
    assert all(a + n <= b for (a, n), (b, _) in zip(regions, regions[1:]))
    # a second set, where nobody asked for one, stays inside as well
    assert max(set_o + rows * D, m + set_ml + rows, l + set_ml + rows) <= end


def test_invalid_arguments():
    assert rl.load_library().rlkv_plan_static_scratch(256, 8, 4, 0, None) == -1
    for bad in [(0, 8, 4), (256, 0, 4), (256, 8, 0), (256, 8, 17)]:
        assert layout(*bad, 0)[0] == -1
