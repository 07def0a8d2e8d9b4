"""Host plans added beside the share plan, without a GPU: lists of whole pairs against the general list of the same pairs, and
the division of the single-group prefill form against the limits of its scratch memory."""
import numpy as np
import pytest

import paper_2510_08525_amd as rl


def whole_plan(rounds, n_wg):
    r = np.ascontiguousarray(rounds, dtype=np.int32)
    begin, first, count = np.zeros(n_wg + 1, np.int32), np.zeros(r.size, np.int32), np.zeros(r.size, np.int32)
    used = rl.load_library().rlkv_plan_whole_pairs(r.ctypes.data, r.size, n_wg, begin.ctypes.data, first.ctypes.data,
                                                   count.ctypes.data)
    return used, begin, first, count


@pytest.mark.parametrize("seed", range(6))
def test_whole_pairs_hold_the_units_of_the_general_list(seed):
    rng = np.random.default_rng(seed)
    for n_wg in (1, 7, 64, 256):
        rounds = rng.integers(0, 20, int(rng.integers(1, 2 * n_wg + 1)))
        keep = np.flatnonzero(rounds)[n_wg:]
        rounds[keep] = 0                                     # at most one pair per workgroup
        used, begin, first, count = whole_plan(rounds, n_wg)
        assert used == int((rounds > 0).sum())
        _, general, _, _ = rl.rlkv_plan_shares(rounds, n_wg)
        assert begin[0] == 0 and begin[-1] == general[-1] and (np.diff(begin) >= 0).all()
        at = 0
        for p, r in enumerate(rounds):                       # units of pair p: [at, at + r + 1) in either list
            if r == 0:
                assert count[p] == 0
                continue
            assert count[p] == 1 and begin[first[p]] == at and begin[first[p] + 1] == at + r + 1
            at += r + 1
        busy = np.flatnonzero(np.diff(begin))
        assert len(busy) == used
        if used > 1:                                         # spread over the grid
            assert busy[-1] - busy[0] >= (used - 1) * (n_wg // used)


def test_whole_pairs_refuse_more_pairs_than_workgroups():
    assert whole_plan([1, 1, 1], 2)[0] == -1 and whole_plan([1, 0, 1], 2)[0] == 2 and whole_plan([-1], 2)[0] == -1


def test_narrow_split_stays_within_grid_and_scratch():
    lib, rng, seen = rl.load_library(), np.random.default_rng(2), set()
    for _ in range(2000):
        G, B, n_full = int(rng.integers(1, 17)), int(rng.integers(1, 9)), int(rng.integers(0, 9))
        t = (rng.integers(0, 700, B) * (rng.random(B) < 0.8)).astype(np.int32)
        c = rng.integers(0, 30000, B).astype(np.int32)
        z = lib.rlkv_plan_narrow_split(256, G, n_full, B, t.ctypes.data, c.ctypes.data, 26)
        seen.add(z)
        assert 1 <= z <= 8
        if z > 1:
            per = 128 // G
            blocks = sum(-(-int(x) // per) for x in t)
            assert blocks * n_full * z <= 256 and -(-int(t.max()) // per) * int((t > 0).sum()) * n_full * z <= 1024
            assert min(int(x) // 32 for x, y in zip(c, t) if y > 0) // z >= 26
    assert seen == set(range(1, 9))
    one = np.ones(1, np.int32)
    assert lib.rlkv_plan_narrow_split(256, 17, 1, 1, one.ctypes.data, one.ctypes.data, 1) == -1
    for minimum in (0, -1):                                  # a share without tiles is none
        assert lib.rlkv_plan_narrow_split(256, 7, 1, 1, one.ctypes.data, one.ctypes.data, minimum) == -1
