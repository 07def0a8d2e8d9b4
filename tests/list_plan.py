"""The work list a decode call plans, recomputed from the library's planning functions (no GPU): its kind, the workgroups it uses, the
most of them that share a pair, and whether their partials are merged inside the attention launch."""
import numpy as np

import paper_2510_08525_amd as rl

TILE, ROUND, SLACK, MERGE_FEW = 32, 4, 32, 32


def plan(dtype, kernel, group, mask, S, R, lengths, cap, gated=False, step=False, n_wg=256):
    """mask: per KV head, 1 = full.  Returns (whole pairs, workgroups used, most partials of a pair, merged inside)."""
    lib = rl.load_library()
    H, B = len(mask), len(lengths)
    n = np.asarray(lengths, np.int32)
    if lib.rlkv_plan_list_kind(kernel, dtype, group, int(gated), int(step), n_wg, H, int(sum(mask)), S + R, B, n.ctypes.data, None):
        return True, 0, 1, False
    limit = [(cap + TILE - 1) // TILE * TILE if m else S + R for m in mask]

    def rounds(tiles):
        return np.asarray([-(-min(int(x) + SLACK, l) // (TILE * tiles)) for x in n for l in limit], np.int32)

    half = rounds(ROUND // 2)
    if dtype == rl.RLKV_F32 and half.sum() <= n_wg and half.max() <= MERGE_FEW:
        used, most = int(half.sum()), int(half.max())                # one half round per workgroup
    else:
        r = rounds(ROUND)
        begin, first, count = np.zeros(n_wg + 1, np.int32), np.zeros(B * H, np.int32), np.zeros(B * H, np.int32)
        used = lib.rlkv_plan_shares(r.ctypes.data, B * H, n_wg, begin.ctypes.data, first.ctypes.data, count.ctypes.data)
        most = int(count.max())
    inside = lib.rlkv_plan_merge_inside(kernel, group, int(gated), n_wg, used, most)
    assert inside >= 0
    return False, used, most, bool(inside)
