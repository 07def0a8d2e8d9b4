"""What each workgroup of a prefill attention launch works on when the chunks of its sequences differ in length."""
import numpy as np
import pytest

import paper_2510_08525_amd as rl


@pytest.mark.parametrize("seed", range(12))
def test_every_block_with_queries_is_one_workgroups(seed):
    """Sequences of any chunk lengths: every block of every (sequence, head) that holds queries belongs to exactly one workgroup,
    none is left without; rows dealt by rows stay on one XCD (linear index % 8), the other full heads' blocks spread evenly,
    also over the 32 shader engines (linear index % 32); every XCD serves full heads before compressed ones."""
    rng = np.random.default_rng(seed)
    for _ in range(8):
        per = int(rng.choice([8, 18, 36, 64, 256]))
        n_full, n_comp, B = int(rng.integers(0, 5)), int(rng.integers(0, 5)), int(rng.choice([1, 2, 3, 8, 17, 128]))
        if n_full + n_comp == 0:
            n_comp = 1
        longest = int(rng.integers(1, 700))
        tokens = np.sort(rng.integers(1, longest + 1, size=B))[::-1].copy()
        if rng.random() < 0.5:
            tokens[: B // 2 + 1] = longest
        if rng.random() < 0.3:
            tokens = rng.permutation(tokens)
        if rng.random() < 0.2:
            tokens[:] = longest
        blocks = [-(-int(t) // per) for t in tokens]
        gx, lead = max(blocks), 0
        while lead < B and blocks[lead] == gx:
            lead += 1
        dealt = 8 * int(rng.integers(0, B * n_full // 8 + 1))
        by_rows = min(dealt, lead * n_full) // 8 * 8
        seen, xcds, heavy_rest, last = {}, {}, [], [(-1,)] * 8
        lin = 0
        while (item := rl.rlkv_plan_prefill_item(lin, per, n_full, n_comp, tokens, dealt)) is not None:
            full, place, head, block = item
            assert 0 <= place < B and 0 <= head < (n_full if full else n_comp) and 0 <= block < blocks[place]
            assert item not in seen
            seen[item] = lin
            row = place * (n_full if full else n_comp) + head
            xcds.setdefault((full, row), set()).add(lin % 8)
            if full and row >= by_rows:
                heavy_rest.append(lin)
            assert (not full, row) >= last[lin % 8] or not full
            last[lin % 8] = (not full, row)
            lin += 1
        assert len(seen) == lin == sum(blocks) * (n_full + n_comp)
        for y in range(by_rows):
            assert xcds[(True, y)] == {y % 8}
        for y in range(lead * n_comp // 8 * 8):
            assert xcds[(False, y)] == {y % 8}
        per_xcd = np.bincount([x % 8 for x in heavy_rest], minlength=8)
        assert per_xcd.max() - per_xcd.min() <= 1
        engines = np.bincount([x % 32 for x in heavy_rest], minlength=32)
        assert engines.max() - engines.min() <= 2


@pytest.mark.parametrize("seed", range(4))
def test_blocks_of_large_grids(seed):
    """Quotients by the sizes of a launch are taken as products with their inverses: exact up to the last index of the largest
    grids, and around every multiple."""
    rng = np.random.default_rng(seed)
    for _ in range(200):
        gx = int(rng.choice([1, 2, 3, 7, 13, 455, 4096, 65535, 65536, int(rng.integers(1, 65537))]))
        gy = int(rng.integers(1, min(65535, (2 ** 31 - 1) // gx) + 1))
        heavy = int(rng.integers(0, gy + 1))
        dealt = 8 * int(rng.integers(0, heavy // 8 + 1))
        rows_h, rows_l, n_b = dealt // 8, (gy - heavy) // 8, (heavy - dealt) * gx
        last = gx * gy - 1
        near = int(rng.integers(0, gy)) * gx
        for lin in {0, last, max(0, last - 7), *(min(last, max(0, near * 8 + d)) for d in (-1, 0, 7, 8)), int(rng.integers(0, last + 1))}:
            k, i = lin % 8, lin // 8
            c_a, c_b, c_c = rows_h * gx, (n_b - k + 7) // 8, rows_l * gx
            if i < c_a:
                want = (i % gx, i // gx * 8 + k)
            elif i < c_a + c_b:
                w = (i - c_a) * 8 + k
                want = (w % gx, dealt + w // gx)
            elif i < c_a + c_b + c_c:
                j = i - c_a - c_b
                want = (j % gx, heavy + j // gx * 8 + k)
            else:
                w = (i - c_a - c_c) * 8 + k - n_b
                want = (w % gx, heavy + 8 * rows_l + w // gx)
            assert rl.rlkv_plan_prefill_block(lin, gx, gy, dealt, heavy) == want, (lin, gx, gy, dealt, heavy)


def test_rejects_bad_arguments():
    for bad in [(0, 0, 1, 0, [5], 0), (-1, 36, 1, 0, [5], 0), (0, 36, -1, 0, [5], 0), (0, 36, 1, 0, [0], 0), (0, 36, 1, 0, [5], -8),
                (0, 36, 1, 0, [5] * 129, 0)]:
        with pytest.raises(rl.RlkvError):
            rl.rlkv_plan_prefill_item(*bad)
