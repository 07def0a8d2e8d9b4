"""The rule that gives a layer a list of whole pairs or one of shares, without a GPU: the measured side of the line on both
sides of it, for the kernels, group sizes, gates and kinds of call that meet it at different lengths."""
import numpy as np
import pytest

import paper_2510_08525_amd as rl

MFMA, VALU, BF16, F32 = rl.RLKV_KERNEL_MFMA, rl.RLKV_KERNEL_VALU, rl.RLKV_BF16, rl.RLKV_F32


def whole(kernel, dtype, q_heads, kv_heads, n_full, batch, n, gated=0, step=0, active=None, window=320):
    n = np.full(batch, n, np.int32) if np.isscalar(n) else np.asarray(n, np.int32)
    a = None if active is None else np.asarray(active, np.uint8)
    return rl.load_library().rlkv_plan_list_whole(kernel, dtype, q_heads // kv_heads, gated, step, 256, kv_heads, n_full, window, batch,
                                                  n.ctypes.data, a.ctypes.data if a is not None else None)


# (q heads, KV heads, full heads, sequences, tokens at which whole pairs were faster, tokens at which shares were); None = no
# such length below 1400
TILED = [(8, 8, 4, 1, 800, 1200), (32, 8, 4, 1, 800, 1200), (32, 8, 4, 2, 600, 1000), (32, 8, 4, 4, 500, 800), (32, 8, 4, 8, 500, 800),
         (32, 8, 4, 16, 800, 1200), (32, 8, 4, 32, 1400, None), (28, 4, 2, 1, 800, 1200), (28, 4, 2, 4, 600, 1000), (28, 4, 2, 16, 500, 800),
         (28, 4, 2, 32, 800, 1200), (12, 4, 2, 8, 500, 800), (16, 1, 1, 1, 700, 1000), (16, 1, 1, 4, 700, 1000), (16, 1, 1, 16, 400, 700),
         (64, 4, 4, 1, 700, 1000), (64, 4, 4, 16, 400, 700), (64, 4, 4, 32, 1000, 1400), (64, 4, 4, 64, 1200, None)]


@pytest.mark.parametrize("Hq,Hkv,full,B,yes,no", TILED, ids=lambda x: str(x))
@pytest.mark.parametrize("step", [0, 1], ids=["decode", "step"])
def test_tiled(Hq, Hkv, full, B, yes, no, step):
    assert whole(MFMA, BF16, Hq, Hkv, full, B, yes, step=step) == 1
    if no:
        assert whole(MFMA, BF16, Hq, Hkv, full, B, no, step=step) == 0


@pytest.mark.parametrize("Hq,Hkv,B,yes,no", [(32, 8, 1, 500, 1000), (32, 8, 4, 300, 600), (28, 4, 1, 500, 800), (28, 4, 4, 300, 600),
                                             (16, 1, 1, 200, 600), (64, 4, 1, 200, 600), (64, 4, 4, 200, 500), (16, 1, 16, 200, 500),
                                             (64, 4, 32, 800, None), (32, 8, 16, 1000, None)], ids=lambda x: str(x))
def test_steps_that_blend(Hq, Hkv, B, yes, no):
    assert whole(MFMA, BF16, Hq, Hkv, Hkv, B, yes, gated=1, step=1) == 1
    if no:
        assert whole(MFMA, BF16, Hq, Hkv, Hkv, B, no, gated=1, step=1) == 0


@pytest.mark.parametrize("Hq,Hkv,full,lengths,want", [
    (8, 8, 4, [500, 316, 182], 1), (8, 8, 4, [700, 442, 255], 1), (28, 4, 2, [600, 379, 219], 1), (28, 4, 2, [1300, 820, 470], 0),
    (64, 4, 4, [700, 442, 255], 0), (32, 8, 8, [4000] + [3800] * 29, 1), (32, 8, 8, [9000] + [3800] * 29, 0), (32, 8, 8, [5000] * 16, 0),
], ids=lambda x: str(x))
def test_ragged_and_long(Hq, Hkv, full, lengths, want):
    assert whole(MFMA, BF16, Hq, Hkv, full, len(lengths), lengths) == want


@pytest.mark.parametrize("dtype,Hq,Hkv,full,B,gated,yes,no", [
    (F32, 8, 8, 4, 1, 0, 128, 260), (F32, 32, 8, 4, 1, 0, 128, 260), (F32, 32, 8, 4, 32, 0, 400, 5000), (F32, 28, 4, 2, 1, 0, 128, 200),
    (F32, 16, 1, 1, 1, 0, 128, 130), (F32, 64, 4, 4, 32, 0, 100, 130), (F32, 28, 4, 4, 64, 0, 400, None), (F32, 32, 8, 4, 1, 1, 128, 200),
    (BF16, 8, 8, 4, 1, 0, 200, 400), (BF16, 32, 8, 4, 1, 0, 200, 260), (BF16, 28, 4, 2, 8, 0, 128, 200), (BF16, 16, 1, 1, 8, 0, 128, 130),
    (BF16, 64, 4, 4, 1, 1, 128, 130), (BF16, 32, 8, 4, 32, 0, 300, None),
], ids=lambda x: str(x))
def test_row_major(dtype, Hq, Hkv, full, B, gated, yes, no):
    for step in (0, 1):
        assert whole(VALU, dtype, Hq, Hkv, full, B, yes, gated=gated, step=step) == 1
        if no:
            assert whole(VALU, dtype, Hq, Hkv, full, B, no, gated=gated, step=step) == 0


def test_only_active_sequences_count():
    assert whole(MFMA, BF16, 32, 8, 4, 40, 100) == 0                       # 320 pairs for 256 workgroups
    assert whole(MFMA, BF16, 32, 8, 4, 40, 100, active=[1] * 32 + [0] * 8) == 1
    assert whole(MFMA, BF16, 32, 8, 4, 2, [300, 9000]) == 0
    assert whole(MFMA, BF16, 32, 8, 4, 2, [300, 9000], active=[1, 0]) == 1
    assert whole(MFMA, BF16, 32, 8, 0, 2, 9000) == 1                       # compressed heads only: 320 rows each


def test_invalid_arguments():
    lib, n = rl.load_library(), np.ones(1, np.int32)
    ok = [MFMA, BF16, 4, 0, 0, 256, 8, 4, 320, 1, n.ctypes.data, None]
    assert lib.rlkv_plan_list_whole(*ok) == 1
    for at, value in ((0, 0), (1, 7), (2, 0), (2, 17), (5, 0), (6, 0), (7, 9), (7, -1), (8, 0), (9, 0), (10, None)):
        assert lib.rlkv_plan_list_whole(*(ok[:at] + [value] + ok[at + 1:])) == -1, at
    bad = np.full(1, -1, np.int32)
    assert lib.rlkv_plan_list_whole(*(ok[:10] + [bad.ctypes.data, None])) == -1
