"""Blending prefill (Eq. 1) in the form with two column groups per wavefront, which chunks of many workgroups take: tiles at the
end of the sinks and at the band's edge fold into both passes, windows shorter than a workgroup's positions leave no hot
tiles to the local one, and the first chunks hold sinks themselves.  Of 9 full heads and 20 sequences of 36 tokens, 360 workgroups
of 128 columns (270 in the last step) would need a second round on 256 CUs, 180 of 256 columns do not; every step asserts that the
library chooses them."""
import numpy as np
import pytest
import torch

import paper_2510_08525_amd as rl
from harness import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,R,page,wide", [(33, 70, 0, False), (64, 31, 64, False), (5, 1, 0, False), (0, 300, 32, False), (40, 24, 0, True)])
def test_two_passes_over_one_accumulator_set(gpu_device, S, R, page, wide):
    B, H = 20, 10
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    c = Case(Hq=7 * H, Hkv=H, B=B, S=S, R=R, dtype=rl.RLKV_BF16, kernel=rl.RLKV_KERNEL_MFMA, mask=[1] * (H - 1) + [0], cap=620,
             seed=S + R, prefill_tokens=36, page_tokens=page, pool_pages=B * 20 if page else 0, arena_fill=0xFF)
    if wide:
        c.v_hist[:, 0, 33] = 65536.0          # beyond fp16: the second pass takes V as stored too
    g = np.asarray([i / 8 for i in range(H - 1)] + [1.0], dtype=np.float32)         # 0, 1/8, ... 1: the last full head does not blend
    c.cache.set_gates(g)
    rel = 2.0 ** -10 if wide else 0.0
    for step, (cached, counts) in enumerate([(0, [36] * B), (36, [36 - b % 3 for b in range(B)]), (300 + S, [36] * B), (523, [36, 3] * (B // 2))]):
        if cached > int(c.n.max()):
            c.append([cached - int(n) for n in c.n])
        assert not rl.rlkv_plan_blend_form(cus, 7, H - 1, counts)
        c.check_prefill(counts, step, f"{cached} cached", gates=g, rel=rel)
    c.check_indices()
    c.close()
