"""Blending prefill (Eq. 1) of few long sequences: every full head's workgroup divided into 2 to 8 shares of the keys outside the
local positions; the last share takes those too and leaves their result beside its accumulators; merged and blended by the kernel
that follows."""
import numpy as np
import pytest

import harness
import paper_2510_08525_amd as rl
from harness import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("page", [0, 64])
@pytest.mark.parametrize("Hq,Hkv,mask,gates,B", [
    (28, 4, [1, 0, 0, 1], [0.3, 1, 1, 1.0], 1),
    (28, 4, [1, 0, 1, 0], [0.0, 1, 0.8, 1], 2),
    (16, 1, [1], [0.5], 1),
    (6, 2, [0, 1], [1, 0.7], 3),
], ids=["one of two full heads blends", "two sequences", "group of 16", "group of 3"])
def test_blending_workgroups_divided(gpu_device, Hq, Hkv, mask, gates, B, page, monkeypatch):
    monkeypatch.setattr(harness, "TUNING", {"prefill_min_share_tiles": 4})
    c = Case(Hq=Hq, Hkv=Hkv, B=B, S=33, R=96, dtype=rl.RLKV_BF16, kernel=rl.RLKV_KERNEL_MFMA, mask=mask, cap=2300, seed=7,
             prefill_tokens=160, page_tokens=page, pool_pages=B * 36 if page else 0, arena_fill=0xFF)
    g = np.asarray(gates, dtype=np.float32)
    c.cache.set_gates(g)
    for step, (cached, counts) in enumerate([(0, [160] * B), (300, [64] * B), (1000, [33] + [160] * (B - 1)), (2000, [90] * B)]):
        if cached > int(c.n.max()):
            c.append([cached - int(n) for n in c.n])
        c.check_prefill(counts, step, f"{cached} cached", gates=g)
        c.check_indices()
    c.check_decode(0, "decode", fused=True, gates=g)
    c.close()
