"""Prefill tiles outside the unmasked loop: each kind of mask a tile can take (none, diagonal, band edge, both, ring slots,
the end of the sinks) over stores long enough that whole ranges of tiles are hopped over, at odd lengths and windows."""
import numpy as np
import pytest

import paper_2510_08525_amd as rl
from harness import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,R", [(33, 70), (64, 31), (5, 1), (0, 300), (40, 24)], ids=lambda x: str(x))
@pytest.mark.parametrize("gated", [False, True], ids=["plain", "gated"])
def test_masks_behind_long_stores(gpu_device, S, R, gated):
    c = Case(Hq=14, Hkv=2, B=2, S=S, R=R, dtype=rl.RLKV_BF16, kernel=rl.RLKV_KERNEL_MFMA, mask=[1, 0], cap=1700, seed=S + R,
             prefill_tokens=128, arena_fill=0xFF)
    g = np.asarray([0.3, 1.0], dtype=np.float32) if gated else None
    if gated:
        c.cache.set_gates(g)
    c.check_prefill([S + 7, 1], 0, "the chunk that ends the sinks", gates=g)
    c.append([1201, 1473])
    for step, counts in enumerate([[128, 65], [1, 128], [33, 30]]):
        c.check_prefill(counts, step + 1, f"chunk {step}", gates=g)
        c.check_indices()
    c.check_decode(0, "decode", fused=True, gates=g)
    c.close()
