"""cfg.prefill_min_share_tiles taken as it is set, in every form of the prefill kernel: a chunk whose shares would have fewer
tiles is not divided, so its outputs have the bits of a cache that never divides."""
import numpy as np
import pytest
import torch

import harness
import paper_2510_08525_amd as rl
from harness import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gates", [None, [0.3, 1, 1, 0.8]], ids=["plain", "blending"])
@pytest.mark.parametrize("minimum,cached", [(100, 4400), (1, 0), (2, 70)], ids=lambda x: str(x))
def test_shares_below_the_minimum_are_not_made(gpu_device, minimum, cached, gates, monkeypatch):
    outs = []
    for tiles in (minimum, 1 << 20):
        monkeypatch.setattr(harness, "TUNING", {"prefill_min_share_tiles": tiles})
        c = Case(Hq=28, Hkv=4, B=1, S=16, R=112, dtype=rl.RLKV_BF16, kernel=rl.RLKV_KERNEL_MFMA, mask=[1, 0, 0, 1], cap=cached + 96,
                 seed=5, prefill_tokens=96)
        g = None if gates is None else np.asarray(gates, dtype=np.float32)
        if g is not None:
            c.cache.set_gates(g)
        if cached:
            c.append([cached])
        c.check_prefill([96], 0, f"shares of at least {tiles} tiles", gates=g)
        outs.append(c.last_out.view(torch.int16).clone())
        c.close()
    assert torch.equal(outs[0], outs[1])
