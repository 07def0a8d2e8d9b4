"""Prefill under softmax scales near the end of the fp32 range, whose reciprocal is a subnormal: scores that are all negative and
rise with the position, so that every tile has to move the reference maximum below zero."""
import numpy as np
import pytest
import torch

import paper_2510_08525_amd as rl
from harness import Case
from inputs import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [3e37, 1e38, 2.3e38])
@pytest.mark.parametrize("gated", [False, True], ids=["plain", "blending"])
def test_scales_with_a_subnormal_reciprocal(gpu_device, gated, scale, monkeypatch):
    c = Case(Hq=8, Hkv=2, B=2, S=5, R=150, dtype=rl.RLKV_BF16, kernel=rl.RLKV_KERNEL_MFMA, mask=[1, 0], cap=480, seed=9,
             prefill_tokens=240, scale=scale, q_prescale=2.0 ** -60, arena_fill=0xFF)
    # scores of about -240 (1 - position / 600), from the first 4 dimensions of K alone; products are 2^-122 and up
    fall = (1.0 - torch.arange(480) / 600.0)[None, None, :, None]
    k = torch.zeros(c.k_hist.shape)
    k[..., :4] = (1e38 / scale) * 2.0 ** -58 * fall * (0.75 + 0.25 * torch.rand(k[..., :4].shape, generator=torch.Generator().manual_seed(1)))
    c.k_hist = (-k).to(torch.bfloat16)
    g = None
    if gated:
        g = np.asarray([0.375, 1.0], dtype=np.float32)
        c.cache.set_gates(g)
    normal = synth.normal
    monkeypatch.setattr(synth, "normal", lambda seed, what, *a, **kw: normal(seed, what, *a, **kw).abs().clamp(0.5, 1.0)
                        if what == synth.T_Q else normal(seed, what, *a, **kw))
    for step, counts in enumerate([[240, 101], [200, 240]]):
        c.check_prefill(counts, step, f"chunk {step}", gates=g)
    c.close()
