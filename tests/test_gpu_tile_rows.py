"""Multi-token appends of the tiled layout: rows pass through LDS into the tile.  Chunks that start and end inside tiles,
wrap a ring more than once, and a V tensor that starts at an odd element (no 16-byte loads)."""
import numpy as np
import pytest
import torch

import paper_2510_08525_amd as rl
from harness import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("v_offset", [0, 1, 4], ids=lambda o: f"v+{o}")
@pytest.mark.parametrize("S,R", [(4, 24), (33, 70), (0, 5)], ids=lambda x: str(x))
def test_append_chunks_any_v_alignment(gpu_device, S, R, v_offset):
    c = Case(Hq=8, Hkv=2, B=2, S=S, R=R, dtype=rl.RLKV_BF16, kernel=rl.RLKV_KERNEL_MFMA, mask=[1, 0], cap=400, seed=31,
             arena_fill=0xFF)
    for step, counts in enumerate([[1, 31], [32, 33], [95, 64], [3, 130]]):
        stride = max(counts)
        k = torch.zeros(c.B, c.Hkv, stride, c.D, dtype=torch.bfloat16)
        flat = torch.zeros(k.numel() + v_offset, dtype=torch.bfloat16)
        v = flat[v_offset:].view(k.shape)
        for b, n in enumerate(counts):
            k[b, :, :n] = c.k_hist[b, :, c.n[b]:c.n[b] + n]
            v[b, :, :n] = c.v_hist[b, :, c.n[b]:c.n[b] + n]
        vd = flat.to(gpu_device)[v_offset:].view(k.shape)
        assert vd.data_ptr() % 16 == 2 * v_offset
        c.cache.append_ragged(0, k.to(gpu_device), vd, np.asarray(counts, dtype=np.int32))
        c.n += np.asarray(counts)
        c.check_indices()
        c.check_decode(step, f"after chunk {step}")
    c.close()
