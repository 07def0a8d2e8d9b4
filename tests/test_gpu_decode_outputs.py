"""Decode outputs go out four to a store where the caller's buffer lies on 8 bytes (fp32: 16), else one by one: the same bits.  Groups at
the edges of a merge pass (8 heads to 256 threads, 16 to 512), pairs of one workgroup (four and eight wavefronts) and pairs of several."""
import numpy as np
import pytest
import torch

import paper_2510_08525_amd as rl
from harness import Case
from inputs import synth

pytestmark = pytest.mark.gpu


KINDS = [(rl.RLKV_BF16, rl.RLKV_KERNEL_MFMA), (rl.RLKV_BF16, rl.RLKV_KERNEL_VALU), (rl.RLKV_F32, rl.RLKV_KERNEL_VALU)]


@pytest.mark.parametrize("dtype,kernel", KINDS, ids=["mfma", "valu-bf16", "valu-f32"])
@pytest.mark.parametrize("gate", [1.0, 0.375])
@pytest.mark.parametrize("group", [1, 8, 9, 16])
@pytest.mark.parametrize("B,cached", [(2, 40), (3, 700), (40, 90)])
def test_output_that_starts_at_any_element(gpu_device, B, cached, group, gate, dtype, kernel):
    H = 2
    c = Case(Hq=group * H, Hkv=H, B=B, S=3, R=50, dtype=dtype, kernel=kernel, mask=[1, 0], cap=cached + 3,
             seed=group + cached, arena_fill=0xFF)
    if gate < 1.0:
        c.cache.set_gates(np.asarray([gate, 1.0], dtype=np.float32))
    c.append([cached - b % 3 for b in range(B)])
    tdt = torch.float32 if dtype == rl.RLKV_F32 else torch.bfloat16
    q = synth.normal(6, synth.T_Q, 0, range(B), range(group * H), 0, 1, 128, dtype=tdt)[:, :, 0].contiguous().to(c.device)
    want = torch.zeros_like(q)
    c.cache.decode_attention(0, q, want, c.scale)
    for offset in (1, 2, 4):
        room = torch.zeros(want.numel() + 16, dtype=tdt, device=c.device)
        got = room[offset:offset + want.numel()].view(want.shape)
        c.cache.decode_attention(0, q, got, c.scale)
        torch.cuda.synchronize()
        assert torch.equal(want, got)
        assert not room[:offset].any() and not room[offset + want.numel():].any()
    if gate == 1.0:
        c.check_decode(0, "against the oracle")
    c.close()
