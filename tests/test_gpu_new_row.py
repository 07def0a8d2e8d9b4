"""A fused step attends over the row it appends, whatever tile, wavefront and register of the first loads the row falls into, and leaves
it in the store: every new K is one query's own direction, so that this query's output is the new V row (a row missing, misplaced or
half written is off by whole units), and a decode call afterwards gives the same.  Groups at the edges of the packed merge."""
import numpy as np
import pytest
import torch

import paper_2510_08525_amd as rl

pytestmark = pytest.mark.gpu

KINDS = [(rl.RLKV_BF16, rl.RLKV_KERNEL_MFMA), (rl.RLKV_BF16, rl.RLKV_KERNEL_VALU), (rl.RLKV_F32, rl.RLKV_KERNEL_VALU)]


@pytest.mark.parametrize("dtype,kernel", KINDS, ids=["mfma", "valu-bf16", "valu-f32"])
@pytest.mark.parametrize("gate", [1.0, 0.5])
@pytest.mark.parametrize("group", [1, 3, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("start,steps", [(0, 140), (700, 40)])
def test_step_attends_over_its_row_and_keeps_it(gpu_device, start, steps, group, gate, dtype, kernel):
    H, B, S, R, D = 2, 2, 5, 70, 128
    tdt = torch.float32 if dtype == rl.RLKV_F32 else torch.bfloat16
    g = torch.Generator().manual_seed(group * 1000 + start)
    cache = rl.Cache(1, group * H, H, D, B, S, R, dtype, [1, 0], [start + steps] * B, kernel=kernel, device=gpu_device, arena_fill=0xFF)
    if gate < 1.0:
        cache.set_gates(np.asarray([gate, 1.0], dtype=np.float32))
    if start:
        k, v = (torch.randn(B, H, start, D, generator=g).to(tdt).to(gpu_device) for _ in range(2))
        cache.append(0, k, v)
    for t in range(steps):
        pick = t % group                                     # the head whose direction the new keys take
        # score of the new row: 2 |q|^2 / sqrt(D), about 22; of the others N(0, 1), of earlier steps' rows N(0, 2)
        q = torch.randn(B, group * H, D, generator=g).to(tdt).float()
        k = (2.0 * q.view(B, H, group, D)[:, :, pick:pick + 1]).to(tdt).to(gpu_device)
        v = torch.randn(B, H, 1, D, generator=g).to(tdt).to(gpu_device)
        qd = q.to(tdt).to(gpu_device)
        out, again = torch.zeros(B, group * H, D, dtype=tdt, device=gpu_device), torch.zeros(B, group * H, D, dtype=tdt, device=gpu_device)
        cache.append_decode(0, k, v, qd, out, 1.0 / D ** 0.5)
        cache.decode_attention(0, qd, again, 1.0 / D ** 0.5)
        got = out.view(B, H, group, D)[:, :, pick].float()
        # (the others' weight together is below 1e-5 of exp(22); rounding of an output below 4: 2^-7)
        assert (got - v[:, :, 0].float()).abs().max().item() < 2e-2, t
        # two lists may cut the sums differently: one rounding of the output
        assert (out.float() - again.float()).abs().max().item() <= (2e-5 if dtype == rl.RLKV_F32 else 4e-2), t
    assert (cache.lengths(0) == start + steps).all()
    cache.close()
