"""Pairs cut into shares are merged by the last workgroup that leaves one, inside the attention launch: call after call the same bits as
the merge launch behind a recorded call gives, for two to 33 partials, groups that fill a wavefront's two heads and that do not,
shares that end in one pair and begin in the next, outputs at any element, and steps whose growth the host counts."""
import numpy as np
import pytest
import torch

import paper_2510_08525_amd as rl
from harness import Case

pytestmark = pytest.mark.gpu

KINDS = [(rl.RLKV_BF16, rl.RLKV_KERNEL_MFMA), (rl.RLKV_F32, rl.RLKV_KERNEL_VALU), (rl.RLKV_BF16, rl.RLKV_KERNEL_VALU)]


@pytest.mark.parametrize("dtype,kernel", KINDS, ids=["mfma", "valu-f32", "valu-bf16"])
@pytest.mark.parametrize("gate", [None, 0.375], ids=["plain", "blending"])
@pytest.mark.parametrize("group", [1, 4, 7, 16])
@pytest.mark.parametrize("lengths", [[1400], [2010], [4100], [3000, 2500, 1400], [1200] * 40], ids=lambda x: f"{len(x)}x{x[0]}")
def test_same_bits_as_the_merge_launch(gpu_device, lengths, group, gate, dtype, kernel):
    B = len(lengths)
    c = Case(Hq=2 * group, Hkv=2, B=B, S=8, R=56, dtype=dtype, kernel=kernel, mask=[1, 0] if B < 40 else [1, 1], cap=max(lengths) + 8,
             seed=group)
    if gate is not None:
        c.cache.set_gates(np.asarray([gate, 1.0], dtype=np.float32))
    while (c.n < np.asarray(lengths)).any():
        c.append([int(min(2048, n - x)) for n, x in zip(lengths, c.n)])
    q = c.make_q(3).to(c.device)
    room = torch.full((q.numel() + 8,), float("nan"), dtype=c.tdtype, device=c.device)
    inside = [room[k:k + q.numel()].view(q.shape) for k in (0, 1)]
    recorded = torch.zeros_like(q)
    c.cache.decode_attention(0, q, recorded, c.scale)             # (plans the list; a call under capture may not)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        c.cache.decode_attention(0, q, recorded, c.scale)         # a recorded call has the merge launch
    recorded.fill_(float("nan"))
    graph.replay()
    torch.cuda.synchronize()
    assert torch.isfinite(recorded.float()).all()
    for _ in range(5):
        for out in inside:
            room.fill_(float("nan"))
            c.cache.decode_attention(0, q, out, c.scale)
            torch.cuda.synchronize()
            assert torch.equal(out, recorded)
    # steps: growth counted by the host, then read by a replay from the list
    c.check_decode(1, "step", fused=True, gates=None if gate is None else np.asarray([gate, 1.0], dtype=np.float32))
    c.check_decode(2, "step", fused=True, gates=None if gate is None else np.asarray([gate, 1.0], dtype=np.float32))
    c.cache.decode_attention(0, q, inside[0], c.scale)
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(inside[0], recorded)
    c.close()
