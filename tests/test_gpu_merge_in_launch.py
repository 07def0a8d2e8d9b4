"""Pairs cut into shares are merged by the last workgroup that leaves one, inside the attention launch: call after call the same bits as
the merge launch behind a recorded call gives, for 3 to 32 partials, groups that fill a wavefront's two heads and that do not,
shares that end in one pair and begin in the next, outputs at any element, and steps whose growth the host counts.  The lists beyond the
lines between the two merges (33 partials; 17, or more than half of the grid, where heads blend or groups are beyond 8; row-major groups
beyond 8) take the merge launch in either kind of call and go through the same."""
import numpy as np
import pytest
import torch

import paper_2510_08525_amd as rl
from harness import Case
from list_plan import plan

pytestmark = pytest.mark.gpu

KINDS = {"mfma": (rl.RLKV_BF16, rl.RLKV_KERNEL_MFMA), "valu-f32": (rl.RLKV_F32, rl.RLKV_KERNEL_VALU), "valu-bf16": (rl.RLKV_BF16, rl.RLKV_KERNEL_VALU)}
S, R = 8, 56


def mask(lengths):
    return [1, 0] if len(lengths) < 40 else [1, 1]


def inside(lengths, group, gate, kind):
    return plan(*KINDS[kind], group, mask(lengths), S, R, lengths, max(lengths) + 8, gated=gate is not None)[3]


ALL = [(lengths, group, gate, kind)
       for lengths in [[900], [1400], [2010], [4100], [7900], [8100], [3000, 2500, 1400], [1200] * 40]
       for group in [1, 4, 7, 16] for gate in [None, 0.375] for kind in KINDS]
name = lambda c: f"{len(c[0])}x{c[0][0]}-{c[1]}-{'plain' if c[2] is None else 'blending'}-{c[3]}"


@pytest.mark.parametrize("case", [c for c in ALL if inside(*c)], ids=name)
def test_same_bits_as_the_merge_launch(gpu_device, case):
    run(*case)


@pytest.mark.parametrize("case", [c for c in ALL if not inside(*c)], ids=name)
def test_lists_beyond_the_lines(gpu_device, case):
    run(*case)


def run(lengths, group, gate, kind):
    dtype, kernel = KINDS[kind]
    B = len(lengths)
    c = Case(Hq=2 * group, Hkv=2, B=B, S=S, R=R, dtype=dtype, kernel=kernel, mask=mask(lengths), cap=max(lengths) + 8, seed=group)
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
