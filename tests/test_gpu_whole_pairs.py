"""Decode over lists of whole pairs (one workgroup per pair, no merge launch) and the lists around them: sizes at the edges
of the eight wavefronts' tiles, the step at which the rule hands over to shares, recorded launches that outlive the kind
of list they were recorded under, steps whose growth only the device knows; the fused step of the row-major stores."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_08525_amd as rl
from harness import Case, to_np, tolerance

pytestmark = pytest.mark.gpu

BF16, F32, MFMA, VALU = rl.RLKV_BF16, rl.RLKV_F32, rl.RLKV_KERNEL_MFMA, rl.RLKV_KERNEL_VALU
KINDS = [(BF16, MFMA), (BF16, VALU), (F32, VALU)]


@pytest.mark.parametrize("dtype,kernel", KINDS, ids=["tiled", "rows bf16", "rows f32"])
@pytest.mark.parametrize("Hq,Hkv,mask", [(8, 2, [1, 0]), (28, 4, [1, 0, 0, 1]), (16, 1, [1]), (2, 2, [0, 1])],
                         ids=lambda x: str(x) if isinstance(x, int) else "")
@pytest.mark.parametrize("n", [1, 31, 127, 255, 511])
def test_steps_at_the_edges_of_tiles(gpu_device, Hq, Hkv, mask, n, dtype, kernel):
    """Stores start as NaN bytes: a row that is not there may reach no sum, in the step that appends least of all."""
    c = Case(Hq=Hq, Hkv=Hkv, B=3, S=4, R=61, dtype=dtype, kernel=kernel, mask=mask, cap=n + 8, seed=n, arena_fill=0xFF)
    c.append([n, max(1, n // 3), max(1, n - 5)])
    for step in range(4):
        c.check_decode(step, f"fused step {step}", fused=True)
        c.check_decode(step, f"decode {step}")
        c.check_indices()
    c.append([2, 2, 2])                       # the list survives a uniform append
    c.check_decode(9, "decode after a uniform append")
    c.check_decode(10, "fused step after a uniform append", fused=True)
    c.check_indices()
    c.close()


@pytest.mark.parametrize("dtype,kernel,at", [(BF16, MFMA, 1536), (F32, VALU, 128), (BF16, VALU, 256)],
                         ids=["tiled", "rows f32", "rows bf16"])
@pytest.mark.parametrize("gated", [False, True], ids=["plain", "gated"])
def test_growth_across_the_rule(gpu_device, dtype, kernel, at, gated):
    """From a list of whole pairs into one of shares, a step at a time."""
    c = Case(Hq=8, Hkv=2, B=2, S=8, R=120, dtype=dtype, kernel=kernel, mask=[1, 1], cap=at + 80, seed=4)
    g = np.asarray([0.4, 1.0], dtype=np.float32) if gated else None
    if gated:
        c.cache.set_gates(g)
    c.append([at - 20, at // 2])
    for step in range(70):
        if step % 10 == 9:
            c.check_decode(step, f"step {step}", fused=True, gates=g)
        else:
            c.append_decode(step)
    c.check_indices()
    c.close()


@pytest.mark.parametrize("page", [0, 64])
@pytest.mark.parametrize("first,second", [(300, 2600), (2600, 300)])
def test_recorded_launch_outlives_its_kind_of_list(gpu_device, page, first, second):
    """Recorded and replayed under lists that a decode call planned, of whole pairs at 300 tokens and of shares at 2600; then
    steps by call again, the first of which follows a prepared step the host cannot know to have run."""
    steps = 3
    cap = max(first, second) + 16
    c = Case(Hq=28, Hkv=4, B=2, S=8, R=56, dtype=BF16, kernel=MFMA, mask=[1, 0, 0, 1], cap=cap, seed=6, page_tokens=page,
             pool_pages=2 * -(-cap // page) if page else 0)
    k = torch.zeros(2, 4, 1, 128, dtype=torch.bfloat16, device=c.device)
    v, q = torch.zeros_like(k), torch.zeros(2, 28, 128, dtype=torch.bfloat16, device=c.device)
    out = torch.zeros_like(q)
    c.append([first, first // 2])
    c.check_decode(40, "the call that plans the first list")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        c.cache.append_decode_launch(0, k, v, q, out, c.scale)

    def replay(step):
        rows = [torch.stack([h[b, :, c.n[b]:c.n[b] + 1] for b in range(2)]) for h in (c.k_hist, c.v_hist)]
        qs = c.make_q(step)
        k.copy_(rows[0]), v.copy_(rows[1]), q.copy_(qs)
        c.cache.append_decode_prepare(0)
        graph.replay()
        torch.cuda.synchronize()
        c.n += 1
        ref = oracle.decode_attention(to_np(c.k_hist), to_np(c.v_hist), c.n, c.mask_layer, to_np(qs), c.S, c.R, c.scale)
        err = np.abs(out.float().cpu().numpy() - ref)
        assert (err <= tolerance(ref, BF16)).all(), f"replay {step}: {err.max():.3e}"

    for s in range(steps):
        replay(s)
    c.check_decode(50, "decode between replays")
    if second > first:
        c.append([second - first - steps, 40])
    else:
        c.cache.reset()
        c.n[:] = 0
        c.append([second, second // 2])
    c.check_decode(41, "the call that plans the second list")
    for s in range(steps):
        replay(10 + s)
    c.check_indices()
    for s in range(3):
        c.check_decode(20 + s, f"step by call {s}", fused=True)
    replay(30)
    c.check_decode(31, "decode after the last replay")
    c.check_indices()
    c.close()
