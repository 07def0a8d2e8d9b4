"""rlkv_decode_attention and rlkv_decode_attention_noalloc recorded into a HIP graph and replayed after the layer's work list
has been rebuilt: as another list of the same kind, or from one of whole pairs into one of shares and back."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_08525_amd as rl
from harness import Case, to_np, tolerance

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("entry", ["decode_attention", "decode_attention_noalloc"])
@pytest.mark.parametrize("dtype,kernel,short,long", [
    (rl.RLKV_BF16, rl.RLKV_KERNEL_MFMA, 300, 2600), (rl.RLKV_F32, rl.RLKV_KERNEL_VALU, 60, 1000),
    (rl.RLKV_BF16, rl.RLKV_KERNEL_VALU, 60, 1000),
], ids=["tiled", "rows f32", "rows bf16"])
@pytest.mark.parametrize("lengths", ["grow", "shrink", "grow on"])
@pytest.mark.parametrize("gated", [False, True], ids=["plain", "gated"])
def test_replay_under_another_list(gpu_device, lengths, dtype, kernel, short, long, entry, gated):
    first, second = {"grow": (short, long), "shrink": (long, short), "grow on": (long, 2 * long)}[lengths]
    c = Case(Hq=28, Hkv=4, B=2, S=8, R=56, dtype=dtype, kernel=kernel, mask=[1, 0, 0, 1], cap=max(first, second) + 16, seed=8)
    g = np.asarray([0.4, 1, 1, 0.7], dtype=np.float32) if gated else None
    if gated:
        c.cache.set_gates(g)
    q = torch.zeros(2, 28, 128, dtype=c.tdtype, device=c.device)
    out = torch.zeros_like(q)
    c.append([first, first // 2])
    c.check_decode(0, "before the recording", gates=g)          # (the list is planned by a direct call)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        getattr(c.cache, entry)(0, q, out, c.scale)

    def replay(step):
        qs = c.make_q(step)
        q.copy_(qs)
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        kv = to_np(c.k_hist), to_np(c.v_hist), c.n
        if gated:
            ref = oracle.decode_attention_gated(*kv, [float(x) if m else 0.0 for x, m in zip(g, c.mask_layer)], to_np(qs), c.S,
                                                c.R, c.scale)
        else:
            ref = oracle.decode_attention(*kv, c.mask_layer, to_np(qs), c.S, c.R, c.scale)
        got = out.float().cpu().numpy()
        assert np.isfinite(got).all(), f"replay {step}: rows not written"
        err = np.abs(got - ref)
        assert (err <= tolerance(ref, dtype)).all(), f"replay {step}: max err {err.max():.3e}"

    replay(1)
    c.append([2, 2])                                             # the list survives a uniform append
    replay(2)
    if second > first:
        c.append([second - first - 2, 40])
    else:
        c.cache.reset()
        c.n[:] = 0
        c.append([second, second // 2])
    c.check_decode(3, "the call that plans the new list", gates=g)
    replay(4)
    c.append([1, 1])
    replay(5)
    c.check_decode(6, "direct call after the replays", gates=g)
    c.close()
