"""Start of a decode launch: the ring slot of a step's new row is a remainder by a product (windows whose inverse is exact, nearly
exact and far from it, down to one slot), and the row-major kernel has a form without blending heads, which a recorded launch must not
take: gates may be set between its replays."""
import numpy as np
import pytest
import torch

import paper_2510_08525_amd as rl

pytestmark = pytest.mark.gpu
D = 128


@pytest.mark.parametrize("dtype", [rl.RLKV_F32, rl.RLKV_BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("sink,recent,first", [(0, 1, 1), (3, 1, 2), (0, 2, 9), (5, 3, 4), (1, 31, 65500), (4, 64, 60), (16, 70, 1200), (2, 257, 511)])
def test_ring_slot_of_a_step(gpu_device, dtype, sink, recent, first):
    tdt = torch.float32 if dtype == rl.RLKV_F32 else torch.bfloat16
    steps = 40
    c = rl.Cache(1, 4, 2, D, 1, sink, recent, dtype, [[1, 0]], [first + steps])
    rows = torch.randn(1, 2, 4096, D, device="cuda", dtype=tdt)
    for at in range(0, first, 4096):
        n = min(4096, first - at)
        c.append(0, rows[:, :, :n].contiguous(), rows[:, :, :n].contiguous())
    q = torch.randn(1, 4, D, device="cuda", dtype=tdt)
    out, new = torch.empty_like(q), rows[:, :, :1].contiguous()
    for n in range(first + 1, first + steps + 1):
        c.append_decode(0, new, new, q, out, 0.1)
        if n % 7 and n < first + steps:
            continue
        want = np.full(sink + recent, -1, dtype=np.int32)
        for p in range(max(0, n - recent), n):
            if p >= sink:
                want[sink + (p - sink) % recent] = p
        want[:min(sink, n)] = np.arange(min(sink, n))
        held = min(n, sink + recent)
        assert (c.slot_positions(0, 1, 0)[:held] == want[:held]).all()
    c.close()


@pytest.mark.parametrize("n", [40, 700])
def test_recorded_launch_follows_gates_set_later(gpu_device, n):
    c = rl.Cache(1, 8, 4, D, 2, 4, 28, rl.RLKV_F32, [[1, 1, 0, 1]], [n] * 2)
    k = torch.randn(2, 4, n, D, device="cuda")
    c.append(0, k, k.flip(2).contiguous())
    q = torch.randn(2, 8, D, device="cuda")
    eager, recorded = torch.empty_like(q), torch.empty_like(q)
    c.decode_attention(0, q, eager, 0.1)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        c.decode_attention(0, q, recorded, 0.1)
    seen = []
    for gates in (None, [0.3, 1.0, 1.0, 0.8], [0.0, 0.5, 1.0, 1.0], None):
        c.set_gates(None if gates is None else np.asarray(gates, np.float32))
        c.decode_attention(0, q, eager, 0.1)
        recorded.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(eager, recorded)
        seen.append(eager.clone())
    assert torch.equal(seen[0], seen[3]) and not torch.equal(seen[0], seen[1]) and not torch.equal(seen[1], seen[2])
    c.close()
