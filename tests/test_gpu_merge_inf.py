"""An Inf in a partial is merged as it is: the merges take partials four at a time, and what stands in for those beyond a pair's last
one may not be a partial with weight zero (0 x Inf = NaN).  Any number of partials, merged in the launch and by a merge launch."""
import numpy as np
import pytest
import torch

import paper_2510_08525_amd as rl
from harness import Case

pytestmark = pytest.mark.gpu

KINDS = [(rl.RLKV_BF16, rl.RLKV_KERNEL_MFMA), (rl.RLKV_F32, rl.RLKV_KERNEL_VALU), (rl.RLKV_BF16, rl.RLKV_KERNEL_VALU)]


@pytest.mark.parametrize("dtype,kernel", KINDS, ids=["mfma", "valu-f32", "valu-bf16"])
@pytest.mark.parametrize("gate", [None, 0.5], ids=["plain", "blending"])
@pytest.mark.parametrize("n", [600, 700, 1000, 1500, 2600])
def test_inf_of_the_first_partial(gpu_device, n, gate, dtype, kernel):
    """The sum of one column over the first 64 rows is beyond the range of fp32 (as is the tiled kernel's, whose weights come in two
    parts of either sign, so that a V of Inf would be NaN there by itself): Inf, in that column alone."""
    c = Case(Hq=4, Hkv=1, B=1, S=80, R=30, dtype=dtype, kernel=kernel, mask=[1], cap=n + 4, seed=15, sink_keys=False)
    c.k_hist[:, :, :64] = 0
    c.v_hist[:, :, :64, 33] = 3e38
    if gate is not None:
        c.cache.set_gates(np.asarray([gate], np.float32))
    c.append([n])
    q = (0.01 * c.make_q(0).float()).to(c.tdtype).to(c.device)
    out = torch.zeros_like(q)
    c.cache.decode_attention(0, q, out, c.scale)
    recorded = torch.zeros_like(q)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        c.cache.decode_attention(0, q, recorded, c.scale)
    graph.replay()
    torch.cuda.synchronize()
    for what, got in (("call", out), ("replay", recorded)):
        got = got.float()
        assert (got[..., 33] == float("inf")).all(), f"{what}: {got[..., 33]}"
        got[..., 33] = 0
        assert torch.isfinite(got).all(), what
    c.close()
