"""Rows that do not count reach no sum, whatever they hold: an Inf in V at a position outside the sink and the recent range stays out of
the local attention of a blending head (it reaches the output through the full attention alone), and an Inf in the last row of a store
is not met again with weight zero by the rows behind it.  Row-major stores; the call and the step give the same."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_08525_amd as rl
from harness import Case, to_np, tolerance

pytestmark = pytest.mark.gpu

KINDS = [(rl.RLKV_F32, rl.RLKV_KERNEL_VALU), (rl.RLKV_BF16, rl.RLKV_KERNEL_VALU)]


def check(c, out, q, gates, column, label):
    got = out.float().cpu().numpy().astype(np.float64)
    assert (got[..., column] == np.inf).all(), f"{label}: {got[..., column]}"
    kv = to_np(c.k_hist), np.where(np.isinf(to_np(c.v_hist)), 0, to_np(c.v_hist)) if c.dtype == rl.RLKV_F32 else to_np(
        torch.where(c.v_hist.isinf(), 0, c.v_hist))
    ref = oracle.decode_attention_gated(*kv, c.n, [float(g) for g in gates], to_np(q), c.S, c.R, c.scale)
    err = np.abs(got - ref)
    err[..., column] = 0
    assert (err <= tolerance(ref, c.dtype)).all(), f"{label}: max err {err.max():.3e}"


@pytest.mark.parametrize("dtype,kernel", KINDS, ids=["f32", "bf16"])
@pytest.mark.parametrize("group", [4, 7, 16])
@pytest.mark.parametrize("n,row,gates", [
    (200, 9, [0.25, 0.75]),          # behind the sink, in a batch with it
    (200, 168, [0.25, 0.75]),        # just ahead of the recent range
    (3000, 9, [0.25, 0.75]), (3000, 2968, [0.25, 0.75]),
    (201, 200, [1.0, 1.0]), (3001, 3000, [1.0, 1.0]),      # the last row of a ragged batch
], ids=lambda x: str(x))
def test_inf_in_a_row_that_does_not_count(gpu_device, n, row, gates, group, dtype, kernel):
    c = Case(Hq=2 * group, Hkv=2, B=1, S=8, R=30, dtype=dtype, kernel=kernel, mask=[1, 1], cap=n + 4, seed=14)
    column = 77
    c.v_hist[:, :, row, column] = float("inf")
    c.cache.set_gates(np.asarray(gates, np.float32))
    c.append([n])
    q, out = c.decode(0)
    check(c, out, q, gates, column, "decode")
    c.cache.reset()
    c.n[:] = 0
    c.append([n - 1])
    q, out = c.append_decode(0)
    check(c, out, q, gates, column, "step")
    c.close()
