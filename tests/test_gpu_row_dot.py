"""Scores of the row-major fp32 kernel: a block of the matrix instruction sums 16 neighbouring columns of a row in four sums of four, which
are added last, and the eight blocks of a row are added after that.  One chain over the 16 would lose what is below half an ulp of a large
product ahead of it, element by element; so would one over columns of several blocks.  A group of one or two heads sums four neighbouring
columns in a lane of the vector ALU, and the lanes of a row after that."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_08525_amd as rl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group", [1, 2, 3])
@pytest.mark.parametrize("fused", [False, True], ids=["decode", "fused step"])
@pytest.mark.parametrize("big,small", [(0, 64), (23, 84), (63, 124),               # in another block
                                       (0, 4), (16, 28), (17, 24), (50, 60), (112, 124)])      # in another four columns of the same one
def test_small_products_behind_a_large_one(gpu_device, big, small, fused, group):
    """q . k = 2048 + 4 x 2^-13 for one key and 2048 for the other.  Each small product is half an ulp of 2048, which a chain
    behind 2048 rounds away (to even); their own sum is two ulps, so that both scores are exact in fp32.  The scale, ln 2,
    makes the factor on the scores exactly 1, so nothing else is rounded before the exponentials (of 0 and 2^-11, 1 ulp each).
    A lost sum moves the output, v0 - v1 = 2 times a weight of slope 1/4, by 2^-11 ln 2 / 2 = 1.7e-4; what is left is a few
    roundings of values up to 1: 1e-6."""
    D, n, scale = 128, 2, float(np.log(2.0))
    k = np.zeros((1, 1, n, D), np.float32)
    v = np.zeros_like(k)
    q = np.zeros((1, group, D), np.float32)
    q[0, :, big] = 1.0
    k[0, 0, :, big] = 2048.0
    q[0, :, small:small + 4] = 1.0
    k[0, 0, 0, small:small + 4] = 2.0 ** -13
    v[0, 0, 0], v[0, 0, 1] = 1.0, -1.0
    c = rl.Cache(1, group, 1, D, 1, 4, 28, rl.RLKV_F32, [1], [8], kernel=rl.RLKV_KERNEL_VALU)
    put = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(gpu_device)
    out = torch.zeros(1, group, D, device=gpu_device)
    if fused:
        c.append(0, put(k[:, :, :1]), put(v[:, :, :1]))
        c.append_decode(0, put(k[:, :, 1:]), put(v[:, :, 1:]), put(q), out, scale)
    else:
        c.append(0, put(k), put(v))
        c.decode_attention(0, put(q), out, scale)
    torch.cuda.synchronize()
    ref = oracle.decode_attention(k, v, np.asarray([n]), [1], q, 4, 28, scale)
    err = np.abs(out.cpu().numpy().astype(np.float64) - ref)
    assert err.max() <= 1e-6, f"max err {err.max():.3e}"
    c.close()
