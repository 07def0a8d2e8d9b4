"""Decode calls and steps whose scores are large: from 2^24 on a score in the log2 domain is a whole number, and its distance from the
product before rounding grows beyond what an exponential takes (128 from 2^31 on).  The row with the largest score has all the weight:
differences between rows are many times the rounding of a score, so that the output is that row's V to the tolerance of the type."""
import pytest

import paper_2510_08525_amd as rl
from harness import Case

pytestmark = pytest.mark.gpu

KINDS = [(rl.RLKV_BF16, rl.RLKV_KERNEL_MFMA), (rl.RLKV_F32, rl.RLKV_KERNEL_VALU), (rl.RLKV_BF16, rl.RLKV_KERNEL_VALU)]


@pytest.mark.parametrize("dtype,kernel", KINDS, ids=["mfma", "valu-f32", "valu-bf16"])
@pytest.mark.parametrize("scale", [1e6, 1e8, 1e9, -1e9, 1e30])
@pytest.mark.parametrize("Hq,Hkv,lengths", [(8, 2, [1, 1]), (14, 2, [64, 17]), (32, 2, [64, 17]), (8, 2, [1500, 700])],
                         ids=["one row", "64 group 7", "64 group 16", "shares"])
def test_the_largest_score_has_all_the_weight(gpu_device, Hq, Hkv, lengths, scale, dtype, kernel):
    c = Case(Hq=Hq, Hkv=Hkv, B=2, S=4, R=28, dtype=dtype, kernel=kernel, mask=[1, 0], cap=max(lengths) + 8, seed=12, scale=scale)
    c.append(lengths)
    c.check_decode(0, "decode")
    c.check_decode(1, "step", fused=True)
    c.check_decode(2, "step", fused=True)
    c.close()


@pytest.mark.parametrize("dtype,kernel", KINDS, ids=["mfma", "valu-f32", "valu-bf16"])
@pytest.mark.parametrize("q_scale", [1e10, -1e10, 1e25])
def test_large_queries(gpu_device, q_scale, dtype, kernel):
    c = Case(Hq=16, Hkv=2, B=2, S=4, R=28, dtype=dtype, kernel=kernel, mask=[1, 0], cap=80, seed=13, q_prescale=q_scale)
    c.append([1, 60])
    c.check_decode(0, "decode")
    c.check_decode(1, "step", fused=True)
    c.close()
