"""Which lists of shares merge their partials inside the attention launch, without a GPU: both sides of every line, and that the lists of
the device tests lie where those say."""
import pytest

import paper_2510_08525_amd as rl
from list_plan import plan

MFMA, VALU, BF16, F32 = rl.RLKV_KERNEL_MFMA, rl.RLKV_KERNEL_VALU, rl.RLKV_BF16, rl.RLKV_F32


# (kernel, group, gated, workgroups used of 256, most partials): merged inside
@pytest.mark.parametrize("case,expected", [
    ((MFMA, 4, 0, 256, 32), 1), ((MFMA, 4, 0, 256, 33), 0), ((VALU, 8, 0, 256, 32), 1), ((VALU, 8, 0, 256, 33), 0),
    ((VALU, 9, 0, 20, 4), 0), ((VALU, 16, 1, 20, 4), 0), ((VALU, 8, 1, 20, 4), 1),
    ((MFMA, 8, 1, 128, 16), 1), ((MFMA, 8, 1, 129, 16), 0), ((MFMA, 8, 1, 128, 17), 0),
    ((MFMA, 9, 0, 128, 16), 1), ((MFMA, 9, 0, 129, 16), 0), ((MFMA, 16, 0, 128, 17), 0), ((VALU, 4, 1, 128, 17), 0),
], ids=lambda x: str(x))
def test_lines(case, expected):
    kernel, group, gated, used, partials = case
    assert rl.load_library().rlkv_plan_merge_inside(kernel, group, gated, 256, used, partials) == expected


def test_invalid_arguments():
    for bad in [(7, 4, 0, 256, 20, 4), (MFMA, 0, 0, 256, 20, 4), (MFMA, 17, 0, 256, 20, 4), (MFMA, 4, 0, 0, 20, 4), (MFMA, 4, 0, 256, 0, 4),
                (MFMA, 4, 0, 256, 257, 4), (MFMA, 4, 0, 256, 20, 0)]:
        assert rl.load_library().rlkv_plan_merge_inside(*bad) == -1


@pytest.mark.parametrize("dtype,kernel,n,partials", [
    (BF16, MFMA, 900, 8), (BF16, MFMA, 1400, 11), (BF16, MFMA, 2010, 16), (BF16, MFMA, 4100, 17), (BF16, MFMA, 7900, 32), (BF16, MFMA, 8100, 33),
    (F32, VALU, 900, 15), (F32, VALU, 1400, 22), (F32, VALU, 2010, 32), (F32, VALU, 4100, 17), (F32, VALU, 7900, 32), (F32, VALU, 8100, 33)])
def test_partials_of_the_device_tests(dtype, kernel, n, partials):
    whole, used, most, inside = plan(dtype, kernel, 4, [1, 0], 8, 56, [n], n + 8)
    assert not whole and most == partials and inside == (partials <= 32) and used == partials + 1
