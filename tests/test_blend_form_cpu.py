"""Which form of the prefill kernel a chunk of a layer that blends takes."""
import numpy as np
import pytest

import paper_2510_08525_amd as rl


@pytest.mark.parametrize("seed", range(4))
def test_form_by_rounds_of_workgroups(seed):
    rng = np.random.default_rng(seed)
    for _ in range(100):
        cu, group, n_full = int(rng.choice([64, 256, 304])), int(rng.integers(1, 17)), int(rng.integers(0, 9))
        tokens = rng.integers(0, int(rng.choice([40, 300, 2000])), size=int(rng.integers(1, 40)))
        rounds = [-(-sum(-(-int(t) // (cols // group)) for t in tokens) * n_full // cu) for cols in (256, 128)]
        assert rl.rlkv_plan_blend_form(cu, group, n_full, tokens) == (3 * rounds[1] < 5 * rounds[0])
        assert not rl.rlkv_plan_blend_form(cu, group, n_full, tokens, allow_narrow=False)


def test_rejects_bad_arguments():
    for bad in [(0, 4, 1, [5]), (256, 0, 1, [5]), (256, 17, 1, [5]), (256, 4, -1, [5]), (256, 4, 1, [-1]), (256, 4, 1, [])]:
        with pytest.raises(rl.RlkvError):
            rl.rlkv_plan_blend_form(*bad)
