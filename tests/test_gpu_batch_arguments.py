"""Token counts of ragged calls: in the kernels' arguments up to 128 sequences, written to the arena by a kernel beyond
(512 values per launch).  Sizes on both sides of both limits; also the work lists of these batches."""
import numpy as np
import pytest

import paper_2510_08525_amd as rl
from harness import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [128, 129, 300])
def test_ragged_counts_of_large_batches(gpu_device, B):
    rng = np.random.default_rng(B)
    c = Case(Hq=2, Hkv=2, B=B, S=2, R=9, dtype=rl.RLKV_BF16, kernel=rl.RLKV_KERNEL_MFMA, mask=[1, 0], cap=64, seed=3,
             prefill_tokens=32, arena_fill=0xFF)
    c.append(rng.integers(1, 20, B))
    c.check_indices()
    counts = rng.integers(0, 33, B)
    counts[0], counts[-1] = 32, 0
    c.check_prefill(counts, 0, "ragged chunk")
    c.check_indices()
    c.check_decode(0, "fused step", fused=True)
    c.close()
