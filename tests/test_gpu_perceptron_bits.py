"""GPU: the perceptron's results are those recorded before its second-layer products moved to the matrix cores, bit for
bit (tests/golden/make_perceptron_bits.py): a sum that rounds differently moves bf16 values next to a rounding boundary,
and momentum and the bf16 shadow carry such a step on."""
import os
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, "golden"))
from make_perceptron_bits import CASES, name, results  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", CASES)
def test_perceptron_keeps_the_recorded_bits(case):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1710_06952_amd as P
    print("perceptron bits %s" % name(case), flush=True)
    with np.load(os.path.join(HERE, "golden", "perceptron_bits.npz")) as rec:
        for k, v in results(P, case).items():
            want = rec[name(case) + "/" + k]
            assert v.dtype == want.dtype and np.array_equal(v, want), k
