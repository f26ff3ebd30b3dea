"""The backward's two pre-pass jobs at the sizes where their plan changes: one launch or partial sums, 64 x 64 or 128 x
128 tiles, K chunks that end ragged in the longer and in the shorter job.  Each output alone keeps the full call's bits
(the plan looks at both jobs whichever run).  Tolerances: the arithmetic bound of the other backward tests."""
import numpy as np
import pytest

import workloads as WL
from oracle import lora_linear_backward_ref
from gpu_helpers import assert_rel, say
from test_gpu_backward import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,r", [
    (2048, 72, 40, 16), (2049, 72, 40, 16),    # the last rows of one launch, the first of partial sums
    (1024, 40, 72, 20), (520, 72, 40, 100),    # the same at ranks 32 and 128
    (300, 2056, 264, 128), (300, 264, 2056, 100),  # 64 x 64 tiles, six ragged chunks and one, in either job
    (1000, 1032, 520, 64),                     # five and three
    (4100, 264, 1032, 128),                    # 128 x 128 tiles, three and one
])
def test_backward_plans(M, K, N, r, dev):
    say("backward plan", M, K, N, r)
    case = WL.gen_backward(1200 + M + K + r, M, K, N, r)
    c = case.lin
    full = _run(case, dev)
    for got, want, name in zip(full, lora_linear_backward_ref(c.x, c.W, c.A, c.B, c.s, case.dy), ("dx", "dA", "dB")):
        assert_rel(got, want, name)
    for i, name in enumerate(("dx", "dA", "dB")):
        assert np.array_equal(_run(case, dev, want=(name,))[i], full[i]), name
