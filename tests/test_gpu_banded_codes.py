"""Banded alignment paths on both sides of the rule that chooses how a step's
code is found: with the values (match - mismatch up to 63) or by comparisons."""
import numpy as np
import pytest

from test_gpu_banded_pair import mixed
from test_gpu_banded_trace import assert_same, gpu_trace, oracle_trace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", [(1, -1, -1), (1, -62, -1), (1, -63, -1), (31, -32, -5),
                                    (32, -32, -5), (63, 0, -127), (2, 1, -1), (127, -127, -127)])
@pytest.mark.parametrize("lo,hi", [(17, 90), (190, 400)])
def test_codes(scheme, lo, hi):
    rng = np.random.default_rng(hi)
    w = mixed(hi, 203, lo, hi)
    ws = rng.integers(0, 49, w.n_tasks).astype(np.int32)
    assert_same(gpu_trace(w, ws, scheme), oracle_trace(w, ws, scheme), "%s" % (scheme,))
