"""Banded scores on both sides of the line between two tasks to a wavefront and
one: match times the store's mean read length up to 16 bits, and past it, with
tasks of either kind, refused ones and bands outside the grid in both."""
import numpy as np
import pytest

from test_gpu_banded import assert_same, run
from test_gpu_banded_pair import mixed

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", [(1, -1, -1), (100, -90, -127), (127, -1, -1)])
@pytest.mark.parametrize("mean", [400, 660, 1500])
def test_long_reads(scheme, mean):
    w = mixed(mean, 203, mean - 300, mean + 300)
    rng = np.random.default_rng(mean)
    got, ref = run(w, rng.integers(0, 49, w.n_tasks).astype(np.int32), scheme)
    print(scheme, mean, scheme[0] * int(w.length.mean()), flush=True)
    assert_same(got, ref, "%s %d" % (scheme, mean))
