"""More evaluated cells than 32 bits hold, in the 1,024-row lists of the lane
tiers: the longest reads, of one base and of that base in 54 of 100 places,
whose band stays some 790 rows wide all along."""
import numpy as np
import pytest

import oracle
from helpers import rand_codes, workload_from
from test_gpu_parity import assert_same

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2001_10049_amd as xd  # noqa: E402


def test_cells_past_32_bits():
    n = 1 << 22
    j = np.arange(n, dtype=np.int64)
    a = np.zeros(n, np.uint8)
    b = np.where((j + 1) * 54 // 100 > j * 54 // 100, 0, 1).astype(np.uint8)
    c = rand_codes(np.random.default_rng(1), 400)
    w = workload_from([a, b, c, c.copy()], [(0, 1, 0, 0, 62), (2, 3, 200, 200, 62)])
    print("oracle", flush=True)
    ref = oracle.align_workload(w)
    assert ref["cells"][0] > 1 << 32
    print("lanes", flush=True)
    at = np.r_[0, np.ones(12_300, np.int64)]  # few of them, and the lane tiers run
    pairs, seeds, x = xd.workload_tensors(w.subset(at), "cuda")
    with xd.ReadStore.from_workload(w) as store:
        out = xd.align_batch(store, pairs, seeds, x=x, k=w.k, persistent=True)
        torch.cuda.synchronize()
        got = {k: v.cpu().numpy() for k, v in out.items()}
    assert_same(got, {k: ref[k][at] for k in got}, label="cells")
