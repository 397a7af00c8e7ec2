"""The seed sort's two forms around the limit between them (64 bits for two read
ids, two positions and, on both strands, a flag): read sets whose longest read
and number of reads set those bits, against the oracle."""
import numpy as np
import pytest

from helpers import mutate_codes, rand_codes
from oracle import overlap as ov

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2001_10049_amd as xd  # noqa: E402


# (reads, longest read): 2 * (17 + 15) = 64 bits, 2 * (17 + 16) = 66, 2 * (8 + 12) = 40
@pytest.mark.parametrize("strands", [1, 2])
@pytest.mark.parametrize("n_reads,longest", [(70_000, 32_000), (70_000, 65_000), (200, 4_000)])
def test_bits(n_reads, longest, strands):
    print("sort", n_reads, longest, strands, flush=True)
    rng = np.random.default_rng(longest + strands)
    genome = rand_codes(rng, longest)
    reads = [genome]
    for q in range(60):
        p = int(rng.integers(0, longest - 2000))
        r = mutate_codes(rng, genome[p:p + int(rng.integers(40, 2000))], 0.05)
        reads.append(3 - r[::-1] if q % 3 == 0 else r)
    few = len(reads) - 20
    reads = reads[:few] + [np.zeros(0, np.uint8)] * (n_reads - len(reads)) + reads[few:]
    length = np.array([len(r) for r in reads], np.uint32)
    off = np.concatenate([[0], np.cumsum(length)[:-1]]).astype(np.uint64)
    codes = np.concatenate(reads).astype(np.uint8)
    ref = ov.find_overlaps(codes, off, length, 17, 2, 8, strands)
    with xd.ReadStore(codes, off, length) as st:
        got = xd.find_overlaps(st, k=17, m=8, strands=strands)
    torch.cuda.synchronize()
    u = lambda t, d: t.cpu().numpy().view(d)  # noqa: E731
    pairs, seed_off, seeds = ref[:3]
    if strands == 2:
        assert np.array_equal(u(got["rc"], np.uint8), ref[4])
    assert len(pairs) > 50 and (np.asarray(pairs)[:, 1] >= n_reads - 20).any()
    assert np.array_equal(u(got["pairs"], np.uint32).reshape(-1, 2), pairs)
    assert np.array_equal(u(got["seed_off"], np.uint64), seed_off)
    assert np.array_equal(u(got["seeds"], np.uint32).reshape(-1, 2), seeds)
