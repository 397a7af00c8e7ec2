"""The filters' layouts by the k-mers' smallest m-mers: a filter only decides
which k-mers are counted, so every k, from one m-mer to a k-mer up to six, both
strands and every filter size have to give the same result; past 2^27 words the
first filter goes by the k-mers themselves."""
import numpy as np
import pytest

from helpers import mutate_codes, rand_codes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2001_10049_amd as xd  # noqa: E402
import synth  # noqa: E402


@pytest.fixture(scope="module")
def store():
    rng = np.random.default_rng(5)
    genome = rand_codes(rng, 700_000)
    genome[1000:3000] = 0  # runs of one base, and a tandem repeat
    genome[5000:9000] = np.resize(np.array([0, 1, 3], np.uint8), 4000)
    reads = []
    for q in range(900):
        p = int(rng.integers(0, 690_000))
        r = genome[p:p + 10_000].copy()
        hit = rng.integers(0, r.size, 300)
        r[hit] = rng.integers(0, 4, 300)
        reads.append(3 - r[::-1] if q % 2 else r)
    reads += [mutate_codes(rng, genome[:500], 0.1), rand_codes(rng, 31), rand_codes(rng, 17)]
    length = np.array([len(r) for r in reads], np.uint32)
    off = np.concatenate([[0], np.cumsum(length)[:-1]]).astype(np.uint64)
    st = xd.ReadStore(np.concatenate(reads).astype(np.uint8), off, length)
    yield st
    st.close()


@pytest.mark.parametrize("strands", [1, 2])
@pytest.mark.parametrize("k", [1, 10, 11, 12, 15, 16, 17, 31])
def test_layouts_agree(store, k, strands):
    print("lines k", k, "strands", strands, flush=True)
    out = [xd.find_overlaps(store, k=k, m=8, bloom_bits=b, strands=strands) for b in (16, 64)]
    torch.cuda.synchronize()
    for key in ("pairs", "seed_off", "seeds") + (("rc",) if strands == 2 else ()):
        assert torch.equal(out[0][key], out[1][key]), key
    for key in ("kmers", "non_singletons", "retained", "occurrences", "pairs", "seeds"):
        assert out[0]["counts"][key] == out[1]["counts"][key], key
    assert out[0]["counts"]["kmers"] * 64 >= 8 * (4 << 20) * 16
    if k >= 15:
        assert out[0]["counts"]["pairs"] > 100


def test_large_filter():
    w = synth.config("c2", n_tasks=1)
    with xd.ReadStore.from_workload(w) as st:
        out = [xd.find_overlaps(st, k=17, m=8, bloom_bits=b) for b in (16, 64)]
        torch.cuda.synchronize()
    assert out[1]["counts"]["kmers"] > 1 << 27  # a word for each at 64 bits
    for key in ("pairs", "seed_off", "seeds"):
        assert torch.equal(out[0][key], out[1][key]), key
    for key in ("non_singletons", "retained", "occurrences"):
        assert out[0]["counts"][key] == out[1]["counts"][key], key
    assert out[0]["counts"]["pairs"] == 803126
