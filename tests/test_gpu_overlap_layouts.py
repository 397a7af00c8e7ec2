"""The two layouts of the candidate stage's filters give the same result: by the
k-mers' smallest m-mers up to 2^27 words of the first filter, by the k-mers
themselves past that.  (On small sets test_gpu_overlap.py compares the first
with the oracle, for k from 1 to 31 and both strands.)"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2001_10049_amd as xd  # noqa: E402
import synth  # noqa: E402


@pytest.fixture(scope="module")
def store():
    # the c2 read set, every other read from the other strand
    w = synth.config("c2", n_tasks=1)
    codes = w.codes.copy()
    for o, n in zip(w.off[1::2], w.length[1::2]):
        codes[int(o):int(o) + int(n)] = 3 - codes[int(o):int(o) + int(n)][::-1]
    st = xd.ReadStore(codes, w.off, w.length)
    yield st
    st.close()


@pytest.mark.parametrize("k,m,strands", [(17, 8, 2), (31, 2, 2), (31, 8, 1), (12, 4, 1)])
def test_both_layouts(store, k, m, strands):
    out = []
    for bits in (16, 64):
        print("layout", k, m, strands, bits, flush=True)
        out.append(xd.find_overlaps(store, k=k, m=m, bloom_bits=bits, strands=strands))
        torch.cuda.synchronize()
        words = (out[-1]["counts"]["kmers"] * bits + 63) // 64
        assert (words > 1 << 27) == (bits == 64), words
    for key in ("pairs", "seed_off", "seeds") + (("rc",) if strands == 2 else ()):
        assert torch.equal(out[0][key], out[1][key]), key
    for key in ("kmers", "non_singletons", "retained", "occurrences", "pairs", "seeds"):
        assert out[0]["counts"][key] == out[1]["counts"][key], key
    assert out[0]["counts"]["pairs"] > 0
