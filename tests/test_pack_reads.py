"""xd_pack_reads around its 16-base steps: lengths at the edges of a word, an
unaligned start, and a code above 3 at every position (CPU only)."""
import numpy as np
import pytest

import paper_2001_10049_amd as xd


@pytest.mark.parametrize("start", [0, 1, 7])
def test_words_hold_the_codes(start):
    rng = np.random.default_rng(start)
    length = np.array([0, 1, 15, 16, 17, 31, 32, 33, 47, 48, 255, 256, 257], np.uint32)
    off = (start + np.concatenate([[0], np.cumsum(length)[:-1]])).astype(np.uint64)
    codes = rng.integers(0, 4, start + int(length.sum()), dtype=np.uint8)
    words, word_off = xd.pack_reads(codes, off, length)
    for r, n in enumerate(length):
        w = words[int(word_off[r]):]
        for u in range((int(n) + 255) // 256 * 256):  # zero-padded to 16 words
            want = codes[int(off[r]) + u] if u < n else 0
            assert (int(w[u // 16]) >> (2 * (u % 16))) & 3 == want, (r, u)


@pytest.mark.parametrize("bad", [4, 128, 255])
def test_a_code_above_3_names_its_base(bad):
    for at in range(50):
        codes = np.zeros(50, np.uint8)
        codes[at] = bad
        with pytest.raises(xd.XdropError, match="read 0 base %d: code %d > 3" % (at, bad)):
            xd.pack_reads(codes, [0], [50])
