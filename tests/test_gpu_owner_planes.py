"""The routing planes and rolled windows of the owner-partitioned count where
they can go wrong: k around the widths of words, planes and digits, read ends
and non-bases at every offset of a 64-position word, reads across tile edges,
and key-space parts of any count; against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from brute import assert_same_table

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def octx(kh):
    c = kh.Context(0)
    yield c
    c.close()


def _reads(rng, n, lo, hi, genome=4000):
    g = "".join(rng.choice(list("ACGT"), genome))
    pairs = []
    for _ in range(n):
        m = int(rng.integers(lo, hi + 1))
        a = int(rng.integers(0, genome - m + 1))
        s = list(g[a:a + m])
        for i in range(m):
            u = rng.random()
            if u < 0.004:
                s[i] = "N"
            elif u < 0.008:
                s[i] = "acgt"[int(rng.integers(0, 4))]
        pairs.append(("".join(s), "".join(chr(33 + int(x)) for x in rng.integers(2, 42, m))))
    return synth.Reads.from_strings(pairs)


@pytest.mark.parametrize("k", [1, 3, 5, 7, 29, 31, 33, 35, 37, 63, 65, 67, 69, 95, 97, 99, 101, 125, 127])
def test_every_width(octx, k):
    rng = np.random.default_rng(k)
    reads = _reads(rng, 400, 1, 300)
    assert_same_table(octx.count(reads, k).to_numpy(), oracle.count(reads, k))


@pytest.mark.parametrize("n", [63, 64, 65, 4095, 4096, 4097, 4096 + 126, 4096 + 127, 8192, 12289])
def test_tile_edges(octx, n):
    """One read (and two) of n bases: windows that end at and cross tile edges."""
    rng = np.random.default_rng(n)
    s = "".join(rng.choice(list("ACGT"), n))
    for parts in ([s, s], [s[:n // 2], s[n // 2:], s]):
        reads = synth.Reads.from_strings([(x, "I" * len(x)) for x in parts])
        for k in (21, 63):
            assert_same_table(octx.count(reads, k, min_count=1).to_numpy(),
                              oracle.count(reads, k, min_count=1))


@pytest.mark.parametrize("shards", [2, 3, 7, 8, 1000, 4294967295])
def test_parts(kh, octx, shards):
    rng = np.random.default_rng(shards % 1000)
    reads = _reads(rng, 150, 60, 200, genome=1500)
    for k in (21, 33, 77, 99):
        whole = oracle.count(reads, k)
        parts = np.array([kh.owner_of(x, shards) for x in whole["keys"]], np.uint64)
        for part in {0, shards - 1, int(parts[0])} if shards > 8 else range(shards):
            got = octx.count(reads, k, owner_shards=shards, owner=int(part)).to_numpy()
            np.testing.assert_array_equal(got["keys"], whole["keys"][parts == part])
            np.testing.assert_array_equal(got["counts"], whole["counts"][parts == part])
            np.testing.assert_array_equal(got["ext"], whole["ext"][parts == part])
