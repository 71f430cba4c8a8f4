"""The single-table path's export sort at the edges of its ways: sets ranked in
one launch (up to 16,384 rows), segments of every length, buckets longer than a
segment, and many keys sharing their top 20 bases; against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from brute import assert_same_table

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sctx(kh):
    c = kh.Context(0)
    c.set_tuning(partitioned=0)
    yield c
    c.close()


def _distinct(rng, n, k, letters="ACGT", prefix=""):
    """n reads of one window each, keys of random order."""
    return synth.Reads.from_strings(
        [(prefix + "".join(s), "I" * k) for s in rng.choice(list(letters), (n, k - len(prefix)))])


@pytest.mark.parametrize("k", [21, 25, 31, 33, 65])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 4097, 16383, 16384, 16385, 16500])
def test_small_sets(sctx, k, n):
    rng = np.random.default_rng(n + k)
    reads = _distinct(rng, n, k)
    assert_same_table(sctx.count(reads, k, min_count=1).to_numpy(),
                      oracle.count(reads, k, min_count=1))


@pytest.mark.parametrize("letters,n", [("ACGT", 300_000), ("AAACGTTT", 120_000),
                                       ("AAAAAAACG", 250_000)])
@pytest.mark.parametrize("k", [21, 33])
def test_segments(sctx, k, letters, n):
    """Even and crowded prefixes: the fullest bucket picks the segment length,
    the last case holds buckets no segment holds."""
    rng = np.random.default_rng(n)
    reads = _distinct(rng, n, k, letters)
    assert_same_table(sctx.count(reads, k, min_count=1).to_numpy(),
                      oracle.count(reads, k, min_count=1))


@pytest.mark.parametrize("n", [50, 3000, 30_000])
def test_shared_prefix(sctx, n):
    """n keys whose first 24 bases agree (the sort key is the first 20)."""
    rng = np.random.default_rng(n)
    reads = _distinct(rng, n, 55, "ACGT", "AAAACCCCGGGGAAAACCCCGGGG")
    t = sctx.count(reads, 55, min_count=1)
    assert sctx.stats()["full_key_sort"] == int(n > 64)
    assert_same_table(t.to_numpy(), oracle.count(reads, 55, min_count=1))
