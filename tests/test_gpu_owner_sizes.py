"""Owners at the edges of what the in-LDS count holds: an owner's records up to
and past a block's share, every key a row, every key twice, one key many times
(past 16-bit tallies), and owners of one record; against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from brute import assert_same_table

pytestmark = pytest.mark.gpu

# records an owner may hold, by record words (k = 21, 55, 77, 99)
RECORDS = {21: 4608, 55: 3584, 77: 2560, 99: 2048}


@pytest.fixture(scope="module")
def octx(kh):
    c = kh.Context(0)
    assert c.tuning()["partitioned"] == 1
    yield c
    c.close()


def _one_owner(rng, k, n):
    """n distinct k-mers that share their first 12 bases and are canonical as
    they stand (they start with A and end in G)."""
    seen = set()
    while len(seen) < n:
        seen.add("AAAAACCGGACA" + "".join(rng.choice(list("ACGT"), k - 13)) + "G")
    return sorted(seen)


def _reads(kmers, rng):
    order = rng.permutation(len(kmers))
    return synth.Reads.from_strings([(kmers[i], "I" * len(kmers[i])) for i in order])


@pytest.mark.parametrize("k", sorted(RECORDS))
@pytest.mark.parametrize("extra", [-1, 0, 1, 700])
def test_every_key_twice(octx, k, extra):
    rng = np.random.default_rng(k)
    n = RECORDS[k] // 2 + extra
    reads = _reads(_one_owner(rng, k, n) * 2, rng)
    want = oracle.count(reads, k)
    assert want["n_rows"] == n
    for bloom in (False, True):
        assert_same_table(octx.count(reads, k, use_bloom=bloom).to_numpy(), want)


@pytest.mark.parametrize("k", sorted(RECORDS))
@pytest.mark.parametrize("extra", [-1, 0, 1])
def test_every_record_a_row(octx, k, extra):
    rng = np.random.default_rng(100 + k)
    reads = _reads(_one_owner(rng, k, RECORDS[k] // 2 + extra), rng)
    assert_same_table(octx.count(reads, k, min_count=1).to_numpy(),
                      oracle.count(reads, k, min_count=1))


@pytest.mark.parametrize("k", sorted(RECORDS))
@pytest.mark.parametrize("extra", [0, 1])
def test_distinct_keys_fill_an_owner(octx, k, extra):
    """As many distinct keys as records (the slots' fullest), few of them rows."""
    rng = np.random.default_rng(200 + k)
    kmers = _one_owner(rng, k, RECORDS[k] + extra - 40)
    reads = _reads(kmers + kmers[:40], rng)
    st = octx.count(reads, k, use_bloom=True)
    assert st.info()["n_rows"] == 40
    assert_same_table(st.to_numpy(), oracle.count(reads, k))


@pytest.mark.parametrize("k", sorted(RECORDS))
@pytest.mark.parametrize("times", [1.01, 1.6, 2.5, 6])
def test_distinct_keys_past_an_owner(octx, k, times):
    """Without the screen, several times an owner's records of distinct keys
    (one key beside them many times): counted in parts; at 6 times the parts
    of short keys do not fit either, which takes the single table."""
    rng = np.random.default_rng(300 + k)
    kmers = _one_owner(rng, k, int(times * RECORDS[k]))
    reads = _reads(kmers + kmers[:40] + kmers[50:51] * 3000, rng)
    table = octx.count(reads, k, use_bloom=False)
    st = octx.stats()
    assert_same_table(table.to_numpy(), oracle.count(reads, k))
    if times < 6:
        assert (st["rebuilds"], st["claimed"], st["passed"]) == (0, len(kmers), len(kmers) + 3040)


@pytest.mark.parametrize("times", [4096, 65535, 65536, 70000])
def test_one_key_many_times(octx, times):
    """A homopolymer run: one key `times` times beside others of its owner."""
    k = 31
    rng = np.random.default_rng(times)
    others = ["A" * 12 + "".join(rng.choice(list("ACG"), 19)) for _ in range(50)]
    reads = synth.Reads.from_strings([("A" * (times + k - 1), "I" * (times + k - 1))]
                                     + [(s, "I" * k) for s in others * 3])
    want = oracle.count(reads, k)
    assert int(want["counts"].max()) == times
    for bloom in (False, True):
        assert_same_table(octx.count(reads, k, use_bloom=bloom).to_numpy(), want)
