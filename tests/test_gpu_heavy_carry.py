"""K-mers of tens of thousands of occurrences and more, nearly all with the same
neighbour, in the paths that count in one table (whose spill tally of T lies next
to the mark that has such k-mers recounted): against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from brute import assert_same_table

pytestmark = pytest.mark.gpu


def _reads(k, times, base, back):
    """`times` copies of a canonical k-mer followed by `base` (back: of the other
    strand, which the base's complement precedes), and a few others."""
    rng = np.random.default_rng(k + times)
    mid = "".join(rng.choice(list("ACGT"), k - 2))
    one = "A" + mid + "G" + base
    if back:
        one = one[::-1].translate(str.maketrans("ACGT", "TGCA"))
    rest = "".join(rng.choice(list("ACGT"), 300))
    some = "".join(rng.choice(list("ACGT"), len(one)))
    flat = np.frombuffer((one * times + rest * 3 + some * 2).encode(), np.uint8).copy()
    lens = [len(one)] * times + [len(rest)] * 3 + [len(some)] * 2
    return synth.Reads(flat, np.full_like(flat, 73), np.concatenate([[0], np.cumsum(lens)]))


@pytest.fixture(scope="module")
def single(kh):
    c = kh.Context(0)
    c.set_tuning(partitioned=0)
    yield c
    c.close()


@pytest.mark.parametrize("back", [False, True])
@pytest.mark.parametrize("base", ["T", "G"])
@pytest.mark.parametrize("times", [32_000, 32_830, 32_832, 40_000, 65_535, 69_700, 100_000,
                                   135_000, 600_000])
def test_one_table(kh, single, times, base, back):
    k = 21
    reads = _reads(k, times, base, back)
    want = oracle.count(reads, k)
    assert int(want["counts"].max()) == times
    for bloom in (False, True):
        got = single.count(reads, k, use_bloom=bloom)
        assert_same_table(got.to_numpy(), want)
        got.free()


@pytest.mark.parametrize("k", [33, 77, 127])
@pytest.mark.parametrize("times", [40_000, 70_000])
def test_wide_keys(single, times, k):
    reads = _reads(k, times, "T", False)
    assert_same_table(single.count(reads, k).to_numpy(), oracle.count(reads, k))


@pytest.mark.parametrize("times", [40_000, 100_000, 400_000])
def test_no_allocation(kh, times):
    import torch
    k = 21
    reads = _reads(k, times, "T", False)
    want = oracle.count(reads, k)
    n = want["n_rows"]
    out = [torch.zeros((n + 8,) + s, dtype=d, device="cuda")
           for s, d in (((1,), torch.int64), ((), torch.int32), ((8,), torch.int32),
                        ((2,), torch.uint8))]
    rows, _ = kh.count_noalloc(kh.DeviceReads.from_host(reads), k, *out)
    assert rows == n
    np.testing.assert_array_equal(out[1][:n].cpu().numpy(), want["counts"])
    np.testing.assert_array_equal(out[2][:n].cpu().numpy(), want["ext"])


@pytest.mark.parametrize("k", [21, 77])
@pytest.mark.parametrize("times", [40_000, 100_000, 130_000])
def test_aggregated(kh, times, k):
    c = kh.Context(0)
    try:
        c.set_tuning(aggregate=1)
        reads = _reads(k, times, "T", False)
        assert_same_table(c.count(reads, k, use_bloom=True).to_numpy(), oracle.count(reads, k))
    finally:
        c.close()


def test_served_in_batches(kh):
    """The count grows over several batches of a sample, past the table's growth."""
    reads = _reads(21, 90_000, "T", False)
    srv = kh.Server([21])
    try:
        for a in range(0, reads.n_reads, 11_000):
            srv.wait(srv.submit(0, reads.slice(a, min(a + 11_000, reads.n_reads))))
        (table,) = srv.finalize(0)
        assert_same_table(table.to_numpy(), oracle.count(reads, 21))
        table.free()
    finally:
        srv.close()
