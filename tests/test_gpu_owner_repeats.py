"""Owners of very many records of few keys (runs of one base, tandem repeats, a
small genome sequenced thousands of times over), unscreened: the rows are those
of the screened count and of the oracle, and the call takes no longer than the
screened one by much (1.5 times, with every such owner counted in parts)."""
import time

import numpy as np
import pytest

import oracle
import synth
from brute import assert_same_table

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def octx(kh):
    c = kh.Context(0)
    assert c.tuning()["partitioned"] == 1
    yield c
    c.close()


def _reads(n, repeats, length=150, seed=1):
    """n reads of a random genome, but the first `repeats` of them of one base
    or of one three-base unit."""
    rng = np.random.default_rng(seed)
    genome = rng.integers(0, 4, n * length // 8)
    at = rng.integers(0, genome.size - length, n)
    seq = np.frombuffer(b"ACGT", np.uint8)[genome[at[:, None] + np.arange(length)]]
    seq[:repeats // 2] = ord("A")
    seq[repeats // 2:repeats] = np.frombuffer(b"CAG" * length, np.uint8)[:length]
    return seq.reshape(-1).copy(), np.arange(n + 1, dtype=np.int64) * length


@pytest.mark.parametrize("k", [1, 3, 7, 21, 55])
def test_repeats_unscreened(octx, k):
    seq, off = _reads(6000, 3000)
    reads = synth.Reads(seq, np.full_like(seq, 73), off)
    want = oracle.count(reads, k)
    for bloom in (False, True):
        assert_same_table(octx.count(reads, k, use_bloom=bloom).to_numpy(), want)


@pytest.mark.parametrize("times", [1.1, 2.5])
def test_repeated_and_distinct_owners(octx, times):
    """600 big owners, every other one (in no order) of 40 keys, the others of
    distinct keys: more than one of either kind for a block, which tries owners
    whole by what its last one held."""
    k, owners, n = 21, 600, int(times * 4608)
    rng = np.random.default_rng(int(10 * times))
    # AAAAA, five bases that name the owner, ten of the key, G: canonical, one
    # k-mer a read
    code = np.zeros((owners, n, k), np.uint8)
    ident = rng.permutation(1024)[:owners]
    for j in range(5):
        code[:, :, 5 + j] = (ident >> (2 * (4 - j)) & 3)[:, None]
    key = rng.integers(0, 4 ** 10, (owners, n))
    key[::2] = key[::2, :40][np.arange(owners // 2)[:, None], rng.integers(0, 40, n)]
    for j in range(10):
        code[:, :, 10 + j] = key >> (2 * j) & 3
    code[:, :, 20] = 2
    seq = np.frombuffer(b"ACGT", np.uint8)[code.reshape(-1, k)]
    seq = seq[rng.permutation(len(seq))].reshape(-1).copy()
    reads = synth.Reads(seq, np.full_like(seq, 73), np.arange(owners * n + 1, dtype=np.int64) * k)
    want = oracle.count(reads, k)
    assert want["n_rows"] > owners * 20
    assert_same_table(octx.count(reads, k, use_bloom=False).to_numpy(), want)


def test_repeats_take_no_parts(kh, octx):
    import torch
    seq, off = _reads(500_000, 100_000)
    seq = torch.from_numpy(seq).cuda()
    reads = kh.DeviceReads(seq, torch.full_like(seq, 73), torch.from_numpy(off).cuda())

    def best(bloom):
        times = []
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            octx.count(reads, 21, use_bloom=bloom).free()
            times.append(time.perf_counter() - t0)
        return min(times)

    assert best(False) < 1.2 * best(True)
