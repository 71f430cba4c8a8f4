"""Packing four bytes at a time: every byte value as a base, quality thresholds
around the ends of a byte's range, read sets of any length modulo 64 and device
buffers at any alignment; against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from brute import assert_same_table

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(kh):
    c = kh.Context(0)
    yield c
    c.close()


def _set(rng, n, letters):
    seq = rng.choice(np.array(letters, np.uint8), n)
    qual = rng.integers(0, 256, n).astype(np.uint8)
    cuts = np.unique(np.concatenate([[0, n], rng.integers(0, n + 1, n // 40)])).astype(np.int64)
    return synth.Reads(seq, qual, cuts)


@pytest.mark.parametrize("offset,cutoff", [(0, 0), (33, 20), (0, 1), (64, 63), (64, 64), (100, 29),
                                           (128, 127), (200, 56), (0, 300)])
def test_thresholds(ctx, offset, cutoff):
    rng = np.random.default_rng(offset + cutoff)
    reads = _set(rng, 20_000, list(b"ACGT"))
    kw = dict(qual_offset=offset, qual_cutoff=cutoff)
    assert_same_table(ctx.count(reads, 5, **kw).to_numpy(), oracle.count(reads, 5, **kw))


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 1000, 4095, 4096, 4113])
def test_lengths_and_bytes(ctx, n):
    rng = np.random.default_rng(n)
    for letters in (list(b"ACGTacgt"), list(b"ACGTACGTACGTACGTN")):
        reads = _set(rng, n, letters)
        assert_same_table(ctx.count(reads, 3, min_count=1).to_numpy(),
                          oracle.count(reads, 3, min_count=1))
    every = _set(rng, n, list(b"ACGTacgt") * 60 + list(range(256)))
    assert_same_table(ctx.count(every, 3, min_count=1).to_numpy(),
                      oracle.count(every, 3, min_count=1))


@pytest.mark.parametrize("shift", [1, 2, 4, 7, 8, 15])
def test_alignment(kh, ctx, shift):
    import torch
    rng = np.random.default_rng(shift)
    reads = _set(rng, 5_003, list(b"ACGTACGTACGTN"))
    dev = kh.DeviceReads.from_host(reads)
    seq = torch.zeros(reads.n_bases + 32, dtype=torch.uint8, device="cuda")
    qual = torch.zeros_like(seq)
    seq[shift:shift + reads.n_bases] = dev.seq
    qual[16 - shift:16 - shift + reads.n_bases] = dev.qual
    moved = kh.DeviceReads(seq[shift:shift + reads.n_bases],
                           qual[16 - shift:16 - shift + reads.n_bases], dev.offsets)
    assert_same_table(ctx.count(moved, 21, min_count=1).to_numpy(),
                      oracle.count(reads, 21, min_count=1))
