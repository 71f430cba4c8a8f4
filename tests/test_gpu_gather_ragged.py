"""Gathered reads of every short length (the copy moves 16-byte pieces at any
alignment, the last of them over the one before) equal the input's reads."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths", [list(range(0, 70)), [0, 0, 1, 0], [255, 256, 257, 271, 272, 1000]])
def test_gather_ragged(kh, lengths):
    import torch
    rng = np.random.default_rng(len(lengths))
    lens = np.array(lengths * 3)
    rng.shuffle(lens)
    pairs = [("".join(rng.choice(list("ACGTN"), n)), "".join(chr(33 + int(x)) for x in
              rng.integers(2, 42, n))) for n in lens]
    reads = synth.Reads.from_strings(pairs)
    ctx = kh.Context(0)
    dev = kh.DeviceReads.from_host(reads)
    order = rng.permutation(reads.n_reads)
    got = ctx.gather_reads(dev, torch.from_numpy(order).to(dev.offsets.device))
    want = synth.Reads.from_strings([pairs[i] for i in order])
    np.testing.assert_array_equal(got.offsets.cpu().numpy(), want.offsets)
    np.testing.assert_array_equal(got.seq.cpu().numpy(), want.seq)
    np.testing.assert_array_equal(got.qual.cpu().numpy(), want.qual)
    ctx.close()
