"""A read set of more than 2^34 bases, which packing takes in two launches: the
windows around where they meet, and at both ends, among bases that are none;
against the oracle on the same windows alone."""
import numpy as np
import pytest

import oracle
import synth
from brute import assert_same_table

pytestmark = pytest.mark.gpu


def test_bases_past_one_launch(kh):
    import torch
    k, meet, n = 31, 1 << 34, (1 << 34) + 5_000
    rng = np.random.default_rng(9)
    text = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, 4_000)]
    # (where it lies, what lies there): the middle one crosses the launches' meeting
    parts = [(0, text[:1_000]), (meet - 700, text[1_000:3_000]), (n - 1_000, text[3_000:])]
    cut = meet - 200  # a read starts inside the middle part
    seq = torch.full((n,), ord("N"), dtype=torch.uint8, device="cuda")
    qual = torch.full((n,), 73, dtype=torch.uint8, device="cuda")
    for at, piece in parts:
        seq[at:at + len(piece)] = torch.from_numpy(piece.copy()).cuda()
    reads = kh.DeviceReads(seq, qual, torch.tensor([0, cut, n], device="cuda"))
    small = [parts[0][1].tobytes() + b"N" + parts[1][1][:500].tobytes(),
             parts[1][1][500:].tobytes() + b"N" + parts[2][1].tobytes()]
    want = oracle.count(synth.Reads.from_strings([(s.decode(), "I" * len(s)) for s in small]), k,
                        min_count=1)
    ctx = kh.Context(0)
    try:
        table = ctx.count(reads, k, min_count=1)
        assert_same_table(table.to_numpy(), want)
        table.free()
    finally:
        ctx.close()
        kh.release_cached(0)
        del reads, seq, qual
        torch.cuda.empty_cache()
