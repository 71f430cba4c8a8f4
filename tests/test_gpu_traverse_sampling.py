"""The traversal with one splitter in 16 and one in 32 (below and above 1.57
million rows): paths of very different lengths and one long cycle; against the
contig oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1_500_000, 1_650_000])
def test_sample_sizes(kh, rows):
    k, step, length = 31, 100, 150
    rng = np.random.default_rng(rows)
    letters = np.frombuffer(b"ACGT", np.uint8)
    pieces = []
    left, size = rows, 400_000
    cyclic = letters[rng.integers(0, 4, size)]  # whole rounds of reads: a cycle of `size` k-mers
    ring = np.concatenate([cyclic, cyclic[:length]])
    pieces.append(ring[np.arange(0, size, step)[:, None] + np.arange(length)])
    left -= size
    while left > 0:  # paths of 1,020 bases and more
        size = min(left, int(10 ** rng.uniform(3.1, 5)))
        n = max(size, 200) // step
        genome = letters[rng.integers(0, 4, n * step + length)]
        pieces.append(genome[np.arange(0, n * step + 1, step)[:, None] + np.arange(length)])
        left -= n * step + length - k + 1
    seq = np.concatenate(pieces)
    seq = np.concatenate([seq, seq]).reshape(-1)
    reads = synth.Reads(seq, np.full_like(seq, 73),
                        np.arange(len(seq) // length + 1, dtype=np.int64) * length)
    ctx = kh.Context(0)
    try:
        table = ctx.count(reads, k)
        assert abs(table.info()["n_rows"] - rows) < 5_000
        contigs = ctx.traverse(table)
        got, want = contigs.to_python(), oracle.traverse(table.to_numpy())
        assert got["n_contigs"] == want["n_contigs"] > 20
        for f in ("seqs", "n_kmers", "depth", "cycle"):
            assert list(got[f]) == list(want[f]), f
        assert any(got["cycle"])
        contigs.free()
        table.free()
    finally:
        ctx.close()
