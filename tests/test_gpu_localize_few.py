"""A handful of reads against a large table: no index of its rows is built for
them, and for some hundreds none with masks (told by the memory the call takes);
the order is the oracle's."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

K = 31


@pytest.fixture(scope="module")
def large(kh):
    """(context, table, contigs, their sequences, most bytes a call asked for)"""
    import torch
    most = [0]

    def alloc(nbytes, device):
        most[0] = max(most[0], nbytes)
        return torch.cuda.caching_allocator_alloc(nbytes, device)

    def free(ptr, nbytes, device):
        torch.cuda.caching_allocator_delete(ptr)

    rng = np.random.default_rng(3)
    n, length = 60_000, 600_000
    genome = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, length)]
    at = np.concatenate([np.arange(0, length - 149, 60), rng.integers(0, length - 149, n)])
    seq = genome[at[:, None] + np.arange(150)]
    flat = np.ascontiguousarray(seq).reshape(-1)
    reads = synth.Reads(flat, np.full_like(flat, 73), np.arange(len(at) + 1, dtype=np.int64) * 150)
    ctx = kh.Context(0, allocator=(alloc, free))
    table = ctx.count(reads, K)
    contigs = ctx.traverse(table)
    assert 2 << 18 < table.info()["n_rows"] < 3 << 18
    yield ctx, table, contigs, contigs.to_python()["seqs"], reads, most
    contigs.free()
    table.free()
    ctx.close()


@pytest.mark.parametrize("foreign", [False, True])
@pytest.mark.parametrize("n,room", [(1, 64 << 10), (2, 1100 << 10), (200, 1100 << 10),
                                    (9000, 4 << 20)])
def test_memory_of_few_reads(kh, large, n, room, foreign):
    ctx, table, contigs, seqs, reads, most = large
    few = reads.slice(7, 7 + n)
    if foreign:
        seq = np.frombuffer(b"ACGTN", np.uint8)[np.random.default_rng(n).integers(0, 5, 150 * n)]
        few = synth.Reads(seq.copy(), few.qual, few.offsets)
    dev = kh.DeviceReads.from_host(few)
    want = oracle.localize(few, seqs, K)
    ctx.trim()
    most[0] = 0
    got = ctx.localize_order(table, contigs, dev)
    assert most[0] <= room
    np.testing.assert_array_equal(got.cpu().numpy(), want)
