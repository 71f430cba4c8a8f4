"""Many keys with the same sort prefix (single table): the full-key sort that
orders them takes no memory beside what the same number of ordinary rows takes,
so that a budget which holds the one holds the other; the rows are the
oracle's, also where they go to the caller's buffers."""
import numpy as np
import pytest

import oracle
import synth
from brute import assert_same_table

pytestmark = pytest.mark.gpu


def _reads(k, n, head, seed):
    """n distinct k-mers twice each, the first bases of all of them `head`."""
    rng = np.random.default_rng(seed)
    seq = rng.integers(0, 4, (n, k))
    seq[:, :len(head)] = ["ACGT".index(c) for c in head]
    seq[:, -1] = 2  # ... G: they start with A, so canonical as they stand
    text = np.frombuffer(b"ACGT", np.uint8)[np.concatenate([seq, seq])].reshape(-1).copy()
    return synth.Reads(text, np.full_like(text, 73), np.arange(2 * n + 1, dtype=np.int64) * k)


@pytest.mark.parametrize("n", [100, 30_000])
@pytest.mark.parametrize("k", [33, 55, 77, 99, 127])
def test_full_key_sort_memory(kh, k, n):
    import torch
    peaks = []
    for head in ("AAAAAC", "A" * 24):  # runs of few rows, one run of all
        sizes = {}
        most = [0]

        def alloc(nbytes, device):
            p = torch.cuda.caching_allocator_alloc(nbytes, device)
            sizes[p] = nbytes
            most[0] = max(most[0], sum(sizes.values()))
            return p

        def free(ptr, nbytes, device):
            del sizes[ptr]
            torch.cuda.caching_allocator_delete(ptr)

        reads = _reads(k, n, head, k)
        ctx = kh.Context(0, allocator=(alloc, free))
        try:
            ctx.set_tuning(partitioned=0)
            table = ctx.count(reads, k)
            assert ctx.stats()["full_key_sort"] == int(len(head) == 24)
            assert_same_table(table.to_numpy(), oracle.count(reads, k))
            table.free()
        finally:
            ctx.close()
        peaks.append(most[0])
    assert peaks[1] <= peaks[0], peaks


def test_caller_buffers(kh):
    """Rows to the caller's own buffers, which hold them alone."""
    import torch
    k, n = 77, 5000
    reads = _reads(k, n, "A" * 24, 5)
    want = oracle.count(reads, k)
    dev = kh.DeviceReads.from_host(reads)
    keys = torch.zeros((n, 3), dtype=torch.int64, device="cuda")
    counts = torch.zeros(n, dtype=torch.int32, device="cuda")
    ext = torch.zeros((n, 8), dtype=torch.int32, device="cuda")
    codes = torch.zeros((n, 2), dtype=torch.uint8, device="cuda")
    rows, _ = kh.count_noalloc(dev, k, keys, counts, ext, codes)
    assert rows == n == want["n_rows"]
    np.testing.assert_array_equal(keys.cpu().numpy().view(np.uint64), want["keys"])
    np.testing.assert_array_equal(counts.cpu().numpy(), want["counts"])
    np.testing.assert_array_equal(ext.cpu().numpy(), want["ext"])
    np.testing.assert_array_equal(codes.cpu().numpy(), want["codes"])
