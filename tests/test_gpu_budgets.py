"""Calls in a context whose budget holds what they cannot do without (their
inputs live in another context) and little beside: merging, pruning and counting
on the owner path, against a context without a budget."""
import numpy as np
import pytest

from brute import assert_same_table

pytestmark = pytest.mark.gpu

MIB = 1 << 20


@pytest.fixture(scope="module")
def free_ctx(kh):
    c = kh.Context(0)
    yield c
    c.close()


def _reads(kh, n, cover, err=0.0, length=150):
    """n reads from a random genome they cover `cover` times, on the GPU."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    size = int(n * length / cover)
    genome = torch.randint(0, 4, (size,), generator=g, device="cuda")
    at = torch.randint(0, size - length + 1, (n,), generator=g, device="cuda")
    code = genome[at[:, None] + torch.arange(length, device="cuda")]
    if err:
        wrong = torch.rand(code.shape, generator=g, device="cuda") < err
        code = (code + wrong * torch.randint(1, 4, code.shape, generator=g, device="cuda")) & 3
    letters = torch.tensor([65, 67, 71, 84], dtype=torch.uint8, device="cuda")
    seq = letters[code].reshape(-1).contiguous()
    return kh.DeviceReads(seq, torch.full_like(seq, 73),
                          torch.arange(n + 1, device="cuda") * length)


def _budgeted(kh, nbytes):
    kh.release_cached(0)
    return kh.Context(0, hbm_budget=int(nbytes))


def _blocks(*sizes):
    """Pool blocks of these sizes (from 2 MiB on in whole ones)."""
    return sum((s + 2 * MIB - 1) // (2 * MIB) * 2 * MIB if s >= 2 * MIB else s + 256
               for s in sizes)


@pytest.mark.parametrize("k", [21, 55])
@pytest.mark.parametrize("contigs", [[], ["ACGGTTTCAGGCAT" * 12]])
def test_merge_holds_the_merged_rows(kh, free_ctx, k, contigs):
    """Few contigs: the merged rows, and half a megabyte."""
    table = free_ctx.count(_reads(kh, 100_000, 8), k)
    rows, W = table.info()["n_rows"], (k + 31) // 32
    want = free_ctx.merge_contigs(table, contigs)
    n = want.info()["n_rows"]
    assert n > 1_000_000 and n - rows < 200
    ctx = _budgeted(kh, _blocks(8 * W * n, 4 * n, 32 * n, 2 * n) + MIB // 2)
    try:
        got = ctx.merge_contigs(table, contigs)
        assert_same_table(got.to_numpy(), want.to_numpy())
        got.free()
    finally:
        ctx.close()
    want.free()
    table.free()


def test_prune_memory(kh, free_ctx):
    """47 bytes a contig for the sweeps, 32 for the kept ones' places, the kept
    ones, and a quarter of a megabyte."""
    table = free_ctx.count(_reads(kh, 60_000, 10, err=0.01), 21, min_count=1)
    contigs = free_ctx.traverse(table)
    nc = contigs.info()["n_contigs"]
    want, report = free_ctx.prune(table, contigs)
    kept, bases = want.info()["n_contigs"], want.info()["total_bases"]
    assert nc > 1_000_000 and kept < nc
    budget = _blocks(8 * nc, nc, nc, nc, 32 * nc, 4 * nc, 8 * nc, 8 * nc, 8 * nc, 8 * nc,
                     8 * kept, 8 * kept, 8 * kept, kept, bases) + MIB // 4
    ctx = _budgeted(kh, budget)
    try:
        got, rep = ctx.prune(table, contigs)
        assert rep == report
        a, b = got.to_numpy(), want.to_numpy()
        for f in a:
            np.testing.assert_array_equal(a[f], b[f])
        got.free()
    finally:
        ctx.close()
    want.free()
    contigs.free()
    table.free()


@pytest.mark.parametrize("k", [21, 55])
def test_owner_count_holds_records_and_rows(kh, free_ctx, k):
    """The packed reads, two record buffers, the rows, and 24 MiB (a third
    of what the windows' planes take beside them while they are routed)."""
    n, length = 1_300_000, 150
    reads = _reads(kh, n, 20)
    want = free_ctx.count(reads, k)
    rows, W, R = want.info()["n_rows"], (k + 31) // 32, (2 * k - 10 + 6 + 63) // 64
    bases = n * length
    records = 8 * R * n * (length + 1 - k)
    plane = bases // 8
    assert 3 * plane > 69 * MIB
    ctx = _budgeted(kh, _blocks(2 * plane, plane, plane, plane, records, records, 8 * W * rows,
                                4 * rows, 32 * rows, 2 * rows) + 24 * MIB)
    try:
        got = ctx.count(reads, k)
        assert ctx.stats()["table_bytes"] == 2 * records  # the owner path, staging in them
        assert_same_table(got.to_numpy(), want.to_numpy())
        got.free()
    finally:
        ctx.close()
    want.free()
