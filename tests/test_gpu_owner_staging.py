"""Room for the owner pass's rows.

The owner pass stages its rows in a record buffer it has read: the smallest
read sets, and sets whose rows fill three quarters of it, fit at the first
attempt (a second pass over every owner takes a staging buffer of its own,
which the table's bytes then show); the rows are those of the single table.
With min_count 1 the rows have a buffer of their own, sized by the windows."""
import pytest

from brute import assert_same_table

pytestmark = pytest.mark.gpu

RECORD_WORDS = {21: 1, 55: 2, 77: 3, 99: 4}


@pytest.fixture(scope="module")
def octx(kh):
    c = kh.Context(0)
    assert c.tuning()["partitioned"] == 1
    yield c
    c.close()


@pytest.fixture(scope="module")
def sctx(kh):
    c = kh.Context(0)
    c.set_tuning(partitioned=0)
    yield c
    c.close()


def _reads(kh, n, cover):
    """n reads of 150 bases from a random genome they cover `cover` times."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    length = int(n * 150 / cover)
    letters = torch.tensor([65, 67, 71, 84], dtype=torch.uint8, device="cuda")
    genome = letters[torch.randint(0, 4, (length,), generator=g, device="cuda")]
    at = torch.randint(0, length - 149, (n,), generator=g, device="cuda")
    seq = genome[at[:, None] + torch.arange(150, device="cuda")].reshape(-1).contiguous()
    return kh.DeviceReads(seq, torch.full_like(seq, 73),
                          torch.arange(n + 1, device="cuda") * 150)


@pytest.mark.parametrize("bloom", [False, True])
@pytest.mark.parametrize("k", sorted(RECORD_WORDS))
@pytest.mark.parametrize("n,cover", [(20, 12), (300, 20), (800, 20), (1400, 20),
                                     (200_000, 12), (200_000, 9)])
def test_rows_fit_staging(kh, octx, sctx, n, cover, k, bloom):
    reads = _reads(kh, n, cover)
    table = octx.count(reads, k, use_bloom=bloom)
    records = 16 * RECORD_WORDS[k] * table.info()["n_windows"]  # two buffers
    assert octx.stats()["table_bytes"] == records
    want = sctx.count(reads, k, use_bloom=False)
    assert_same_table(table.to_numpy(), want.to_numpy())
    table.free()
    want.free()


@pytest.mark.parametrize("k", sorted(RECORD_WORDS))
@pytest.mark.parametrize("n,cover", [(20, 4), (1000, 4), (30_000, 0.2), (200_000, 0.2)])
def test_every_window_a_row(kh, sctx, n, cover, k):
    """min_count 1 in a context whose budget holds the records (two buffers), a
    quarter more rows than windows, the table itself, and 64 MiB for the rest."""
    reads = _reads(kh, n, cover)
    row = 8 * ((k + 31) // 32) + 38
    windows = n * (151 - k)
    most = 16 * RECORD_WORDS[k] * windows + windows * 5 // 4 * row + 512
    ctx = kh.Context(0, hbm_budget=most + windows * row + (64 << 20))
    try:
        table = ctx.count(reads, k, min_count=1)
        st = ctx.stats()  # the owner path's statistics: two record buffers and the staging
        assert most - 64 * row <= st["table_bytes"] <= most
        want = sctx.count(reads, k, min_count=1)
        assert_same_table(table.to_numpy(), want.to_numpy())
        table.free()
        want.free()
    finally:
        ctx.close()


@pytest.mark.parametrize("times", [1.1, 2.5])
def test_parts_fit_staging(kh, octx, sctx, times):
    """Unscreened owners counted in parts (600, of one-time keys nearly all) take
    room for the rows they have, not for a table full of them."""
    import torch
    k, owners, n = 21, 600, int(times * 4608)
    g = torch.Generator(device="cuda")
    g.manual_seed(int(10 * times))
    # AAAAA, five bases that name the owner, ten of the key, G: canonical
    ident = torch.randperm(1024, generator=g, device="cuda")[:owners].repeat_interleave(n)
    key = torch.randint(0, 4 ** 10, (owners * n,), generator=g, device="cuda")
    cols = [torch.zeros_like(key)] * 5 + [ident >> 2 * j & 3 for j in range(5)]
    cols += [key >> 2 * j & 3 for j in range(10)] + [torch.full_like(key, 2)]
    code = torch.stack(cols, 1)[torch.randperm(owners * n, generator=g, device="cuda")]
    letters = torch.tensor([65, 67, 71, 84], dtype=torch.uint8, device="cuda")
    seq = letters[code].reshape(-1).contiguous()
    reads = kh.DeviceReads(seq, torch.full_like(seq, 73),
                           torch.arange(owners * n + 1, device="cuda") * k)
    table = octx.count(reads, k, use_bloom=False)
    assert octx.stats()["rebuilds"] == 0
    assert octx.stats()["table_bytes"] == 16 * owners * n
    want = sctx.count(reads, k, use_bloom=False)
    assert_same_table(table.to_numpy(), want.to_numpy())
    table.free()
    want.free()
