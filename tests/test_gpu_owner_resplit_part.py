"""A key-space part whose owners are split finer (a testing hook gives them few
slots) emits its records again: the windows' planes are formed anew, in a record
buffer where that has room for them (few parts) and beside it (many)."""
import pytest

import oracle
import synth
from brute import assert_same_table

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [21, 77])
@pytest.mark.parametrize("shards,slots,scale", [(2, 400, 0.004), (32, 200, 0.02)])
def test_resplit_of_a_part(kh, monkeypatch, shards, slots, scale, k):
    reads = synth.config(2, scale=scale)
    want = oracle.count_shard(reads, k, shards, 1)
    monkeypatch.setenv("KMERHIP_OWNER_SLOTS", str(slots))
    ctx = kh.Context(0)
    try:
        table = ctx.count(reads, k, owner_shards=shards, owner=1)
        assert ctx.stats()["rebuilds"] >= 1
        assert_same_table(table.to_numpy(), want)
        table.free()
    finally:
        ctx.close()
