"""The traversal's splitter walks where they can go wrong: cycles with and
without a splitter beside paths of every short length, chains of many
splitters, keys that crowd one bucket of the row index, and the 64-bit state
numbers; against the contig oracle."""
import numpy as np
import pytest

import brute
import synth
from test_gpu_traverse import _check
from test_traverse_pins import _random_genome, _reads, _tile

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tctx(kh):
    c = kh.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("k", [21, 33, 65, 97])
def test_cycles_and_paths(tctx, monkeypatch, k, wide):
    if wide:
        monkeypatch.setenv("KMERHIP_TRAVERSE_WIDE", "1")
    rng = np.random.default_rng(31 + k)
    L = k + 9
    strings = []
    # cycles of 2 .. 700 k-mers: most of the short ones hold no splitter
    for n in [max(2, x) for x in (2, 3, 5, 8, 13, 21, 40, 64, 65, 128, 300, 700)] * 2:
        g = _random_genome(rng, n)
        strings += _tile(g * (L // n + 2) if n < L else g, L, circular=n >= L)[:max(n, 1)]
    for n in list(range(1, 20)) + [63, 64, 65, 1000]:  # paths of n k-mers
        g = _random_genome(rng, k + n - 1)
        strings += [g] if len(g) < L else _tile(g, L)
    got = _check(tctx, tctx.count(_reads(strings), k))
    assert got["cycle"].any() and not got["cycle"].all()


def test_long_chain_and_crowded_prefix(tctx):
    """One path of 40,000 k-mers, and 2,000 keys that share their first 13 bases."""
    rng = np.random.default_rng(5)
    g = _random_genome(rng, 40_000)
    strings = [g[p:p + 400] for p in range(0, len(g) - 399, 200)]
    strings += ["A" * 13 + _random_genome(rng, 18) for _ in range(2000)]
    got = _check(tctx, tctx.count(_reads(strings), 31))
    assert max(len(s) for s in got["seqs"]) > 30_000


@pytest.mark.parametrize("n", [1, 2, 3, 64, 65])
def test_few_rows(tctx, n):
    rng = np.random.default_rng(n)
    g = _random_genome(rng, 31 + n - 1)
    got = _check(tctx, tctx.count(_reads([g, brute.revcomp(g)]), 31))
    assert got["n_contigs"] == 1
