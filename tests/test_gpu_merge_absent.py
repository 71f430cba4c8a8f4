"""The merge's screen of the contigs' windows against the table's rows: every
key width, contigs that are all in the table, none of them, or some, windows
at the edges of tiles, new k-mers before the first and after the last row, and
k-mers repeated often; against the merge oracle."""
import numpy as np
import pytest

import synth
from test_gpu_merge import _check
from test_traverse_pins import _random_genome, _reads, _tile

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mctx(kh):
    c = kh.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("k", [5, 21, 31, 33, 63, 65, 95, 97, 127])
def test_some_windows_new(mctx, k):
    rng = np.random.default_rng(100 + k)
    g = _random_genome(rng, 3000)
    t = mctx.count(_reads(_tile(g[:2000], 150)), k)
    contigs = [g[:400], g[900:3000], "A" * (k + 5), "T" * k, "G" * (k + 1),
               g[100:100 + k], g[:k - 1], "", g[2500:2500 + k] + "N" + g[2600:2700 + k],
               (g[2700:2700 + k + 3] + "N") * 70, g[500:600 + k].lower()]
    _check(mctx, t, contigs)


@pytest.mark.parametrize("n", [1023, 1024, 1025, 2048 + 20, 4097])
def test_tile_edges(mctx, n):
    rng = np.random.default_rng(n)
    g = _random_genome(rng, n)
    t = mctx.count(_reads([g[n // 3:n // 2]]), 21)
    _check(mctx, t, [g])


def test_nothing_new_and_all_new(mctx):
    rng = np.random.default_rng(3)
    g, h = _random_genome(rng, 5000), _random_genome(rng, 5000)
    t = mctx.count(_reads(_tile(g, 100)), 33)
    assert _check(mctx, t, [g])["n_rows"] == t.info()["n_rows"]
    _check(mctx, t, [h])
    many = "ACGTTGCATG" * 1200  # ten k-mers, 1,200 times each: counts over 63
    _check(mctx, t, [many, h[:300]] * 4)
