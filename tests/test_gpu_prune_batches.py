"""Pruning runs its sweeps several to a batch: loops that end inside the first
batch, at a batch's edge and many batches later, contig counts around a block,
and contigs of every short length copied; against the pruning oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pctx(kh):
    c = kh.Context(0)
    yield c
    c.close()


@pytest.fixture(scope="module")
def walked(pctx):
    out = []
    for k, scale in ((21, 0.004), (55, 0.002), (9, 0.0005)):
        reads = synth.config(2, scale=scale)
        t = pctx.count(reads, k, min_count=2, t_min_ext=1)
        out.append((k, t, pctx.traverse(t)))
    yield out
    for _, t, c in out:
        c.free()
        t.free()


@pytest.mark.parametrize("alpha,beta", [(0.1, 0.2), (0.001, 0.3), (1000.0, 1.0), (0.5, 0.0),
                                        (0.06, 10.0), (0.05, 0.5)])
def test_batches(pctx, walked, alpha, beta):
    for k, t, c in walked:
        d = c.to_python()
        kept, rep, at = pctx.prune(t, c, alpha=alpha, beta=beta, removed_at=True)
        want, sweeps = oracle.prune(d["seqs"], k, d["depth"], alpha, beta)
        print(k, alpha, beta, rep, flush=True)
        np.testing.assert_array_equal(at, want)
        assert rep["sweeps"] == sweeps and rep["removed"] == int((want >= 0).sum())
        assert kept.to_python()["seqs"] == [s for s, x in zip(d["seqs"], want) if x < 0]
        kept.free()
