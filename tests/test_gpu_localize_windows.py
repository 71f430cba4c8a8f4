"""Localisation of reads whose first window on a contig lies at the edges of
what a block looks up at once: behind 0 .. 100 foreign bases, behind N, in the
read's last window, with a second contig further on, or nowhere; against the
oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lctx(kh):
    c = kh.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("crowded", [0, 90])
@pytest.mark.parametrize("k", [5, 21, 33, 77, 127])
def test_first_hit(kh, lctx, k, crowded):
    """`crowded` further contigs share a prefix, more rows than the index masks."""
    rng = np.random.default_rng(k + crowded)

    def junk(n):
        return "".join(rng.choice(list("ACGT"), n))

    genomes = [junk(3 * k + 40) for _ in range(6)]
    genomes += ["A" * 14 + junk(k + 6) for _ in range(crowded)]
    table = lctx.count(synth.Reads.from_strings([(g, "I" * len(g)) for g in genomes * 2]), k)
    contigs = lctx.traverse(table)
    texts = ["", junk(k - 1), junk(k), junk(300), "N" * 200, genomes[0][:k]]
    for at in [0, 1, 2, 14, 15, 16, 17, 31, 32, 33, 48, 100]:
        texts += ["A" * 14 + junk(k), junk(at) + "A" * 13 + junk(2 * k)]
        for i, g in enumerate(genomes[:12]):
            other = genomes[(i + 1 + at) % len(genomes)]
            texts += [junk(at) + g[7:7 + k],                      # the read's last window
                      junk(at) + g[3:] + other,                   # another contig behind
                      junk(at // 2) + "N" + junk(at) + g[:k + 5] + "N" + junk(9)]
    texts = [texts[i] for i in rng.permutation(len(texts))] * 3
    reads = synth.Reads.from_strings([(s, "I" * len(s)) for s in texts])
    want = oracle.localize(reads, contigs.to_python()["seqs"], k)
    got = lctx.localize_order(table, contigs, kh.DeviceReads.from_host(reads))
    np.testing.assert_array_equal(got.cpu().numpy(), want)
    contigs.free()
    table.free()


@pytest.mark.parametrize("room", [1 << 20, 64 << 10])
def test_smaller_index(kh, room):
    """No block of `room` bytes or more to be had, fewer than the index of these
    rows takes: the same order by longer searches."""
    import torch
    limit = [1 << 40]

    def alloc(nbytes, device):
        return torch.cuda.caching_allocator_alloc(nbytes, device) if nbytes < limit[0] else 0

    def free(ptr, nbytes, device):
        torch.cuda.caching_allocator_delete(ptr)

    ctx = kh.Context(0, allocator=(alloc, free))
    try:
        reads = synth.config(2, scale=0.01)
        table = ctx.count(reads, 21)
        contigs = ctx.traverse(table)
        few = synth.Reads.from_strings(reads.strings()[:500])
        want = oracle.localize(few, contigs.to_python()["seqs"], 21)
        dev = kh.DeviceReads.from_host(few)
        assert table.info()["n_rows"] > room
        ctx.trim()
        limit[0] = room
        got = ctx.localize_order(table, contigs, dev)
        np.testing.assert_array_equal(got.cpu().numpy(), want)
        limit[0] = 1 << 40
        contigs.free()
        table.free()
    finally:
        ctx.close()
