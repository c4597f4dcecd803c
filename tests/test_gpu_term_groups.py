"""Term queries resolved in groups of 64 (single terms and term sets) at the
sizes where the grouping can go wrong: batches around a multiple of 64, answers
of one word to past a chunk of 16, rows of 1 to 256 words with B on either side
of a multiple of 64, one to eight repetitions, an index whose group masks do not
fit LDS (the general path), and batches that are cut into slices or fill the
chip. Bit-exact against the oracle."""
import numpy as np
import pytest

import gen
import oracle
from paper_1910_04358_amd import rambo as rb
from tests.gpu_util import to_dev, to_host_u64

pytestmark = pytest.mark.gpu

# (K, B, R, m, eta)
SHAPES = [
    (64, 1, 1, 4_099, 1),         # one cell, one repetition, one word
    (513, 33, 2, 1 << 13, 2),     # nine words, the last of one document
    (1024, 64, 8, 9_001, 3),      # exactly one chunk of 16 words
    (1100, 128, 3, 1 << 13, 4),   # the widest row a lane holds
    (700, 129, 6, 1 << 12, 2),    # the narrowest that lanes share
    (2000, 5000, 3, 1 << 11, 2),  # rows of 256 words, groups of 16 waves
    (300, 8192, 8, 1 << 9, 1),    # group masks past 160 KB
]


def build(shape, seed):
    K, B, R, m, eta = shape
    dm = gen.TermDocModel(seed=seed, n_docs=K, mean_terms=40, vocab=30_000)
    terms, offs = dm.docs()
    idx = rb.Rambo(K, B, R, m, eta, seed, opaque_terms=True)
    idx.insert_batch(to_dev(np.arange(K, dtype=np.uint64)), to_dev(offs), to_dev(terms))
    idx.sync()
    o = oracle.Oracle(K, B, R, m, eta, seed)
    o.build_term_docs(terms, offs)
    return idx, o, dm, terms, offs


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "K%d-B%d-R%d" % s[:3])
def test_groups_equal_oracle(shape):
    idx, o, dm, terms, offs = build(shape, 8100 + shape[1])
    q, _ = dm.term_queries(5, 193, 0.7)
    want = o.query_terms(q, oracle.MODE_ALG2)
    pt, po, _ = dm.phrases(6, 190, 1, 8, 0.7)
    # a set of several rounds of terms that all of one document holds, and an empty one
    long = np.tile(terms[offs[3]:offs[4]], 12)
    pt = np.concatenate([pt, long])
    po = np.concatenate([po, [po[-1] + long.size] * 2]).astype(np.uint64)
    swant, _ = o.query_termsets(pt, po, oracle.MODE_ALG2, early_exit=True)
    for resolve in (rb.RESOLVE_AUTO, rb.RESOLVE_DENSE):
        idx.set_resolve(resolve)
        for n in (1, 63, 64, 65, 193):
            assert np.array_equal(to_host_u64(idx.query_kmers(to_dev(q[:n]))), want[:n]), n
        for ee in (True, False):
            idx.set_early_exit(ee)
            for n in (1, 5, 192):
                got = to_host_u64(idx.query_term_sets(to_dev(pt), to_dev(po[-n - 1:])))
                assert np.array_equal(got, swant[-n:]), (n, ee)
    assert idx.sync() == rb.OK_EMPTYQ
    idx.close()


@pytest.mark.parametrize("B", [40, 150])
def test_batches_that_fill_the_chip(B):
    shape = (200, B, 2, 1 << 13, 2)
    idx, o, dm, terms, offs = build(shape, 8300 + B)
    q, _ = dm.term_queries(7, 140_001, 0.5)
    assert np.array_equal(to_host_u64(idx.query_kmers(to_dev(q))), o.query_terms(q, oracle.MODE_ALG2))
    pt, po, _ = dm.phrases(8, 70_001, 1, 5, 0.5)
    want, _ = o.query_termsets(pt, po, oracle.MODE_ALG2, early_exit=True)
    assert np.array_equal(to_host_u64(idx.query_term_sets(to_dev(pt), to_dev(po))), want)
    idx.close()


@pytest.mark.parametrize("shape", [(1, 5000, 3, 1 << 11, 2), (1500, 2048, 8, 1 << 11, 1), (2049, 4950, 4, 1 << 11, 2),
                                   (1030, 8192, 2, 1 << 11, 2)], ids=lambda s: "K%d-B%d-R%d" % s[:3])
def test_half_groups_equal_oracle(shape):
    """Groups of 32 terms: masks of 64 terms would take more than half the LDS.
    Batches around multiples of 32; answers of one word, of half a chunk more
    than one, of one word more than two; every number of probed repetitions."""
    idx, o, dm, terms, offs = build(shape, 8400 + shape[1])
    q, _ = dm.term_queries(9, 20_003, 0.7)
    want = o.query_terms(q, oracle.MODE_ALG2)
    for n in (1, 31, 32, 33, 95, 20_003):
        assert np.array_equal(to_host_u64(idx.query_kmers(to_dev(q[:n]))), want[:n]), n
    idx.close()
