"""Bulk insertion (bits sorted by region of the rows before they are set) where
it can go wrong: regions of one row word to many, m that is no power of two,
more than three hash functions, several passes over the documents, documents
that are empty, short, hold other letters or ids past K, a first offset that is
not 0, a small insertion from a large buffer, insertions on two streams at once
and under graph capture. Whole indexes, bit-exact against the oracle or against
the same documents inserted one by one (which takes the direct path)."""
import numpy as np
import pytest

import gen
import oracle
from paper_1910_04358_amd import rambo as rb
from tests.gpu_util import cuda, to_dev

pytestmark = pytest.mark.gpu

# (K, B, R, m, eta): documents of 80 kbp, 2.4 million positions or more
SHAPES = [
    (30, 1, 1, 1 << 17, 4),       # one-word rows, one cell
    (30, 100, 2, 100_003, 2),     # a bucket past the last row
    (30, 40, 3, 65_537, 3),       # two-word rows
    (30, 1100, 2, 9_001, 2),      # rows of 64 words, few regions
    (30, 32, 2, 3_000_017, 16),   # many regions, many hash functions
    (40, 1000, 1, 1 << 20, 2),    # regions of one full tile of the rows
    (40, 1000, 1, (1 << 20) + 5, 2),  # of two tiles
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B%d-R%d-m%d-eta%d" % s[1:])
def test_bulk_insert_equals_oracle(shape):
    K, B, R, m, eta = shape
    seed = 8500 + B
    dm = gen.DocModel(seed=B, n_docs=K, length=80_000, docs_per_anc=5, mu_lo=0.02, mu_hi=0.02)
    docs = dm.docs(0, K)
    o = oracle.Oracle(K, B, R, m, eta, seed)
    o.build_docs(docs, dm.length, 0, K)
    want = o.bits()
    offs = np.arange(K + 1, dtype=np.uint64) * np.uint64(dm.length)
    ids = np.arange(K, dtype=np.uint64)
    idx = rb.Rambo(K, B, R, m, eta, seed)
    idx.insert_seqs(to_dev(ids), to_dev(docs), to_dev(offs))
    assert idx.sync() == rb.OK
    assert np.array_equal(idx.bfu_major(), want)
    idx.close()
    codes = [dm.window_codes(d) for d in range(K)]
    koff = np.concatenate([[0], np.cumsum([c.size for c in codes])]).astype(np.uint64)
    idx = rb.Rambo(K, B, R, m, eta, seed)
    idx.insert_batch(to_dev(ids), to_dev(koff), to_dev(np.concatenate(codes)))
    assert idx.sync() == rb.OK
    assert np.array_equal(idx.bfu_major(), want)
    idx.close()


def one_by_one(idx, ids, docs, offs):
    for i in range(ids.size):
        s = docs[int(offs[i]):int(offs[i + 1])]
        if s.size:
            idx.insert_seqs(to_dev(ids[i:i + 1]), to_dev(s), to_dev(np.array([0, s.size], dtype=np.uint64)))


def ragged(seed, n, K, mean):
    """Documents of 0 to 2 mean bases, some with other letters, some with ids past K."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, 2 * mean, n)
    lens[::7] = rng.integers(0, 40, lens[::7].size)
    lens[3:6] = 0
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
    docs = rng.choice(np.frombuffer(b"ACGTacgt", np.uint8), int(offs[-1]))
    docs[rng.integers(0, docs.size, docs.size // 500)] = ord("N")
    ids = rng.integers(0, K, n).astype(np.uint64)
    ids[5] = K  # empty: not counted
    return ids, docs, offs


def test_several_passes_and_ragged_documents():
    import torch
    K, B, R, m, eta, seed = 64, 20, 2, 1 << 21, 3, 8601
    ids, docs, offs = ragged(1, 200, K, 150_000)   # about 27 million positions, 80 million bits a repetition
    a, b = (rb.Rambo(K, B, R, m, eta, seed) for _ in range(2))
    pre = np.frombuffer(b"ACGTN" * 7, np.uint8)  # the first offset is 35
    a.insert_seqs(to_dev(ids), to_dev(np.concatenate([pre, docs])), to_dev(offs + np.uint64(35)))
    one_by_one(b, ids, docs, offs)
    assert a.sync() == rb.OK and b.sync() == rb.OK
    assert np.array_equal(a.copy_rows(), b.copy_rows())
    # a small insertion from the large buffer, one of its ids past K
    big = to_dev(docs)
    sub = np.array([K, 7], dtype=np.uint64)
    o2 = np.array([0, 100, 50_100], dtype=np.uint64)
    a.insert_seqs(to_dev(sub), big, to_dev(o2))
    with pytest.raises(rb.RamboError):
        a.sync()
    b.insert_seqs(to_dev(sub[1:]), to_dev(docs[100:50_100]), to_dev(np.array([0, 50_000], dtype=np.uint64)))
    b.sync()
    assert np.array_equal(a.copy_rows(), b.copy_rows())
    torch.cuda.synchronize()
    a.close()
    b.close()


def test_two_streams_and_capture():
    import torch
    K, B, R, m, eta, seed = 64, 20, 2, 1 << 16, 3, 8602
    parts = [ragged(s, 40, K, 80_000) for s in (2, 3, 4)]
    a, b = (rb.Rambo(K, B, R, m, eta, seed) for _ in range(2))
    dev = [tuple(to_dev(x) for x in p) for p in parts]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for k in range(2):
        a.insert_seqs(*dev[k], stream=streams[k])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        a.insert_seqs(*dev[2])
    for _ in range(2):
        g.replay()
    torch.cuda.synchronize()
    a.sync()
    for p in parts:
        one_by_one(b, *p)
    b.sync()
    assert np.array_equal(a.copy_rows(), b.copy_rows())
    a.close()
    b.close()
