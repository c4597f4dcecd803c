"""Single terms that no document holds, in groups that hold no other term and in
groups that do, on rows that a lane holds whole: zeros over whatever the answers'
memory held, for answers of one word to several slices; against the oracle."""
import numpy as np
import pytest

import gen
import oracle
from paper_1910_04358_amd import rambo as rb
from tests.gpu_util import to_dev, to_host_u64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,B,R", [(40, 20, 1), (700, 40, 2), (5_001, 100, 3), (2_000, 128, 8)])
def test_terms_that_no_document_holds(K, B, R):
    import torch
    m, eta, seed = 1 << 14, 2, 8500 + B
    dm = gen.TermDocModel(seed=seed, n_docs=K, mean_terms=12, vocab=30_000)
    terms, offs = dm.docs()
    idx = rb.Rambo(K, B, R, m, eta, seed, opaque_terms=True)
    idx.insert_batch(to_dev(np.arange(K, dtype=np.uint64)), to_dev(offs), to_dev(terms))
    o = oracle.Oracle(K, B, R, m, eta, seed)
    o.build_term_docs(terms, offs)
    rng = np.random.default_rng(K)
    q = rng.integers(1 << 40, 1 << 61, 40_000).astype(np.uint64)
    q[640] = terms[0]
    q[1_000:1_064] = terms[:64]
    want = o.query_terms(q[:2_000], oracle.MODE_ALG2)
    assert want[640].any()
    qd = to_dev(q)
    for at, n in ((0, 1), (1, 63), (0, 64), (0, 65), (640, 1), (600, 100), (990, 70), (0, 2_000)):
        out = torch.full((n, idx.W), -1, dtype=torch.int64, device="cuda")
        assert np.array_equal(to_host_u64(idx.query_kmers(qd[at:at + n].contiguous(), out=out)), want[at:at + n]), (at, n)
    out = torch.full((q.size, idx.W), -1, dtype=torch.int64, device="cuda")
    assert np.array_equal(to_host_u64(idx.query_kmers(qd, out=out))[:2_000], want)
    idx.close()
