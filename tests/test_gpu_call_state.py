"""What a handle keeps between calls and reports about them."""
import numpy as np
import pytest

import gen
from paper_1910_04358_amd import rambo as rb
from tests.gpu_util import build_gpu_seqs, reads_to_dev

pytestmark = pytest.mark.gpu


def index_and_reads(sizes, B=100, m=1 << 18):
    K, R, eta, seed = 70, 3, 2, 9100
    dm = gen.DocModel(seed=91, n_docs=K, length=3_000, docs_per_anc=7, mu_lo=0.01, mu_hi=0.01)
    idx = rb.Rambo(K, B, R, m, eta, seed)
    build_gpu_seqs(idx, dm, 0, K)
    rm = gen.ReadModel(qseed=92, src_lo=0, src_hi=K, len_kind=0, median=90, sigma=0.9, lo=20, hi=2_900, err_hi=0.003)
    return idx, [reads_to_dev(gen.reads(dm, rm, n, i0=n)) for n in sizes]


def test_batch_times_are_of_the_last_batched_call():
    import torch
    idx, (large, small) = index_and_reads((400_000, 5_000))
    idx.set_mode(rb.MODE_BATCHED)
    idx.set_tune(rb.Tune(4, 1024, 16, 4, 1, 2))
    idx.query_seqs(*large, check=False)
    times = idx.last_batch_ms()
    idx.set_mode(rb.MODE_PLAIN)
    for _ in range(3):
        idx.query_seqs(*small, check=False)  # (takes the batched launches, and their state)
        assert idx.last_batch_ms() == times
    idx.set_mode(rb.MODE_BATCHED)
    idx.query_seqs(*small, check=False)
    again = idx.last_batch_ms()
    assert again != times and again[0] < times[0]
    torch.cuda.synchronize()
    idx.close()
