"""Batches whose work items are cut by the windows that the scout pass leaves: from
batches that leave nothing to batches whose every window is probed, one after the
other on the same queue state, with and without the scout pass, in one workgroup's
queue and in larger ones, for rows that a lane holds and rows that lanes share.
The reference takes no queue: the same reads in calls of 1,000, which a team of waves
answers read by read, and the oracle for the first of them."""
import numpy as np
import pytest

import gen
from paper_1910_04358_amd import rambo as rb
from tests.gpu_util import build_gpu_seqs, build_oracle, make_reads, to_dev, to_host_u64

pytestmark = pytest.mark.gpu


def by_teams(idx, seqs, offs, n):
    """The answers of calls of 1,000 reads in the plain form."""
    import torch
    idx.set_mode(rb.MODE_PLAIN)
    out = torch.empty((n, idx.W), dtype=torch.int64, device="cuda")
    for i in range(0, n, 1_000):
        j = min(n, i + 1_000)
        idx.query_seqs(seqs, offs[i:j + 1], out=out[i:j], check=False)
    return out


@pytest.mark.parametrize("B", [100, 300, 2_000])
def test_items_follow_the_windows_left(B):
    import torch
    K, R, m, eta, seed = 70, 3, 1 << 19, 2, 8960 + B
    dm = gen.DocModel(seed=B + 19, n_docs=K, length=9_000, docs_per_anc=7, mu_lo=0.01, mu_hi=0.01)
    idx = rb.Rambo(K, B, R, m, eta, seed)
    build_gpu_seqs(idx, dm, 0, K)
    o = build_oracle((K, B, R, m, eta, seed), dm)
    rng = np.random.default_rng(B)
    docs = [dm.doc(d) for d in range(K)]

    def reads(n, L, held):
        rs = []
        for i in range(n):
            a = int(rng.integers(0, 9_000 - L + 1))
            s = docs[int(rng.integers(0, K))][a:a + L]
            rs.append(s if rng.random() < held else bytes(rng.choice(np.frombuffer(b"ACGT", np.uint8), L)))
        return make_reads(rs)

    # windows left / 1,500: 0 to about 50, 500, 5,000 and more
    batches = [reads(3_000, 60, 0.0), reads(2_500, 2_000, 0.02), reads(6_000, 700, 0.25), reads(3_000, 8_900, 1.0),
               reads(1_900, 5_000, 0.5), reads(2_049, 31, 0.5), reads(1_000, 8_000, 1.0), reads(9_000, 400, 1.0)]
    dev = [(to_dev(s), to_dev(f), f.size - 1) for s, f in batches]
    want = [by_teams(idx, *d) for d in dev]
    for (s, f), w in zip(batches, want):
        ow, _ = o.query_seqs(s, f[:41])
        assert np.array_equal(to_host_u64(w[:40]), ow)
    idx.set_mode(rb.MODE_BATCHED)
    for sched, most in ((2, 4096), (2, 192), (1, 4096), (0, 1024), (2, 1024)):
        t = idx.get_tune()
        t.seg, t.sched, t.tile = 4, sched, most
        idx.set_tune(t)
        for k in (0, 3, 0, 1, 2, 4, 5, 6, 7, 3, 5):
            got = torch.full_like(want[k], -1)
            idx.query_seqs(dev[k][0], dev[k][1], out=got, check=False)
            assert torch.equal(got, want[k]), (sched, most, k)
    idx.set_mode(rb.MODE_PLAIN)
    for k in range(len(dev)):
        assert torch.equal(idx.query_seqs(dev[k][0], dev[k][1], check=False), want[k]), k
    idx.sync()
    idx.close()


@pytest.mark.parametrize("B,n", [(100, 2_048), (100, 4_097), (100, 600_000), (300, 70_000)])
def test_queues_of_every_size_equal_teams(B, n):
    import torch
    K, R, m, eta, seed = 70, 3, 1 << 18, 2, 8980 + B
    dm = gen.DocModel(seed=B + 29, n_docs=K, length=3_000, docs_per_anc=7, mu_lo=0.01, mu_hi=0.01)
    idx = rb.Rambo(K, B, R, m, eta, seed)
    build_gpu_seqs(idx, dm, 0, K)
    rm = gen.ReadModel(qseed=n, src_lo=0, src_hi=K, len_kind=0, median=90, sigma=0.9, lo=20, hi=2_900, err_lo=0.0,
                       err_hi=0.003)
    r = gen.reads(dm, rm, n)
    seqs, offs = to_dev(r.seqs), to_dev(r.offsets)
    want = by_teams(idx, seqs, offs, n)
    assert torch.equal(idx.query_seqs(seqs, offs, check=False), want)
    idx.set_mode(rb.MODE_BATCHED)
    for sched in (2, 1):
        for tile in (64, 2048):
            t = idx.get_tune()
            t.seg, t.tile, t.sched = 4, tile, sched
            idx.set_tune(t)
            got = torch.full_like(want, -1)
            idx.query_seqs(seqs, offs, out=got, check=False)
            assert torch.equal(got, want), (sched, tile)
    idx.sync()
    idx.close()
