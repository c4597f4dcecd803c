"""The plain form with one wave per read, which batches of more than 4,096 reads take
under graph capture and in the no-allocation call: for rows of 1 to 256 words (a lane
a term, and 2 to 64 lanes), every probe schedule and resolve, with and without early
exit, as bitsets and as id lists; against the oracle."""
import ctypes

import numpy as np
import pytest

import gen
from paper_1910_04358_amd import rambo as rb
from tests.gpu_util import build_gpu_seqs, build_oracle, make_reads, to_dev, to_host_u64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,B,R,m,eta", [(60, 20, 2, 1 << 16, 3), (60, 64, 1, 1 << 16, 2), (130, 100, 5, 1 << 16, 2),
                                         (70, 200, 8, 1 << 15, 1), (70, 400, 4, 1 << 15, 4), (80, 1_000, 6, 1 << 14, 2),
                                         (60, 2_000, 3, 1 << 14, 2), (60, 4_000, 2, 1 << 13, 2), (33_000, 8_192, 2, 1 << 13, 1)])
def test_one_wave_per_read_equals_oracle(K, B, R, m, eta):
    import torch
    nd, seed, n = min(K, 90), 9300 + B, 4_200
    dm = gen.DocModel(seed=B + 3, n_docs=nd, length=3_000, docs_per_anc=9, mu_lo=0.01, mu_hi=0.01)
    idx = rb.Rambo(K, B, R, m, eta, seed)
    build_gpu_seqs(idx, dm, 0, nd)
    o = build_oracle((K, B, R, m, eta, seed), dm)
    rm = gen.ReadModel(qseed=B + 4, src_lo=0, src_hi=nd, len_kind=0, median=110, sigma=0.9, lo=31, hi=2_900, err_lo=0.0,
                       err_hi=0.005)
    r = gen.reads(dm, rm, n - 7)
    d0 = dm.doc(0)
    edge = [d0, b"", b"ACGT" * 7, b"N" * 200, d0[:31], d0[100:163], d0[:1500] + b"N" + d0[1501:]]
    seqs, offs = make_reads(edge + [r.read(i) for i in range(r.n)])
    want, _ = o.query_seqs(seqs, offs)
    bits = np.unpackbits(want.view(np.uint8), axis=1, bitorder="little")[:, :K]
    total = int(bits.sum())
    sd, od = to_dev(seqs), to_dev(offs)
    out = torch.empty((n, idx.W), dtype=torch.int64, device="cuda")
    ids = torch.empty(total, dtype=torch.int32, device="cuda")
    ioff = torch.empty(n + 1, dtype=torch.int64, device="cuda")
    p = [ctypes.c_void_p(t.data_ptr()) for t in (sd, od, out, ids, ioff)]
    for sched in (2, 1, 0):
        t = idx.get_tune()
        t.sched = sched
        idx.set_tune(t)
        for resolve, ee in ((rb.RESOLVE_AUTO, True), (rb.RESOLVE_DENSE, False), (rb.RESOLVE_CANDIDATE, True)):
            idx.set_resolve(resolve)
            idx.set_early_exit(ee)
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                idx.query_seqs(sd, od, out=out, check=False)
            for _ in range(3):
                out.fill_(-1)
                g.replay()
                torch.cuda.synchronize()
                assert np.array_equal(to_host_u64(out), want), (sched, resolve, ee)
            ids.fill_(-1)
            st = rb.lib().rambo_query_seqs_ids_noalloc(idx._h, p[0], p[1], n, p[2], p[3], p[4], total, None)
            assert st == rb.OK_EMPTYQ
            assert np.array_equal(np.diff(ioff.cpu().numpy()), bits.sum(axis=1)), (sched, resolve, ee)
            assert np.array_equal(ids.cpu().numpy(), np.nonzero(bits)[1]), (sched, resolve, ee)
            del g
    idx.sync()
    idx.close()


def test_scans_past_4096_workgroups():
    """4.3 million reads: the sums of the scans' workgroups are scanned in a launch of
    their own, for the id lists' offsets and for the queue of a batch with long reads
    in many items."""
    import torch
    K, B, R, m, eta, seed, n = 40, 20, 2, 1 << 16, 2, 9390, 4_300_001
    dm = gen.DocModel(seed=93, n_docs=K, length=2_000, docs_per_anc=8, mu_lo=0.01, mu_hi=0.01)
    idx = rb.Rambo(K, B, R, m, eta, seed)
    build_gpu_seqs(idx, dm, 0, K)
    o = build_oracle((K, B, R, m, eta, seed), dm)
    rng = np.random.default_rng(5)
    docs = np.frombuffer(b"".join(dm.doc(d) for d in range(K)), np.uint8)
    lens = np.full(n, 31, dtype=np.uint64)
    lens[::1_000] = 1_500
    lens[1::1_000] = 30
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
    at = (rng.integers(0, K, n) * 2_000 + rng.integers(0, 400, n)).astype(np.int64)
    pos = np.repeat(at - offs[:-1].astype(np.int64), lens.astype(np.int64)) + np.arange(int(offs[-1]))
    seqs = docs[pos]
    bad = rng.integers(0, seqs.size, seqs.size // 60)
    seqs[bad] = ord("A")
    sd, od = to_dev(seqs), to_dev(offs)
    want = torch.empty((n, idx.W), dtype=torch.int64, device="cuda")
    for i in range(0, n, 1_000):  # (teams of waves: no queue, no scan)
        idx.query_seqs(sd, od[i:min(n, i + 1_000) + 1], out=want[i:i + 1_000], check=False)
    ow, _ = o.query_seqs(seqs, offs[:3_001])
    assert np.array_equal(to_host_u64(want[:3_000]), ow)
    bits = np.unpackbits(to_host_u64(want).view(np.uint8), axis=1, bitorder="little")[:, :K]
    total = int(bits.sum())
    idx.set_mode(rb.MODE_BATCHED)
    for sched in (2, 1):
        idx.set_tune(rb.Tune(1, 64, 16, 4, 1, sched))
        assert torch.equal(idx.query_seqs(sd, od, check=False), want), sched
        ids, ioff = idx.query_seqs_ids(sd, od, ids_cap=total, check=False)
        assert np.array_equal(np.diff(ioff.cpu().numpy()), bits.sum(axis=1)), sched
        assert np.array_equal(ids.cpu().numpy(), np.nonzero(bits)[1]), sched
    idx.sync()
    idx.close()
