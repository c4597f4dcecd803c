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


def test_ids_total_of_a_rejected_call_is_zero():
    import ctypes
    import torch
    idx, ((seqs, offs),) = index_and_reads((300,))
    total = rb.lib().rambo_last_ids_total
    ids, off = idx.query_seqs_ids(seqs, offs, ids_cap=70 * 300, check=False)
    assert ids.numel() == total() > 0
    with pytest.raises(rb.RamboError):  # too small: the total is known
        idx.query_seqs_ids(seqs, offs, ids_cap=1, check=False)
    assert total() == ids.numel()
    scratch = torch.empty((300, idx.W), dtype=torch.int64, device="cuda")
    p = [ctypes.c_void_p(t.data_ptr()) for t in (seqs, offs, scratch, ids, off)]
    lib = rb.lib()
    for call in (lib.rambo_query_seqs_ids, lib.rambo_query_seqs_ids_noalloc):
        def good():
            call(idx._h, p[0], p[1], 300, p[2], p[3], p[4], ids.numel(), None)
            assert total() == ids.numel()
        good()
        assert call(None, p[0], p[1], 300, p[2], p[3], p[4], ids.numel(), None) == rb.EINVAL
        assert total() == 0
        good()
        assert call(idx._h, None, p[1], 300, p[2], p[3], p[4], ids.numel(), None) == rb.EINVAL
        assert total() == 0
        good()
        assert call(idx._h, p[0], p[1], 300, p[2], p[3], None, ids.numel(), None) == rb.EINVAL
        assert total() == 0
    good()
    terms = rb.Rambo(10, 4, 1, 64, 1, 1, opaque_terms=True)
    assert lib.rambo_query_seqs_ids(terms._h, p[0], p[1], 300, p[2], p[3], p[4], 0, None) == rb.EINVAL
    assert total() == 0
    terms.close()
    idx.close()


def test_more_streams_than_queue_states():
    """Batches of changing sizes on 20 streams, all in flight at once: the calls past
    the 16th wait for states that others hold."""
    import torch
    sizes = (30_000, 5_000, 12_000, 60_000)
    idx, sets = index_and_reads(sizes)
    idx.set_mode(rb.MODE_PLAIN)
    want = []
    for seqs, offs in sets:  # (in calls of 1,000, which take no queue)
        n = offs.numel() - 1
        out = torch.empty((n, idx.W), dtype=torch.int64, device="cuda")
        for i in range(0, n, 1_000):
            idx.query_seqs(seqs, offs[i:min(n, i + 1_000) + 1], out=out[i:i + 1_000], check=False)
        want.append(out)
    idx.set_mode(rb.MODE_BATCHED)
    idx.set_tune(rb.Tune(4, 1024, 16, 4, 1, 2))
    streams = [torch.cuda.Stream() for _ in range(20)]
    outs = []
    torch.cuda.synchronize()
    for rep in range(3):
        for j, st in enumerate(streams):
            k = (j + rep) % 4
            out = torch.empty_like(want[k])
            out.record_stream(st)
            outs.append((k, idx.query_seqs(*sets[k], out=out, stream=st, check=False)))
    torch.cuda.synchronize()
    assert all(torch.equal(o, want[k]) for k, o in outs)
    idx.close()


def test_fold_gives_back_what_calls_kept():
    """The scratch of a bulk insertion and the queue states of batches do not stand in
    the way of the folded rows."""
    import torch
    from tests.gpu_util import to_dev

    def free_bytes():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    K, B, R, m, eta, L, n = 150, 64, 2, 1 << 21, 3, 80_000, 300_000
    docs = torch.randint(0, 4, (K * L,), device="cuda", dtype=torch.uint8)
    docs = torch.tensor(list(b"ACGT"), dtype=torch.uint8, device="cuda")[docs.to(torch.int64)]
    ids = to_dev(np.arange(K, dtype=np.uint64))
    off = to_dev(np.arange(K + 1, dtype=np.uint64) * np.uint64(L))
    roff = to_dev(np.arange(n + 1, dtype=np.uint64) * np.uint64(31))
    out = torch.empty((n, 3), dtype=torch.int64, device="cuda")
    for _ in range(2):  # (the first loads the kernels)
        idx = rb.Rambo(K, B, R, m, eta, 9101)
        fresh = free_bytes()
        idx.insert_seqs(ids, docs, off)
        idx.query_seqs(docs, roff, out=out, check=False)
        want = out.clone()
        kept = fresh - free_bytes()
        idx.fold()
        rows = R * m * 4  # (64 cells of two words to 32 of one)
        left = fresh + rows - free_bytes()
        assert torch.equal(idx.query_seqs(docs, roff, check=False) & want, want)
        idx.close()
    assert kept > 100 << 20, kept
    assert left < 8 << 20, (kept, left)
