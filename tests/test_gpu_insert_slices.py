"""Insertions of a few documents out of a large buffer cost what the documents
cost, in time and in memory, and the scratch of a bulk insertion stays within its
documented size; documents that turn out shorter than the estimate that chooses
the bulk path are inserted all the same (against the same documents one by one)."""
import time

import numpy as np
import pytest

from paper_1910_04358_amd import rambo as rb
from tests.gpu_util import to_dev
from tests.test_gpu_bulk_insert import one_by_one

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def bases(n):
    import torch
    return torch.tensor(list(b"ACGT"), dtype=torch.uint8, device="cuda")[torch.randint(0, 4, (n,), device="cuda")]


def free_bytes():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def seconds(f):
    import torch
    best = 1e9
    for _ in range(10):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


def test_one_document_of_a_large_buffer():
    import torch
    K, B, R, m, eta, L = 1_000, 32, 4, 1 << 24, 3, 20_000
    idx = rb.Rambo(K, B, R, m, eta, 8701)
    big = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
    for i in range(0, big.numel(), 1 << 26):
        big[i:i + (1 << 26)] = bases(1 << 26)
    ids = torch.zeros(1, dtype=torch.int64, device="cuda")
    off = torch.tensor([L, 2 * L], dtype=torch.int64, device="cuda")
    small = big[L:2 * L].clone()
    off0 = torch.tensor([0, L], dtype=torch.int64, device="cuda")
    own = seconds(lambda: idx.insert_seqs(ids, small, off0))
    before = free_bytes()
    part = seconds(lambda: idx.insert_seqs(ids, big, off))
    assert before - free_bytes() < 16 * MIB
    # the bits are set already: both are one launch that looks (the launches of a
    # bulk insertion of 1 GiB, hundreds, take milliseconds even when they find nothing)
    assert part < 4 * own + 100e-6, (part, own)
    idx.sync()
    idx.close()


def test_scratch_stays_within_its_documented_size():
    K, B, R, m, eta, L = 740, 20, 2, 1 << 21, 3, 124_600
    offs = to_dev(np.arange(K + 1, dtype=np.uint64) * np.uint64(L))
    ids = to_dev(np.arange(K, dtype=np.uint64))
    docs = bases(K * L)
    for _ in range(2):  # (the first loads the kernels)
        idx = rb.Rambo(K, B, R, m, eta, 8702)
        before = free_bytes()
        idx.insert_seqs(ids, docs, offs)
        taken = before - free_bytes()
        idx.sync()
        idx.close()
    assert 64 * MIB < taken <= 256 * MIB, taken  # (the rows are smaller)


@pytest.mark.parametrize("n,L", [(40, 1_000), (64, 50), (17, 30)])
def test_short_documents_of_a_large_buffer(n, L):
    K, B, R, m, eta, seed = 64, 20, 3, 1 << 21, 3, 8703
    rng = np.random.default_rng(n)
    docs = rng.choice(np.frombuffer(b"ACGT", np.uint8), 16 * MIB)
    offs = (np.arange(n + 1) * L + 12_345).astype(np.uint64)
    ids = rng.integers(0, K, n).astype(np.uint64)
    a, b = (rb.Rambo(K, B, R, m, eta, seed) for _ in range(2))
    a.insert_seqs(to_dev(ids), to_dev(docs), to_dev(offs))
    one_by_one(b, ids, docs, offs)
    assert a.sync() == rb.OK and b.sync() == rb.OK
    assert np.array_equal(a.copy_rows(), b.copy_rows())
    a.close()
    b.close()
