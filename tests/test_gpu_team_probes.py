"""Plain-form batches of a few reads to some thousands, of reads that end early: a
read with errors is ended by few probes however long it is, as with one wave per
read (counted by the probe counter), under every number of waves per read and for
narrow and split rows; answers against the oracle, with reads long enough for
every step of the scouting."""
import numpy as np
import pytest

import gen
from paper_1910_04358_amd import rambo as rb
from tests.gpu_util import build_gpu_seqs, build_oracle, make_reads, to_dev, to_host_u64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,B,R,eta", [(60, 100, 5, 2), (90, 300, 6, 2), (60, 1000, 1, 3), (60, 8192, 2, 1)])
def test_reads_that_end_early_take_few_probes(K, B, R, eta):
    import torch
    m = 1 << 21
    dm = gen.DocModel(seed=B + 15, n_docs=K, length=12_000, docs_per_anc=6, mu_lo=0.01, mu_hi=0.01)
    idx = rb.Rambo(K, B, R, m, eta, 8710 + B)
    build_gpu_seqs(idx, dm, 0, K)
    o = build_oracle((K, B, R, m, eta, 8710 + B), dm)
    rng = np.random.default_rng(B)

    def read(L, errors):
        d = np.frombuffer(dm.doc(int(rng.integers(0, K))), np.uint8).copy()
        s = d[(a := int(rng.integers(0, d.size - L + 1))):a + L]
        at = rng.integers(0, L, errors)
        s[at] = np.frombuffer(b"TGAC", np.uint8)[(s[at] >> 1) & 3]  # (another base)
        return s.tobytes()

    probes = torch.zeros(1, dtype=torch.int64, device="cuda")
    for n in (16, 257, 600, 1_200):
        # 10 errors in 10,000 bases, one in 1,500 and in 31, none
        lens = [(10_000, 10), (2_100, 3), (1_015, 2), (31, 1), (64, 0), (1_984, 0), (1_985, 0), (2_050, 0), (9_000, 0)]
        kinds = [lens[i % len(lens)] for i in range(n)]
        reads = [read(*k) for k in kinds[:54]]
        reads = [reads[i % 54] for i in range(n)]
        seqs, offs = make_reads(reads)
        sd, od = to_dev(seqs), to_dev(offs)
        want, _ = o.query_seqs(*make_reads(reads[:54]))
        want = np.concatenate([want] * (n // 54 + 1))[:n]
        for ee in (True, False):
            idx.set_early_exit(ee)
            assert np.array_equal(to_host_u64(idx.query_seqs(sd, od)), want), (n, ee)
        idx.set_early_exit(True)
        assert want[4].any() and want[8].any()
        # long reads with errors alone: within 64 windows 31 apart of the read's
        # first 2,000 and the rest of those (9,970 windows each otherwise)
        seqs, offs = make_reads([read(10_000, 40) for _ in range(40)] * (n // 40 + 1))
        offs = offs[:n + 1]
        idx.set_probe_counter(probes)
        probes.zero_()
        got = to_host_u64(idx.query_seqs(to_dev(seqs), to_dev(offs)))
        assert not got.any()
        torch.cuda.synchronize()
        assert int(probes) <= n * eta * 400, (n, int(probes) / n / eta)
        idx.set_probe_counter(None)
    idx.close()
