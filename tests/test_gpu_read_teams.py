"""Plain-form queries at the batch sizes where the number of waves per read
changes (16, 8, 4, then one wave), as bitsets and as id lists, with and without
early exit and under every resolve: reads of 0 windows to many more than the
waves of a team take at once. Rows of 4 words (a lane a term), of 16 (4 lanes)
and of 256 words (64 lanes, masks that leave room for fewer waves), answers of
one word and of more than a team resolves densely. Bit-exact against the
oracle."""
import numpy as np
import pytest

import gen
from paper_1910_04358_amd import rambo as rb
from tests.gpu_util import build_gpu_seqs, build_oracle, make_reads, to_dev, to_host_u64

pytestmark = pytest.mark.gpu

# (K, B, R, m, eta): the last resolves by candidates straight into the answer
SHAPES = [(60, 100, 5, 1 << 17, 2), (700, 300, 6, 1 << 16, 3), (96, 8192, 8, 1 << 13, 2), (40_000, 200, 2, 1 << 18, 2)]
SIZES = (1, 16, 288, 289, 512, 513, 4096, 4097)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "K%d-B%d-R%d" % s[:3])
def test_every_team_size_equals_oracle(shape):
    K, B, R, m, eta = shape
    nd = min(K, 90)
    dm = gen.DocModel(seed=B + 5, n_docs=nd, length=4_000, docs_per_anc=9, mu_lo=0.01, mu_hi=0.01)
    idx = rb.Rambo(K, B, R, m, eta, 8700 + B)
    build_gpu_seqs(idx, dm, 0, nd)
    o = build_oracle((K, B, R, m, eta, 8700 + B), dm)
    rm = gen.ReadModel(qseed=B + 6, src_lo=0, src_hi=nd, len_kind=0, median=120, sigma=0.9, lo=31, hi=3_500,
                       err_lo=0.0, err_hi=0.005)
    r = gen.reads(dm, rm, 4_090)
    d0 = dm.doc(0)
    edge = [d0, b"", b"ACGT" * 7, b"N" * 200, d0[:31], d0[100:163], d0[:1500] + b"N" + d0[1501:]]
    seqs, offs = make_reads(edge + [r.read(i) for i in range(r.n)])
    want, _ = o.query_seqs(seqs, offs)
    bits = np.unpackbits(want.view(np.uint8), axis=1, bitorder="little")[:, :K]
    assert bits.any(axis=1).sum() > 500
    sd = to_dev(seqs)
    for n in SIZES:
        od = to_dev(offs[:n + 1])
        for resolve in (rb.RESOLVE_AUTO, rb.RESOLVE_DENSE, rb.RESOLVE_CANDIDATE):
            idx.set_resolve(resolve)
            for ee in (True, False):
                idx.set_early_exit(ee)
                got = to_host_u64(idx.query_seqs(sd, od))
                assert np.array_equal(got, want[:n]), (n, resolve, ee)
                ids, ioff = idx.query_seqs_ids(sd, od, ids_cap=int(bits[:n].sum()))
                ioff = ioff.cpu().numpy()
                assert np.array_equal(np.diff(ioff), bits[:n].sum(axis=1)), (n, resolve, ee)
                assert np.array_equal(ids.cpu().numpy(), np.nonzero(bits[:n])[1]), (n, resolve, ee)
                assert idx.last_status == (rb.OK_EMPTYQ if n > 1 else rb.OK)
    idx.sync()
    idx.close()
