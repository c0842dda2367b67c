"""The positions of a k-means iteration sorted by centre, where the sort's stretches change: one stretch and a second of one position,
32 stretches of exactly 1024 and of one more, a broken last one; many members of one centre; two sequences of unequal
length.  Exact products and sums, so the first update is the oracle's bit for bit whatever the order inside a centre."""
import numpy as np
import pytest

import oracle
from ctkvr_inputs import Batch, bf16_bits_to_f32, paginate, small_workload
from tests import harness as H
from tests.test_gpu_kmeans import _lattice_batch

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2512_15550_amd as ck


@pytest.mark.parametrize("h,g,lens,C,crowd", [(4, 1, (1025,), 33, 0), (2, 2, (32768,), 65, 0), (4, 1, (32769,), 40, 5000),
                                              (8, 1, (40003,), 31, 700), (2, 1, (34000, 1500), 64, 0)])
def test_first_update_over_many_stretches(h, g, lens, C, crowd):
    parts = [_lattice_batch(1200 + s + C, s, h, g, C, 64, 4, 48) for s in lens]
    seqs = [p.seqs[0] for p in parts]
    rng = np.random.Generator(np.random.Philox(1300 + C))
    if crowd:
        for sq in seqs:
            at = rng.permutation(sq.s)[:crowd]
            sq.q_full[at] = sq.q_full[at[0]]
            sq.q_tail = sq.q_full[sq.s - C:]
    wl = small_workload("km_stretches", "bf16", h, g, lens, tuple(range(len(lens))), C, 0, 4, 64, 48, 2)
    bt = Batch(wl=wl, seqs=seqs, paged=paginate(seqs, wl.page_size, 9))
    init = np.stack([np.stack([np.sort(rng.permutation(sq.s)[:C]) for _ in range(g)]) for sq in seqs]).astype(np.int32)
    db = H.device_batch(bt)
    qf, cu = H.device_full_queries(bt)
    for _ in range(2):   # the second build finds the first one's scratch
        idx = ck.ctkvr_build_index(H.params_of(wl, centroid_mode=ck.KMEANS, kmeans_iters=1, build_algo=ck.BUILD_MFMA), qf, cu, False,
                                   db.k_pages, db.block_table, db.ctx_lens, init_pos=torch.from_numpy(init).cuda())
        cen = bf16_bits_to_f32(ck.ctkvr_index_centroids(idx))
        ck.ctkvr_free(idx)
        for b, sq in enumerate(seqs):
            Qc, _, _ = oracle.kmeans_centroids(sq.q_full, g, init[b], iters=1)
            assert np.array_equal(cen[b], Qc), (lens, b)
