"""The candidate route of the matrix-core build where its threshold and its selection change form: keys spread over many
buckets of the sample's histogram, crowded into one, and below its range; many and few segments, candidates near the most a
block holds, a resident window; every group size."""
import numpy as np
import pytest

from ctkvr_inputs import Batch, gen_batch, paginate, round_to_dtype, small_workload
from tests import harness as H

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2512_15550_amd as ck


@pytest.mark.parametrize("h,g,s,C,rho,keys,n_init,n_local", [
    (1, 1, 9001, 40, 256, 1.0, 0, 0), (4, 2, 12000, 33, 300, 1.0, 5, 200), (4, 1, 30033, 129, 700, 1.0, 0, 0), (8, 1, 12001, 40, 300, 1.0, 0, 0),
    (2, 1, 66000, 17, 2730, 1.0, 0, 0), (4, 1, 20000, 600, 400, 1.0, 0, 0),
    (4, 1, 12000, 40, 300, 2.0 ** -8, 0, 0), (2, 1, 9001, 40, 256, 2.0 ** -6, 9, 300),     # one or two buckets hold all keys
    (4, 1, 12000, 40, 300, 64.0, 0, 0), (8, 1, 9000, 33, 256, 64.0, 0, 0)])                # most keys lie below the histogram
def test_candidates_give_the_lists_of_all_keys(h, g, s, C, rho, keys, n_init, n_local, monkeypatch):
    wl = small_workload("candidates", "bf16", h, g, (s,), (700 + s,), C, 0, 4, rho, 60, 1)
    bt = gen_batch(wl)
    sq = bt.seqs[0]
    sq.K[:] = round_to_dtype(sq.K.astype(np.float64) * keys, "bf16")
    bt = Batch(wl=wl, seqs=[sq], paged=paginate([sq], wl.page_size, 5))
    db = H.device_batch(bt)
    got = []
    for cand in ("0", "1"):
        monkeypatch.setenv("CTKVR_BUILD_CANDIDATES", cand)
        idx = ck.ctkvr_build_index(H.params_of(wl, build_algo=ck.BUILD_MFMA, n_init=n_init, n_local=n_local), db.q_prefill, db.cu_seqlens,
                                   True, db.k_pages, db.block_table, db.ctx_lens)
        assert ck.ctkvr_index_build_route(idx) == (cand == "1", 0)   # and no chunk handed back
        got.append(ck.ctkvr_index_lists(idx)[0, :, :C])
        ck.ctkvr_free(idx)
    assert np.array_equal(got[0], got[1])
    assert got[0].min() >= n_init and got[0].max() < s - n_local and (np.diff(got[0], axis=-1) > 0).all()
