"""The exact build's lists where their block changes form: 512 threads with 8 and with 32 keys each (to 4096 and to 16384
positions), 1024 threads beyond; lengths that end inside a group of 64, a resident window, equal keys; every group size."""
import numpy as np
import pytest

import oracle
from ctkvr_inputs import Batch, gen_batch, gen_lattice_sequence, paginate, small_workload
from tests import harness as H

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2512_15550_amd as ck


@pytest.mark.parametrize("dtype,h,g,s,rho,lattice,n_init,n_local", [
    ("bf16", 4, 1, 4096, 300, False, 0, 0), ("bf16", 4, 1, 4097, 300, False, 0, 0), ("f32", 2, 1, 4160, 500, False, 4, 100),
    ("bf16", 8, 1, 9001, 700, False, 0, 0), ("bf16", 4, 1, 12000, 900, True, 0, 0), ("bf16", 1, 1, 16384, 1000, False, 64, 256),
    ("bf16", 4, 1, 16385, 1000, False, 0, 0), ("bf16", 2, 1, 20033, 800, True, 0, 0)])
def test_exact_lists_equal_the_oracles(dtype, h, g, s, rho, lattice, n_init, n_local):
    C = 17
    wl = small_workload("exact_lists", dtype, h, g, (s,), (1400 + s,), C, 0, 4, rho, 64, 1)
    if lattice:
        sq = gen_lattice_sequence(1400 + s, s, h, g, 128, C, 1, denom=2, span=1)
        bt = Batch(wl=wl, seqs=[sq], paged=paginate([sq], wl.page_size, 5))
    else:
        bt = gen_batch(wl)
        sq = bt.seqs[0]
    db = H.device_batch(bt)
    idx = ck.ctkvr_build_index(H.params_of(wl, n_init=n_init, n_local=n_local), db.q_prefill, db.cu_seqlens, True, db.k_pages, db.block_table,
                               db.ctx_lens)
    got = ck.ctkvr_index_lists(idx)[0]
    ck.ctkvr_free(idx)
    assert np.array_equal(got, oracle.build_lists(sq.K, oracle.centroids_last_c(sq.q_tail, C), rho, n_init=n_init, n_local=n_local))


@pytest.mark.parametrize("dtype,h,g,s,C,rho", [
    ("bf16", 4, 1, 16400, 257, 200), ("f32", 2, 1, 16385, 300, 100), ("bf16", 1, 1, 33000, 540, 200),   # more lists than CUs: two blocks a CU
    ("bf16", 8, 1, 16900, 260, 200), ("bf16", 8, 1, 40001, 33, 400)])                                  # eight heads: one
def test_exact_lists_of_long_contexts_by_how_many_there_are(dtype, h, g, s, C, rho):
    wl = small_workload("exact_many", dtype, h, g, (s,), (1500 + s,), C, 0, 4, rho, 64, 1)
    bt = gen_batch(wl)
    sq = bt.seqs[0]
    db = H.device_batch(bt)
    idx = ck.ctkvr_build_index(H.params_of(wl), db.q_prefill, db.cu_seqlens, True, db.k_pages, db.block_table, db.ctx_lens)
    got = ck.ctkvr_index_lists(idx)[0]
    ck.ctkvr_free(idx)
    assert np.array_equal(got, oracle.build_lists(sq.K, oracle.centroids_last_c(sq.q_tail, C), rho))
