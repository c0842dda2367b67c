"""The matrix-core build kernels at the edges of their tiles: key steps of 64 that end after 1, 31, 32, 33 or 63 keys,
centroid tiles of one row more or less than they hold, every group size; in k-means the same for points and centres, and
centres of more members than one block sums; lists of long contexts; and the fp32 matrix instruction itself."""
import os

import numpy as np
import pytest

import oracle
from ctkvr_inputs import Batch, bf16_bits_to_f32, gen_batch, gen_lattice_sequence, paginate, small_workload
from ctkvr_inputs.kmeans_init import kmeanspp_for_sequence
from tests import harness as H
from tests.test_gpu_kmeans import _lattice_batch
from tests.test_gpu_parity import _check_lists_within_band

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2512_15550_amd as ck


@pytest.mark.parametrize("h,g,s,C", [(2, 2, 1024 + 1, 257), (4, 4, 2048 - 33, 33), (4, 2, 1024 + 31, 129), (8, 4, 3072 + 32, 63),
                                     (8, 2, 2048 + 33, 65), (4, 1, 1024 - 1, 31), (8, 1, 2048 + 63, 32), (16, 2, 1024 + 64, 33)])
def test_matrix_core_lists_at_tile_edges(h, g, s, C, monkeypatch):
    """Inputs whose dot products are exact in fp32: only the denominators' sums separate the lists from the oracle's
    (the derived band), and the two routes rank the same keys."""
    rho = 300
    wl = small_workload("tile_edges", "bf16", h, g, (s,), (90 + s,), C, 0, 4, rho, 60, 1)
    sq = gen_lattice_sequence(90 + s, s, h, g, 128, C, 1)
    bt = Batch(wl=wl, seqs=[sq], paged=paginate([sq], wl.page_size, 5))
    db = H.device_batch(bt)
    got = []
    for cand in ("0", "1"):
        monkeypatch.setenv("CTKVR_BUILD_CANDIDATES", cand)
        idx = ck.ctkvr_build_index(H.params_of(wl, build_algo=ck.BUILD_MFMA), db.q_prefill, db.cu_seqlens, True, db.k_pages,
                                   db.block_table, db.ctx_lens)
        got.append(ck.ctkvr_index_lists(idx)[0])
        ck.ctkvr_free(idx)
    assert np.array_equal(got[0], got[1])
    n_diff, _, _ = _check_lists_within_band(got[0], sq, oracle.centroids_last_c(sq.q_tail, C), wl, exact_dots=True)
    assert n_diff <= 0.001 * got[0].size


@pytest.mark.parametrize("h,g,s,C,crowd", [(2, 2, 511, 65, 0), (4, 4, 1025, 33, 0), (4, 2, 513, 64, 0), (8, 4, 257, 127, 0),
                                           (8, 2, 769, 63, 0), (8, 2, 2000, 65, 1281), (8, 1, 1409, 33, 0), (8, 1, 1300, 31, 769),
                                           (2, 2, 1800, 20, 1024), (4, 2, 1500, 40, 257)])
def test_kmeans_first_update_at_tile_edges(h, g, s, C, crowd):
    """Exact products and sums, so the first update is the oracle's bit for bit; with `crowd` that many positions hold
    one vector, hence one centre."""
    bt = _lattice_batch(900 + s + C, s, h, g, C, 64, 4, 48)
    sq = bt.seqs[0]
    if crowd:
        at = np.random.Generator(np.random.Philox(901)).permutation(s)[:crowd]
        sq.q_full[at] = sq.q_full[at[0]]
        sq.q_tail = sq.q_full[s - C:]
    init = kmeanspp_for_sequence(sq.q_full, g, C, seed=7)
    for iters in (1, 1):   # the second build finds the first one's accumulators
        Qc, _, _ = oracle.kmeans_centroids(sq.q_full, g, init, iters=iters)
        db = H.device_batch(bt)
        qf, cu = H.device_full_queries(bt)
        ip = torch.from_numpy(np.ascontiguousarray(init[None], np.int32)).cuda()
        idx = ck.ctkvr_build_index(H.params_of(bt.wl, centroid_mode=ck.KMEANS, kmeans_iters=iters), qf, cu, False, db.k_pages,
                                   db.block_table, db.ctx_lens, init_pos=ip)
        cen = bf16_bits_to_f32(ck.ctkvr_index_centroids(idx))
        ck.ctkvr_free(idx)
        assert np.array_equal(cen[0], Qc)


@pytest.mark.parametrize("s,lattice", [(16385, False), (32768, True), (32769, False), (40001, False), (65600, True)])
def test_every_key_lists_of_long_contexts(s, lattice, monkeypatch):
    """One block per list over all its keys, beyond 16384 positions (64 keys a thread in registers) and beyond 32768 (1024
    threads, later keys read again): the lists of the candidate route, which selects otherwise, and the oracle's within the band;
    on the lattice many keys are equal."""
    h, g, C, rho = 8, 2, 33, 700
    wl = small_workload("long_lists", "bf16", h, g, (s,), (60 + s,), C, 0, 4, rho, 60, 1)
    if lattice:
        sq = gen_lattice_sequence(60 + s, s, h, g, 128, C, 1, denom=2, span=1)
        bt = Batch(wl=wl, seqs=[sq], paged=paginate([sq], wl.page_size, 5))
    else:
        bt = gen_batch(wl)
        sq = bt.seqs[0]
    db = H.device_batch(bt)
    got = {}
    for cand in ("0", "1"):
        monkeypatch.setenv("CTKVR_BUILD_CANDIDATES", cand)
        idx = ck.ctkvr_build_index(H.params_of(wl, build_algo=ck.BUILD_MFMA), db.q_prefill, db.cu_seqlens, True, db.k_pages,
                                   db.block_table, db.ctx_lens)
        by_cand, redone = ck.ctkvr_index_build_route(idx)
        assert by_cand == (cand == "1") and (lattice or not redone)
        got[cand] = ck.ctkvr_index_lists(idx)[0]
        ck.ctkvr_free(idx)
    assert np.array_equal(got["0"], got["1"])
    pairs = np.array([[kv, j] for kv in range(g) for j in (0, 1, 16, 31, 32)], np.int32)
    _check_lists_within_band(got["0"], sq, oracle.centroids_last_c(sq.q_tail, C), wl, pairs=pairs, exact_dots=lattice)


def test_fp32_matrix_instruction_is_a_chain_of_fused_multiply_adds():
    """What the exact list build's bit-reproducibility rests on (the program compares 2 M results with fmaf)."""
    import subprocess
    from paper_2512_15550_amd.build import PROBE_DIR
    r = subprocess.run([os.path.join(PROBE_DIR, "mfma_chain_probe")], capture_output=True, text=True, timeout=60)
    print(r.stdout, flush=True)
    assert r.returncode == 0 and r.stdout.count(": 0 of 524288") == 4, r.stdout + r.stderr
