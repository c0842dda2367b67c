"""The build's small launches where their forms change: threshold and selection of the candidate route by blocks of different
sizes, the lengths of more sequences than one launch carries, prompt queries that start on any element, sequences with fewer
centroids than the table has rows, and k-means sums whose rounds lie inside and outside the range that 32 bits take."""
import numpy as np
import pytest

import oracle
from ctkvr_inputs import bf16_bits_to_f32, gen_batch, small_workload
from ctkvr_inputs.kmeans_init import kmeanspp_for_sequence
from tests import harness as H
from tests.test_gpu_kmeans import _lattice_batch

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2512_15550_amd as ck


# one sample in sixteen positions, by runs of 32: 2048 samples end at 32768 positions; 4096 candidates at lists of 1024
@pytest.mark.parametrize("G,s,rho", [(4, 32768, 1024), (4, 32769, 1024), (2, 32768, 1025), (1, 33281, 1025), (8, 9000, 1024), (4, 131072, 2048)])
def test_candidates_give_the_lists_of_all_keys_at_the_edges_of_their_blocks(G, s, rho, monkeypatch):
    wl = small_workload("cand_blocks", "bf16", G, 1, (s,), (810 + G,), 40, 0, 4, rho, 60, 1)
    db = H.device_batch(gen_batch(wl))
    got = []
    for cand in ("0", "1"):
        monkeypatch.setenv("CTKVR_BUILD_CANDIDATES", cand)
        idx = ck.ctkvr_build_index(H.params_of(wl, build_algo=ck.BUILD_MFMA), db.q_prefill, db.cu_seqlens, True, db.k_pages, db.block_table,
                                   db.ctx_lens)
        assert ck.ctkvr_index_build_route(idx) == (cand == "1", 0)
        got.append(ck.ctkvr_index_lists(idx)[0])
        ck.ctkvr_free(idx)
    assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("batch", [170, 171])   # three arrays of 512 integers in all travel with one launch
def test_lengths_of_many_sequences(batch):
    lens = tuple(64 + (37 * b) % 90 for b in range(batch))
    wl = small_workload("many", "bf16", 2, 1, lens, tuple(range(820, 820 + batch)), 0, 16, 2, 20, 16, 1)
    bt = gen_batch(wl)
    db = H.device_batch(bt)
    idx = ck.ctkvr_build_index(H.params_of(wl), db.q_prefill, db.cu_seqlens, True, db.k_pages, db.block_table, db.ctx_lens)
    oi = H.oracle_index(bt)
    lists = ck.ctkvr_index_lists(idx)
    for b, sq in enumerate(bt.seqs):
        assert np.array_equal(lists[b, :, :wl.centroids_of(sq.s)], oi.lists[b])
    H.run_decode_parity(bt, oi, idx, db)
    ck.ctkvr_free(idx)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shift", [1, 2, 4])
def test_prompt_queries_on_any_element(dtype, shift):
    """Unequal numbers of centroids, none a multiple of a block's sixteen rows: the same index as from aligned rows."""
    wl = small_workload("shifted", dtype, 8, 2, (900, 333), (830, 831), 0, 19, 4, 64, 40, 1)
    bt = gen_batch(wl)
    db = H.device_batch(bt)
    room = torch.empty(db.q_prefill.numel() + shift, dtype=db.q_prefill.dtype, device="cuda")
    moved = room[shift:].view(db.q_prefill.shape)
    moved.copy_(db.q_prefill)
    oi = H.oracle_index(bt)
    want, _ = oi.padded(wl)
    for q in (db.q_prefill, moved):
        idx = ck.ctkvr_build_index(H.params_of(wl), q, db.cu_seqlens, True, db.k_pages, db.block_table, db.ctx_lens)
        assert np.array_equal(ck.ctkvr_index_centroids(idx), want)
        H.run_decode_parity(bt, oi, idx, db)
        ck.ctkvr_free(idx)


@pytest.mark.parametrize("h,g,s,C", [(1, 1, 700, 20), (4, 2, 901, 33), (8, 2, 1100, 24), (8, 1, 650, 17)])
def test_kmeans_sums_below_and_beyond_128(h, g, s, C):
    """Lattice values (to 1) times 64, 128 and 256 beside others as they are: exact products and sums, the oracle's centres bit for bit."""
    bt = _lattice_batch(840 + s, s, h, g, C, 48, 3, 32)
    sq = bt.seqs[0]
    rng = np.random.Generator(np.random.Philox(841))
    sq.q_full *= np.choose(rng.integers(0, 6, s), [1.0, 1.0, 1.0, 64.0, 128.0, 256.0]).astype(np.float32)[:, None, None]
    sq.q_tail = sq.q_full[s - C:]
    assert np.abs(sq.q_full).max() > 128.0
    init = kmeanspp_for_sequence(sq.q_full, g, C, seed=9)
    Qc, _, _ = oracle.kmeans_centroids(sq.q_full, g, init, iters=1)
    db = H.device_batch(bt)
    qf, cu = H.device_full_queries(bt)
    ip = torch.from_numpy(np.ascontiguousarray(init[None], np.int32)).cuda()
    idx = ck.ctkvr_build_index(H.params_of(bt.wl, centroid_mode=ck.KMEANS, kmeans_iters=1), qf, cu, False, db.k_pages, db.block_table,
                               db.ctx_lens, init_pos=ip)
    assert np.array_equal(bf16_bits_to_f32(ck.ctkvr_index_centroids(idx))[0], Qc)
    ck.ctkvr_free(idx)
