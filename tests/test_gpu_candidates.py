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


@pytest.mark.parametrize("lens,h,g,C,rho,flat", [
    ((12000, 2001, 5003), 8, 2, 0, 1000, None),     # short ones beside a long one: every key, or most, a candidate
    ((3000, 3100), 4, 4, 1100, 256, None), ((3000, 3100), 4, 4, 1100, 256, 0), ((3100, 3000), 4, 4, 1100, 256, 1)])   # two chunks, one handed back
def test_ragged_batches_and_single_chunks_handed_back(lens, h, g, C, rho, flat, monkeypatch):
    wl = small_workload("cand_ragged", "bf16", h, g, lens, tuple(range(730, 730 + len(lens))), C, 64, 4, rho, 60, 1)
    bt = gen_batch(wl)
    if flat is not None:
        bt.seqs[flat].K[:] = bt.seqs[flat].K[:, :1]
        bt = Batch(wl=wl, seqs=bt.seqs, paged=paginate(bt.seqs, wl.page_size, 7))
    db = H.device_batch(bt)
    got = []
    for cand in ("0", "1"):
        monkeypatch.setenv("CTKVR_BUILD_CANDIDATES", cand)
        idx = ck.ctkvr_build_index(H.params_of(wl, build_algo=ck.BUILD_MFMA), db.q_prefill, db.cu_seqlens, True, db.k_pages, db.block_table,
                                   db.ctx_lens)
        assert ck.ctkvr_index_build_route(idx) == (cand == "1", int(cand == "1" and flat is not None))
        lists = ck.ctkvr_index_lists(idx)
        got.append([lists[b, :, :wl.centroids_of(s)].copy() for b, s in enumerate(lens)])
        ck.ctkvr_free(idx)
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("s,C,rho,want", [(30000, 1000, 700, True), (29000, 1000, 700, False), (30000, 1000, 255, False), (16000, 2000, 1700, False)])
def test_the_route_is_chosen_by_keys_and_their_share(s, C, rho, want, monkeypatch):
    """Two KV heads: 60 M keys or more, ten of them for each one listed."""
    monkeypatch.delenv("CTKVR_BUILD_CANDIDATES", raising=False)
    wl = small_workload("cand_rule", "bf16", 2, 2, (s,), (760,), C, 0, 4, rho, 60, 1)
    db = H.device_batch(gen_batch(wl))
    idx = ck.ctkvr_build_index(H.params_of(wl, build_algo=ck.BUILD_MFMA), db.q_prefill, db.cu_seqlens, True, db.k_pages, db.block_table, db.ctx_lens)
    assert ck.ctkvr_index_build_route(idx)[0] == want
    ck.ctkvr_free(idx)


@pytest.mark.parametrize("lens,h,g,C,flat,chunks", [
    ((5003,), 8, 4, 70, [(0, 0), (0, 2), (0, 3)], 1),                 # runs of one and of two pairs beside one that stands
    ((4000, 5003), 4, 4, 1100, [(0, 3), (1, 0), (1, 2)], 2),          # the last pair of one chunk and the first of the next
    ((5003, 2500), 16, 2, 40, [(1, 1)], 1)])                          # eight heads
def test_only_what_failed_is_handed_back_with_its_statistics(lens, h, g, C, flat, chunks, monkeypatch):
    """Keys of some (sequence, KV head) pairs all equal: ranked by the route of all keys from the statistics of the first round."""
    wl = small_workload("cand_pairs", "bf16", h, g, lens, tuple(range(770, 770 + len(lens))), C, 0, 4, 256, 60, 1)
    bt = gen_batch(wl)
    for b, kv in flat:
        bt.seqs[b].K[kv] = bt.seqs[b].K[kv, :1]
    bt = Batch(wl=wl, seqs=bt.seqs, paged=paginate(bt.seqs, wl.page_size, 7))
    db = H.device_batch(bt)
    got = []
    for cand in ("0", "1"):
        monkeypatch.setenv("CTKVR_BUILD_CANDIDATES", cand)
        idx = ck.ctkvr_build_index(H.params_of(wl, build_algo=ck.BUILD_MFMA), db.q_prefill, db.cu_seqlens, True, db.k_pages, db.block_table,
                                   db.ctx_lens)
        assert ck.ctkvr_index_build_route(idx) == (cand == "1", chunks if cand == "1" else 0)
        got.append(ck.ctkvr_index_lists(idx))
        ck.ctkvr_free(idx)
    assert np.array_equal(*got)


@pytest.mark.parametrize("s,rho", [(131072, 2048), (200001, 2048), (262144, 2048), (262144, 1024)])
def test_flat_scores_of_long_contexts_fit_their_candidates(s, rho, monkeypatch):
    """Scores so alike that a bucket of the sample's histogram holds a good part of what is wanted: nothing is handed back."""
    wl = small_workload("cand_flat", "bf16", 4, 1, (s,), (780,), 129, 0, 4, rho, 60, 1)
    sq = gen_batch(wl).seqs[0]
    k = sq.K
    for scale in (0.03, 0.02, 0.015, 0.01):
        sq.K = round_to_dtype(k.astype(np.float64) * scale, "bf16")
        db = H.device_batch(Batch(wl=wl, seqs=[sq], paged=paginate([sq], wl.page_size, 5)))
        got = []
        for cand in ("0", "1"):
            monkeypatch.setenv("CTKVR_BUILD_CANDIDATES", cand)
            idx = ck.ctkvr_build_index(H.params_of(wl, build_algo=ck.BUILD_MFMA), db.q_prefill, db.cu_seqlens, True, db.k_pages,
                                       db.block_table, db.ctx_lens)
            assert ck.ctkvr_index_build_route(idx) == (cand == "1", 0), scale
            got.append(ck.ctkvr_index_lists(idx))
            ck.ctkvr_free(idx)
        assert np.array_equal(*got)


@pytest.mark.parametrize("lens,g,C,rho,want", [
    ((98304,), 1, 16, 256, True), ((98303,), 1, 16, 256, False),                # few lists: by their length
    ((32769,), 4, 228, 512, False), ((33000,), 4, 228, 512, True),              # 30.0 M keys, just under and over
    ((32768,), 4, 230, 512, False), ((33000,), 4, 228, 1100, False),            # (not longer than 32768; fewer than 32 for each one listed)
    ((100000, 30000), 1, 16, 256, False)])
def test_the_route_of_few_long_lists(lens, g, C, rho, want, monkeypatch):
    monkeypatch.delenv("CTKVR_BUILD_CANDIDATES", raising=False)
    wl = small_workload("cand_long", "bf16", g, g, lens, tuple(range(790, 790 + len(lens))), C, 0, 4, rho, 60, 1)
    db = H.device_batch(gen_batch(wl))
    lists = []
    for forced in (None, "0"):
        if forced:
            monkeypatch.setenv("CTKVR_BUILD_CANDIDATES", forced)
        idx = ck.ctkvr_build_index(H.params_of(wl, build_algo=ck.BUILD_MFMA), db.q_prefill, db.cu_seqlens, True, db.k_pages, db.block_table,
                                   db.ctx_lens)
        assert ck.ctkvr_index_build_route(idx) == (want and not forced, 0)
        lists.append(ck.ctkvr_index_lists(idx))
        ck.ctkvr_free(idx)
    assert np.array_equal(*lists)


@pytest.mark.parametrize("s,want", [(475136, True), (475137, False)])
def test_the_route_ends_where_the_sample_is_too_small(s, want, monkeypatch):
    """1 in 58 positions sampled: 52 of them at the threshold, and 2.5 sqrt(52) more, stand for 4061 of the 4096 keys that fit; 1 in 59: for 4131."""
    monkeypatch.delenv("CTKVR_BUILD_CANDIDATES", raising=False)
    wl = small_workload("cand_end", "bf16", 1, 1, (s,), (810,), 3, 0, 2, 1024, 60, 1)
    db = H.device_batch(gen_batch(wl))
    idx = ck.ctkvr_build_index(H.params_of(wl, build_algo=ck.BUILD_MFMA), db.q_prefill, db.cu_seqlens, True, db.k_pages, db.block_table, db.ctx_lens)
    assert ck.ctkvr_index_build_route(idx)[0] == want
    ck.ctkvr_free(idx)


@pytest.mark.parametrize("s,rho", [(700001, 2048), (1 << 20, 300)])
def test_forced_candidates_of_the_longest_contexts(s, rho, monkeypatch):
    """Bitmaps beyond what once shared the memory with the candidates: the lists of all keys, handed back or not."""
    wl = small_workload("cand_longest", "bf16", 1, 1, (s,), (811,), 9, 0, 2, rho, 60, 1)
    db = H.device_batch(gen_batch(wl))
    lists = []
    for cand in ("0", "1"):
        monkeypatch.setenv("CTKVR_BUILD_CANDIDATES", cand)
        idx = ck.ctkvr_build_index(H.params_of(wl, build_algo=ck.BUILD_MFMA), db.q_prefill, db.cu_seqlens, True, db.k_pages, db.block_table, db.ctx_lens)
        assert ck.ctkvr_index_build_route(idx)[0] == (cand == "1")
        lists.append(ck.ctkvr_index_lists(idx))
        ck.ctkvr_free(idx)
    assert np.array_equal(*lists)
