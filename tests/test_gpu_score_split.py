"""The prologue of the scoring launch (Algorithm 2 line 4: recalled ids and their rows) where it changes form: pages smaller than the
eight ids of a byte of the bitmap, pages larger than a block's ids, block tables that fit beside the bitmap and not (beyond
4096 entries), contexts whose bitmap is kept (to 4096 words) and read again (beyond), lengths that end inside a word, few
recalled ids for many blocks; by id range and by rank."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2512_15550_amd as ck
from ctkvr_inputs import gen_batch, small_workload
from tests import harness as H
from tests.test_gpu_share_tail import _inputs, _run


@pytest.mark.parametrize("by_rank", [0, 1])
@pytest.mark.parametrize("h,g,lens,page,rho,n_probe", [(2, 1, (301,), 1, 40, 3), (4, 2, (1003, 77), 2, 30, 4), (8, 2, (2021,), 4, 200, 6),
                                                       (8, 2, (2049, 513), 8, 256, 4), (8, 1, (40007,), 256, 900, 5),
                                                       (2, 2, (70001, 9000), 16, 700, 4), (4, 1, (131072,), 32, 3000, 4),
                                                       (4, 1, (132001,), 16, 5000, 4), (4, 1, (9001,), 16, 3, 2), (1, 1, (64,), 16, 64, 2)])
def test_recalled_ids_and_rows_match_the_oracle(h, g, lens, page, rho, n_probe, by_rank, monkeypatch):
    monkeypatch.setenv("CTKVR_SCORE_BY_RANK", str(by_rank))
    wl = small_workload("score_split", "bf16", h, g, lens, tuple(800 + i for i in range(len(lens))), 8, 0, n_probe, rho, min(rho, 100), 2, page_size=page)
    bt = gen_batch(wl)
    db = H.device_batch(bt)
    idx = ck.ctkvr_build_index(H.params_of(wl), db.q_prefill, db.cu_seqlens, True, db.k_pages, db.block_table, db.ctx_lens)
    try:
        H.run_decode_parity(bt, H.oracle_index(bt), idx, db)
    finally:
        ck.ctkvr_free(idx)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("h,g,batch,rho", [(8, 8, 2, 1024), (16, 8, 2, 1024), (32, 8, 2, 1024), (64, 8, 2, 1024), (8, 8, 2, 1025), (16, 8, 2, 1025),
                                           (32, 8, 2, 1025), (64, 8, 2, 1025), (32, 8, 3, 1025), (5, 5, 1, 1300), (4, 4, 1, 1300)])
def test_blocks_of_few_ids_by_rank(dtype, h, g, batch, rho, monkeypatch):
    """Four rounds of rows in flight or twelve, on both sides of the lines between them (256 CUs): 16 units of 32 blocks with at most 64 ids
    a block, or 65; 24 units, and more than two blocks a CU; four and five units, and fewer blocks."""
    monkeypatch.setenv("CTKVR_SCORE_BY_RANK", "1")
    lens = tuple(3201 + 13 * i for i in range(batch))
    wl = small_workload("few_ids", dtype, h, g, lens, tuple(850 + i for i in range(batch)), 4, 0, 2, rho, 100, 1)
    bt = gen_batch(wl)
    db = H.device_batch(bt)
    idx = ck.ctkvr_build_index(H.params_of(wl), db.q_prefill, db.cu_seqlens, True, db.k_pages, db.block_table, db.ctx_lens)
    try:
        assert ck.ctkvr_index_info(idx)["l_stride"] == 2 * rho
        H.run_decode_parity(bt, H.oracle_index(bt), idx, db)
    finally:
        ck.ctkvr_free(idx)


@pytest.mark.parametrize("B,g,s,rho,n_probe", [(9, 4, 22277, 514, 10), (1, 5, 131072, 4000, 8)])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_streamed_rows_by_rank_and_by_id_range_give_the_same_bits(G, B, g, s, rho, n_probe, monkeypatch):
    """More than 128 MiB of keys (non-temporal loads), more and fewer than two blocks a CU by rank."""
    p = ck.Params(batch=B, n_q_heads=G * g, n_kv_heads=g, n_centroids=16, list_len=rho, n_probe=n_probe, top_k=300, dtype=ck.BF16)
    assert B * g * s * 256 > 128 << 20
    data = _inputs("bf16", B, G, g, s, rho, 300, 1.0, 0, 4300, C=16)
    got = []
    for by_rank in ("0", "1"):
        monkeypatch.setenv("CTKVR_SCORE_BY_RANK", by_rank)
        got.append(_run(p, s, data, {"CTKVR_TAIL": "0"}, monkeypatch))
    for a, b in zip(*got):
        assert all(np.array_equal(x, y) for x, y in zip(a, b))
