"""GPU parity of the dynamic centroid update (Algorithm 2 line 12): decode steps with an
update after each, on the GPU through the C ABI and in the oracle, from the same index.
Every step's integers must stay bit-equal (so a wrong slot, list or centroid shows up in the
next step's probe), and at the end the two indexes must hold the same lists and centroids."""
import numpy as np
import pytest

from ctkvr_inputs import gen_batch, small_workload
from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ck():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2512_15550_amd as ck
    ck.load_library()
    return ck


CASES = [
    # name, dtype, h, g, ctx_lens, C, div, C', rho, rho', steps
    ("same_budget", "bf16", 8, 2, (1000,), 24, 0, 4, 64, 64, 6),
    ("wraps_around", "bf16", 4, 2, (800,), 5, 0, 2, 48, 48, 12),        # more updates than slots
    ("list_longer", "bf16", 8, 2, (1500,), 16, 0, 4, 120, 50, 5),       # rho > rho': second ranking with budget rho
    ("list_shorter", "f32", 4, 2, (1200,), 12, 0, 3, 40, 90, 5),        # rho < rho'
    ("ragged_batch", "bf16", 8, 2, (700, 1333, 2049), 0, 100, 3, 80, 80, 9),   # C_i = 7, 13, 20: slots differ per sequence
    ("multi_tile", "bf16", 16, 4, (9000,), 96, 0, 12, 700, 300, 3),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_update_keeps_gpu_and_oracle_indexes_equal(ck, case):
    name, dtype, h, g, lens, C, div, n_probe, rho, top_k, steps = case
    wl = small_workload(name, dtype, h, g, lens, tuple(range(700, 700 + len(lens))), C, div, n_probe, rho, top_k, steps)
    print(f"[dcu {name}] generating", flush=True)
    bt = gen_batch(wl)
    oi = H.oracle_index(bt)
    db = H.device_batch(bt)
    cen, lst = oi.padded(wl)
    idx = ck.ctkvr_index_load(H.params_of(wl), db.ctx_lens, cen, lst)
    print(f"[dcu {name}] {steps} steps with update", flush=True)
    st = H.run_decode_parity(bt, oi, idx, db, update=True)
    ref_cen, ref_lst = oi.padded(wl)
    got_lst, got_cen = ck.ctkvr_index_lists(idx), ck.ctkvr_index_centroids(idx)
    for b, sq in enumerate(bt.seqs):
        Cb = wl.centroids_of(sq.s)
        assert np.array_equal(got_lst[b, :, :Cb], ref_lst[b, :, :Cb]), f"lists of sequence {b} differ after the updates"
        assert np.array_equal(got_cen[b, :, :Cb], ref_cen[b, :, :Cb]), f"centroids of sequence {b} differ after the updates"
    assert not np.array_equal(ref_lst, lst), "the updates changed nothing"
    print(f"[dcu {name}] ok {st}", flush=True)
    ck.ctkvr_free(idx)


def test_update_at_full_size_32k(ck):
    """cfg2 (32K context, C = 512, C' = 32, rho = rho' = 1024) in the launch shape bench.py times."""
    from ctkvr_inputs import workload
    wl = workload("cfg2")
    print("[dcu cfg2] generating", flush=True)
    bt = gen_batch(wl, n_decode=6)
    oi = H.oracle_index(bt)
    db = H.device_batch(bt)
    cen, lst = oi.padded(wl)
    idx = ck.ctkvr_index_load(H.params_of(wl), db.ctx_lens, cen, lst)
    print("[dcu cfg2] 6 steps with update", flush=True)
    st = H.run_decode_parity(bt, oi, idx, db, update=True, check_candidates=False)
    ref_cen, ref_lst = oi.padded(wl)
    assert np.array_equal(ck.ctkvr_index_lists(idx), ref_lst)
    assert np.array_equal(ck.ctkvr_index_centroids(idx), ref_cen)
    print(f"[dcu cfg2] ok {st}", flush=True)
    ck.ctkvr_free(idx)


def test_update_needs_a_decode_step_first(ck):
    import torch
    wl = small_workload("dcu_err", "bf16", 4, 2, (300,), (1,), 8, 0, 2, 32, 16, 1)
    bt = gen_batch(wl)
    oi = H.oracle_index(bt)
    db = H.device_batch(bt)
    cen, lst = oi.padded(wl)
    idx = ck.ctkvr_index_load(H.params_of(wl), db.ctx_lens, cen, lst)
    q = H.to_dev(np.stack([sq.q_decode[0] for sq in bt.seqs]), wl)
    with pytest.raises(ck.CtkvrError) as ei:
        ck.ctkvr_centroid_update(idx, q)
    assert ei.value.code == -1
    out = torch.empty((wl.batch, wl.h, wl.d), dtype=torch.float32, device="cuda")
    ck.ctkvr_decode_step(idx, q, db.k_pages, db.v_pages, db.block_table, out)
    ck.ctkvr_centroid_update(idx, q)
    with pytest.raises(ck.CtkvrError):
        ck.ctkvr_centroid_update(idx, q)     # one update per step
    torch.cuda.synchronize()
    ck.ctkvr_free(idx)


# recalled keys (probes x list length, lists that do not overlap), the update's budget being the list length: what one block keeps
# in registers and beyond, whole and broken rounds of later keys, both sides of the line to the chip-wide passes (l_stride 49152)
SECOND = [(8, 1024, 500), (3, 2731, 900), (12, 1024, 300), (11, 1119, 300), (13, 1567, 2000), (12, 4096, 800), (12, 4097, 800),
          (13, 5000, 1000), (31, 1900, 2500)]


def _second_ranking(ck, batch, s, g, n_probe, rho, top_k, equal):
    """The slot's lists after an update with budget top_k != rho against what a step of budget rho selects, id for id."""
    import torch
    h, C = 2 * g, 40
    rng = np.random.Generator(np.random.Philox(950 + n_probe + rho))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rho)
    n_pages = (s + 15) // 16

    def rows(*shape):
        x = torch.randn(shape, generator=gen, device="cuda")
        return (x.round() if equal else x).to(torch.bfloat16)

    k, v = rows(batch * n_pages, g, 16, 128), rows(batch * n_pages, g, 16, 128)
    table = torch.arange(batch * n_pages, dtype=torch.int32, device="cuda").view(batch, n_pages)
    q = rows(batch, h, 128)
    if equal:
        q = torch.where(torch.arange(128, device="cuda") < 12, q, torch.zeros_like(q))   # scores on a coarse lattice
    cen = rows(batch, h, C, 128).view(torch.int16).cpu().numpy().view(np.uint16)
    lists = np.empty((batch, g, C, rho), np.int32)
    for b in range(batch):
        for kv in range(g):   # rows of a permutation, so that any n_probe of its s // rho rows are disjoint
            part = np.sort(rng.permutation(s)[:(s // rho) * rho].reshape(-1, rho), axis=1)
            lists[b, kv] = part[np.arange(C) % part.shape[0]]
    got = {}
    for budget in (top_k, rho):
        p = ck.Params(batch=batch, n_q_heads=h, n_kv_heads=g, n_centroids=C, list_len=rho, n_probe=n_probe, top_k=budget)
        idx = ck.ctkvr_index_load(p, [s] * batch, cen, lists)
        out = torch.empty((batch, h, 128), device="cuda")
        sel = torch.empty((batch, g, budget), dtype=torch.int32, device="cuda")
        nc = torch.empty((batch, g), dtype=torch.int32, device="cuda")
        ck.ctkvr_decode_step(idx, q, k, v, table, out, out_sel=sel, out_ncand=nc)
        if budget == top_k:
            ck.ctkvr_centroid_update(idx, q)
            new = ck.ctkvr_index_lists(idx)
            assert np.array_equal(new[:, :, 1:], lists[:, :, 1:])
        else:
            want = sel.cpu().numpy()
        L = nc.cpu().numpy()
        ck.ctkvr_free(idx)
    print(f"[dcu second] L {L.min()}..{L.max()} of {min(s, n_probe * rho)}", flush=True)
    for b in range(batch):
        for kv in range(g):
            n = min(L[b, kv], rho)
            assert np.array_equal(new[b, kv, 0, :n], want[b, kv, :n])
            assert (new[b, kv, 0, n:] == new[b, kv, 0, n - 1]).all()


@pytest.mark.parametrize("step", ["tail", "keyclass", "separate", "share"])
@pytest.mark.parametrize("g,n_probe,rho,top_k,equal", [(2, *c, False) for c in SECOND] + [(8, 12, 1024, 300, False), (8, 13, 4000, 700, False),
                         (2, 12, 1024, 300, True), (2, 13, 5000, 1000, True)])
def test_second_ranking_is_the_selection_of_a_step_with_that_budget(ck, g, n_probe, rho, top_k, equal, step, monkeypatch):
    monkeypatch.setenv("CTKVR_TAIL", {"tail": "1", "share": "2"}.get(step, "0"))
    if step in ("keyclass", "separate"):
        monkeypatch.setenv("CTKVR_KEYCLASS", "1" if step == "keyclass" else "0")
    _second_ranking(ck, 1, 65537, g, n_probe, rho, top_k, equal)


@pytest.mark.parametrize("n_probe,rho", [(12, 4096), (15, 4000)])
def test_second_ranking_where_groups_of_a_batch_step_in_different_forms(ck, n_probe, rho, monkeypatch):
    """Two sequences of four KV heads in one group (tail_kernel), three in the other (share_tail_kernel)."""
    monkeypatch.setenv("CTKVR_DECODE_GROUPS", "2")
    _second_ranking(ck, 5, 61000, 4, n_probe, rho, 700, False)
