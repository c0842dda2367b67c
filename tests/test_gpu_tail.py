"""What follows the scoring in one launch (tail_kernel) against the separate launches it replaces: the same integers bit
for bit and outputs within rounding, where its branches change -- the recalled keys a block keeps in registers (8192) and
beyond, every key kept (top_k >= L), few recalled keys, a crowded deciding bucket (equal keys), one to 64 units, every
group size, and a block that never sees its siblings' sums and takes them all itself."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2512_15550_amd as ck
from ctkvr_inputs import Batch, gen_batch, gen_lattice_sequence, paginate, small_workload
from ctkvr_inputs.device import device_batch, params_of, to_dev

CASES = {  # dtype, h, g, ctx_lens, C, n_probe, rho, top_k, lattice
    "ordinary": ("bf16", 8, 2, (3000,), 48, 6, 200, 160, False),
    "one_unit_f32": ("f32", 4, 1, (900,), 24, 4, 64, 48, False),
    "beyond_registers": ("bf16", 8, 2, (20000, 9000), 64, 24, 2400, 1000, False),
    "rounds_of_later_keys": ("bf16", 8, 2, (12289, 16447), 32, 32, 8000, 900, False),   # whole and broken rounds of eight
    "just_past_registers": ("bf16", 4, 1, (8257,), 32, 32, 6000, 700, False),
    "every_key_kept": ("bf16", 8, 2, (700,), 24, 2, 60, 300, False),
    "equal_keys": ("bf16", 8, 2, (4000,), 32, 8, 600, 500, True),
    "group_1_many_units": ("bf16", 16, 16, (2000, 1500, 900, 800), 40, 5, 128, 100, False),
    "group_2": ("bf16", 16, 8, (2500,), 40, 5, 256, 300, False),
    "group_8": ("bf16", 16, 2, (6000, 3111), 64, 10, 400, 600, False),
}


def _steps(wl, bt, env, monkeypatch):
    for k in ("CTKVR_TAIL", "CTKVR_TAIL_SPINS", "CTKVR_KEYCLASS"):
        monkeypatch.delenv(k, raising=False)
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    db = device_batch(bt)
    idx = ck.ctkvr_build_index(params_of(wl), db.q_prefill, db.cu_seqlens, True, db.k_pages, db.block_table, db.ctx_lens)
    got = []
    for st in range(2):
        out = torch.full((wl.batch, wl.h, wl.d), float("nan"), device="cuda")
        lse = torch.full((wl.batch, wl.h), float("nan"), device="cuda")
        sel = torch.full((wl.batch, wl.g, wl.top_k), -5, dtype=torch.int32, device="cuda")
        ncand = torch.full((wl.batch, wl.g), -5, dtype=torch.int32, device="cuda")
        q = to_dev(np.stack([sq.q_decode[st] for sq in bt.seqs]), wl)
        ck.ctkvr_decode_step(idx, q, db.k_pages, db.v_pages, db.block_table, out, lse, sel, ncand)
        torch.cuda.synchronize()
        got.append([t.cpu().numpy() for t in (out, lse, sel, ncand)])
    ck.ctkvr_free(idx)
    return got


@pytest.mark.parametrize("name", CASES)
def test_one_launch_equals_the_separate_ones(name, monkeypatch):
    dtype, h, g, lens, C, n_probe, rho, top_k, lattice = CASES[name]
    wl = small_workload("tail_" + name, dtype, h, g, lens, tuple(range(700, 700 + len(lens))), C, 0, n_probe, rho, top_k, 2)
    if lattice:
        seqs = [gen_lattice_sequence(s, n, h, g, 128, C, 2, denom=2, span=1) for s, n in zip(wl.seeds, lens)]
        bt = Batch(wl=wl, seqs=seqs, paged=paginate(seqs, 16, 3))
    else:
        bt = gen_batch(wl)
    ref = _steps(wl, bt, {"CTKVR_TAIL": "0"}, monkeypatch)
    if name in ("beyond_registers", "rounds_of_later_keys"):
        assert ref[0][3].max() > 8192
    for env in ({"CTKVR_TAIL": "1"}, {"CTKVR_TAIL": "1", "CTKVR_TAIL_SPINS": "0"}):
        for st, (a, b) in enumerate(zip(_steps(wl, bt, env, monkeypatch), ref)):
            assert np.array_equal(a[2], b[2]) and np.array_equal(a[3], b[3]), f"{env} step {st}: selection differs"
            assert np.allclose(a[0], b[0], rtol=2e-5, atol=2e-5 * np.abs(b[0]).max()), f"{env} step {st}"
            assert np.allclose(a[1], b[1], rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("g,s,one", [(2, 32768, True), (2, 32769, False), (8, 65536, True), (8, 65537, False)])
def test_the_choice_on_both_sides_of_its_lines(g, s, one, monkeypatch):
    """tail_kernel up to l_stride 32768, or 65536 with a multiple of eight units, and share_tail_kernel beyond; the same integers in
    every form, and the bits of the attention, which each form sums in its own order, tell which form ran.  CTKVR_TAIL=0 is the
    separate launches: the bits they have with either way to the selection."""
    h, C, n_probe, rho, top_k = 4 * g, 40, 24, 3000, 700
    gen = torch.Generator(device="cuda")
    gen.manual_seed(s)
    n_pages = (s + 15) // 16
    k = torch.randn((n_pages, g, 16, 128), generator=gen, device="cuda").to(torch.bfloat16)
    v = torch.randn((n_pages, g, 16, 128), generator=gen, device="cuda").to(torch.bfloat16)
    q = torch.randn((1, h, 128), generator=gen, device="cuda").to(torch.bfloat16)
    table = torch.randperm(n_pages, generator=gen, device="cuda").to(torch.int32).view(1, -1)
    cen = torch.randn((1, h, C, 128), generator=gen, device="cuda").to(torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)
    rng = np.random.Generator(np.random.Philox(s))
    lists = np.stack([np.sort(rng.choice(s, rho, replace=False)) for _ in range(g * C)]).astype(np.int32).reshape(1, g, C, rho)
    p = ck.Params(batch=1, n_q_heads=h, n_kv_heads=g, n_centroids=C, list_len=rho, n_probe=n_probe, top_k=top_k)
    got = {}
    forms = {None: {}, "0": {"CTKVR_TAIL": "0"}, "1": {"CTKVR_TAIL": "1"}, "2": {"CTKVR_TAIL": "2"}, "two": {"CTKVR_KEYCLASS": "0"},
             "merged": {"CTKVR_KEYCLASS": "1"}}
    for tail, env in forms.items():
        monkeypatch.delenv("CTKVR_TAIL", raising=False)
        monkeypatch.delenv("CTKVR_KEYCLASS", raising=False)
        for name, value in env.items():
            monkeypatch.setenv(name, value)
        idx = ck.ctkvr_index_load(p, [s], cen, lists)
        assert ck.ctkvr_index_info(idx)["l_stride"] == s
        out = torch.full((1, h, 128), float("nan"), device="cuda")
        sel = torch.full((1, g, top_k), -5, dtype=torch.int32, device="cuda")
        ck.ctkvr_decode_step(idx, q, k, v, table, out, out_sel=sel)
        got[tail] = (out.cpu().numpy(), sel.cpu().numpy())
        ck.ctkvr_free(idx)
    for tail in forms:
        assert np.array_equal(got[tail][1], got["1"][1])
        assert np.allclose(got[tail][0], got["1"][0], rtol=2e-5, atol=2e-5 * np.abs(got["1"][0]).max())
    assert np.array_equal(got["0"][0], got["two"][0]) and np.array_equal(got["0"][0], got["merged"][0])
    assert not np.array_equal(got["0"][0], got["1"][0]) and not np.array_equal(got["0"][0], got["2"][0])
    # (share_tail_kernel's bits differ between calls where a wait expires)
    assert np.array_equal(got[None][0], got["1"][0]) == one and not np.array_equal(got[None][0], got["0"][0])
