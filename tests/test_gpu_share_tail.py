"""What follows the scoring with a unit's recalled keys shared out over its blocks (share_tail_kernel) against the separate
launches: the same integers bit for bit and outputs within rounding, where its branches change -- one to eight blocks a unit, keys
beyond those in registers, a wave with more picks than it takes at a time, shares without keys, every key kept, flat scores (a
second histogram), a bucket of 129 to 512 keys (likewise; so many equal ones are ranked all the same), scores below the histogram's range (a second
and a third, or a block goes on alone), equal keys (likewise), a head whose picks' weights vanish, the
resident window, groups of sequences side by side, the static scratch, and blocks that never see their siblings' words."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2512_15550_amd as ck

SEPARATE = {"CTKVR_TAIL": "0", "CTKVR_KEYCLASS": "0"}
CASES = {  # dtype, batch, G, g, s, lists' length, probes, top_k, scale of the queries, number of resident tokens
    "eight_blocks": ("bf16", 1, 4, 8, 9000, 700, 12, 500, 1.0, 0),
    "four_blocks_f32": ("f32", 6, 2, 8, 5003, 700, 12, 333, 1.0, 0),
    "two_blocks_g8": ("bf16", 12, 8, 8, 4001, 300, 16, 640, 1.0, 0),
    "one_block": ("bf16", 17, 1, 8, 3001, 300, 9, 100, 1.0, 0),
    "later_keys_and_many_picks": ("bf16", 17, 4, 8, 10007, 2000, 24, 4000, 1.0, 0),
    "later_keys_g8": ("bf16", 1, 8, 2, 60001, 4000, 40, 1500, 1.0, 0),
    "most_keys_picked": ("bf16", 1, 4, 2, 20000, 2000, 20, 8191, 1.0, 0),
    "shares_without_keys": ("bf16", 1, 4, 2, 1000, 70, 3, 65, 1.0, 0),
    "every_key": ("bf16", 2, 4, 8, 3000, 100, 3, 301, 1.0, 0),
    "flat_scores": ("bf16", 1, 4, 8, 30000, 3000, 16, 1000, 0.01, 0),
    "equal_keys": ("bf16", 1, 4, 8, 5000, 300, 8, 700, 0.0, 0),
    "crowded_bucket": ("bf16", 4, 4, 8, 4099, 350, 12, 1024, 1.0, 0),
    "few_equal_keys": ("bf16", 2, 4, 8, 450, 100, 8, 200, 0.0, 0),
    "below_the_range": ("bf16", 1, 2, 8, 2000, 300, 8, 1100, 40.0, 0),
    "many_below_the_range": ("bf16", 1, 1, 2, 120001, 20000, 40, 8000, 26.0, 0),
    "below_both_ranges": ("bf16", 1, 2, 8, 3000, 300, 8, 900, 300.0, 0),
    "last_bucket_decides": ("f32", 1, 1, 8, 900, 100, 5, 300, 60.0, 0),
    "weights_vanish": ("bf16", 1, 2, 8, 3000, 300, 8, 1, 40.0, 0),
    "window": ("bf16", 5, 4, 8, 4100, 300, 12, 400, 1.0, 96),
}


def _inputs(dtype, B, G, g, s, rho, top_k, scale, win, seed, C=48):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    h, n_pages = G * g, (s + 15) // 16
    k = torch.randn((B * n_pages, g, 16, 128), generator=gen, device="cuda").to(dt)
    v = torch.randn((B * n_pages, g, 16, 128), generator=gen, device="cuda").to(dt)
    q = (scale * torch.randn((B, h, 128), generator=gen, device="cuda")).to(dt)
    if scale == 0.0:
        q[...] = 1e-30       # every score rounds to the same small number's neighbourhood: long runs of equal keys
    table = torch.randperm(B * n_pages, generator=gen, device="cuda").to(torch.int32).view(B, n_pages)
    cen = torch.randn((B, h, C, 128), generator=gen, device="cuda").to(dt)
    cen = cen.view(torch.int16).cpu().numpy().view(np.uint16) if dtype == "bf16" else cen.cpu().numpy()
    rng = np.random.Generator(np.random.Philox(seed))
    ids = np.arange(win, s - win)
    lists = np.stack([np.sort(rng.choice(ids, rho, replace=False)) for _ in range(g * C)]).astype(np.int32)
    lists = np.ascontiguousarray(np.broadcast_to(lists.reshape(1, g, C, rho), (B, g, C, rho)))
    return k, v, q, table, cen, lists


def _run(p, s, data, env, monkeypatch, static=False):
    for name in ("CTKVR_TAIL", "CTKVR_KEYCLASS", "CTKVR_TAIL_SPINS", "CTKVR_SHARE_LATE", "CTKVR_DECODE_GROUPS"):
        monkeypatch.delenv(name, raising=False)
    for name, value in env.items():
        monkeypatch.setenv(name, value)
    k, v, q, table, cen, lists = data
    idx = ck.ctkvr_index_load(p, [s] * p.batch, cen, lists)
    got = []
    for st in range(2):      # the second step finds what the first left behind
        qs = q if st == 0 else q.roll(1, dims=1).contiguous()
        out = torch.full((p.batch, p.n_q_heads, 128), float("nan"), device="cuda")
        lse = torch.full((p.batch, p.n_q_heads), float("nan"), device="cuda")
        sel = torch.full((p.batch, p.n_kv_heads, p.top_k), -5, dtype=torch.int32, device="cuda")
        ncand = torch.full((p.batch, p.n_kv_heads), -5, dtype=torch.int32, device="cuda")
        step = ck.ctkvr_decode_step_static if static else ck.ctkvr_decode_step
        step(idx, qs, k, v, table, out, lse, sel, ncand)
        torch.cuda.synchronize()
        got.append([t.cpu().numpy() for t in (out, lse, sel, ncand)])
    ck.ctkvr_free(idx)
    return got


def _same(got, ref, what):
    # the same fp32 terms in another order: sums of n terms differ by some sqrt(n) 2^-24 of the largest, n <= 8191
    for st, (a, b) in enumerate(zip(got, ref)):
        assert np.array_equal(a[3], b[3]) and np.array_equal(a[2], b[2]), f"{what} step {st}: selection differs"
        assert np.allclose(a[0], b[0], rtol=2e-5, atol=2e-5 * np.abs(b[0]).max()), f"{what} step {st}"
        assert np.allclose(a[1], b[1], rtol=1e-5, atol=1e-5), f"{what} step {st}"


def _params(name):
    dtype, B, G, g, s, rho, n_probe, top_k, scale, win = CASES[name]
    p = ck.Params(batch=B, n_q_heads=G * g, n_kv_heads=g, n_centroids=48, list_len=rho, n_probe=n_probe, top_k=top_k,
                  dtype=ck.BF16 if dtype == "bf16" else ck.F32, n_init=win, n_local=win)
    return p, s, _inputs(dtype, B, G, g, s, rho, top_k, scale, win, 4000 + len(name))


@pytest.mark.parametrize("name", CASES)
def test_shared_out_keys_equal_the_separate_launches(name, monkeypatch):
    p, s, data = _params(name)
    ref = _run(p, s, data, SEPARATE, monkeypatch)
    if name == "every_key":
        assert ref[0][3].max() <= p.top_k
    if name == "later_keys_g8":
        assert ref[0][3].max() > 8 * 512 * 8        # more than eight blocks keep
    _same(_run(p, s, data, {"CTKVR_TAIL": "2"}, monkeypatch), ref, "shared out")
    _same(_run(p, s, data, {"CTKVR_TAIL": "2", "CTKVR_TAIL_SPINS": "0"}, monkeypatch), ref, "alone")


@pytest.mark.parametrize("block", ["", ":0", ":1"])
@pytest.mark.parametrize("wait", [0, 1, 2, 3])
@pytest.mark.parametrize("name", ["two_blocks_g8", "four_blocks_f32", "eight_blocks", "many_below_the_range"])
def test_a_wait_that_expires_in_every_block_or_in_one(name, wait, block, monkeypatch):
    """Of the sums, the histograms, the deciding bucket's keys or the outputs: all blocks of a unit go on alone, or one does and the
    others, which wait for what it never writes, follow it or have finished."""
    p, s, data = _params(name)
    _same(_run(p, s, data, {"CTKVR_TAIL": "2", "CTKVR_SHARE_LATE": f"{wait}{block}"}, monkeypatch), _run(p, s, data, SEPARATE, monkeypatch),
          f"wait {wait}{block}")


def test_shared_out_keys_of_groups_and_on_the_static_scratch(monkeypatch):
    p, s, data = _params("four_blocks_f32")
    ref = _run(p, s, data, SEPARATE, monkeypatch)
    _same(_run(p, s, data, {"CTKVR_TAIL": "2", "CTKVR_DECODE_GROUPS": "3"}, monkeypatch), ref, "three groups")
    p, s, data = _params("eight_blocks")
    ref = _run(p, s, data, SEPARATE, monkeypatch)
    _same(_run(p, s, data, {"CTKVR_TAIL": "2"}, monkeypatch, static=True), ref, "static scratch")


@pytest.mark.parametrize("top_k", [8191, 8192])
def test_the_choice_on_both_sides_of_the_largest_budget(top_k, monkeypatch):
    """Larger batches take share_tail_kernel up to budgets of 8191 and the separate launches beyond: the same integers, and the bits of
    the attention tell which form ran (the separate launches' are the same in every call)."""
    p = ck.Params(batch=4, n_q_heads=16, n_kv_heads=8, n_centroids=48, list_len=4000, n_probe=8, top_k=top_k, dtype=ck.BF16)
    data = _inputs("bf16", 4, 2, 8, 20000, 4000, top_k, 1.0, 0, 4100)
    ref = _run(p, 20000, data, SEPARATE, monkeypatch)
    assert ref[0][3].min() > top_k
    got = _run(p, 20000, data, {}, monkeypatch)
    _same(got, ref, "default")
    assert np.array_equal(got[0][0], ref[0][0]) == (top_k > 8191)


@pytest.mark.parametrize("batch,G,s", [(8, 1, 53248), (8, 1, 53249), (16, 2, 51200), (16, 2, 51201)])
def test_the_choice_on_both_sides_of_the_line_of_one_block_a_unit(batch, G, s, monkeypatch):
    """136 units, 16 of 256 CUs more than half: the separate launches beyond 53248 slots a unit; 272 units, 32 of 512 in two rounds:
    beyond 51200."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the line is that of 256 CUs")
    p = ck.Params(batch=batch, n_q_heads=17 * G, n_kv_heads=17, n_centroids=8, list_len=7000, n_probe=8, top_k=900, dtype=ck.BF16)
    data = _inputs("bf16", batch, G, 17, s, 7000, 900, 1.0, 0, 4200, C=8)
    ref = _run(p, s, data, SEPARATE, monkeypatch)
    got = _run(p, s, data, {}, monkeypatch)
    _same(got, ref, "default")
    assert np.array_equal(got[0][0], ref[0][0]) == (s % 2 == 1)
