"""Measured cases of the CTkvr hot path: decode steps (centroid-then-token retrieval with sparse attention) and the
ways an index comes to be (exact build, matrix-core build, k-means build, load from host memory).

Inputs follow the recipe of ``ctkvr_inputs``, drawn on the GPU: keys N(0, 1) with RoPE at their position, values
N(0, 1), post-RoPE queries of a per-head Gaussian random walk (step 0.05), so that neighbouring queries are similar;
the KV cache in pages whose physical order is a random permutation.  Head shapes, context lengths and retrieval
parameters are those of the repository's workloads (``ctkvr_inputs.workload``, ``bench.py``) and ranges around them.

A decode pass is one call per generated token with every output asked for; the queries of a state continue the walk
and are taken in turn.  A build pass is what one prompt costs a server: the index is built (or loaded), the first
token is decoded on it, and the index is given back; where it is kept for later prompts it is copied to the host.
"""
import math

import numpy as np
import torch

import paper_2512_15550_amd as ck

WALK_STEP = 0.05
ROPE_BASE = 10000.0
N_QUERIES = 64          # decode queries of a state; a step takes the next one

_DEFAULTS = {
    "kind": "decode",   # decode | build | load
    "dtype": "bf16", "h": 32, "g": 8, "page": 16,
    "batch": 1, "ctx_lo": 32768, "ctx_hi": 32768, "ctx_seed": 0,   # context lengths: uniform in [ctx_lo, ctx_hi]
    "centroids": 512, "centroid_div": 0,     # C, or C = ctx / centroid_div where centroids is 0
    "probe": 32, "list_len": 1024, "top_k": 1024,
    "n_init": 0, "n_local": 0, "decoded": 0,   # resident window; tokens decoded since the index was built
    "update": False,                         # decode only: the dynamic centroid update after every step
    "algo": "exact", "kmeans": 0,            # build only: list build on the vector units or the matrix cores; Lloyd iterations
    "export": False,                         # build only: the centroids and lists are also copied to the host
}


def _case(name, **over):
    return dict(_DEFAULTS, name=name, **over)


def listed():
    return [
        # the smallest step in use: a short fp32 context, two KV heads; launches and latency are all of it
        _case("decode_4k_f32", dtype="f32", h=8, g=2, ctx_lo=4096, ctx_hi=4096, centroids=64, probe=8, list_len=256, top_k=256),
        # the ordinary step: one sequence of 32K tokens on a layer of 32 query and 8 KV heads
        _case("decode_32k"),
        # the largest step: four sequences of 128K tokens
        _case("decode_128k_b4", batch=4, ctx_lo=131072, ctx_hi=131072, centroids=2048, probe=64, list_len=2048, top_k=2048),
        # a server's running batch: 16 sequences of unequal, odd lengths, as many centroids as each is worth
        _case("decode_ragged_b16", batch=16, ctx_lo=8192, ctx_hi=65536, ctx_seed=4, centroids=0, centroid_div=64),
        # the paper's own operating point (four probes, long lists) on a layer of four KV heads
        _case("decode_32k_4kv", g=4, centroids=2048, probe=4, list_len=1280, top_k=512),
        # the whole of a generation step as the paper runs it: resident window with the tokens decoded so far, sparse
        # attention, merge, then the update of the centroids by the step's own query
        _case("decode_window_update", centroids=2048, probe=4, list_len=2560, top_k=1024, n_init=128, n_local=512,
              decoded=100, update=True),
        # time to first token of a short fp32 prompt that many requests share: its index also goes to host memory
        _case("build_4k_f32", kind="build", dtype="f32", h=8, g=2, ctx_lo=4096, ctx_hi=4096, centroids=64, probe=8,
              list_len=256, top_k=256, export=True),
        # time to first token of an ordinary prompt, with the default (bit-reproducible) list build
        _case("build_32k", kind="build"),
        # ... of a ragged batch of three prompts on the matrix cores, with a resident window
        _case("build_mfma_ragged", kind="build", algo="mfma", batch=3, ctx_lo=9000, ctx_hi=30000, ctx_seed=7, centroids=0,
              centroid_div=64, n_init=64, n_local=256),
        # ... of a 128K prompt on the matrix cores
        _case("build_mfma_128k", kind="build", algo="mfma", ctx_lo=131072, ctx_hi=131072, centroids=2048, probe=64,
              list_len=2048, top_k=2048),
        # ... with k-means centroids (ten Lloyd iterations from given start positions)
        _case("build_kmeans_128k", kind="build", algo="mfma", kmeans=10, ctx_lo=131072, ctx_hi=131072, centroids=2048,
              probe=64, list_len=2048, top_k=2048),
        # a prompt whose index was built before and kept in host memory
        _case("load_32k", kind="load"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    c = dict(_DEFAULTS)
    kind = rng.choice(["decode"] * 7 + ["build"] * 4 + ["load"])
    c["kind"] = kind
    c["dtype"] = "f32" if rng.random() < 0.15 else "bf16"
    c["h"], c["g"] = rng.choice([(32, 8), (32, 8), (32, 8), (32, 4), (32, 4), (8, 2), (8, 8), (16, 8), (40, 10)])
    c["page"] = rng.choice([16, 16, 16, 32, 64])
    batch = 1
    if kind == "decode" and rng.random() < 0.5:
        batch = _log_int(rng, 2, 16)
    elif kind == "build" and rng.random() < 0.25:
        batch = rng.randint(2, 4)
    c["batch"] = batch
    hi_all = {"decode": 131072, "build": 131072, "load": 49152}[kind]
    f32 = c["dtype"] == "f32"
    if f32:
        hi_all = 32768
    if kind == "build":
        mode = "exact" if f32 else rng.choice(["exact", "exact", "mfma", "mfma", "kmeans"])
        c["algo"] = "exact" if mode == "exact" else "mfma"
        c["kmeans"] = rng.randint(5, 10) if mode == "kmeans" else 0
    # tokens of the batch: up to the largest listed case's
    hi = min(hi_all, (524288 if kind == "decode" else 131072) // batch)
    if c["h"] == c["g"]:
        hi = min(hi, 65536)
    top = _log_int(rng, 3000, hi)
    c["ctx_hi"] = top
    c["ctx_lo"] = top if batch == 1 or rng.random() < 0.4 else max(2048, top // rng.randint(2, 6))
    c["ctx_lo"] = min(c["ctx_lo"], top)
    c["ctx_seed"] = rng.randrange(1 << 20)
    lo = c["ctx_lo"]
    if rng.random() < 0.5:
        c["centroids"], c["centroid_div"] = 0, rng.choice([32, 64, 64])
        n_c = lo // c["centroid_div"]
    else:
        c["centroids"] = max(32, min(2048, lo // rng.choice([16, 32, 64])))
        n_c = c["centroids"]
    if rng.random() < 0.4:      # few probes, lists longer than the budget
        c["probe"] = rng.randint(2, 8)
        c["top_k"] = min(_log_int(rng, 128, 1024), lo // 8)
        c["list_len"] = min(int(2.5 * c["top_k"]), lo // 2)
    else:
        c["probe"] = min(_log_int(rng, 8, 64), max(2, n_c // 2))
        c["top_k"] = min(_log_int(rng, 200, 2048), lo // 8)
        c["list_len"] = c["top_k"]
    if rng.random() < 0.25 and lo >= 4096:
        c["n_init"], c["n_local"] = rng.choice([(128, 512), (64, 256), (4, 1000)])
        c["list_len"] = min(c["list_len"], lo - c["n_init"] - c["n_local"])
        if kind == "decode":
            c["decoded"] = rng.randint(0, 300)
    if kind == "decode":
        c["update"] = rng.random() < 0.2
    if kind == "build":
        # no more than the largest listed builds: 2.2 TFLOP of scores on the matrix cores, 0.55 in the exact arithmetic
        most = 5.5e11 if c["algo"] == "exact" else 2.2e12
        while _score_flops(c) > most:
            if c["centroids"]:
                c["centroids"] = max(64, c["centroids"] // 2)
            else:
                c["centroid_div"] *= 2
            c["probe"] = min(c["probe"], max(2, min(_n_cent(c, s) for s in _ctx_lens(c)) // 2))
            if c["centroids"] == 64 or c["centroid_div"] > 512:
                break
        c["export"] = rng.random() < 0.5 and sum(_list_bytes(c, s) for s in _ctx_lens(c)) < 2 ** 24
    return c


# ------------------------------------------------------------------------------
# sizes
# ------------------------------------------------------------------------------
def _ctx_lens(case):
    r = np.random.RandomState(case["ctx_seed"])
    return [int(x) for x in r.randint(case["ctx_lo"], case["ctx_hi"] + 1, size=case["batch"])]


def _n_cent(case, s):
    return case["centroids"] or s // case["centroid_div"]


def _list_bytes(case, s):
    return case["g"] * _n_cent(case, s) * case["list_len"] * 4


def _score_flops(case):
    return sum(2.0 * case["h"] * _n_cent(case, s) * s * 128 for s in _ctx_lens(case))


def _params(case):
    return ck.Params(batch=case["batch"], n_q_heads=case["h"], n_kv_heads=case["g"], head_dim=128, page_size=case["page"],
                     dtype=ck.BF16 if case["dtype"] == "bf16" else ck.F32, n_centroids=case["centroids"],
                     centroid_div=case["centroid_div"], list_len=case["list_len"], n_probe=case["probe"], top_k=case["top_k"],
                     centroid_mode=ck.KMEANS if case["kmeans"] else ck.LAST_C, kmeans_iters=case["kmeans"],
                     build_algo=ck.BUILD_MFMA if case["algo"] == "mfma" else ck.BUILD_EXACT,
                     n_init=case["n_init"], n_local=case["n_local"])


# ------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------
def _rope(x, pos):
    """x [n, heads, 128] fp32, in place of the recipe's rotate-half pairing (i, i + 64) at positions pos [n]."""
    theta = ROPE_BASE ** (-torch.arange(64, dtype=torch.float64, device=x.device) / 64.0)
    ang = pos.to(torch.float64)[:, None] * theta
    c, s = torch.cos(ang).float()[:, None, :], torch.sin(ang).float()[:, None, :]
    a, b = x[..., :64], x[..., 64:]
    return torch.cat([a * c - b * s, b * c + a * s], dim=-1)


def _walk(gen, start, n, h):
    """Post-RoPE queries at positions start .. start + n - 1, [n, h, 128] fp32."""
    inc = torch.randn((n, h, 128), generator=gen, device="cuda")
    inc[0] *= math.sqrt(1.0 + WALK_STEP * WALK_STEP * start)
    inc[1:] *= WALK_STEP
    return _rope(torch.cumsum(inc, dim=0), torch.arange(start, start + n, device="cuda"))


def _inputs(case, seed):
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    h, g, page, lens = case["h"], case["g"], case["page"], _ctx_lens(case)
    tokens = [s + case["decoded"] for s in lens]
    pages = [-(-t // page) for t in tokens]
    pool = sum(pages) + 3
    perm = torch.randperm(pool, generator=gen, device="cuda")
    k_pages = torch.zeros((pool, g, page, 128), dtype=dt, device="cuda")
    v_pages = torch.zeros_like(k_pages)
    table = torch.full((len(lens), max(pages)), -1, dtype=torch.int32, device="cuda")
    prefill, decode, at = [], [], 0
    for i, (s, n_pg) in enumerate(zip(lens, pages)):
        phys = perm[at:at + n_pg]
        at += n_pg
        table[i, :n_pg] = phys.to(torch.int32)
        n = n_pg * page
        k = _rope(torch.randn((n, g, 128), generator=gen, device="cuda"), torch.arange(n, device="cuda"))
        k_pages[phys] = k.view(n_pg, page, g, 128).transpose(1, 2).to(dt)
        del k
        v = torch.randn((n, g, 128), generator=gen, device="cuda")
        v_pages[phys] = v.view(n_pg, page, g, 128).transpose(1, 2).to(dt)
        del v
        first = 0 if case["kmeans"] else s - _n_cent(case, s)
        skip = case["decoded"]   # decode queries come after the tokens decoded so far
        w = _walk(gen, first, s - first + skip + N_QUERIES, h).to(dt)
        prefill.append(w[:s - first].contiguous())
        decode.append(w[s - first + skip:].contiguous())
    cu = np.zeros(len(lens) + 1, np.int32)
    cu[1:] = np.cumsum([p.shape[0] for p in prefill])
    st = {"case": case, "params": _params(case), "k": k_pages, "v": v_pages, "table": table,
          "lens": np.array(lens, np.int32), "q_prefill": torch.cat(prefill), "cu": cu,
          "q": torch.stack(decode, dim=1).contiguous(), "step": 0, "init_pos": None}   # q [step][batch][h][128]
    if case["kmeans"]:
        c_max = max(_n_cent(case, s) for s in lens)
        pos = torch.zeros((len(lens), g, c_max), dtype=torch.int32, device="cuda")
        for i, s in enumerate(lens):
            for kv in range(g):
                n_c = _n_cent(case, s)
                pos[i, kv, :n_c] = torch.randperm(s, generator=gen, device="cuda")[:n_c].sort().values.to(torch.int32)
        st["init_pos"] = pos
    b = len(lens)
    st["out"] = {"out": torch.empty((b, h, 128), dtype=torch.float32, device="cuda"),
                 "lse": torch.empty((b, h), dtype=torch.float32, device="cuda"),
                 "sel": torch.empty((b, g, case["top_k"]), dtype=torch.int32, device="cuda"),
                 "ncand": torch.empty((b, g), dtype=torch.int32, device="cuda"),
                 "probe": torch.empty((b, g, case["probe"]), dtype=torch.int32, device="cuda")}
    st["cur"] = torch.tensor(tokens, dtype=torch.int32, device="cuda") if case["decoded"] else None
    return st


def _build(st):
    return ck.ctkvr_build_index(st["params"], st["q_prefill"], st["cu"], not st["case"]["kmeans"], st["k"], st["table"],
                                st["lens"], init_pos=st["init_pos"])


def prepare(case, seed):
    case = dict(_DEFAULTS, **case)
    st = _inputs(case, seed)
    if case["kind"] == "decode":
        st["index"] = _build(st)
        st["q_prefill"] = None
    elif case["kind"] == "load":
        idx = _build(st)
        st["centroids"], st["lists"] = ck.ctkvr_index_centroids(idx), ck.ctkvr_index_lists(idx)
        ck.ctkvr_free(idx)
        st["q_prefill"] = None
    return st


# ------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------
def _decode(st, idx):
    o, q = st["out"], st["q"][st["step"] % N_QUERIES]
    st["step"] += 1
    if st["cur"] is None:
        ck.ctkvr_decode_step(idx, q, st["k"], st["v"], st["table"], o["out"], out_lse=o["lse"], out_sel=o["sel"],
                             out_ncand=o["ncand"], out_probe=o["probe"])
    else:
        ck.ctkvr_decode_step_window(idx, q, st["k"], st["v"], st["table"], st["cur"], o["out"], out_lse=o["lse"],
                                    out_sel=o["sel"], out_ncand=o["ncand"], out_probe=o["probe"])
    if st["case"]["update"]:
        ck.ctkvr_centroid_update(idx, q)
    return o


def run(st):
    kind = st["case"]["kind"]
    if kind == "decode":
        return _decode(st, st["index"])
    if kind == "build":
        idx = _build(st)
    else:
        idx = ck.ctkvr_index_load(st["params"], st["lens"], st["centroids"], st["lists"])
    out = _decode(st, idx)
    if st["case"]["export"]:
        out = dict(out, centroids=ck.ctkvr_index_centroids(idx), lists=ck.ctkvr_index_lists(idx))
    ck.ctkvr_free(idx)
    return out


# ------------------------------------------------------------------------------
# what a pass cannot do without, and how close two correct implementations come
# ------------------------------------------------------------------------------
def _step_work(case):
    """Centroid table and inverse norms, the probed lists, every recalled key row once per KV head (the probed lists
    overlap: about a quarter of their entries are distinct on these inputs), the selected value rows, the window."""
    e = 2 if case["dtype"] == "bf16" else 4
    h, g = case["h"], case["g"]
    nbytes = flops = 0.0
    for s in _ctx_lens(case):
        c = _n_cent(case, s)
        recalled = min(s, max(case["list_len"], 0.25 * case["probe"] * case["list_len"]))
        sel = min(case["top_k"], recalled)
        win = case["n_init"] + case["n_local"] + case["decoded"]
        nbytes += h * c * (128 * e + 4) + g * case["probe"] * case["list_len"] * 4
        nbytes += g * (recalled * (128 * e + 4) + sel * (128 * e + 4) + win * 2 * 128 * e) + 2 * h * 128 * 4
        flops += 2.0 * 128 * h * (c + recalled + sel + 2 * win)
        if case["update"]:
            nbytes += g * case["list_len"] * 4 + h * 128 * e
    return nbytes, flops


def work(case):
    case = dict(_DEFAULTS, **case)
    nbytes, flops = _step_work(case)
    if case["kind"] == "decode":
        return {"bytes": nbytes, "flops": flops}
    e = 2 if case["dtype"] == "bf16" else 4
    for s in _ctx_lens(case):
        c = _n_cent(case, s)
        nbytes += case["h"] * c * (2 * 128 * e + 4) + _list_bytes(case, s)   # queries in, centroids and lists out
        if case["export"]:
            nbytes += 2 * (case["h"] * c * 128 * e + _list_bytes(case, s))
        if case["kind"] == "build":
            nbytes += case["g"] * s * 128 * e + case["kmeans"] * case["h"] * s * 128 * e
    if case["kind"] == "build":
        flops += (1 + case["kmeans"]) * _score_flops(case)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Ids are whole numbers of one fixed arithmetic: the same everywhere.  The attention is summed in fp32.
    # The matrix-core list build may resolve a near-tie at the end of a list either way: an id in a thousand may shift.
    case = dict(_DEFAULTS, **case)
    if case["algo"] == "mfma":
        return {"rel": 1e-4, "max": 4e-3, "differ": 0.01}
    return {"rel": 1e-5, "max": 4e-4}
