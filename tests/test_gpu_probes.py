"""The probed centroids (Algorithm 2 line 3) where their selection changes form: a wave's share of 64, 128, 256, 512 and
2048 ids by the table's size, the candidates of one to four waves, 64 probes and more (by the block, at every number of
ids a thread holds), fewer centroids than the table
holds; and values that crowd -- copies of a few vectors (ties go to the lowest id) and values some units in the last place
apart."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2512_15550_amd as ck


def _centroids(kind, rng, h, C):
    if kind == "random":
        return rng.standard_normal((h, C, 128)).astype(np.float32)
    few = rng.standard_normal((h, 5, 128)).astype(np.float32)
    x = few[:, rng.integers(0, 5, size=C)]
    if kind == "near":   # some units in the last place of one element apart
        x[:, :, 7] = (x[:, :, 7].view(np.int32) + rng.integers(0, 40, size=(h, C)).astype(np.int32)).view(np.float32)
    return np.ascontiguousarray(x)


@pytest.mark.parametrize("kind", ["random", "copies", "near"])
@pytest.mark.parametrize("C,n_probe", [(2, 1), (9, 8), (64, 8), (65, 64), (65, 1), (129, 9), (256, 64), (257, 32), (512, 32),
                                       (513, 5), (1024, 64), (1025, 17), (2048, 4), (2048, 64), (2049, 8), (5000, 40), (300, 65),
                                       (2100, 100), (100, 100), (200, 65), (256, 100), (900, 80), (1500, 70)])
def test_probes_equal_the_oracles(kind, C, n_probe):
    h, g, rho = 4, 2, 8
    rng = np.random.Generator(np.random.Philox(1000 + C + n_probe))
    n_c = [C, max(C // 2, n_probe)]   # the second sequence has fewer centroids than the table holds

    ctx = [4 * n for n in n_c]
    params = ck.Params(batch=2, n_q_heads=h, n_kv_heads=g, head_dim=128, page_size=16, dtype=ck.F32, n_centroids=0, centroid_div=4,
                       list_len=min(rho, min(ctx)), n_probe=n_probe, top_k=min(rho, min(ctx)))
    rho = params.list_len
    pages = [-(-n // 16) for n in ctx]
    k = torch.randn((sum(pages), g, 16, 128), device="cuda")
    table = torch.zeros((2, max(pages)), dtype=torch.int32, device="cuda")
    table[0, :pages[0]] = torch.arange(pages[0])
    table[1, :pages[1]] = torch.arange(pages[0], sum(pages))
    cen = np.zeros((2, h, max(n_c), 128), np.float32)
    for b in range(2):
        cen[b, :, :n_c[b]] = _centroids(kind, rng, h, n_c[b])
    lists = np.broadcast_to(np.arange(rho, dtype=np.int32), (2, g, max(n_c), rho)).copy()
    idx = ck.ctkvr_index_load(params, ctx, cen, lists)
    try:
        out = torch.empty((2, h, 128), device="cuda")
        probe = torch.full((2, g, n_probe), -7, dtype=torch.int32, device="cuda")
        for step in range(2):
            q = rng.standard_normal((2, h, 128)).astype(np.float32)
            if step:   # a query that is one of the centroids
                q = np.ascontiguousarray(cen[:, :, 0])
            ck.ctkvr_decode_step(idx, torch.from_numpy(q).cuda(), k, k, table, out, out_probe=probe)
            torch.cuda.synchronize()
            for b in range(2):
                _, want = oracle.recall(q[b], np.ascontiguousarray(cen[b, :, :n_c[b]]), g, n_probe)
                assert np.array_equal(probe[b].cpu().numpy(), want), (kind, C, n_probe, step, b)
    finally:
        ck.ctkvr_free(idx)
