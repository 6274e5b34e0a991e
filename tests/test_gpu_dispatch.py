"""GPU parity at the edges of the size rules that choose between forms of a kernel.  Every
intermediate against the oracle, on one group where the shape is large."""

import numpy as np
import pytest
import torch

import paper_2602_07721_amd as pk
import workloads
from parity import GpuRun, check_attention, check_head, check_index, oracle_group

pytestmark = pytest.mark.gpu
SCALE = 1.0 / np.sqrt(128.0)


def _run(batch, hkv, G, n, bud, flags=0, seed=71, K=None, Q=None):
    """Retrieve on the GPU, two (sequence, KV head) groups checked in full; the run and its read-back."""
    print(f"[dispatch] {batch} x {hkv} x {G}, n {n}, budget {bud}, flags {flags}", flush=True)
    wc = workloads.Config("dispatch", batch=batch, n_kv_heads=hkv, q_per_kv=G, n=n, n_cand=bud[0], n_collide=bud[1],
                          top_k=bud[2], seed=seed)
    law, V = workloads.layer_kv(wc)
    K = law if K is None else K
    Q = workloads.layer_queries(wc, K)[0] if Q is None else Q
    signs = workloads.rotation_signs(wc.seed)
    budget = pk.Budget(*bud, flags=flags)
    run = GpuRun(K, V, Q, signs, G, budget, SCALE, capacity=n + 5).retrieve()
    inter = run.intermediates()
    fused = run.retrieve_attend()
    again = run.intermediates()
    for name in ("cand", "cand_score", "idx", "score", "thresh"):
        np.testing.assert_array_equal(inter[name].view(np.uint32), again[name].view(np.uint32))
    np.testing.assert_array_equal(fused.view(np.uint32), run.attend(run.out_idx).view(np.uint32))
    ids, rec, cnt = run.host_index()
    for s, h in {(0, 0), (batch - 1, hkv - 1)}:
        orc = oracle_group(K[s, h], signs)
        check_index(ids[s, h], rec[s, h], cnt[s, h], orc)
        for g in range(G):
            check_head(inter, s, h, g, G, Q[s, h * G + g], orc, signs, budget, n)
            check_attention(fused[s, h * G + g], Q[s, h * G + g], K[s, h], V[s, h], inter["idx"][s, h * G + g], SCALE)
    return run, inter


@pytest.mark.parametrize("batch,hkv,G,n,bud", [
    # the scan reads a chunk in rounds of 2048 keys
    (1, 1, 4, 2047, (200, 400, 30)), (1, 1, 3, 2049, (200, 400, 30)), (1, 2, 4, 4096 + 2048, (300, 600, 40)),
    # 512 rerank blocks (512 threads each), 576 and 2048 (256 threads), 2080 (past one round)
    (2, 8, 4, 8 * 4096 - 5, (700, 1400, 64)), (2, 8, 4, 8 * 4096 + 3, (700, 1400, 64)),
    (16, 8, 4, 4 * 4096, (300, 600, 32)), (13, 8, 5, 3 * 4096 + 1, (300, 600, 32)),
    # past one round of blocks: 16 chunks, the most whose threshold the rerank derives there, and 17
    (1, 9, 16, 16 * 4096, (600, 1200, 40)), (1, 9, 16, 16 * 4096 + 9, (600, 1200, 40)),
    # 32 chunks, the most whose threshold the rerank derives, and 33
    (1, 1, 2, 32 * 4096, (2048, 4096, 100)), (1, 1, 2, 32 * 4096 + 1, (2048, 4096, 100)),
])
def test_chunk_and_grid_edges(batch, hkv, G, n, bud):
    _run(batch, hkv, G, n, bud)


@pytest.mark.parametrize("batch,hkv,G,n,bud", [(1, 1, 4, 2049, (200, 400, 30)), (1, 2, 4, 70001, (3000, 6000, 64)),
                                               (2, 8, 4, 8 * 4096 + 3, (700, 1400, 64)), (1, 1, 1, 32 * 4096, (60000, 90000, 64))])
def test_forced_recount_equals_the_histogram(batch, hkv, G, n, bud):
    _, inter = _run(batch, hkv, G, n, bud)
    run, again = _run(batch, hkv, G, n, bud, flags=pk.EXACT_RECOUNT)
    assert np.all(again["thresh"][..., 5] == 1)
    for name in ("cand", "cand_score", "idx", "score"):
        np.testing.assert_array_equal(inter[name].view(np.uint32), again[name].view(np.uint32))
    _check_chunks(run, again, batch, hkv, G, n)


def _check_chunks(run, inter, batch, hkv, G, n):
    """The per-chunk counts of three rows below each chunk, as the workspace layout documents them."""
    L = run.layout
    rows = batch * hkv * G
    base = run.ws[L["chunk_base"]:L["chunk_base"] + 8 * rows * L["n_chunks"]].cpu().numpy().view(np.int32)
    base = base.reshape(batch, hkv * G, L["n_chunks"], 2)
    for s, r in {(0, 0), (0, G - 1), (batch - 1, hkv * G - 1)}:
        S, theta = inter["S"][s, r, :n].astype(np.int64), inter["thresh"][s, r, 0]
        for c in range(L["n_chunks"]):
            assert base[s, r, c, 0] == np.sum(S[:c * 4096] > theta) and base[s, r, c, 1] == np.sum(S[:c * 4096] == theta)


def _clustered(batch, hkv, n, clusters, in_runs, seed):
    """Keys of several modes, their centres 2 sigma apart per coordinate, mixed or one run per mode."""
    r = np.random.default_rng(seed)
    K = np.empty((batch, hkv, n, 128), dtype=np.float16)
    for s in range(batch):
        for h in range(hkv):
            centres = np.sqrt(2.0) * r.standard_normal((clusters, 128), dtype=np.float32)
            of = np.arange(n) * clusters // n if in_runs else r.integers(0, clusters, n)
            K[s, h] = r.standard_normal((n, 128), dtype=np.float32) + centres[of]
    return K


@pytest.mark.parametrize("batch,hkv,G,n,modes,in_runs", [
    # rerank blocks of 512 threads: one whole chunk, ragged, 32 chunks; of 256 threads: 9, 4 and 16 chunks
    (1, 1, 4, 4096, 16, False), (1, 2, 4, 5 * 4096 + 77, 16, False), (1, 2, 4, 5 * 4096 + 77, 16, True),
    (1, 1, 3, 33000, 24, True), (1, 1, 4, 32 * 4096, 16, True), (2, 8, 4, 9 * 4096 - 100, 16, True),
    (9, 8, 8, 3 * 4096 + 5, 16, True), (1, 9, 16, 16 * 4096 - 1, 16, False)])
def test_floor_above_the_threshold(batch, hkv, G, n, modes, in_runs):
    # keys of several modes and many candidates: the floor lies above most heads' thresholds, by 1 to 4
    C = n // 8
    bud = (C, 2 * C, min(C, 64))
    K = _clustered(batch, hkv, n, modes, in_runs, 9)
    run, inter = _run(batch, hkv, G, n, bud, K=K)
    below = inter["thresh"][..., 4] - inter["thresh"][..., 0]
    print(f"  floor - theta: {np.bincount(below[below > 0])[1:]}", flush=True)
    assert inter["thresh"][..., 5].any()
    _check_chunks(run, inter, batch, hkv, G, n)
    _, forced = _run(batch, hkv, G, n, bud, flags=pk.EXACT_RECOUNT, K=K)
    for name in ("cand", "cand_score", "idx", "score"):
        np.testing.assert_array_equal(inter[name].view(np.uint32), forced[name].view(np.uint32))


@pytest.mark.parametrize("n,near,C", [(4096 + 900, 0.15, 0.2), (3 * 4096 - 3, 0.3, 0.35), (9000, 0.05, 0.1),
                                      (20000, 0.4, 0.45), (32 * 4096 - 17, 0.15, 0.2)])
def test_floor_far_above_the_threshold(n, near, C):
    # fewer than C keys lie by the query and the others opposite: the former alone raise the floor, and the threshold
    # lies among the few scores of the latter, so the search goes on to halving
    batch, hkv, G = 1, 1, 4
    r = np.random.default_rng(n)
    x = r.standard_normal(128)
    side = np.where(r.random(n) < near, 1.0, -1.0)[:, None]
    K = (side * x + 0.4 * r.standard_normal((n, 128))).astype(np.float16)[None, None]
    gaps = []
    for collide in (near, 1.5 * near):
        bud = (int(C * n), int(collide * n), 32)
        run, inter = _run(batch, hkv, G, n, bud, K=K, Q=(x + 0.4 * r.standard_normal((1, G, 128))).astype(np.float16))
        assert (inter["thresh"][..., 5] == 1).all()
        gaps += (inter["thresh"][..., 4] - inter["thresh"][..., 0]).ravel().tolist()
        _check_chunks(run, inter, batch, hkv, G, n)
        _, forced = _run(batch, hkv, G, n, bud, flags=pk.EXACT_RECOUNT, K=K, Q=run.Q.cpu().numpy())
        for name in ("cand", "cand_score", "idx", "score"):
            np.testing.assert_array_equal(inter[name].view(np.uint32), forced[name].view(np.uint32))
    print(f"  floor - theta: {sorted(gaps)}", flush=True)
    assert max(gaps) > 4


def _call_us(K, G, C, k, flags=0):
    b, h, n, _ = K.shape
    gen = torch.Generator(device="cuda").manual_seed(4)
    q = K[:, :, torch.randint(0, n, (G,), generator=gen, device="cuda")].reshape(b, h * G, 128).contiguous()
    cfg = pk.Config(h, G, n, workloads.rotation_signs(5))
    index = pk.Index.empty(cfg, b)
    pk.encode(cfg, index, K)
    budget = pk.Budget(C, 2 * C, k, flags=flags)
    idx, _, ws = pk.retrieve(cfg, index, q, n, budget)
    times = []
    for _ in range(9):
        t0, t1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        t0.record()
        for _ in range(20):
            pk.retrieve(cfg, index, q, n, budget, out_idx=idx, workspace=ws)
        t1.record()
        torch.cuda.synchronize()
        times.append(t0.elapsed_time(t1) * 50)
    return float(np.median(times))


@pytest.mark.parametrize("b,n", [(2, 131072), (12, 65536)])
def test_a_floor_above_the_threshold_costs_no_second_scan(b, n):
    # A histogram of the row in every rerank block made these calls 3 to 5 times those of one mode; with one count
    # per row, or a short search per block, they take up to 1.4 times them.  Twice leaves room for the clock.
    print(f"[high floor] {b} x 8 x 4, {n} keys", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(3)
    one = torch.randn(b, 8, n, 128, generator=gen, device="cuda", dtype=torch.float16)
    centres = 2 ** 0.5 * torch.randn(b, 8, 16, 128, generator=gen, device="cuda", dtype=torch.float16)
    of = torch.randint(0, 16, (b, 8, n, 1), generator=gen, device="cuda").expand(b, 8, n, 128)
    C = min(n // 8, 16384)
    plain = _call_us(one, 4, C, 256)
    many = _call_us(one + torch.gather(centres, 2, of), 4, C, 256)
    forced = _call_us(one, 4, C, 256, flags=pk.EXACT_RECOUNT)
    print(f"  one mode {plain:.1f} us, 16 modes {many:.1f}, forced recount {forced:.1f}", flush=True)
    assert many < 2 * plain and forced < 2 * plain


@pytest.mark.parametrize("batch,hkv,G,n,bud", [
    # top-k blocks of 256, 512 and 1024 threads: 1024 / 1025, 2048 / 2049 and 4096 / 4097
    # candidates, lists of 128 / 129 and 256 / 257 rows
    (1, 1, 3, 3000, (1024, 2048, 128)), (1, 1, 3, 3000, (1024, 2048, 129)), (1, 1, 3, 3000, (1025, 2048, 128)),
    (1, 1, 2, 6000, (2048, 4096, 256)), (1, 1, 2, 6000, (2048, 4096, 257)), (1, 1, 2, 6000, (2049, 4096, 1)),
    # more than 256 rows: 8 candidates per thread
    (17, 4, 4, 2500, (2048, 4096, 128)), (17, 4, 4, 2500, (2049, 4096, 128)), (17, 4, 4, 4200, (4096, 6000, 256)),
    (17, 4, 4, 4200, (4097, 6000, 200)), (17, 4, 4, 1100, (1024, 2000, 5)),
])
def test_top_k_block_edges(batch, hkv, G, n, bud):
    _run(batch, hkv, G, n, bud)


@pytest.mark.parametrize("batch,hkv,G", [(4, 8, 4), (11, 3, 4), (4, 4, 8), (11, 1, 10), (3, 11, 1), (8, 8, 4), (13, 5, 2),
                                         (11, 3, 7), (6, 8, 4), (7, 7, 4), (8, 3, 7), (5, 5, 8)])
def test_query_block_edges(batch, hkv, G):
    # 32, 33, 48, 49 and 50, 64 and 65 quads of query heads: 1 and 4 subspaces per block, rankings by
    # 64-bit and by 32-bit keys; partial quads
    _run(batch, hkv, G, 1500, (200, 400, 20))


def test_tied_rankings_by_short_keys():
    # queries with a few equal coordinates: most proxies tie, exactly or within 24 bits
    batch, hkv, G, n = 17, 4, 4, 700
    wc = workloads.Config("ties", batch=batch, n_kv_heads=hkv, q_per_kv=G, n=n, n_cand=90, n_collide=180, top_k=9, seed=73)
    K, V = workloads.layer_kv(wc)
    Q, _ = workloads.layer_queries(wc, K)
    r = np.random.default_rng(5)
    Q[:8] = (r.integers(-1, 2, size=Q[:8].shape) * (r.random(Q[:8].shape) < 0.03)).astype(np.float16)
    Q[8] = Q[8, :, :1] * (r.random(Q[8].shape) < 0.1) + (2.0 ** -20 * r.integers(-1, 2, size=Q[8].shape)).astype(np.float16)
    signs = workloads.rotation_signs(73)
    budget = pk.Budget(90, 180, 9)
    run = GpuRun(K, V, Q, signs, G, budget, SCALE).retrieve()
    inter = run.intermediates()
    for s in (0, 5, 8, 16):
        for h in range(hkv):
            orc = oracle_group(K[s, h], signs)
            for g in range(G):
                check_head(inter, s, h, g, G, Q[s, h * G + g], orc, signs, budget, n)


@pytest.mark.parametrize("batch,C,k", [(1, 700, 50), (1, 2000, 200), (9, 2000, 100), (9, 4000, 200)])
def test_equal_estimates_take_the_radix_passes(batch, C, k):
    # a zero query: every estimate is 0, so the boundary bin holds all of them
    n, hkv, G = 5000, 8, 4
    wc = workloads.Config("zero", batch=batch, n_kv_heads=hkv, q_per_kv=G, n=n, n_cand=C, n_collide=2 * C, top_k=k, seed=72)
    K, V = workloads.layer_kv(wc)
    Q, _ = workloads.layer_queries(wc, K)
    Q[:, ::3] = 0
    run = GpuRun(K, V, Q, workloads.rotation_signs(72), G, pk.Budget(C, 2 * C, k), SCALE).retrieve()
    inter = run.intermediates()
    np.testing.assert_array_equal(run.retrieve_attend().view(np.uint32), run.attend(run.out_idx).view(np.uint32))
    for s in range(batch):
        for h in range(hkv * G):
            c, e = inter["cand"][s, h], inter["cand_score"][s, h]
            np.testing.assert_array_equal(inter["idx"][s, h], np.sort(c[np.lexsort((c, -e))[:k]]))
            assert h % 3 or not e.any()


@pytest.mark.parametrize("batch,C,k,bins", [
    # top-k blocks of 256, 512 and 1024 threads, at 4 and at 8 candidates per thread
    (1, 1000, 102, 512), (1, 2000, 202, 1024), (1, 4000, 302, 2048), (1, 7000, 202, 2048),
    (9, 2000, 102, 512), (9, 4000, 202, 1024)])
def test_distinct_estimates_of_one_bin_take_the_radix_passes(batch, C, k, bins):
    # one key of a thousand times the others' size stretches [min, max], so that the other estimates fall in one
    # bin; every other key comes four times, so that equal estimates lie across the k-th place (no multiple of 4)
    n, hkv, G = 8000, 8, 4
    print(f"[radix] {batch} x {hkv} x {G}, C {C}, k {k}", flush=True)
    wc = workloads.Config("one bin", batch=batch, n_kv_heads=hkv, q_per_kv=G, n=n // 4, n_cand=C, n_collide=2 * C,
                          top_k=k, seed=74)
    K, V = (np.tile(x, (1, 1, 4, 1)) for x in workloads.layer_kv(wc))
    r = np.random.default_rng(6)
    Q = (K[:, :, 17, None] + 0.1 * r.standard_normal((batch, hkv, G, 128))).astype(np.float16)
    K[:, :, 17] *= np.float16(60000) / np.abs(K[:, :, 17]).max(axis=-1, keepdims=True)
    run = GpuRun(K, V, Q.reshape(batch, hkv * G, 128), workloads.rotation_signs(74), G, pk.Budget(C, 2 * C, k),
                 SCALE).retrieve()
    inter = run.intermediates()
    fused = run.retrieve_attend()
    np.testing.assert_array_equal(run.out_idx.cpu().numpy(), inter["idx"])
    np.testing.assert_array_equal(fused.view(np.uint32), run.attend(run.out_idx).view(np.uint32))
    shared = 0
    for s in range(batch):
        for h in range(hkv * G):
            c, e = inter["cand"][s, h], inter["cand_score"][s, h]
            order = np.lexsort((c, -e))
            np.testing.assert_array_equal(inter["idx"][s, h], np.sort(c[order[:k]]))
            # more than 64 estimates, many of them distinct, in the bin of the k-th: the passes over its digits run
            of = np.minimum(bins - 1, (e - e.min()) * np.float32(bins) / (e.max() - e.min())).astype(np.int64)
            among = e[of == of[order[k - 1]]]
            assert len(among) > 64 and len(np.unique(among)) > 48
            shared += e[order[k - 1]] == e[order[k]]
    assert shared > batch * hkv * G // 2
