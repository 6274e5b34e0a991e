"""GPU parity of the encode kernel where its transform and its bins can go wrong: key counts at
the edges of a 16-key tile and of a block, both ways of counting clusters, and keys whose
coordinates reach the limits of the exact float16 split (rounding boundary 8, size limit 4096,
subnormals, zeros of both signs, infinities next to ordinary keys).  Every byte against the oracle."""

import numpy as np
import pytest
import torch

import paper_2602_07721_amd as pk
import workloads
from parity import SLOT, check_index, oracle_group

pytestmark = pytest.mark.gpu


def _edge_keys(n, seed):
    """Keys [n][128] float16, each of one kind, the kinds mixed inside every 16-key tile."""
    r = np.random.default_rng(seed)
    K = r.standard_normal((n, 128)) * np.exp2(r.integers(-14, 6, size=(n, 128)))
    kind = np.arange(n) % 9
    few = r.integers(-2, 3, size=(n, 128)) * (r.random((n, 128)) < 0.05)
    K = np.where((kind == 1)[:, None], few, K)  # many transformed coordinates exactly 0
    at8 = np.array([8.0, -8.0, 7.996, -7.996, 8.008, 15.99, 16.0, -4.0])
    K = np.where((kind == 2)[:, None], r.choice(at8, size=(n, 128)), K)
    K = np.where((kind == 3)[:, None], r.choice([1023.5, -4094.0, 2.0 ** -24, 0.00781], size=(n, 128)), K)
    K = np.where((kind == 4)[:, None], r.choice([2.0 ** -24, -(2.0 ** -24), 2.0 ** -14, 3e-6], size=(n, 128)), K)
    K = np.where((kind == 5)[:, None], np.where(r.random((n, 128)) < 0.5, 0.0, -0.0), K)
    K = np.where((kind == 6)[:, None], r.standard_normal((n, 128)) + 40.0 * (np.arange(128) % 37 == 0), K)
    return K.astype(np.float16)


def _large(K, every):
    """Coordinates past the split's limit (4096 and the largest float16) in every `every`-th key."""
    K = K.copy()
    K[::every, 5] = np.float16(4096.0)
    K[every // 2::every, 77] = np.float16(-65504.0)
    return K


def _check(K, flags=0, seed=3):
    b, h, n, _ = K.shape
    signs = workloads.rotation_signs(seed)
    cfg = pk.Config(h, 4, n, signs, flags=flags)
    index = pk.Index.empty(cfg, b)
    pk.encode(cfg, index, torch.from_numpy(K).cuda())
    torch.cuda.synchronize()
    ids, rec = SLOT[index.ids.cpu().numpy()], index.rec.cpu().numpy()
    counts = index.counts.cpu().numpy().view(np.uint32)
    for s in range(b):
        for j in range(h):
            orc = oracle_group(K[s, j], signs, not flags & pk.NO_ROTATION, not flags & pk.NO_ALPHA_CORRECTION)
            check_index(ids[s, j], rec[s, j], counts[s, j], orc)
    return index


@pytest.mark.parametrize("b,h,n", [(1, 1, 1), (1, 2, 15), (1, 1, 16), (2, 1, 17), (1, 3, 64), (1, 1, 65), (1, 2, 1025),
                                   (3, 1, 5003), (2, 2, 30011)])
def test_edge_values_at_tile_and_block_edges(b, h, n):
    print(f"[encode] {b} x {h} x {n}", flush=True)
    K = np.stack([_edge_keys(n, 100 * s + j) for s in range(b) for j in range(h)]).reshape(b, h, n, 128)
    _check(K)


@pytest.mark.parametrize("flags", [0, pk.NO_ROTATION, pk.NO_ALPHA_CORRECTION])
@pytest.mark.parametrize("every", [3, 50])
def test_large_coordinates_take_the_general_transform(flags, every):
    print(f"[encode] flags {flags}, every {every}", flush=True)
    _check(_large(_edge_keys(1000, 9), every).reshape(1, 1, 1000, 128), flags)


def test_infinite_keys_leave_their_tile_neighbours_alone():
    K = _edge_keys(200, 12)
    bad = np.arange(7, 200, 20)
    K[bad, 3] = np.float16(np.inf)
    K[bad[::2], 90] = np.float16(np.nan)
    signs = workloads.rotation_signs(3)
    cfg = pk.Config(1, 4, 200, signs)
    index = pk.Index.empty(cfg, 1)
    pk.encode(cfg, index, torch.from_numpy(K.reshape(1, 1, 200, 128)).cuda())
    ids, rec = SLOT[index.ids.cpu().numpy()][0, 0], index.rec.cpu().numpy()[0, 0]
    ok = np.setdiff1d(np.arange(200), bad)
    orc = oracle_group(K[ok], signs)
    counts = np.stack([np.bincount(ids[ok, s], minlength=256) for s in range(16)])
    check_index(ids[ok], rec[ok], counts, orc)
    assert (index.counts.cpu().numpy().sum(axis=-1) == 200).all()


@pytest.mark.parametrize("t", [1, 16, 17, 300])
def test_append_continues_the_counts(t):
    K = _edge_keys(700 + t, 21).reshape(1, 1, -1, 128)
    whole = _check(K)
    cfg = pk.Config(1, 4, 700 + t, workloads.rotation_signs(3))
    index = pk.Index.empty(cfg, 1)
    Kd = torch.from_numpy(K).cuda()
    pk.encode(cfg, index, Kd[:, :, :700].contiguous())
    pk.append(cfg, index, Kd[:, :, 700:].contiguous(), 700)
    for name in ("ids", "rec", "counts"):
        assert torch.equal(getattr(index, name), getattr(whole, name)), name


@pytest.mark.parametrize("t,name", [(1, "append"), (16, "append"), (17, "append"), (1023, "append"), (1024, "encode")])
def test_profile_names_appends_by_their_size(t, name):
    cfg = pk.Config(2, 4, t, workloads.rotation_signs(3))
    index = pk.Index.empty(cfg, 1)
    index.counts.zero_()
    K = torch.randn(1, 2, t, 128, device="cuda").half()
    pk.profile_enable(True)
    pk.profile_reset()
    try:
        pk.append(cfg, index, K, 0)
        assert set(pk.profile_read()) == {name}
    finally:
        pk.profile_enable(False)
        pk.profile_reset()


@pytest.mark.parametrize("n,share", [(16, 1.0), (130, 0.5), (1000, 1.0), (150000, 0.5), (150000, 1.0)])
def test_large_coordinates_beside_the_limit(n, share):
    # a share of the 16-key tiles has keys of coordinates on both sides of 4096, some in every place of the key;
    # 150000 keys give a wave 4 tiles, which it sees as all large from the first and the middle one
    print(f"[encode] n {n}, share {share}", flush=True)
    r = np.random.default_rng(n)
    K = r.standard_normal((n, 128), dtype=np.float32)
    tile = np.arange(n) // 16
    pick = (r.random(tile[-1] + 1) < share)[tile] & (r.random(n) < 0.5)
    values = np.array([4094.0, -4094.0, 4096.0, -4096.0, 65504.0, -65504.0, 5000.0, 2.0 ** -24, -0.0])
    big = r.choice(values, size=(int(pick.sum()), 128))
    K[pick] = np.where(r.random(big.shape) < r.random((len(big), 1)), big, K[pick])
    _check(K.astype(np.float16).reshape(1, 1, n, 128))


def test_large_keys_cost_no_second_transform():
    # Keys past the split's limit in every tile take one transform of three operands, 1.3 times the ordinary keys'
    # time.  After the ordinary one, as a call of its own, it was 2.2 to 2.4 times.
    def us(K):
        cfg = pk.Config(8, 4, K.shape[2], workloads.rotation_signs(3))
        index = pk.Index.empty(cfg, 1)
        times = []
        for _ in range(10):
            t0, t1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            t0.record()
            for _ in range(10):
                pk.encode(cfg, index, K)
            t1.record()
            torch.cuda.synchronize()
            times.append(t0.elapsed_time(t1) * 100)
        return float(np.median(times))

    gen = torch.Generator(device="cuda").manual_seed(2)
    K = torch.randn(1, 8, 131072, 128, generator=gen, device="cuda", dtype=torch.float16)
    large = K.clone()
    large[:, :, ::16, 5] = 5000.0
    plain, past = us(K), us(large)
    print(f"[encode] ordinary keys {plain:.1f} us, a coordinate of 5000 in every tile {past:.1f}", flush=True)
    assert past < 1.7 * plain
