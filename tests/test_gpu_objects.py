"""The object kernel -- tiles whose frontier lies at the leaves or up to two
levels above -- against the oracle: strip and word edges, wide and flat
segments, the switches to a level-1 and a level-2 frontier, small and large
batches."""
import numpy as np
import pytest

import oracle
from gpu_common import build, log, render
from helpers import parity
from test_gpu_aa import check_aa, render_aa

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "needs a GPU"
    return t


@pytest.fixture(scope="module")
def hv():
    from paper_2005_12489_amd import hv as m
    return m


Z, TX, TY = 5, 11, 17  # the tile under test


def objects(kind, n, seed):
    """n objects in and around the tile, in normalised coordinates; segments of
    every kind of length and slope."""
    rng = np.random.default_rng(seed)
    p = rng.uniform(-80.0, 336.0, (n, 2))           # tile pixels
    if kind == 0:
        q = p
    else:
        length = rng.choice([0.0, 0.4, 3.0, 14.0, 90.0, 900.0], n, p=[0.05, 0.35, 0.35, 0.15, 0.07, 0.03])
        ang = rng.choice([0.0, np.pi / 2, np.pi, 3e-6, 2e-3], n)
        ang = np.where(rng.random(n) < 0.3, ang, rng.uniform(0, 2 * np.pi, n))
        q = np.concatenate([p, p + length[:, None] * np.stack([np.cos(ang), np.sin(ang)], 1)], 1)
    world = 256.0 * 2 ** Z
    return (q + np.tile([256.0 * TX, 256.0 * TY], q.shape[1] // 2)) / world


TILES = np.array([[Z, TX, TY], [Z, TX + 1, TY], [Z + 1, 2 * TX + 1, 2 * TY], [Z - 1, TX // 2, TY // 2]])


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("n", [1, 17, 250, 4096, 4200, 30_000, 120_000])
def test_masks(hv, torch, kind, n):
    obj = objects(kind, n, 7 * n + kind)
    ref = oracle.OracleIndex(obj, kind, merc01=True)
    log(f"objects kind={kind} n={n}")
    h = build(hv, torch, obj, kind | hv.HV_INPUT_MERC01)
    for r in (0.3, 1.0, 2.5) + ((20.0, 64.0) if n <= 250 else ()) if n < 100_000 else (0.3, 0.9):
        tri = ref.render(TILES, r)["tri"]
        for L in (None, dict(region=32, waves_per_wg=1, objs_per_lane=2, cand_cap=128)):
            log(f"  r={r} launch={L}")
            mism, amb, lit = parity(render(hv, torch, h, TILES, r, L), tri)
            assert mism == 0, f"r={r}: {mism} mismatches of {lit} lit"
    hv.hv_free(h)


@pytest.mark.parametrize("requests", [1, 65, 1100])
def test_batch_sizes(hv, torch, requests):
    """Strips and launches depend on the batch's size; masks do not."""
    obj = objects(1, 5000, 3)
    tiles = np.resize(TILES, (requests, 3))
    h = build(hv, torch, obj, 1 | hv.HV_INPUT_MERC01)
    log(f"batch of {requests}")
    tri = oracle.OracleIndex(obj, 1, merc01=True).render(TILES[:requests], 1.25)["tri"]
    bits = render(hv, torch, h, tiles, 1.25)
    hv.hv_free(h)
    for k in range(requests):
        mism, _, _ = parity(bits[k], tri[k % len(TILES)])
        assert mism == 0, f"request {k}: {mism} mismatches"


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("n", [17, 6000, 120_000])
def test_anti_aliased(hv, torch, kind, n):
    obj = objects(kind, n, n + kind)
    ref = oracle.OracleIndex(obj, kind, merc01=True)
    h = build(hv, torch, obj, kind | hv.HV_INPUT_MERC01)
    for r in (0.5, 2.0) + ((30.0,) if n < 100 else ()) if n < 100_000 else (0.5,):
        log(f"aa objects kind={kind} n={n} r={r}")
        got = render_aa(hv, torch, h, TILES, r, {"region": 32, "objs_per_lane": 2, "aa_split": -1})
        check_aa(got, ref.render_aa(TILES, r), f"objects kind={kind} n={n} r={r}")
    hv.hv_free(h)


@pytest.mark.parametrize("aa", [0, 1])
@pytest.mark.parametrize("length", [0.0, 3.0, 40.0])
def test_choice(hv, torch, length, aa):
    """Which tiles go by strips depends on the frontier's size and level, the
    radius, the objects' extent and the batch's size; values do not.  Frontiers
    of about 8, 32, 64 and 160 nodes, leaves small and large to the radius."""
    rng = np.random.default_rng(int(length))
    launches = (None, dict(region=32, waves_per_wg=1, objs_per_lane=2, cand_cap=128))
    for n in (130, 560, 1100, 2700, 9000):
        p = rng.uniform(-20.0, 276.0, (n, 2))
        a = rng.uniform(0, 2 * np.pi, n)
        d = length * np.stack([np.cos(a), np.sin(a)], 1)
        obj = (np.concatenate([p, p + d], 1) if length else p)
        obj = (obj + np.tile([256.0 * TX, 256.0 * TY], obj.shape[1] // 2)) / (256.0 * 2 ** Z)
        kind = int(length > 0)
        ref = oracle.OracleIndex(obj, kind, merc01=True)
        h = build(hv, torch, obj, kind | hv.HV_INPUT_MERC01)
        for r in (0.5, 1.0, 2.0, 2.1, 5.9, 6.1) if n < 9000 else (0.5, 2.1, 6.1):
            want = ref.render_aa(TILES, r) if aa else ref.render(TILES, r)["tri"]
            for requests in (4, 17, 65, 193) if n < 9000 else (17, 193):
                for L in launches:
                    log(f"choice length={length} aa={aa} n={n} r={r} requests={requests} launch={L}")
                    tiles = np.resize(TILES, (requests, 3))
                    got = (render_aa(hv, torch, h, tiles, r, dict(L or {"region": 32, "objs_per_lane": 2}, aa_split=-1))
                           if aa else render(hv, torch, h, tiles, r, L))
                    for k in range(4, requests):
                        assert np.array_equal(got[k], got[k % 4]), f"request {k} of {requests}"
                    if aa:
                        check_aa(got[:4], want, f"n={n} r={r} {requests} {L}")
                    else:
                        mism, _, lit = parity(got[:4], want)
                        assert mism == 0, f"n={n} r={r} {requests} {L}: {mism} mismatches of {lit} lit"
        hv.hv_free(h)


@pytest.mark.parametrize("kind,aa", [(0, 0), (1, 0), (0, 1)])
def test_large_radius(hv, torch, kind, aa):
    """A tile of many objects and a radius that lights all of it costs no more than
    a few times what a small radius does: regions light their pixels and leave the
    other objects (1 to 3 times; 10 to 25 times where every object in reach went
    over every strip)."""
    n = 15_000 * 16
    p = np.random.default_rng(8).uniform(0, 4, (n, 2)) + 8.0  # 15,000 a tile at zoom 5
    obj = (p if kind == 0 else np.concatenate([p, p + 3.0 / 256], 1)) / 32.0
    h = build(hv, torch, obj, kind | hv.HV_INPUT_MERC01)
    tiles = np.array([[5, 8 + k % 4, 8 + k // 4] for k in range(16)] * 16)
    out = torch.empty((len(tiles), hv.HV_AA_BYTES if aa else 8192), dtype=torch.uint8, device="cuda")
    ms = []
    for r in (2.0, 16.0):
        log(f"large radius kind={kind} aa={aa} r={r}")
        reqs = hv.requests(h, tiles, r)
        time = hv.hv_time_aa if aa else hv.hv_time_kernels
        ms.append(min(time(reqs, out, dict(region=32, waves_per_wg=4, objs_per_lane=2, cand_cap=512, aa_split=-1) if aa
                           else None, reps=3)[1] for _ in range(4)))
    hv.hv_free(h)
    log(f"r=2 {ms[0]:.3f} ms, r=16 {ms[1]:.3f} ms")
    assert ms[1] < 5 * ms[0]
