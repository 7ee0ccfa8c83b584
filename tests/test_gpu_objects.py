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
