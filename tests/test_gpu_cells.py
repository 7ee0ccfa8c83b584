"""Pixels settled from the occupancy cells, against the oracle: every distance
of cell size and radius at which they are used, the world's edges, segments
over many cells, and the sets for which they are not used."""
import numpy as np
import pytest

import oracle
from gpu_common import build, log, render
from helpers import parity

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


N = 131_072  # cells down to zoom 3


def dataset(name):
    """(objects in normalised coordinates, kind)."""
    rng = np.random.default_rng(len(name))
    p = np.concatenate([rng.uniform(0, 1, (N // 4, 2)), 0.3 + 0.02 * rng.normal(size=(N - N // 4, 2))])
    p = np.clip(p, 0.0, 1.0)
    if name == "points":
        return p, 0
    if name == "edges of the world":
        p[::3, 0] = rng.choice([0.0, 1.0], len(p[::3]))
        p[1::3, 1] = rng.choice([0.0, 1.0], len(p[1::3]))
        return p, 0
    if name == "outside":  # one object beyond the world: the cells are not used
        p[7] = (1.002, 0.5)
        return p, 0
    ang = rng.uniform(0, 2 * np.pi, N)
    size = 10.0 ** rng.uniform(-5, -2.5, N)
    if name == "long segments":
        size[:40] = 0.7
    if name == "too many long segments":  # the cells then settle no pixel as unlit
        size[: N // 8] = 0.2
    q = np.clip(p + size[:, None] * np.stack([np.cos(ang), np.sin(ang)], 1), 0.0, 1.0)
    return np.concatenate([p, q], 1), 1


@pytest.mark.parametrize("name", ["points", "edges of the world", "outside", "segments", "long segments",
                                  "too many long segments"])
def test_settled(hv, torch, name):
    obj, kind = dataset(name)
    ref = oracle.OracleIndex(obj, kind, merc01=True)
    log(f"cells {name}")
    h = build(hv, torch, obj, kind | hv.HV_INPUT_MERC01)
    # a shallow frontier keeps the tiles in region mode, whatever they hold
    shapes = [dict(region=rs, waves_per_wg=w, objs_per_lane=2, cand_cap=128 * w, cull_nodes=1)
              for rs, w in ((32, 1), (32, 4), (64, 2))]
    tiles = np.array([[0, 0, 0], [1, 0, 0], [1, 1, 1], [2, 1, 1], [2, 3, 0], [3, 2, 2], [3, 7, 7], [4, 4, 4]])
    for r in (0.1, 0.19, 0.5, 0.75, 1.5, 2.0, 7.5, 14.9, 15.0, 15.1):
        tri = ref.render(tiles, r)["tri"]
        for L in [None] + shapes:
            log(f"  r={r} launch={L}")
            mism, amb, lit = parity(render(hv, torch, h, tiles, r, L), tri)
            assert mism == 0, f"r={r} {L}: {mism} mismatches of {lit} lit"
    hv.hv_free(h)


def test_many_long_segments(hv, torch):
    """More segments over many cells than the list of them holds: the cells have
    none of them and settle little, and the accept pass lights the tiles as it
    does for a set without cells (the same with one segment beyond the world)."""
    rng = np.random.default_rng(6)
    n = 3_000_000  # cells down to zoom 5, these 60 of them long
    p = rng.uniform(0.25, 0.5, (n, 2))
    a = rng.uniform(0, 2 * np.pi, n)
    obj = np.concatenate([p, np.clip(p + 60 / 8192 * np.stack([np.cos(a), np.sin(a)], 1), 0, 1)], 1)
    r = 8.0
    tiles = np.stack([np.full(64, 5), 8 + np.arange(64) % 8, 8 + np.arange(64) // 8], 1)
    L = dict(region=32, waves_per_wg=1, objs_per_lane=2, cand_cap=96, cull_nodes=64)
    out = torch.empty((64, 8192), dtype=torch.uint8, device="cuda")
    ref = oracle.OracleIndex(obj, 1, merc01=True)
    ms = []
    for name in ("long", "without cells"):
        if name == "without cells":
            obj[-1] = (1.1, 1.1, 1.2, 1.2)
        h = build(hv, torch, obj, 1 | hv.HV_INPUT_MERC01)
        log(f"many long segments: {name}")
        if name == "long":
            for rr in (0.5, 1.5, r):
                mism, _, lit = parity(render(hv, torch, h, tiles[:4], rr, L), ref.render(tiles[:4], rr)["tri"])
                assert mism == 0, f"r={rr}: {mism} mismatches of {lit} lit"
        reqs = hv.requests(h, tiles, r)
        ms.append(min(hv.hv_time_kernels(reqs, out, L, reps=3)[1] for _ in range(4)))
        hv.hv_free(h)
    log(f"long {ms[0]:.3f} ms, without cells {ms[1]:.3f} ms")
    assert ms[0] < 1.35 * ms[1]


def test_many_long_among_short_segments(hv, torch):
    """As above, among short ones: the cells light regions with many of those,
    which skip the accept pass, and settle the others little, which take it."""
    rng = np.random.default_rng(7)
    n, n_long = 2_600_000, 1_100_000  # cells down to zoom 5, these 64 px wide there
    p = rng.uniform(0.25, 0.5, (n, 2))
    p[n_long:, 0] = 0.25 + 0.125 * rng.uniform(0, 1, n - n_long) ** 4  # few in the east
    a = rng.uniform(0, 2 * np.pi, n)
    size = np.where(np.arange(n) < n_long, 64 / 8192, 1e-5)
    obj = np.concatenate([p, np.clip(p + size[:, None] * np.stack([np.cos(a), np.sin(a)], 1), 0, 1)], 1)
    ref = oracle.OracleIndex(obj, 1, merc01=True)
    h = build(hv, torch, obj, 1 | hv.HV_INPUT_MERC01)
    tiles = np.array([[5, 8, 8], [5, 9, 12], [5, 11, 9], [5, 13, 13], [6, 17, 20], [6, 30, 31]])
    log("many long segments among short ones")
    for r in (0.5, 1.5, 8.0):
        tri = ref.render(tiles, r)["tri"]
        for L in (dict(region=32, waves_per_wg=1, objs_per_lane=2, cand_cap=96, cull_nodes=16),
                  dict(region=64, waves_per_wg=4, objs_per_lane=2, cand_cap=512, cull_nodes=16)):
            mism, _, lit = parity(render(hv, torch, h, tiles, r, L), tri)
            assert mism == 0, f"r={r} {L}: {mism} mismatches of {lit} lit"
    hv.hv_free(h)


@pytest.mark.parametrize("kind", [0, 1, 2])
def test_unused_cells_are_given_back(hv, torch, kind):
    """An index with an object beyond the world cannot use its cells, and does not keep
    their memory: the finest level has 4^k cells, as many as 32 for each of 2^18 objects
    allow, so 2^22 (bits)."""
    n = 1 << 18
    rng = np.random.default_rng(kind)
    p = rng.uniform(0.2, 0.8, (n, 2))
    d = 1e-4 * rng.normal(size=(n, 2))
    obj = p if kind == 0 else np.concatenate([p, p + d], 1)
    held = []
    for outside in (False, True):
        if outside:
            obj[:3] += 1.0
        log(f"unused cells kind={kind} outside={outside}")
        hv.hv_trim()  # (no reused block)
        if kind == 2:
            ring = obj.reshape(-1, 4, 4).copy()  # rings of four edges
            ring[:, :, 2:] = np.roll(ring[:, :, :2], -1, axis=1)
            first = np.arange(0, n + 1, 4, dtype=np.int64)
            t = torch.from_numpy(ring.reshape(-1, 4)).cuda()
            h = hv.hv_polygon_index_build(t, first, hv.HV_INPUT_MERC01)
        else:
            h = build(hv, torch, obj, kind | hv.HV_INPUT_MERC01)
        held.append(hv.hv_index_info(h)["device_bytes"])
        hv.hv_free(h)
    log(f"held {held}")
    assert held[0] - held[1] >= (1 << 22) // 8
