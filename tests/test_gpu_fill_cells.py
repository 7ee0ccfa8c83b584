"""Pixels settled from the polygons' cells, against the oracle: zooms around the
finest level, polygons drawn at every level, holes, the world's edges, polygons
too large to draw and polygons beyond the world."""
import numpy as np
import pytest

import oracle
from gpu_common import log
from helpers import parity, unpack_masks

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


def ring(c, radius, k, rng):
    """A closed star ring of k vertices, as edges."""
    a = np.sort(rng.uniform(0, 2 * np.pi, k))
    r = radius * rng.uniform(0.4, 1.0, k)
    v = np.clip(np.stack([c[0] + r * np.cos(a), c[1] + r * np.sin(a)], 1), 0.0, 1.0)
    return np.concatenate([v, np.roll(v, -1, axis=0)], 1)


def polygons(name):
    """(edges in normalised coordinates, offsets): 2,100 polygons, cells down to zoom 2 or 3."""
    rng = np.random.default_rng(len(name))
    out = []
    for p in range(2100):
        c = rng.uniform(0.0, 1.0, 2) if name == "edges of the world" else rng.uniform(0.3, 0.6, 2)
        size = 10.0 ** rng.uniform(-5, -1.3 if p % 100 == 0 else -2.3)
        parts = [ring(c, size, int(rng.integers(3, 30)), rng)]
        if p % 5 == 0:  # a hole
            parts.append(ring(c, 0.3 * size, 7, rng))
        out.append(np.concatenate(parts))
    if name == "too large":
        out.append(ring((0.5, 0.5), 0.49, 40, rng)[:, :])
    if name == "outside":
        out.append(ring((0.5, 0.5), 0.01, 9, rng) + 0.6)
    first = np.concatenate([[0], np.cumsum([len(e) for e in out])]).astype(np.int64)
    return np.concatenate(out), first


@pytest.mark.parametrize("name", ["clusters", "edges of the world", "too large", "outside"])
def test_settled(hv, torch, name):
    edges, first = polygons(name)
    ref = oracle.OraclePolygons(edges, first, merc01=True)
    log(f"fill cells {name}: {len(edges)} edges")
    h = hv.hv_polygon_index_build(torch.from_numpy(edges).cuda(), first, hv.HV_INPUT_MERC01)
    rng = np.random.default_rng(1)
    tiles = [(0, 0, 0), (1, 0, 0), (1, 1, 1), (2, 1, 1), (2, 0, 3)]
    for z in (3, 4, 5, 7, 10):
        at = edges[rng.integers(0, len(edges), 3), :2].clip(0, 0.999999)
        tiles += [(z, int(x * 2 ** z), int(y * 2 ** z)) for x, y in at]
    tiles = np.array(tiles)
    tri = ref.render(tiles)["tri"]
    for L in (None, dict(region=64, waves_per_wg=4, cand_cap=256), dict(region=32, waves_per_wg=1, cand_cap=64, cull_nodes=1)):
        log(f"  launch={L}")
        out = torch.full((len(tiles), 8192), 0xA5, dtype=torch.uint8, device="cuda")
        hv.hv_render_fill(h, tiles, out, L)
        torch.cuda.synchronize()
        mism, amb, lit = parity(unpack_masks(out.cpu().numpy()), tri)
        log(f"  lit={lit} ambiguous={amb} mismatches={mism}")
        assert mism == 0, f"{L}: {mism} mismatches"
    hv.hv_free(h)


@pytest.mark.parametrize("region", [32, 64])
@pytest.mark.parametrize("waves", [1, 4])
def test_shapes_of_large_batches(hv, torch, region, waves):
    """More tiles than a small call's, each its own workgroups and dealt over 7; and a
    small call dealt over 7: as the oracle, and all alike."""
    edges, first = polygons("clusters")
    ref = oracle.OraclePolygons(edges, first, merc01=True)
    h = hv.hv_polygon_index_build(torch.from_numpy(edges).cuda(), first, hv.HV_INPUT_MERC01)
    few = np.array([(0, 0, 0), (2, 1, 1), (4, 6, 7), (9, 200, 210), (3, 0, 0)])
    tri = ref.render(few)["tri"]
    L = dict(region=region, waves_per_wg=waves, cand_cap=64 * waves)
    for n, grid in ((5, 7), (66, 0), (66, 7), (130, 3)):
        log(f"fill region={region} waves={waves} n={n} grid={grid}")
        tiles = few[np.arange(n) % len(few)]
        out = torch.full((n, 8192), 0xA5, dtype=torch.uint8, device="cuda")
        hv.hv_render_fill(h, tiles, out, dict(L, grid_wgs=grid))
        torch.cuda.synchronize()
        bits = unpack_masks(out.cpu().numpy())
        for k in range(n):
            mism, _, lit = parity(bits[k], tri[k % len(few)])
            assert mism == 0, f"tile {k} of {n}, grid {grid}: {mism} mismatches of {lit} lit"
    hv.hv_free(h)
