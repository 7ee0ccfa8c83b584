"""Calls at the edges of the small-call launches: 32 and 33 requests (a walk of
its own in every workgroup, or a frontier kernel), 64 and 65 (requests in the
kernels' arguments, or in a workspace), 4 and 5 indexes in one call."""
import numpy as np
import pytest

import oracle
from gpu_common import log
from helpers import parity, unpack_masks
from test_gpu_aa import check_aa, render_aa
from test_gpu_fill_cells import polygons
from test_gpu_objects import TILES, objects

pytestmark = pytest.mark.gpu

R = 1.5


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "needs a GPU"
    return t


@pytest.fixture(scope="module")
def hv():
    from paper_2005_12489_amd import hv as m
    return m


@pytest.fixture(scope="module")
def world(hv, torch):
    """Five indexes and what each draws on the four tiles."""
    hs, tri, aa = [], [], []
    for k, (kind, n) in enumerate([(0, 90), (1, 700), (0, 20_000), (1, 6000), (0, 3)]):
        obj = objects(kind, n, 50 + k)
        ref = oracle.OracleIndex(obj, kind, merc01=True)
        tri.append(ref.render(TILES, R)["tri"])
        aa.append(ref.render_aa(TILES, R))
        hs.append(hv.hv_index_build(torch.from_numpy(obj).cuda(), kind | hv.HV_INPUT_MERC01))
    yield np.array(hs, dtype=np.uint64), tri, aa
    for h in hs:
        hv.hv_free(int(h))


@pytest.mark.parametrize("indexes", [1, 4, 5])
@pytest.mark.parametrize("n", [1, 16, 17, 32, 33, 64, 65])
def test_masks_and_values(hv, torch, world, n, indexes):
    hs, tri, aa = world
    d = (np.arange(n) + 1) % indexes
    t = (np.arange(n) * 3) % len(TILES)
    log(f"{n} requests of {indexes} indexes")
    out = torch.full((n, 8192), 0xA5, dtype=torch.uint8, device="cuda")
    hv.hv_render_batch(hv.requests(hs[d], TILES[t], np.full(n, R)), out)
    torch.cuda.synchronize()
    bits = unpack_masks(out.cpu().numpy())
    val = render_aa(hv, torch, hs[d], TILES[t], R)
    for k in range(n):
        assert parity(bits[k], tri[d[k]][t[k]])[0] == 0, f"request {k} of {n}"
        check_aa(val[k:k + 1], {f: aa[d[k]][f][t[k]:t[k] + 1] for f in ("val", "amb", "sure")}, f"request {k} of {n}")


@pytest.mark.parametrize("n", [1, 16, 17, 32, 33, 64, 65])
def test_fill(hv, torch, n):
    edges, first = polygons("clusters")
    ref = oracle.OraclePolygons(edges, first, merc01=True)
    h = hv.hv_polygon_index_build(torch.from_numpy(edges).cuda(), first, hv.HV_INPUT_MERC01)
    tiles = np.array([[2, 1, 1], [6, 25, 30], [9, 200, 210], [0, 0, 0]])
    tri = ref.render(tiles)["tri"]
    t = np.arange(n) % len(tiles)
    log(f"filling {n} tiles")
    out = torch.full((n, 8192), 0xA5, dtype=torch.uint8, device="cuda")
    hv.hv_render_fill(h, tiles[t], out)
    torch.cuda.synchronize()
    bits = unpack_masks(out.cpu().numpy())
    hv.hv_free(h)
    for k in range(n):
        assert parity(bits[k], tri[t[k]])[0] == 0, f"tile {k} of {n}"
