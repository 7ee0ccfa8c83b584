"""Queues smaller than a leaf step's objects, with several waves to a workgroup:
the step's parts are queued and drained in turn, and every wave has to take the
same turn.  (A wave that read the queue's length after another had queued more
took another one, and the workgroup's barriers no longer matched.)"""
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


# a queue that one part of a step fills, one between, and one short of the step
SHAPES = [dict(region=rs, waves_per_wg=w, objs_per_lane=o, cand_cap=c)
          for rs, w, o, cs in ((32, 2, 2, (128, 129, 255)), (32, 2, 4, (128, 300)), (32, 4, 2, (256, 300)),
                               (32, 4, 4, (256, 1000)), (64, 2, 4, (128,)), (64, 4, 2, (256, 511)))
          for c in cs]
TILES = np.array([[0, 0, 0], [1, 0, 1], [2, 1, 1], [3, 3, 2]])


@pytest.mark.parametrize("kind", [0, 1])
def test_small_queues(hv, torch, kind):
    rng = np.random.default_rng(90 + kind)
    p = rng.uniform(0.2, 0.6, (40_000, 2))
    obj = p if kind == 0 else np.concatenate([p, p + rng.normal(0, 2e-3, p.shape)], 1)
    ref = oracle.OracleIndex(obj, kind, merc01=True)
    h = build(hv, torch, obj, kind | hv.HV_INPUT_MERC01)
    tri, aa = ref.render(TILES, 0.4)["tri"], ref.render_aa(TILES, 0.4)
    for L in SHAPES:
        # (a cull depth of one node leaves the tiles to the regions)
        log(f"small queue kind={kind} {L}")
        mism, _, lit = parity(render(hv, torch, h, TILES, 0.4, dict(L, cull_nodes=1)), tri)
        assert mism == 0, f"{L}: {mism} mismatches of {lit} lit"
        check_aa(render_aa(hv, torch, h, TILES, 0.4, dict(L, cull_nodes=1, aa_split=-1)), aa, f"{L}")
    hv.hv_free(h)


def test_wide_segments(hv, torch):
    """Segments over most of a region's pixels: the queue's tests take the region
    kernel no longer than a wavefront per block, which tests every object's whole
    range and lights nothing ahead of the tests (0.87 of its time; 1.34 where the
    units of the tests were listed anew for each part of the list)."""
    rng = np.random.default_rng(4)
    p = rng.uniform(0, 1, (200_000, 2))
    a = rng.uniform(0, 2 * np.pi, len(p))
    obj = np.concatenate([p, np.clip(p + 30 / 8192 * np.stack([np.cos(a), np.sin(a)], 1), 0, 1)], 1)
    tiles = np.stack([np.full(256, 5), rng.integers(0, 32, 256), rng.integers(0, 32, 256)], 1)
    h = build(hv, torch, obj, 1 | hv.HV_INPUT_MERC01)
    tri = oracle.OracleIndex(obj, 1, merc01=True).render(tiles[:4], 32.0)["tri"]
    out = torch.empty((256, 8192), dtype=torch.uint8, device="cuda")
    ms = []
    for L in (dict(region=32, waves_per_wg=1, objs_per_lane=2, cand_cap=96), dict(region=0, block=16, waves_per_wg=2)):
        L["cull_nodes"] = 1
        log(f"wide segments {L}")
        assert parity(render(hv, torch, h, tiles[:4], 32.0, L), tri)[0] == 0, L
        reqs = hv.requests(h, tiles, 32.0)
        ms.append(min(hv.hv_time_kernels(reqs, out, L, reps=3)[1] for _ in range(4)))
    hv.hv_free(h)
    log(f"regions {ms[0]:.3f} ms, blocks {ms[1]:.3f} ms")
    assert ms[0] < 1.1 * ms[1]


@pytest.mark.parametrize("rs,aa,cap", [(32, 0, 1340), (64, 0, 1332), (32, 1, 1332)])
def test_largest_queue(hv, torch, rs, aa, cap):
    """The largest queue within 64 KiB: 48 bytes an entry, 1 KiB of stack for an index
    of one level, 16 bytes of control and the mask rows (four sets if anti-aliased)."""
    obj = np.random.default_rng(3).uniform(0, 1, (12, 2))
    h = build(hv, torch, obj, hv.HV_INPUT_MERC01)
    L = dict(region=rs, waves_per_wg=4, objs_per_lane=4)
    call = render_aa if aa else render
    call(hv, torch, h, TILES, 2.0, dict(L, cand_cap=cap))
    with pytest.raises(hv.HvError):
        call(hv, torch, h, TILES, 2.0, dict(L, cand_cap=cap + 1))
    hv.hv_free(h)
