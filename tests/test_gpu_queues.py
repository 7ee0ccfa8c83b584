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
