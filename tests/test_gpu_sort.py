"""The build's sort at the edges of its tiles and with equal keys, and builds in
memory that an earlier index gave back."""
import numpy as np
import pytest

from gpu_common import build, log
from helpers import hilbert_np

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


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("n,distinct", [(1, 1), (64, 3), (1023, 1023), (1024, 5), (8191, 8191), (8192, 300),
                                        (8193, 8193), (70_001, 40), (300_007, 300_007)])
def test_order(hv, torch, kind, n, distinct):
    """A stable sort by the key of the box centre, every object stored once,
    boxes and levels exact -- for a fresh index and for one built in the memory
    of a freed one."""
    rng = np.random.default_rng(n + kind)
    w = 4 if kind else 2
    pool = rng.uniform(0, 1, (distinct, w))
    for k in range(2):
        obj = pool[rng.integers(0, distinct, n)] if distinct < n else rng.permutation(pool)
        log(f"sort kind={kind} n={n} distinct={distinct} build {k}")
        h = build(hv, torch, obj, kind | hv.HV_INPUT_MERC01)
        info = hv.hv_index_info(h)
        order = hv.hv_index_read(h, hv.HV_READ_ORDER).astype(np.int64)
        P = hv.hv_index_read(h, hv.HV_READ_OBJECTS)
        boxes = [hv.hv_index_read(h, hv.HV_READ_NODES, lvl) for lvl in range(info["levels"])]
        hv.hv_free(h)
        assert np.array_equal(P, obj[order])
        lo, hi = P.reshape(n, -1, 2).min(1), P.reshape(n, -1, 2).max(1)
        c = 0.5 * (lo + hi) if kind else lo
        s = 2.0 ** info["key_bits"]
        q = np.clip(np.floor(c * s), 0, s - 1)
        key = hilbert_np(q[:, 0], q[:, 1], info["key_bits"])
        expect = np.lexsort((order, key))  # by key, then by input place
        assert np.array_equal(expect, np.arange(n)) and np.array_equal(np.sort(order), np.arange(n))
        box = np.concatenate([lo, hi], 1)
        for got in boxes:
            at = np.arange(0, len(box), 16)
            box = np.concatenate([np.minimum.reduceat(box[:, :2], at), np.maximum.reduceat(box[:, 2:], at)], 1)
            assert np.array_equal(got, box)
