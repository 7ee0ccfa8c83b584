"""The work a program has this library do, as cases that can be timed.

A case is a dict of plain values:

  path      the entry point: "tiles" (hv_render_tiles), "batch" (hv_render_batch),
            "batcher" (hv_batcher_run on a batcher made beforehand), "aa"
            (hv_render_batch_aa), "fill" (hv_render_fill), "load" (hv_index_build
            of data that has just arrived, and its first masks)
  data      "uniform" points, "clustered" points, "lines" (random-walk polylines
            as segments), "edges" (star-polygon edges), "polygons" (the same
            polygons for filling), "two" (lines and clustered points together)
  n         objects of the data set (edges of "polygons"; of "two": segments)
  zlo, zhi  zooms of the requests; equal for one zoom
  pick      "all" (every tile of the zoom), "screen" (a block of neighbouring
            tiles around an object), "mixed" (each tile around an object)
  tiles     requests of a call
  rlo, rhi  radius or half-width of the requests, px; equal for one style
  tuned     whether the batcher was given the shape that hv_autotune picks for
            large mixed batches instead of the default

Masks are bits and anti-aliased values whole numbers 0-4: outputs compare byte
for byte.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2005_12489_amd import hv

# what hv_autotune picks for the mixed batches of the 2e8 edges and of the 1e9
# points: one single-wave workgroup per 32 px region, queues of 96 objects
TUNED = {"block": 0, "cand_cap": 96, "waves_per_wg": 1, "grid_wgs": 1 << 20, "region": 32, "objs_per_lane": 2}


def _case(name, path, data, n, zlo, zhi, pick, tiles, rlo, rhi, tuned=False):
    c = {"path": path, "data": data, "n": n, "zlo": zlo, "zhi": zhi, "pick": pick, "tiles": tiles, "rlo": rlo,
         "rhi": rhi, "tuned": tuned}
    return dict(c, name=name) if name else c


def listed():
    return [
        # one tile of a small point set, asked for alone: the smallest call
        _case("tile_points_1e4", "tiles", "uniform", 10_000, 4, 4, "mixed", 1, 2.0, 2.0),
        # a small point set's whole zoom level in one call
        _case("tiles_points_1e4", "tiles", "uniform", 10_000, 4, 4, "all", 256, 2.0, 2.0),
        # a map view: a screen of neighbouring tiles of the linestrings
        _case("screen_lines_1e7", "batch", "lines", 10_000_000, 7, 7, "screen", 21, 0.75, 0.75),
        # a whole zoom level of the linestrings, thin lines
        _case("tiles_lines_1e7", "tiles", "lines", 10_000_000, 6, 6, "all", 4096, 0.5, 0.5),
        # the headline workload: mixed requests over planet-scale polygon edges,
        # through a kept batcher in its autotuned shape
        _case("batcher_edges_2e8", "batcher", "edges", 200_000_000, 2, 20, "mixed", 4096, 0.5, 2.5, True),
        # the largest set: mixed requests over clustered points, default shape
        _case("batch_points_1e9", "batch", "clustered", 1_000_000_000, 0, 18, "mixed", 10_000, 1.0, 3.0),
        # a server's loop under load: one small batch over two resident sets
        _case("serve_two_sets", "batcher", "two", 10_000_000, 0, 20, "mixed", 61, 0.5, 3.0),
        # anti-aliased zoom level of the linestrings
        _case("aa_lines_1e7", "aa", "lines", 10_000_000, 6, 6, "all", 4096, 0.5, 0.5),
        # anti-aliased mixed requests over polygon edges
        _case("aa_edges_2e7", "aa", "edges", 20_000_003, 2, 20, "mixed", 777, 0.5, 2.5),
        # filling: mixed requests over the planet-scale polygons
        _case("fill_polygons_2e8", "fill", "polygons", 200_000_000, 2, 20, "mixed", 4096, 0.0, 0.0),
        # filling a map view of a smaller set
        _case("fill_screen_2e7", "fill", "polygons", 20_000_003, 6, 6, "screen", 21, 0.0, 0.0),
        # linestrings arrive: index them and show the world down to zoom 2
        _case("load_lines_1e7", "load", "lines", 10_000_000, 0, 2, "all", 21, 0.5, 0.5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["tiles", "batch", "batcher", "aa", "fill", "load"])
    if path == "fill":
        data, n = "polygons", _log(rng, 3e4, 2e8)
    else:
        kinds = ["uniform", "clustered", "lines", "edges"] + (["two"] if path in ("batch", "batcher") else [])
        data = rng.choice(kinds)
        n = _log(rng, 1e4, {"aa": 5e7, "load": 1e8, "tiles": 2e8}.get(path, 1e7 if data == "two" else 2e8))
    points = data in ("uniform", "clustered")
    rlo, rhi = (0.0, 0.0) if path == "fill" else (1.0, 3.0) if points else (0.5, 2.5)
    if path == "load":
        z = rng.randint(0, 2)
        return _case(None, path, data, n, 0, z, "all", (4 ** (z + 1) - 1) // 3, rhi / 2, rhi / 2)
    tiles = _log(rng, 6, 600 if path == "aa" else 4096)
    pick = rng.choice(["screen", "mixed", "mixed"])
    if pick == "screen":
        tiles = min(tiles, 64)
        z = rng.randint(max(3, math.ceil(math.log(n / 65536, 4))), 14)  # not all of it covered
        r = rng.choice([0.5, 0.75, 1.0, 2.0, 4.0]) if rhi else 0.0
        return _case(None, path, data, n, z, z, pick, tiles, r, r)
    if path == "tiles":  # one style for all
        rlo = rhi = rng.uniform(rlo, rhi)
    zlo = rng.randint(0, 8)
    return _case(None, path, data, n, zlo, rng.randint(zlo + 4, 20), pick, tiles, rlo, rhi,
                 path == "batcher" and rng.random() < 0.5)


# ------------------------------------------------------------------- inputs
def _uniform(g, m, lo, hi):
    return torch.rand(m, generator=g, device="cuda", dtype=torch.float64).mul_(hi - lo).add_(lo)


def _normal(g, m, sigma=1.0):
    return torch.randn(m, generator=g, device="cuda", dtype=torch.float64).mul_(sigma)


def _randint(g, m, lo, hi):
    return torch.randint(lo, hi, (m,), generator=g, device="cuda")


def _fold(x, lo, hi):
    """Reflects values into [lo, hi]."""
    w = hi - lo
    y = torch.remainder(x - lo, 2.0 * w)
    return torch.where(y > w, 2.0 * w - y, y).add_(lo)


def _offsets(counts):
    """Exclusive prefix sums of integers, with the total at the end."""
    return torch.cat([counts.new_zeros(1), torch.cumsum(counts, 0)])


def _points(g, n, clustered):
    out = torch.empty((n, 2), device="cuda", dtype=torch.float64)
    hot_lon, hot_lat = _uniform(g, 1000, -180.0, 180.0), _uniform(g, 1000, -80.0, 80.0)
    sigma = 10.0 ** _uniform(g, 1000, -2.0, 0.0)
    for lo in range(0, n, 50_000_000):
        m = min(50_000_000, n - lo)
        lon, lat = _uniform(g, m, -180.0, 180.0), _uniform(g, m, -85.0, 85.0)
        if clustered:  # nine in ten around a hotspot
            k = _randint(g, m, 0, 1000)
            hot = torch.rand(m, generator=g, device="cuda") < 0.9
            s = sigma[k]
            lon = torch.where(hot, _fold(hot_lon[k].add_(_normal(g, m).mul_(s)), -180.0, 180.0), lon)
            lat = torch.where(hot, _fold(hot_lat[k].add_(_normal(g, m).mul_(s)), -85.0, 85.0), lat)
        out[lo:lo + m, 0] = lon
        out[lo:lo + m, 1] = lat
    return out


_GRID = 2.0 ** 40  # running sums are taken in integers: exact in any order


def _lines(g, n):
    """Random-walk polylines of 2 to 50 vertices around 64 centres, split into n segments."""
    p = n // 20 + 64
    first = _offsets(_randint(g, p, 1, 50))
    while int(first[-1]) < n:
        first = _offsets(_randint(g, len(first) + 64, 1, 50))
    first = first[first < n]
    p = len(first)
    counts = torch.diff(first, append=first.new_tensor([n]))
    owner = torch.repeat_interleave(torch.arange(p, device="cuda"), counts, output_size=n)
    c = _randint(g, p, 0, 64)
    out = torch.empty((n, 4), device="cuda", dtype=torch.float64)
    step = torch.exp(_normal(g, n) + math.log(0.01))
    head = _uniform(g, n, 0.0, 2.0 * math.pi)
    for axis, (d, lo, hi, centre) in enumerate(((step * torch.cos(head), -180.0, 180.0, 180.0),
                                                (step * torch.sin(head), -85.0, 85.0, 80.0))):
        start = _uniform(g, 64, -centre, centre)[c] + _normal(g, p, 2.0)
        q = (d * _GRID).to(torch.int64)
        end = torch.cumsum(q, 0)
        base = (end - q)[first]
        end -= base[owner]
        at = start[owner]
        out[:, axis] = _fold(at + (end - q).to(torch.float64) / _GRID, lo, hi)
        out[:, 2 + axis] = _fold(at + end.to(torch.float64) / _GRID, lo, hi)
    return out


def _polygons(g, n):
    """Star polygons of 4 to 200 vertices around 256 centres, about n edges (ring after
    ring, the closing edge included), and the polygons' offsets."""
    p = max(1, n // 102)
    k = _randint(g, p, 4, 201)
    first = _offsets(k)
    nv = int(first[-1])
    owner = torch.repeat_interleave(torch.arange(p, device="cuda"), k, output_size=nv)
    c = _randint(g, p, 0, 256)
    lon = _uniform(g, 256, -180.0, 180.0)[c] + _normal(g, p, 2.0)
    lat = _uniform(g, 256, -80.0, 80.0)[c] + _normal(g, p, 2.0)
    rho = torch.exp(_normal(g, p) + math.log(0.05))
    # rising angles: running sums of exponential gaps over the ring's whole turn
    gap = (-torch.log1p(-_uniform(g, nv, 0.0, 1.0))).add_(1e-9).mul_(2.0 ** 24).to(torch.int64)
    run = torch.cumsum(gap, 0)
    base = (run - gap)[first[:-1]]
    turn = (run[first[1:] - 1] - base).to(torch.float64) + 1.0
    run -= base[owner]
    ang = run.to(torch.float64).div_(turn[owner]).mul_(2.0 * math.pi)
    del gap, run
    rad = _uniform(g, nv, 0.5, 1.0).mul_(rho[owner])
    out = torch.empty((nv, 4), device="cuda", dtype=torch.float64)
    for axis, v in enumerate((_fold(lon[owner] + rad * torch.cos(ang), -180.0, 180.0),
                              _fold(lat[owner] + rad * torch.sin(ang), -85.0, 85.0))):
        out[:, axis] = v
        out[:-1, 2 + axis] = v[1:]
        out[first[1:] - 1, 2 + axis] = v[first[:-1]]
    return out, first


def _data(case, g):
    """[(objects, kind, polygon offsets or None)] of the case's data set."""
    n, data = case["n"], case["data"]
    if data in ("uniform", "clustered"):
        return [(_points(g, n, data == "clustered"), hv.HV_POINTS, None)]
    if data == "lines":
        return [(_lines(g, n), hv.HV_SEGMENTS, None)]
    if data == "two":
        return [(_lines(g, n), hv.HV_SEGMENTS, None), (_points(g, 10 * n, True), hv.HV_POINTS, None)]
    edges, first = _polygons(g, n)
    return [(edges, hv.HV_POLYGON_EDGES, first if data == "polygons" else None)]


def _tile_of(lonlat, z):
    """The tiles (z, x, y) that hold the given locations (one zoom for each)."""
    side = 2.0 ** z
    lat = np.radians(lonlat[:, 1])
    x = np.clip(np.floor((lonlat[:, 0] + 180.0) / 360.0 * side), 0, side - 1)
    y = np.clip(np.floor((0.5 - np.arcsinh(np.tan(lat)) / (2.0 * math.pi)) * side), 0, side - 1)
    return np.stack([z, x, y], axis=1).astype(np.int32)


def _tiles(case, sets, rng):
    """(data set of each request, tiles, radii)."""
    if case["pick"] == "all":
        t = np.concatenate([np.stack([np.full(4 ** z, z), np.tile(np.arange(1 << z), 1 << z),
                                      np.repeat(np.arange(1 << z), 1 << z)], axis=1)
                            for z in range(case["zlo"], case["zhi"] + 1)]).astype(np.int32)
        which = np.zeros(len(t), dtype=np.int64)
    else:
        m = case["tiles"]
        which = rng.integers(0, len(sets), m)
        z = rng.integers(case["zlo"], case["zhi"] + 1, m)
        at = np.empty((m, 2))
        for s, (obj, _, _) in enumerate(sets):
            k = np.flatnonzero(which == s)
            at[k] = obj[torch.from_numpy(rng.integers(0, len(obj), len(k))).cuda(), :2].cpu().numpy()
        t = _tile_of(at, z)
        if case["pick"] == "screen":  # seven wide, around the first anchor
            k = np.arange(m)
            side = 1 << case["zlo"]
            t[:, 1] = np.clip(t[0, 1] - min(m - 1, 6) // 2, 0, side - 7) + k % 7
            t[:, 2] = np.clip(t[0, 2] - (m - 1) // 14, 0, side - 1) + k // 7
            t[:, 1:] %= side
    r = rng.uniform(case["rlo"], case["rhi"], len(t)) if case["rhi"] > case["rlo"] else np.full(len(t), case["rlo"])
    return which, t, r


class _Owned:
    """Frees a handle of the library when its last user is gone."""

    def __init__(self, handle, free):
        self.handle, self._free = handle, free

    def __del__(self):
        self._free(self.handle)


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rng = np.random.default_rng(seed)
    sets = _data(case, g)
    which, tiles, r = _tiles(case, sets, rng)
    state = {"path": case["path"], "tiles": hv.tiles_array(tiles), "r": float(r[0])}
    width = hv.HV_AA_BYTES if case["path"] == "aa" else hv.HV_MASK_BYTES
    state["out"] = torch.empty((len(tiles), width), dtype=torch.uint8, device="cuda")
    if case["path"] == "load":
        state["objects"], state["kind"], _ = sets[0]
        return state
    owned = []
    for obj, kind, first in sets:
        if first is not None:
            owned.append(_Owned(hv.hv_polygon_index_build(obj, first.cpu().numpy()), hv.hv_free))
        else:
            owned.append(_Owned(hv.hv_index_build(obj, kind), hv.hv_free))
    state["indexes"] = owned
    if case["path"] in ("batch", "batcher", "aa"):
        handles = np.array([o.handle for o in owned], dtype=np.uint64)
        state["requests"] = hv.requests(handles[which], tiles, r)
    if case["path"] == "batcher":
        state["batcher"] = _Owned(hv.hv_batcher_create(len(tiles), len(owned), 8, TUNED if case["tuned"] else None),
                                  hv.hv_batcher_free)
    return state


def run(state):
    path, out = state["path"], state["out"]
    if path == "tiles":
        hv.hv_render_tiles(state["indexes"][0].handle, state["tiles"], state["r"], out)
    elif path == "batch":
        hv.hv_render_batch(state["requests"], out)
    elif path == "batcher":
        hv.hv_batcher_run(state["batcher"].handle, state["requests"], out)
    elif path == "aa":
        hv.hv_render_batch_aa(state["requests"], out)
    elif path == "fill":
        hv.hv_render_fill(state["indexes"][0].handle, state["tiles"], out)
    else:
        index = hv.hv_index_build(state["objects"], state["kind"])
        hv.hv_render_tiles(index, state["tiles"], state["r"], out)
        torch.cuda.current_stream().synchronize()  # an index is freed only once its renders are done
        hv.hv_free(index)
    return out


# Per tile and per object of the set, what must be read to certify the unlit
# pixels (bytes) and to test them and the lit ones (flops): the oracle's counts
# for the repository's workloads (c1-c4 and filling), whose sets have the
# given number of objects.
_NEED = {"uniform": (10_000, 640.0, 3.7e3), "clustered": (1_000_000_000, 4.5e4, 8e5), "lines": (10_000_000, 1.14e4, 5e4),
         "edges": (200_000_000, 1.24e5, 4.1e6), "two": (10_000_000, 1.14e4, 5e4), "polygons": (200_000_000, 2.6e6, 1.24e6)}


def work(case):
    n, tiles = case["n"], case["tiles"]
    size = 16.0 if case["data"] in ("uniform", "clustered") else 32.0
    ref, nbytes, flops = _NEED[case["data"]]
    share = min(1.0, n / ref)
    out = tiles * (32.0 + (hv.HV_AA_BYTES if case["path"] == "aa" else hv.HV_MASK_BYTES))
    w = {"bytes": out + tiles * nbytes * share, "flops": tiles * flops * share}
    if case["path"] == "aa":
        w["flops"] *= 4.0
    if case["path"] == "load":  # the objects in, the index (objects, order, boxes) out
        w["bytes"] += n * (2.0 * size + 4.0 + 48.0 / 15.0)
        w["flops"] += n * size / 8.0 * 20.0
    return w


def exact(case, seed):
    """Every output is a bit mask or a whole number 0-4: none has a value in floating point to be near to."""
    return None
