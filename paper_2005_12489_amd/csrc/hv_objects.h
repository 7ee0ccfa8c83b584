// Tiles with few objects in reach, object by object.
//
// Where a tile's frontier (k_tile_frontier) lies at the leaves, one level above
// them or, without cells to settle it, two levels above with few nodes, at most
// 262,144 objects can reach the tile.  If they are small and accepts would not
// do most of the work (by_objects), walking the tree for each of its regions
// would test the same nodes and read the same leaves over and over, a memory
// latency at a time.  Here a workgroup takes a strip
// of the tile -- whole pixel rows, so that the mask is written in whole lines --
// and goes over the frontier's objects once, a lane to an object: Algorithm 1's
// per-pixel box filter seen from the object's side gives the pixels in reach,
// every one of which takes the exact FP64 test.
//
// What bounds it: VALU issue (some 60 instructions per object in reach of the
// tile, then 15 per pixel in reach of the object), with the objects' loads
// hidden behind the other waves' arithmetic.
#pragma once

#include "hv_internal.h"

namespace hv {
namespace {

constexpr int kStripThreads = 256;
constexpr int kUnits = 256;          // (object, row) pairs a wave lists at a time
constexpr int kLaneRows = 15;        // objects over more rows or columns of pixels are taken one by one
constexpr int kLaneCols = 12;
constexpr float kReachEps = 1e-3f;   // px: widens every pixel range (FP32, tile-local: rounding is below 1e-4)
constexpr double kSlack = 1e-4;      // px: samples of a wide object's row this near to r are tested, others are not
constexpr double kFlat = 1e-5;       // |dy| / |d| up to which a segment counts as parallel to the rows

// A wave's objects, one per lane.
struct Staged {
    double2 a[64];    // first point (tile-local px)
    double2 d[64];    // segment direction
    double inv[64];   // 1 / |direction|^2 (0 for a zero-length segment)
    uint32_t rg[64];  // pixels in reach: ilo | ihi << 8 | jlo << 16 | jhi << 22 (rows of the strip)
    uint16_t units[kUnits];  // object | row << 6
};

template <int AA>
struct StripLds {
    Staged w[kStripThreads / 64];
    uint32_t mask[(AA ? 4 : 1) * kStripRows * 8];  // sub-sample m at m * kStripRows * 8
    uint32_t nodes[kFrontier], leaves[kFrontier];
    uint32_t upper[kObjectUpper];  // a level-2 frontier's nodes
    int n_nodes, n_leaves, n_upper;
};

// Lights columns c0 .. c1 of a mask row.
__device__ inline void light_run(uint32_t *row, int c0, int c1) {
    for (int w = c0 >> 5; w <= (c1 >> 5); ++w) {
        const int f = max(c0 - 32 * w, 0), t = min(c1 - 32 * w, 31);
        const uint32_t m = (0xffffffffu >> (31 - t)) & (0xffffffffu << f);
        if ((row[w] & m) != m) atomicOr(&row[w], m);
    }
}

// Rows [j0, j0 + rows) of request t's tile.
template <int SEG, int AA>
__device__ __forceinline__ void strip(const DevIndex &ix, const DevReq &rq, int64_t t, int fcount, int flevel, int j0,
                                      int rows, const uint32_t *__restrict__ frontier, uint8_t *out, StripLds<AA> &L) {
    constexpr int NM = AA ? 4 : 1, MW = kStripRows * 8;
    const int tid = threadIdx.x, lane = tid & 63;
    Staged &W = L.w[__builtin_amdgcn_readfirstlane(tid >> 6)];
    const double r = rq.r, r2 = r * r;
    const double S = ldexp(256.0, rq.z), iS = ldexp(1.0, -8 - rq.z);
    const double ox = 256.0 * (double)rq.x, oy = 256.0 * (double)rq.y;
    const double m = (AA ? r + 0.25 : r) + kCullPad;
    const double qx0 = (ox + (0.5 - m)) * iS, qx1 = (ox + (255.5 + m)) * iS;
    const double qy0 = ((oy + (double)j0) + (0.5 - m)) * iS;
    const double qy1 = ((oy + (double)j0) + ((double)rows - 0.5 + m)) * iS;
    const float reach = (float)(AA ? r + 0.25 : r) + kReachEps;
    // from an object's box to its range of pixels in the strip
    const float xlo = -reach - 0.5f, xhi = reach - 0.5f;
    const float ylo = xlo - (float)j0, yhi = xhi - (float)j0, last = (float)(rows - 1);

    for (int k = tid; k < NM * MW; k += kStripThreads) L.mask[k] = 0;
    if (tid == 0) L.n_nodes = L.n_upper = 0;
    __syncthreads();
    auto meets = [&](const double4 &b) { return b.x <= qx1 && b.z >= qx0 && b.y <= qy1 && b.w >= qy0; };
    {
        bool hit = false;
        uint32_t node = 0;
        if (tid < fcount) {
            node = frontier[t * kFrontier + tid];
            hit = meets(ix.nodes[ix.meta[flevel] + node]);
        }
        uint32_t *const to = flevel == 2 ? L.upper : flevel ? L.nodes : L.leaves;
        const int pos = wave_alloc(flevel == 2 ? &L.n_upper : &L.n_nodes, __ballot(hit), lane);
        if (hit) to[pos] = node;
    }
    __syncthreads();

    // exact FP64 squared distance from a sample (tile-local px) to object c
    auto dist2 = [&](const double2 &a, const double2 &d, double inv, double px, double py) -> double {
        const double wx = px - a.x, wy = py - a.y;
        if (SEG) {
            double tt = (wx * d.x + wy * d.y) * inv;
            tt = fmin(fmax(tt, 0.0), 1.0);
            const double ex = wx - tt * d.x, ey = wy - tt * d.y;
            return ex * ex + ey * ey;
        }
        return wx * wx + wy * wy;
    };
    // the pixels ilo .. ihi (at most kLaneCols) of row j
    auto test_pixels = [&](int c, int ilo, int ihi, int j) {
        const int w0 = ilo >> 5, sh = ilo & 31;
        const bool two = (ihi >> 5) != w0;
        const uint32_t want = (2u << (ihi - ilo)) - 1u;  // bit k: column ilo + k
        uint32_t done = ~0u;
#pragma unroll
        for (int mm = 0; mm < NM; ++mm) {
            const uint32_t *row = L.mask + mm * MW + j * 8 + w0;
            done &= __builtin_amdgcn_alignbit(two ? row[1] : 0u, row[0], (uint32_t)sh);
        }
        uint32_t todo = want & ~done;
        if (!todo) return;
        const double2 a = W.a[c];
        double2 d = make_double2(0.0, 0.0);
        double inv = 0.0;
        if (SEG) {
            d = W.d[c];
            inv = W.inv[c];
        }
        uint32_t bits[NM];
#pragma unroll
        for (int mm = 0; mm < NM; ++mm) bits[mm] = 0;
        const double py = (double)(j0 + j) + 0.5;
        while (todo) {
            const int k = __builtin_ctz(todo);
            todo &= todo - 1u;
            const double px = (double)(ilo + k) + 0.5;
            const uint32_t bit = 1u << k;
#pragma unroll
            for (int mm = 0; mm < NM; ++mm) {
                const double sx = AA ? ((mm & 1) ? 0.25 : -0.25) : 0.0, sy = AA ? ((mm & 2) ? 0.25 : -0.25) : 0.0;
                if (dist2(a, d, inv, px + sx, py + sy) <= r2) bits[mm] |= bit;
            }
        }
#pragma unroll
        for (int mm = 0; mm < NM; ++mm) {
            uint32_t *row = L.mask + mm * MW + j * 8 + w0;
            const uint64_t b = (uint64_t)bits[mm] << sh;
            if ((uint32_t)b) atomicOr(&row[0], (uint32_t)b);
            if ((uint32_t)(b >> 32)) atomicOr(&row[1], (uint32_t)(b >> 32));
        }
    };
    // The pixels ilo .. ihi of row j, however many.  Every decision is the exact
    // FP64 test's, but few samples need one: an object grown by a radius is
    // convex, so a row of samples meets it in one run.  Outside the run for
    // r + kSlack no sample is within r, inside that for r - kSlack all are, FP32
    // rounding included (at radii up to 64 px and columns up to 320 it moves a run's end by
    // less than 6e-5 px), and the few between the two are tested.
    static_assert(HV_MAX_RADIUS <= 64.0 && kSlack >= 1e-4, "the slack covers FP32's rounding of a run's ends");
    auto test_run = [&](int c, int ilo, int ihi, int j) {
        const double2 a = W.a[c];
        double2 d = make_double2(0.0, 0.0);
        double inv = 0.0, idy = 0.0, u = 0.0;
        bool flat = false;
        if (SEG) {
            d = W.d[c];
            inv = W.inv[c];
            // 1 / |d| and 1 / dy: the hardware's approximation and a Newton step
            const double l2 = d.x * d.x + d.y * d.y;
            double q = __builtin_amdgcn_rsq(l2);
            q = fma(0.5 * q, fma(-l2 * q, q, 1.0), q);
            flat = !(fabs(d.y) * q > kFlat);  // zero-length segments too
            idy = __builtin_amdgcn_rcp(d.y);
            idy = fma(idy, fma(-d.y, idy, 1.0), idy);
            u = r * d.x * (d.y < 0.0 ? -q : q);
        }
        const float more2 = (float)((r + kSlack) * (r + kSlack));
        const float less2 = r > 2.0 * kSlack ? (float)((r - kSlack) * (r - kSlack)) : -1.0f;
#pragma unroll
        for (int sy = 0; sy < (AA ? 2 : 1); ++sy) {
            const double py = (double)(j0 + j) + 0.5 + (AA ? (sy ? 0.25 : -0.25) : 0.0);
            const double wy = py - a.y, ax = a.x - 0.5;
            // the larger run's ends in columns (pixel centres at whole
            // numbers), and how far the smaller one's lie inside
            float xl, xr, ml, mr;
            bool each;  // the smaller run may be empty
            if (SEG) {
                // The farthest point of the grown segment along the row is
                // around t = (wy -+ u) / dy of the segment, u = r dx / |d| with
                // dy's sign, or around an endpoint (t clamped to [0, 1]; the
                // extent is concave in t).  Segments all but parallel to the
                // row take their endpoints.
                double tl = fmin(fmax((wy - u) * idy, 0.0), 1.0);
                double tr = fmin(fmax((wy + u) * idy, 0.0), 1.0);
                if (flat) {
                    tl = d.x > 0.0 ? 0.0 : 1.0;
                    tr = 1.0 - tl;
                }
                const double el = wy - tl * d.y, er = wy - tr * d.y;
                float sl = (float)(el * el), sr = (float)(er * er);
                const float kl = less2 - sl, kr = less2 - sr;
                if (flat) sl = sr = el * er < 0.0 ? 0.0f : fminf(sl, sr);
                const float ql = more2 - sl, qr = more2 - sr;
                if (ql < 0.0f || qr < 0.0f) continue;
                each = kl < 0.0f || kr < 0.0f;
                const float hl = __builtin_amdgcn_sqrtf(ql), hr = __builtin_amdgcn_sqrtf(qr);
                xl = (float)(ax + tl * d.x) - hl;
                xr = (float)(ax + tr * d.x) + hr;
                ml = hl - __builtin_amdgcn_sqrtf(fmaxf(kl, 0.0f)) + 1e-4f;
                mr = hr - __builtin_amdgcn_sqrtf(fmaxf(kr, 0.0f)) + 1e-4f;
            } else {
                const float e2 = (float)(wy * wy), q = more2 - e2, k = less2 - e2;
                if (q < 0.0f) continue;
                each = k < 0.0f;
                const float h = __builtin_amdgcn_sqrtf(q);
                xl = (float)ax - h;
                xr = (float)ax + h;
                ml = mr = h - __builtin_amdgcn_sqrtf(fmaxf(k, 0.0f)) + 1e-4f;
            }
#pragma unroll
            for (int sx = 0; sx < (AA ? 2 : 1); ++sx) {
                const float off = AA ? (sx ? 0.25f : -0.25f) : 0.0f;
                const float fl = fminf(fmaxf(ceilf(xl - off), (float)ilo), 256.0f);
                const float fr = fmaxf(fminf(floorf(xr - off), (float)ihi), -1.0f);
                if (!(fl <= fr)) continue;
                int c0 = (int)fl, c1 = (int)fr;
                uint32_t *const row = L.mask + (AA ? 2 * sy + sx : 0) * MW + j * 8;
                auto hit = [&](int x) { return dist2(a, d, inv, (double)x + 0.5 + (double)off, py) <= r2; };
                if (each) {
                    for (int x = c0; x <= c1; ++x)
                        if (hit(x)) light_run(row, x, x);
                    continue;
                }
                while (c0 <= c1 && (float)c0 - (xl - off) < ml && !hit(c0)) ++c0;
                while (c0 <= c1 && (xr - off) - (float)c1 < mr && !hit(c1)) --c1;
                if (c0 <= c1) light_run(row, c0, c1);
            }
        }
    };

    auto load = [&](int64_t o) -> double4 {
        if (SEG) return reinterpret_cast<const double4 *>(ix.obj)[o];
        const double2 p = reinterpret_cast<const double2 *>(ix.obj)[o];
        return make_double4(p.x, p.y, p.x, p.y);
    };
    // The objects of the leaves listed.
    auto take_leaves = [&](int n_leaves) {
        const int total = n_leaves * kLeaf;
        auto object_of = [&](int k) -> int64_t {
            return k < total ? (int64_t)L.leaves[k / kLeaf] * kLeaf + k % kLeaf : ix.n;
        };
        int64_t o = object_of(tid);
        double4 next = o < ix.n ? load(o) : make_double4(0.0, 0.0, 0.0, 0.0);
        for (int base = 0; base < total; base += kStripThreads) {
            const bool have = o < ix.n;
            const double4 g = next;
            o = object_of(base + kStripThreads + tid);
            if (o < ix.n) next = load(o);
            // tile-local pixel frame; scaling by S is exact
            const double ua = g.x * S - ox, va = g.y * S - oy;
            const double ub = SEG ? g.z * S - ox : ua, vb = SEG ? g.w * S - oy : va;
            const float fa = (float)ua, ga = (float)va, fb = (float)ub, gb = (float)vb;
            const float flo_i = fmaxf(ceilf(fminf(fa, fb) + xlo), 0.0f), fhi_i = fminf(floorf(fmaxf(fa, fb) + xhi), 255.0f);
            const float flo_j = fmaxf(ceilf(fminf(ga, gb) + ylo), 0.0f), fhi_j = fminf(floorf(fmaxf(ga, gb) + yhi), last);
            const bool keep = have && flo_i <= fhi_i && flo_j <= fhi_j;
            const int ilo = (int)flo_i, ihi = (int)fhi_i, jlo = (int)flo_j, jhi = (int)fhi_j;
            const bool wide = keep && (ihi - ilo >= kLaneCols || jhi - jlo >= kLaneRows);
            const uint32_t count = keep && !wide ? (uint32_t)(jhi - jlo + 1) : 0u;
            if (keep) {
                W.a[lane] = make_double2(ua, va);
                W.rg[lane] = (uint32_t)ilo | (uint32_t)ihi << 8 | (uint32_t)jlo << 16 | (uint32_t)jhi << 22;
                if (SEG) {
                    const double dx = ub - ua, dy = vb - va, l2 = dx * dx + dy * dy;
                    W.d[lane] = make_double2(dx, dy);
                    // 1 / l2: the hardware reciprocal and two Newton steps
                    double iv = __builtin_amdgcn_rcp(l2);
                    iv = fma(iv, fma(-l2, iv, 1.0), iv);
                    iv = fma(iv, fma(-l2, iv, 1.0), iv);
                    W.inv[lane] = l2 > 0.0 ? iv : 0.0;
                }
            }
            // the rows of the wave's objects, listed one after another, so
            // that the lanes stay busy whatever the objects' sizes
            int first = 0, rows_all = 0;
#pragma unroll
            for (int b = 0; (1 << b) <= kLaneRows; ++b) {
                const uint64_t bm = __ballot((count >> b) & 1u);
                first += (int)lanes_below(bm) << b;
                rows_all += __popcll(bm) << b;
            }
            for (int w0 = 0; w0 < rows_all; w0 += kUnits) {
                __builtin_amdgcn_wave_barrier();
                for (int k = 0; k < (int)count; ++k) {
                    const int at = first + k - w0;
                    if (at >= 0 && at < kUnits) W.units[at] = (uint16_t)(lane | (jlo + k) << 6);
                }
                __builtin_amdgcn_wave_barrier();
                const int nu = min(rows_all - w0, kUnits);
                for (int q = lane; q < nu; q += 64) {
                    const uint32_t e = W.units[q];
                    const uint32_t rg = W.rg[e & 63];
                    test_pixels((int)(e & 63), (int)(rg & 255), (int)((rg >> 8) & 255), (int)(e >> 6));
                }
            }
            __builtin_amdgcn_wave_barrier();
            // an object over many pixels: its rows straight to the lanes
            for (uint64_t bm = __ballot(wide); bm; bm &= bm - 1) {
                const int c = __builtin_ctzll(bm);
                const uint32_t rg = W.rg[c];
                const int j = (int)((rg >> 16) & 63) + lane;
                if (j <= (int)(rg >> 22)) test_run(c, (int)(rg & 255), (int)((rg >> 8) & 255), j);
            }
            __builtin_amdgcn_wave_barrier();
        }
    };
    // The children (of level `lvl`) that meet the strip of up to
    // kStripThreads / kFan nodes at a time.
    auto expand = [&](const uint32_t *nodes, int base, int n, int lvl, uint32_t *to, int *count) {
        if (tid == 0) *count = 0;
        __syncthreads();
        const int k = base + tid / kFan;
        bool hit = false;
        int64_t child = 0;
        if (k < n) {
            child = (int64_t)nodes[k] * kFan + tid % kFan;
            hit = child < ix.meta[kMaxLevels + lvl] && meets(ix.nodes[ix.meta[lvl] + child]);
        }
        const int pos = wave_alloc(count, __ballot(hit), lane);
        if (hit) to[pos] = (uint32_t)child;
        __syncthreads();
    };
    constexpr int kStep = kStripThreads / kFan;
    if (flevel == 0) {
        take_leaves(L.n_nodes);
    } else {
        for (int up = 0;; up += kStep) {
            if (flevel == 2) {
                if (up >= L.n_upper) break;
                expand(L.upper, up, L.n_upper, 1, L.nodes, &L.n_nodes);
            }
            const int n_nodes = L.n_nodes;
            for (int base = 0; base < n_nodes; base += kStep) {
                expand(L.nodes, base, n_nodes, 0, L.leaves, &L.n_leaves);
                take_leaves(L.n_leaves);
                __syncthreads();
            }
            if (flevel != 2) break;
        }
    }
    __syncthreads();
    if (AA) {
        // one byte per pixel: the number of its sub-samples within r
        uint32_t *const o = reinterpret_cast<uint32_t *>(out + t * (int64_t)HV_AA_BYTES + j0 * 256);
        for (int k = tid; k < rows * 64; k += kStripThreads) {
            const int row = k >> 6, col = 4 * (k & 63), w = row * 8 + (col >> 5);
            uint32_t v = 0;
#pragma unroll
            for (int mm = 0; mm < NM; ++mm) {
                const uint32_t b = L.mask[mm * MW + w] >> (col & 31);
                v += (b & 1u) | (b & 2u) << 7 | (b & 4u) << 14 | (b & 8u) << 21;
            }
            o[k] = v;
        }
    } else {
        uint4 *const o = reinterpret_cast<uint4 *>(out + t * (int64_t)HV_MASK_BYTES + j0 * 32);
        for (int k = tid; k < rows * 2; k += kStripThreads) o[k] = reinterpret_cast<const uint4 *>(L.mask)[k];
    }
    __syncthreads();
}

// The object kernel's work items: the strips of the tiles whose frontier lies
// above the leaves first, then of those with a frontier of leaves.
__device__ inline int64_t object_items(const DevBatch &B, int leaf_strips, int node_strips) {
    return (int64_t)B.hdr->node_tiles * node_strips + (int64_t)B.hdr->leaf_tiles * leaf_strips;
}

template <int AA>
__device__ __forceinline__ void object_item(const DevBatch &B, int64_t u, int leaf_strips, int node_strips, uint8_t *out,
                                            StripLds<AA> &L) {
    static_assert(256 / kLeafStrips <= kStripRows && 256 / kNodeStrips <= kStripRows, "a strip fits its rows in LDS");
    const int64_t node_items = (int64_t)B.hdr->node_tiles * node_strips, cap = B.hdr->n_req;
    const bool node = u < node_items;
    const int64_t v = node ? u : u - node_items;
    const int strips = node ? node_strips : leaf_strips;
    const int64_t t = (node ? B.elist : B.list)[cap - 1 - v / strips];
    const int rows = 256 / strips, j0 = (int)(v % strips) * rows;
    const DevReq rq = B.reqs[t];
    const DevIndex ix = B.ixs[rq.index];
    const int fcount = B.fmeta[4 * t], flevel = B.fmeta[4 * t + 1];
    if (ix.seg) strip<1, AA>(ix, rq, t, fcount, flevel, j0, rows, B.frontier, out, L);
    else strip<0, AA>(ix, rq, t, fcount, flevel, j0, rows, B.frontier, out, L);
    if (threadIdx.x == 0 && atomicAdd(&B.done[t], 1u) == (uint32_t)strips - 1u) B.ts[t] = wall_clock64();
}

}  // namespace
}  // namespace hv
