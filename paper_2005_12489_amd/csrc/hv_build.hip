// GPU index build: project -> Hilbert keys -> LSD radix sort -> gather ->
// bottom-up packing of a Hilbert-packed R-tree.
//
// The paper keeps one R-tree per object kind, whose entries are points,
// segments or polygon edges rather than whole objects (Sec. 3.1), built
// with Boost on the CPU.  Here the tree is packed on the GPU: objects are
// ordered along a Hilbert curve through their bounding-box centres (the
// Hilbert-packed R-tree of Kamel and Faloutsos, 1993), cut into leaves of
// kLeaf consecutive objects, and each upper level groups kFan consecutive
// nodes.  Children are implicit (node i of level k owns nodes
// i*kFan .. i*kFan+kFan-1 of level k-1), so the tree has no pointers and
// every level is one contiguous array of FP64 boxes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "hv_internal.h"

namespace hv {
namespace {

constexpr int kST = 512;            // radix-sort threads per block
constexpr int kSKeys = 16;          // keys per thread
constexpr int kSTile = kST * kSKeys;
constexpr int kRT = 256;            // scan threads per block
constexpr int kRIPT = 16;           // counts per thread
constexpr int kRTile = kRT * kRIPT;
constexpr double kMaxLat = 85.0511287798066;
constexpr double kPi = 3.14159265358979323846;

// ------------------------------------------------------------ projection
// lon/lat (deg) -> normalised Web-Mercator X (east), Y (south, 0 = north).
// Contraction is off so that every kernel that projects an object gets the same
// bits: the sort key and the stored coordinates are computed apart.
__device__ inline void mercator(double lon, double lat, double &X, double &Y) {
#pragma clang fp contract(off)
    lat = fmin(fmax(lat, -kMaxLat), kMaxLat);
    const double phi = lat * (kPi / 180.0);
    X = (lon + 180.0) / 360.0;
    Y = 0.5 - log(tan(kPi / 4.0 + phi / 2.0)) / (2.0 * kPi);
}

// Hilbert index of (x, y) on a 2^bits grid (xy -> d: at each level take the
// quadrant's position along the curve, then rotate / reflect the remaining
// low bits into that quadrant's frame).
__device__ inline uint64_t hilbert_d(uint32_t x, uint32_t y, int bits) {
    uint64_t d = 0;
    for (int b = bits - 1; b >= 0; --b) {
        const uint32_t rx = (x >> b) & 1u, ry = (y >> b) & 1u;
        d |= (uint64_t)((3u * rx) ^ ry) << (2 * b);
        if (ry == 0) {
            if (rx == 1) { x = ~x; y = ~y; }
            const uint32_t t = x; x = y; y = t;
        }
    }
    return d;
}

__device__ inline uint32_t quantise(double c, int bits) {
    const double s = ldexp(1.0, bits);
    double q = floor(c * s);
    q = fmin(fmax(q, 0.0), s - 1.0);
    return (uint32_t)q;
}

// An object's projected coordinates.
template <int W>
__device__ inline void project(const double *__restrict__ in, int64_t i, int merc, double *p) {
    double v[W];
    if constexpr (W == 2) {
        const double2 g = reinterpret_cast<const double2 *>(in)[i];
        v[0] = g.x, v[1] = g.y;
    } else {
        const double4 g = reinterpret_cast<const double4 *>(in)[i];
        v[0] = g.x, v[1] = g.y, v[2] = g.z, v[3] = g.w;
    }
#pragma unroll
    for (int c = 0; c < W; c += 2) {
        if (merc) { p[c] = v[c]; p[c + 1] = v[c + 1]; }
        else mercator(v[c], v[c + 1], p[c], p[c + 1]);
    }
}

// The Hilbert key of every object's box centre: its low 8 bits (the first digit
// sorted by) and the rest, at most 32 bits.
template <int W>
__global__ __launch_bounds__(256) void k_project_key(const double *__restrict__ in, int64_t n, int merc,
                                                     uint8_t *__restrict__ low, uint32_t *__restrict__ high, int bits,
                                                     int *err) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    bool bad = false;
#pragma unroll
    for (int c = 0; c < W; c += 2) {
        const double x = in[i * W + c], y = in[i * W + c + 1];
        bad |= !isfinite(x) || !isfinite(y) || (!merc && (fabs(x) > 180.0 || fabs(y) > 90.0));
    }
    if (bad) atomicOr(err, 1);
    double p[W];
    project<W>(in, i, merc, p);
    double cx = p[0], cy = p[1];
    if constexpr (W == 4) {
        cx = 0.5 * (fmin(p[0], p[2]) + fmax(p[0], p[2]));
        cy = 0.5 * (fmin(p[1], p[3]) + fmax(p[1], p[3]));
    }
    const uint64_t key = hilbert_d(quantise(cx, bits), quantise(cy, bits), bits);
    low[i] = (uint8_t)key;
    high[i] = (uint32_t)(key >> 8);
}

// Least and greatest of 16 neighbouring lanes' boxes, in every lane.
__device__ inline double4 box16(double4 b) {
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
        b.x = fmin(b.x, __shfl_xor(b.x, o, 64));
        b.y = fmin(b.y, __shfl_xor(b.y, o, 64));
        b.z = fmax(b.z, __shfl_xor(b.z, o, 64));
        b.w = fmax(b.w, __shfl_xor(b.w, o, 64));
    }
    return b;
}

__device__ inline double4 edge_box(const double *p) {
    return make_double4(fmin(p[0], p[2]), fmin(p[1], p[3]), fmax(p[0], p[2]), fmax(p[1], p[3]));
}

__device__ inline double4 box_union(const double4 &a, const double4 &b) {
    return make_double4(fmin(a.x, b.x), fmin(a.y, b.y), fmax(a.z, b.z), fmax(a.w, b.w));
}

// Bounding box of each polygon's projected edges, written as the diagonal
// segment (min X, min Y) - (max X, max Y), whose own box is the polygon's box;
// 16 lanes to a polygon.  Flags coordinates that are not finite or outside
// [-180, 180] x [-90, 90].
__global__ __launch_bounds__(256) void k_polygon_boxes(const double *__restrict__ edges,
                                                       const int64_t *__restrict__ first, int64_t npoly, int merc,
                                                       double *__restrict__ diag, int *err) {
    const int64_t p = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 4;
    const int c = threadIdx.x & 15;
    double4 box = make_double4(INFINITY, INFINITY, -INFINITY, -INFINITY);
    bool bad = false;
    if (p < npoly)
        for (int64_t e = first[p] + c; e < first[p + 1]; e += 16) {
            const double4 v = reinterpret_cast<const double4 *>(edges)[e];
            bad |= !isfinite(v.x) || !isfinite(v.y) || !isfinite(v.z) || !isfinite(v.w);
            if (!merc) bad |= fabs(v.x) > 180.0 || fabs(v.y) > 90.0 || fabs(v.z) > 180.0 || fabs(v.w) > 90.0;
            double q[4];
            project<4>(edges, e, merc, q);
            box = box_union(box, edge_box(q));
        }
    if (bad) atomicOr(err, 1);
    box = box16(box);
    if (p < npoly && c == 0) reinterpret_cast<double4 *>(diag)[p] = box;
}

// Conservative float box of each run of kEdgeChunk consecutive edges of the
// edge array (runs may straddle polygons): min rounded down, max rounded up,
// so that every edge of the run lies inside it exactly.
__device__ inline float float_down(double d) {
    float f = (float)d;
    if ((double)f > d) f = nextafterf(f, -INFINITY);
    return f;
}
__device__ inline float float_up(double d) {
    float f = (float)d;
    if ((double)f < d) f = nextafterf(f, INFINITY);
    return f;
}

// Eight lanes to a run.
__global__ __launch_bounds__(256) void k_edge_chunks(const double *__restrict__ edges, int64_t n,
                                                     float4 *__restrict__ chunks) {
    static_assert(kEdgeChunk == 8, "a chunk is 8 neighbouring lanes");
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double4 b = make_double4(INFINITY, INFINITY, -INFINITY, -INFINITY);
    if (e < n) {
        const double4 g = reinterpret_cast<const double4 *>(edges)[e];
        b = make_double4(fmin(g.x, g.z), fmin(g.y, g.w), fmax(g.x, g.z), fmax(g.y, g.w));
    }
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) {
        b.x = fmin(b.x, __shfl_xor(b.x, o, 64));
        b.y = fmin(b.y, __shfl_xor(b.y, o, 64));
        b.z = fmax(b.z, __shfl_xor(b.z, o, 64));
        b.w = fmax(b.w, __shfl_xor(b.w, o, 64));
    }
    if (e < n && e % kEdgeChunk == 0)
        chunks[e / kEdgeChunk] = make_float4(float_down(b.x), float_down(b.y), float_up(b.z), float_up(b.w));
}

// Union of each run of kChunkSuper chunk boxes (already outward-rounded):
// the upper level of the two-level box hierarchy over a polygon's edges.
__global__ __launch_bounds__(256) void k_super_chunks(const float4 *__restrict__ chunks, int64_t nchunk,
                                                      float4 *__restrict__ supers) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= (nchunk + kChunkSuper - 1) / kChunkSuper) return;
    float4 b = chunks[s * kChunkSuper];
    const int64_t c1 = min(nchunk, (s + 1) * kChunkSuper);
    for (int64_t c = s * kChunkSuper + 1; c < c1; ++c) {
        const float4 q = chunks[c];
        b = make_float4(fminf(b.x, q.x), fminf(b.y, q.y), fmaxf(b.z, q.z), fmaxf(b.w, q.w));
    }
    supers[s] = b;
}

// Projects each polygon's edges from input order into the tree's order: wave w
// of the grid moves sorted polygon w, whose edges start at src_first[order[w]]
// in `src` and at dst_first[w] in `dst`.
__global__ __launch_bounds__(256) void k_permute_polygons(const double4 *__restrict__ src,
                                                          const int64_t *__restrict__ src_first,
                                                          const uint32_t *__restrict__ order,
                                                          const int64_t *__restrict__ dst_first, int64_t npoly, int merc,
                                                          double4 *__restrict__ dst) {
    const int64_t k = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (k >= npoly) return;
    const int64_t p = order[k];
    const int64_t s0 = src_first[p], cnt = src_first[p + 1] - s0, d0 = dst_first[k];
    for (int64_t e = lane; e < cnt; e += 64) {
        double q[4];
        project<4>(reinterpret_cast<const double *>(src), s0 + e, merc, q);
        dst[d0 + e] = make_double4(q[0], q[1], q[2], q[3]);
    }
}

// ------------------------------------------------------------ scans
__device__ inline uint32_t lanes_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Exclusive scan over the block (blockDim a multiple of 64, <= 1024).
// ws: 16 words of LDS.  All threads must call it.
__device__ uint32_t block_excl_scan(uint32_t v, uint32_t *total, uint32_t *ws) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) ws[w] = x;
    __syncthreads();
    if (w == 0) {
        uint32_t s = lane < nw ? ws[lane] : 0u;
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            const uint32_t y = __shfl_up(s, o, 64);
            if (lane >= o) s += y;
        }
        if (lane < nw) ws[lane] = s;
    }
    __syncthreads();
    const uint32_t off = w ? ws[w - 1] : 0u;
    *total = ws[nw - 1];
    __syncthreads();
    return off + x - v;
}

__global__ __launch_bounds__(256) void k_scan_reduce(const uint32_t *__restrict__ a, int64_t m,
                                                     uint32_t *__restrict__ part) {
    __shared__ uint32_t ws[16];
    const int64_t base = (int64_t)blockIdx.x * kRTile;
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kRIPT; ++k) {
        const int64_t idx = base + k * kRT + threadIdx.x;
        if (idx < m) s += a[idx];
    }
    uint32_t tot;
    block_excl_scan(s, &tot, ws);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

__global__ __launch_bounds__(1024) void k_scan_partials(uint32_t *part, int64_t np) {
    __shared__ uint32_t ws[16];
    uint32_t carry = 0;
    for (int64_t b = 0; b < np; b += 1024) {
        const int64_t idx = b + threadIdx.x;
        const uint32_t v = idx < np ? part[idx] : 0u;
        uint32_t tot;
        const uint32_t e = block_excl_scan(v, &tot, ws);
        if (idx < np) part[idx] = carry + e;
        carry += tot;
    }
}

__global__ __launch_bounds__(256) void k_scan_down(uint32_t *__restrict__ a, int64_t m,
                                                   const uint32_t *__restrict__ part) {
    __shared__ uint32_t ws[16];
    const int64_t base = (int64_t)blockIdx.x * kRTile + (int64_t)threadIdx.x * kRIPT;
    uint32_t v[kRIPT];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kRIPT; ++k) {
        v[k] = base + k < m ? a[base + k] : 0u;
        s += v[k];
    }
    uint32_t tot;
    uint32_t e = block_excl_scan(s, &tot, ws) + part[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kRIPT; ++k) {
        if (base + k < m) a[base + k] = e;
        e += v[k];
    }
}

// ------------------------------------------------------------ radix sort
// Digit histogram of one block's tile; counts are digit-major so that one
// exclusive scan gives every (digit, block) its output offset.  FIRST: the
// digit is the key's low byte, kept apart.
template <bool FIRST>
__global__ __launch_bounds__(kST) void k_radix_hist(const uint8_t *__restrict__ low, const uint32_t *__restrict__ keys,
                                                    int64_t n, int shift, uint32_t *__restrict__ counts, int64_t nb) {
    __shared__ uint32_t h[256];
    if (threadIdx.x < 256) h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * kSTile;
#pragma unroll
    for (int k = 0; k < kSKeys; ++k) {
        const int64_t idx = t0 + k * kST + threadIdx.x;
        if (idx < n) atomicAdd(&h[FIRST ? low[idx] : (keys[idx] >> shift) & 255u], 1u);
    }
    __syncthreads();
    if (threadIdx.x < 256) counts[(int64_t)threadIdx.x * nb + blockIdx.x] = h[threadIdx.x];
}

// Stable scatter of (key, object) pairs.  A wave ranks kSKeys * 64 consecutive
// keys in input order: lanes holding the same digit find each other with eight
// ballots, and per-digit counts carry the order from one 64 to the next.  The
// tile is then brought into digit order in LDS, so that a digit's keys -- 32
// on average -- go out as one run of whole lines.  (Written lane by lane, each
// to its own line, a pass over 1e9 pairs took 26 ms.)  FIRST: the digit is the
// key's low byte and the objects are in input order.
template <bool FIRST>
__global__ __launch_bounds__(kST) void k_radix_scatter(const uint8_t *__restrict__ low, const uint32_t *__restrict__ kin,
                                                       const uint32_t *__restrict__ vin, uint32_t *__restrict__ kout,
                                                       uint32_t *__restrict__ vout, int64_t n, int shift,
                                                       const uint32_t *__restrict__ offs, int64_t nb) {
    constexpr int kWaves = kST / 64;
    __shared__ uint32_t sorted[kSTile];
    __shared__ uint8_t digit_of[kSTile];
    __shared__ uint16_t wc[kWaves][256];  // keys of a digit seen by a wave; then where its first goes in the tile
    __shared__ uint32_t goff[256];        // where the tile's first key of a digit goes, less its place in the tile
    __shared__ uint32_t ws[16];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    for (int k = tid; k < kWaves * 256; k += kST) wc[0][k] = 0;
    __syncthreads();
    const int64_t w0 = (int64_t)blockIdx.x * kSTile + (int64_t)w * (64 * kSKeys);
    const int count = (int)min((int64_t)kSTile, n - (int64_t)blockIdx.x * kSTile);
    uint32_t key[kSKeys], val[kSKeys];
    uint16_t rank[kSKeys];
    uint8_t dig[kSKeys];
#pragma unroll
    for (int k = 0; k < kSKeys; ++k) {
        const int64_t idx = w0 + k * 64 + lane;
        const bool valid = idx < n;
        key[k] = valid ? kin[idx] : 0u;
        val[k] = FIRST ? (uint32_t)idx : valid ? vin[idx] : 0u;
        dig[k] = FIRST ? (valid ? low[idx] : 0) : (uint8_t)(key[k] >> shift);
    }
#pragma unroll
    for (int k = 0; k < kSKeys; ++k) {
        const bool valid = w0 + k * 64 + lane < n;
        const uint32_t d = dig[k];
        uint64_t m = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            m &= bit ? bb : ~bb;
        }
        const uint32_t below = lanes_below(m), seen = wc[w][d];
        rank[k] = (uint16_t)(seen + below);
        __builtin_amdgcn_wave_barrier();
        if (valid && below == 0) wc[w][d] = (uint16_t)(seen + (uint32_t)__popcll(m));
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    {
        uint32_t total = 0, sum = 0;
        if (tid < 256)
#pragma unroll
            for (int q = 0; q < kWaves; ++q) total += wc[q][tid];
        uint32_t all;
        sum = block_excl_scan(tid < 256 ? total : 0u, &all, ws);
        if (tid < 256) {
            goff[tid] = offs[(int64_t)tid * nb + blockIdx.x] - sum;
#pragma unroll
            for (int q = 0; q < kWaves; ++q) {
                const uint32_t c = wc[q][tid];
                wc[q][tid] = (uint16_t)sum;
                sum += c;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSKeys; ++k)
        if (w0 + k * 64 + lane < n) {
            const uint32_t at = wc[w][dig[k]] + rank[k];
            rank[k] = (uint16_t)at;
            sorted[at] = key[k];
            digit_of[at] = dig[k];
        }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSKeys; ++k) {
        const int i = k * kST + tid;
        if (i < count) kout[goff[digit_of[i]] + i] = sorted[i];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSKeys; ++k)
        if (w0 + k * 64 + lane < n) sorted[rank[k]] = val[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSKeys; ++k) {
        const int i = k * kST + tid;
        if (i < count) vout[goff[digit_of[i]] + i] = sorted[i];
    }
}

// ------------------------------------------------------------ gather + pack
// Projects the objects once more, now in sorted order, and packs the leaves:
// each leaf's box and representative, the first vertex of its first object.
template <int W>
__global__ __launch_bounds__(256) void k_gather_leaves(const double *__restrict__ in, const uint32_t *__restrict__ order,
                                                       int64_t n, int merc, double *__restrict__ obj,
                                                       double4 *__restrict__ leaf, double2 *__restrict__ rep) {
    static_assert(kLeaf == 16, "a leaf is 16 neighbouring lanes");
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double4 b = make_double4(INFINITY, INFINITY, -INFINITY, -INFINITY);
    if (i < n) {
        double p[W];
        project<W>(in, order[i], merc, p);
        if constexpr (W == 2) {
            reinterpret_cast<double2 *>(obj)[i] = make_double2(p[0], p[1]);
            b = make_double4(p[0], p[1], p[0], p[1]);
        } else {
            reinterpret_cast<double4 *>(obj)[i] = make_double4(p[0], p[1], p[2], p[3]);
            b = make_double4(fmin(p[0], p[2]), fmin(p[1], p[3]), fmax(p[0], p[2]), fmax(p[1], p[3]));
        }
        if (i % kLeaf == 0) rep[i / kLeaf] = make_double2(p[0], p[1]);
    }
    b = box16(b);
    if (i < n && i % kLeaf == 0) leaf[i / kLeaf] = b;
}

// The median over 64 of n segments, spread over the sorted order, of the larger
// side of their boxes; a wavefront.
__device__ inline void median_extent(const double4 *__restrict__ obj, int64_t n, double *__restrict__ extent) {
    const int lane = threadIdx.x & 63;
    const double4 g = obj[n * lane / 64];
    const float mine = (float)fmax(fabs(g.z - g.x), fabs(g.w - g.y));
    int rank = 0;
    for (int k = 0; k < 64; ++k) {
        const float v = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(mine), k));
        rank += v < mine || (v == mine && k < lane);
    }
    if (rank == 32) *extent = mine;
}

// A level's boxes and representatives from its children's.  Node i of level l
// owns the sorted objects [i * 16^(l + 1), (i + 1) * 16^(l + 1)), so its
// representative is its first child's.  The launch of the root's level, one
// workgroup, also takes the n objects' extent.
__global__ __launch_bounds__(256) void k_level(const double4 *__restrict__ child, const double2 *__restrict__ child_rep,
                                               int64_t nchild, double4 *__restrict__ parent,
                                               double2 *__restrict__ parent_rep, const double4 *__restrict__ obj,
                                               int64_t n, double *__restrict__ extent) {
    static_assert(kFan == 16, "a node is 16 neighbouring lanes");
    if (extent && blockIdx.x == 0 && threadIdx.x < 64) median_extent(obj, n, extent);
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const double4 b = box16(i < nchild ? child[i] : make_double4(INFINITY, INFINITY, -INFINITY, -INFINITY));
    if (i < nchild && i % kFan == 0) {
        parent[i / kFan] = b;
        parent_rep[i / kFan] = child_rep[i];
    }
}

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Bits per axis of the Hilbert grid: enough for ~16 cells per object on
// average, a multiple of 4 so that the key is a whole number of digits.
constexpr int key_bits_for(int64_t n) {
    int lg = 0;
    while ((int64_t(1) << lg) < n && lg < 62) ++lg;
    int kb = (lg + 1) / 2 + 4;
    kb = (kb + 3) / 4 * 4;
    return std::max(8, kb);
}

static_assert(2 * key_bits_for(HV_MAX_OBJECTS) <= 40, "keys are sorted as 8 and 32 bits");

// Offsets of the arrays of one block.
struct Carve {
    size_t bytes = 0;
    size_t take(size_t b) {
        const size_t at = bytes;
        bytes += (b + 255) & ~size_t(255);
        return at;
    }
};

struct Scratch {
    unsigned char *p = nullptr;
    size_t bytes = 0;
    ~Scratch() {
        if (p) device_release(p, bytes);
    }
    hipError_t alloc(size_t want) {
        if (want == 0) return hipSuccess;
        return device_acquire(reinterpret_cast<void **>(&p), want, &bytes);
    }
};

// A block of their own for the cells, which are given back if they turn out to
// be of no use.  (They are an aid only: without memory for them, none.)
void acquire_cells(IndexArrays *a, size_t bytes) {
    if (device_acquire(reinterpret_cast<void **>(&a->cells), bytes, &a->cell_bytes) != hipSuccess) (void)hipGetLastError();
}

BuildResult hip_fail(hipError_t e) {
    (void)hipGetLastError();
    if (e == hipErrorOutOfMemory) return {HV_ENOMEM, "out of device memory"};
    return {HV_EHIP, hipGetErrorString(e)};
}

}  // namespace

void free_poly_arrays(PolyArrays *p) {
    if (p->block) device_release(p->block, p->block_bytes);
    *p = PolyArrays{};
}

BuildResult build_polygons(const double *edges, int64_t n, const int64_t *first, int64_t npoly, int flags,
                           hipStream_t st, IndexArrays *tree, PolyArrays *poly) {
    const int merc = (flags & HV_INPUT_MERC01) != 0;
    *tree = IndexArrays{};
    *poly = PolyArrays{};
    poly->npoly = npoly;
    poly->n_edges = n;
    tree->seg = 1;
    if (npoly == 0) return {HV_OK, ""};
    auto bail = [&](hipError_t e) {
        free_poly_arrays(poly);
        free_index_arrays(tree);
        return hip_fail(e);
    };
    // The polygons' boxes, from the edges as they are; once the tree has sorted
    // the polygons, the edges are projected into the tree's order, so that the
    // polygons of one region lie close together in memory.
    const int64_t nchunk = cdiv(n, kEdgeChunk), nsuper = cdiv(nchunk, kChunkSuper);
    Carve index, work;
    const size_t o_edges = index.take(sizeof(double) * 4 * (size_t)n);
    const size_t o_first = index.take(sizeof(int64_t) * (size_t)(npoly + 1));
    const size_t o_chunks = index.take(sizeof(float4) * (size_t)nchunk);
    const size_t o_supers = index.take(sizeof(float4) * (size_t)nsuper);
    const size_t o_in = work.take(sizeof(int64_t) * (size_t)(npoly + 1));
    const size_t o_diag = work.take(sizeof(double) * 4 * (size_t)npoly), o_flags = work.take(sizeof(CellFlags));
    Scratch scratch;
    hipError_t e;
    if ((e = scratch.alloc(work.bytes)) != hipSuccess) return bail(e);
    int64_t *const in_first = reinterpret_cast<int64_t *>(scratch.p + o_in);
    double *const diag = reinterpret_cast<double *>(scratch.p + o_diag);
    CellFlags *const flg = reinterpret_cast<CellFlags *>(scratch.p + o_flags);
    if ((e = hipMemcpyAsync(in_first, first, sizeof(int64_t) * (size_t)(npoly + 1), hipMemcpyHostToDevice, st)) !=
        hipSuccess)
        return bail(e);
    if ((e = hipMemsetAsync(flg, 0, sizeof(CellFlags), st)) != hipSuccess) return bail(e);
    hipLaunchKernelGGL(k_polygon_boxes, dim3((uint32_t)cdiv(npoly, 16)), dim3(256), 0, st, edges, in_first, npoly, merc,
                       diag, &flg->bad);
    if ((e = hipGetLastError()) != hipSuccess) return bail(e);
    int herr = 0;
    if ((e = hipMemcpyAsync(&herr, &flg->bad, sizeof(int), hipMemcpyDeviceToHost, st)) != hipSuccess) return bail(e);
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return bail(e);
    if (herr) {
        free_poly_arrays(poly);
        return {HV_EINVAL, "edges hold a non-finite coordinate, |lon| > 180 or |lat| > 90"};
    }
    const BuildResult r = build_index(diag, HV_SEGMENTS | HV_INPUT_MERC01, npoly, st, tree, false);
    if (r.status != HV_OK) {
        free_poly_arrays(poly);
        return r;
    }
    // offsets in the tree's order (host prefix sums over the sorted counts)
    std::vector<uint32_t> order((size_t)npoly);
    std::vector<int64_t> sorted_first((size_t)npoly + 1);
    if ((e = hipMemcpy(order.data(), tree->order, sizeof(uint32_t) * (size_t)npoly, hipMemcpyDeviceToHost)) !=
        hipSuccess)
        return bail(e);
    sorted_first[0] = 0;
    for (int64_t k = 0; k < npoly; ++k) {
        const uint32_t p = order[(size_t)k];
        sorted_first[(size_t)k + 1] = sorted_first[(size_t)k] + (first[p + 1] - first[p]);
    }
    const int top = cell_top(n);
    if ((e = device_acquire(&poly->block, index.bytes, &poly->block_bytes)) != hipSuccess) return bail(e);
    if (top >= 0) acquire_cells(tree, 2 * sizeof(uint32_t) * (size_t)cell_level_words(top + 1));
    unsigned char *const block = static_cast<unsigned char *>(poly->block);
    poly->edges = reinterpret_cast<double *>(block + o_edges);
    poly->first = reinterpret_cast<int64_t *>(block + o_first);
    poly->chunks = reinterpret_cast<float4 *>(block + o_chunks);
    poly->supers = reinterpret_cast<float4 *>(block + o_supers);
    if ((e = hipMemcpyAsync(poly->first, sorted_first.data(), sizeof(int64_t) * (size_t)(npoly + 1),
                            hipMemcpyHostToDevice, st)) != hipSuccess)
        return bail(e);
    hipLaunchKernelGGL(k_permute_polygons, dim3((uint32_t)cdiv(npoly, 4)), dim3(256), 0, st,
                       reinterpret_cast<const double4 *>(edges), in_first, tree->order, poly->first, npoly, merc,
                       reinterpret_cast<double4 *>(poly->edges));
    if (nchunk > 0) {
        hipLaunchKernelGGL(k_edge_chunks, dim3((uint32_t)cdiv(nchunk * kEdgeChunk, 256)), dim3(256), 0, st, poly->edges,
                           n, poly->chunks);
        hipLaunchKernelGGL(k_super_chunks, dim3((uint32_t)cdiv(nsuper, 256)), dim3(256), 0, st, poly->chunks,
                           nchunk, poly->supers);
    }
    if ((e = hipGetLastError()) != hipSuccess) return bail(e);
    CellFlags found = {};
    if (tree->cells) {
        if ((e = build_poly_cells(poly->edges, poly->first, tree->obj, npoly, top, tree->cells, flg, st)) != hipSuccess)
            return bail(e);
        if ((e = hipMemcpyAsync(&found, flg, sizeof found, hipMemcpyDeviceToHost, st)) != hipSuccess) return bail(e);
    }
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return bail(e);
    if (found.outside) {
        free_cells(tree);
    } else if (tree->cells) {
        tree->cell_top = top;
        tree->cell_gaps = found.gaps;
    }
    return r;
}

void free_cells(IndexArrays *a) {
    if (a->cells) device_release(a->cells, a->cell_bytes);
    a->cells = nullptr;
    a->cell_bytes = 0;
    a->cell_top = -1;
}

void free_index_arrays(IndexArrays *a) {
    free_cells(a);
    if (a->block) device_release(a->block, a->block_bytes);
    *a = IndexArrays{};
}

#define HV_TRY(expr)                          \
    do {                                      \
        hipError_t e_ = (expr);               \
        if (e_ != hipSuccess) {               \
            free_index_arrays(out);           \
            return hip_fail(e_);              \
        }                                     \
    } while (0)

BuildResult build_index(const double *objects, int kind_flags, int64_t n, hipStream_t st, IndexArrays *out,
                        bool with_cells) {
    const int kind = kind_flags & 0xff;
    const int merc = (kind_flags & HV_INPUT_MERC01) != 0;
    const int seg = kind != HV_POINTS;
    const int W = seg ? 4 : 2;
    *out = IndexArrays{};
    out->n = n;
    out->seg = seg;
    if (n == 0) return {HV_OK, ""};  // empty index: no device memory at all

    // node-level sizes
    int levels = 0;
    int64_t cnt = cdiv(n, kLeaf), total = 0;
    for (;;) {
        if (levels == kMaxLevels) return {HV_EINVAL, "too many tree levels"};
        out->level_off[levels] = total;
        out->level_cnt[levels] = cnt;
        total += cnt;
        ++levels;
        if (cnt == 1) break;
        cnt = cdiv(cnt, kFan);
    }
    out->levels = levels;
    out->nodes_total = total;
    const int bits = key_bits_for(n);
    out->key_bits = bits;
    const int passes = (2 * bits + 7) / 8;
    const int64_t nb = cdiv(n, kSTile);
    const int64_t ncount = 256 * nb;
    const int64_t npart = cdiv(ncount, kRTile);

    // All arrays of the index but the cells in one block.
    const size_t obj_bytes = sizeof(double) * W * (size_t)n, order_bytes = sizeof(uint32_t) * (size_t)n;
    const size_t node_bytes = sizeof(double4) * (size_t)total, rep_bytes = sizeof(double2) * (size_t)total;
    const size_t meta_bytes = sizeof(int64_t) * kMetaWords;
    const int top = with_cells ? cell_top(n) : -1;
    const size_t long_bytes = top >= 0 && seg ? cell_long_bytes(n) : 0;
    Carve index;
    const size_t o_obj = index.take(obj_bytes), o_order = index.take(order_bytes), o_nodes = index.take(node_bytes);
    const size_t o_rep = index.take(rep_bytes), o_meta = index.take(meta_bytes);
    const size_t o_flags = index.take(sizeof(CellFlags));
    // The sort works in the objects' own array, which is only written after
    // it; sets too small for that (the arrays are aligned) get scratch of their own,
    // as does the list of segments over many cells.
    Carve sort;
    const size_t o_low = sort.take((size_t)n), o_k0 = sort.take(order_bytes), o_k1 = sort.take(order_bytes);
    const size_t o_v1 = sort.take(order_bytes), o_counts = sort.take(sizeof(uint32_t) * (size_t)ncount);
    const size_t o_part = sort.take(sizeof(uint32_t) * (size_t)npart);
    Scratch scratch;
    HV_TRY(device_acquire(&out->block, index.bytes, &out->block_bytes));
    if (top >= 0) {
        if (scratch.alloc(long_bytes) == hipSuccess) acquire_cells(out, sizeof(uint32_t) * (size_t)cell_level_words(top + 1));
        else (void)hipGetLastError();
    }
    const bool cells = out->cells != nullptr;
    unsigned char *const block = static_cast<unsigned char *>(out->block);
    out->obj = reinterpret_cast<double *>(block + o_obj);
    out->order = reinterpret_cast<uint32_t *>(block + o_order);
    out->nodes = reinterpret_cast<double4 *>(block + o_nodes);
    out->rep = reinterpret_cast<double2 *>(block + o_rep);
    out->meta = reinterpret_cast<int64_t *>(block + o_meta);
    CellFlags *const flags = reinterpret_cast<CellFlags *>(block + o_flags);
    if (cells) out->cell_top = top;
    Scratch small;
    unsigned char *work = reinterpret_cast<unsigned char *>(out->obj);
    if (sort.bytes > obj_bytes) {
        HV_TRY(small.alloc(sort.bytes));
        work = small.p;
    }

    {
        int64_t meta[kMetaWords] = {};
        for (int l = 0; l < levels; ++l) {
            meta[l] = out->level_off[l];
            meta[kMaxLevels + l] = out->level_cnt[l];
        }
        HV_TRY(hipMemcpyAsync(out->meta, meta, sizeof(meta), hipMemcpyHostToDevice, st));
        HV_TRY(hipStreamSynchronize(st));
    }
    HV_TRY(hipMemsetAsync(flags, 0, sizeof(CellFlags), st));
    const dim3 g((uint32_t)cdiv(n, 256)), t(256);
    uint8_t *const low = work + o_low;
    uint32_t *kin = reinterpret_cast<uint32_t *>(work + o_k0), *kout = reinterpret_cast<uint32_t *>(work + o_k1);
    uint32_t *const v1 = reinterpret_cast<uint32_t *>(work + o_v1);
    uint32_t *const counts = reinterpret_cast<uint32_t *>(work + o_counts);
    uint32_t *const part = reinterpret_cast<uint32_t *>(work + o_part);
    if (seg) hipLaunchKernelGGL(k_project_key<4>, g, t, 0, st, objects, n, merc, low, kin, bits, &flags->bad);
    else hipLaunchKernelGGL(k_project_key<2>, g, t, 0, st, objects, n, merc, low, kin, bits, &flags->bad);
    HV_TRY(hipGetLastError());

    // the last pass writes the stored order
    uint32_t *vin = nullptr, *vout = passes % 2 ? out->order : v1;
    for (int p = 0; p < passes; ++p) {
        const int shift = 8 * (p - 1);
        const dim3 gs((uint32_t)nb), ts(kST);
        if (p == 0) hipLaunchKernelGGL(k_radix_hist<true>, gs, ts, 0, st, low, kin, n, 0, counts, nb);
        else hipLaunchKernelGGL(k_radix_hist<false>, gs, ts, 0, st, low, kin, n, shift, counts, nb);
        hipLaunchKernelGGL(k_scan_reduce, dim3((uint32_t)npart), dim3(kRT), 0, st, counts, ncount, part);
        hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(1024), 0, st, part, npart);
        hipLaunchKernelGGL(k_scan_down, dim3((uint32_t)npart), dim3(kRT), 0, st, counts, ncount, part);
        if (p == 0)
            hipLaunchKernelGGL(k_radix_scatter<true>, gs, ts, 0, st, low, kin, vin, kout, vout, n, 0, counts, nb);
        else hipLaunchKernelGGL(k_radix_scatter<false>, gs, ts, 0, st, low, kin, vin, kout, vout, n, shift, counts, nb);
        HV_TRY(hipGetLastError());
        std::swap(kin, kout);
        vin = vout;
        vout = vin == v1 ? out->order : v1;
    }

    if (seg)
        hipLaunchKernelGGL(k_gather_leaves<4>, g, t, 0, st, objects, out->order, n, merc, out->obj, out->nodes, out->rep);
    else
        hipLaunchKernelGGL(k_gather_leaves<2>, g, t, 0, st, objects, out->order, n, merc, out->obj, out->nodes, out->rep);
    for (int l = 1; l < levels; ++l) {
        const int64_t c = out->level_off[l - 1], nc = out->level_cnt[l - 1], at = out->level_off[l];
        double *const extent = seg && l == levels - 1 ? reinterpret_cast<double *>(out->meta + kMetaExtent) : nullptr;
        hipLaunchKernelGGL(k_level, dim3((uint32_t)cdiv(nc, 256)), t, 0, st, out->nodes + c, out->rep + c, nc,
                           out->nodes + at, out->rep + at, reinterpret_cast<const double4 *>(out->obj), n, extent);
    }
    HV_TRY(hipGetLastError());
    if (cells)
        HV_TRY(build_cells(out->obj, n, seg, top, out->cells, flags, reinterpret_cast<uint32_t *>(scratch.p), st));
    CellFlags found;
    HV_TRY(hipMemcpyAsync(&found, flags, sizeof found, hipMemcpyDeviceToHost, st));
    HV_TRY(hipStreamSynchronize(st));
    out->cell_gaps = found.gaps;
    if (found.outside) free_cells(out);
    if (found.bad) {
        free_index_arrays(out);
        return {HV_EINVAL, "objects hold a non-finite coordinate, |lon| > 180 or |lat| > 90"};
    }
    return {HV_OK, ""};
}

}  // namespace hv
