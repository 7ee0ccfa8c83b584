// Occupancy cells of an index: one bit per cell of a 2^(8 + l) x 2^(8 + l)
// grid over the world for every level l = 0 .. top, set iff some object
// touches the cell.  A cell of level l is a pixel of zoom l, so in a tile of
// zoom z the cells of level z + k are 2^k to a pixel side, and one look at the
// bits around a pixel decides most pixels of a tile dense in objects: an
// occupied cell wholly inside the radius lights the pixel, and with no
// occupied cell in reach none does.  Only pixels between the two need the
// tree.
//
// Guarantee (kept with room to spare by the query's margin of 1e-3 cells): an
// occupied cell lies within 1e-6 cells of a point of some object, and every
// point of every object lies within 1e-6 cells of an occupied cell.
#include <algorithm>

#include "hv_internal.h"

namespace hv {
namespace {

constexpr int kLongCells = 56;          // segments over more cells go to the long list
constexpr int64_t kLongCap = 1 << 20;   // its most entries
constexpr int kBlock = 128;             // a workgroup marks blocks of kBlock x kBlock cells in LDS
constexpr int kHalo = 40;               // rows around a block (and one word on either side) that its segments reach
constexpr int kMarkChunk = 4096;        // objects of a workgroup

struct Line {  // a segment in cells, the upper end first
    double x0, y0, x1, y1, slope;  // slope: dx / dy, used only where r0 < r1
    int r0, r1;
};

__device__ inline int cell_of(double u, int g) { return min((int)u, g - 1); }  // 0 <= u <= g

// Clamps a coordinate to [0, 1]; false if it lies outside by more than the
// projection's rounding at the poles and the antimeridian (1.4e-7 cells of the
// finest level), or is not a number.
__device__ inline bool in_world(double &v) {
    const bool in = v >= -1e-12 && v <= 1.0 + 1e-12;
    v = fmin(fmax(v, 0.0), 1.0);
    return in;
}

__device__ inline Line line_of(double4 s, double G, int g) {
    (void)in_world(s.x), (void)in_world(s.y), (void)in_world(s.z), (void)in_world(s.w);
    Line l;
    const bool down = s.y <= s.w;
    l.x0 = (down ? s.x : s.z) * G;
    l.y0 = (down ? s.y : s.w) * G;
    l.x1 = (down ? s.z : s.x) * G;
    l.y1 = (down ? s.w : s.y) * G;
    l.r0 = cell_of(l.y0, g);
    l.r1 = cell_of(l.y1, g);
    l.slope = (l.x1 - l.x0) / (l.y1 - l.y0);
    return l;
}

__device__ inline void mark(uint32_t *w, uint32_t m) {
    // bits are only ever set: one that is seen set needs no atomic
    if ((*reinterpret_cast<volatile uint32_t *>(w) & m) != m) atomicOr(w, m);
}

// The cells of row r that the line touches; word (xw, y) is base[xw * stride + y].
__device__ inline void mark_row(const Line &l, int r, int g, int64_t stride, uint32_t *base) {
    double a = r == l.r0 ? l.x0 : l.x0 + ((double)r - l.y0) * l.slope;
    double b = r == l.r1 ? l.x1 : l.x0 + ((double)(r + 1) - l.y0) * l.slope;
    const double lo = fmin(l.x0, l.x1), hi = fmax(l.x0, l.x1);
    a = fmin(fmax(a, lo), hi);
    b = fmin(fmax(b, lo), hi);
    const int c0 = cell_of(fmin(a, b), g), c1 = cell_of(fmax(a, b), g);
    for (int w = c0 >> 5; w <= (c1 >> 5); ++w) {
        const int f = max(c0 - 32 * w, 0), t = min(c1 - 32 * w, 31);
        mark(base + w * stride + r, (0xffffffffu >> (31 - t)) & (0xffffffffu << f));
    }
}

// A wave's lines, and pairs (lane | row - r0 << 6) of the rows they touch.
constexpr int kUnits = 256;
struct WaveLines {
    double x0[64], y0[64], x1[64], y1[64], slope[64];
    int r0[64], r1[64];
    uint16_t units[kUnits];
};

// Marks the rows of the wave's lines (rows = 0: none), dealt over its lanes: a
// lane per line waits for the longest of 64 (10M segments 0.38 ms).
__device__ inline void mark_rows(const Line &l, int rows, int g, int64_t stride, uint32_t *base, WaveLines &w, int lane) {
    w.x0[lane] = l.x0, w.y0[lane] = l.y0, w.x1[lane] = l.x1, w.y1[lane] = l.y1, w.slope[lane] = l.slope;
    w.r0[lane] = l.r0, w.r1[lane] = l.r1;
    int first = 0, total = 0;
#pragma unroll
    for (int b = 0; (1 << b) <= kLongCells; ++b) {
        const uint64_t m = __ballot((rows >> b) & 1);
        first += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)) << b;
        total += __popcll(m) << b;
    }
    for (int u0 = 0; u0 < total; u0 += kUnits) {
        __builtin_amdgcn_wave_barrier();
        for (int k = max(u0 - first, 0); k < rows && first + k - u0 < kUnits; ++k)
            w.units[first + k - u0] = (uint16_t)(lane | k << 6);
        __builtin_amdgcn_wave_barrier();
        for (int u = lane; u < min(total - u0, kUnits); u += 64) {
            const int e = w.units[u], c = e & 63;
            const Line q{w.x0[c], w.y0[c], w.x1[c], w.y1[c], w.slope[c], w.r0[c], w.r1[c]};
            mark_row(q, q.r0 + (e >> 6), g, stride, base);
        }
    }
    __builtin_amdgcn_wave_barrier();
}

// A workgroup takes kMarkChunk objects in the tree's (Hilbert) order, in which
// the objects of one block of cells, a block's side being a power of two,
// follow each other: it marks them in LDS block by block and writes out the
// words with a bit.  Marking each object in memory took 675 ms for 1e9 points,
// its atomics running at 1.6 per ns.
template <int W>
__global__ __launch_bounds__(256) void k_cells_mark(const double *__restrict__ obj, int64_t n, int level,
                                                    uint32_t *cells, CellFlags *flags, uint32_t *longs) {
    constexpr int H = W == 2 ? 0 : kHalo, HW = W == 2 ? 0 : 1;
    constexpr int kRows = kBlock + 2 * H, kCols = kBlock / 32 + 2 * HW;
    __shared__ uint32_t lds[kRows * kCols];
    __shared__ WaveLines wave[W == 2 ? 1 : 4];
    __shared__ unsigned long long found[3];  // long segments, their cells, their first slot in the list
    const int tid = threadIdx.x, lane = tid & 63;
    const int g = 256 << level;
    const int64_t stride = cell_stride(level);
    uint32_t *const base = cells + cell_level_words(level) + cell_origin(level);
    for (int k = tid; k < kRows * kCols; k += 256) lds[k] = 0;
    const int64_t end = min(n, ((int64_t)blockIdx.x + 1) * kMarkChunk);
    for (int64_t p = (int64_t)blockIdx.x * kMarkChunk; p < end;) {
        // the block of the first object left, and the objects of it that follow
        double v[W];
        auto block_of = [&](int64_t i) -> uint32_t {
#pragma unroll
            for (int c = 0; c < W; ++c) v[c] = obj[i * W + c];
            double cx = v[0], cy = v[1];
            if constexpr (W == 4) {
                cx = 0.5 * (fmin(v[0], v[2]) + fmax(v[0], v[2]));
                cy = 0.5 * (fmin(v[1], v[3]) + fmax(v[1], v[3]));
            }
            (void)in_world(cx), (void)in_world(cy);
            return (uint32_t)(cell_of(cx * g, g) / kBlock) << 16 | (uint32_t)(cell_of(cy * g, g) / kBlock);
        };
        const uint32_t blk = block_of(p);
        const int bx = (int)(blk >> 16) * kBlock, by = (int)(blk & 0xffffu) * kBlock;
        uint32_t *const at = lds - (int64_t)(bx / 32 - HW) * kRows - (by - H);  // word (xw, y) of the level at xw * kRows + y
        for (;;) {
            if (tid < 3) found[tid] = 0;
            __syncthreads();
            const int64_t i = p + tid;
            const bool mine = i < end && block_of(i) == blk;
            unsigned long long slot = ~0ull;
            Line line;
            int rows = 0;
            if (mine) {
                bool in = true;
#pragma unroll
                for (int c = 0; c < W; ++c) in = in_world(v[c]) && in;
                if (!in) {
                    flags->outside = 1;
                } else if constexpr (W == 2) {
                    const int cx = cell_of(v[0] * g, g), cy = cell_of(v[1] * g, g);
                    mark(at + (cx >> 5) * kRows + cy, 1u << (cx & 31));
                } else {
                    const Line l = line_of(make_double4(v[0], v[1], v[2], v[3]), (double)g, g);
                    const int count = l.r1 - l.r0 + abs(cell_of(l.x1, g) - cell_of(l.x0, g)) + 1;
                    if (count > kLongCells) {
                        slot = atomicAdd(&found[0], 1ull);
                        atomicAdd(&found[1], (unsigned long long)count);
                    } else {
                        line = l;
                        rows = l.r1 - l.r0 + 1;
                    }
                }
            }
            if constexpr (W == 4) mark_rows(line, rows, g, kRows, at, wave[tid >> 6], lane);
            const int took = __syncthreads_count(mine);
            if (W == 4 && found[0]) {
                if (tid == 0) {
                    found[2] = atomicAdd(&flags->n_long, found[0]);
                    atomicAdd(&flags->long_cells, found[1]);
                }
                __syncthreads();
                if (slot != ~0ull && found[2] + slot < (unsigned long long)kLongCap)
                    longs[found[2] + slot] = (uint32_t)i;
            }
            __syncthreads();
            p += took;
            if (took < 256) break;
        }
        for (int k = tid; k < kRows * kCols; k += 256) {
            const uint32_t m = lds[k];
            if (m) {
                atomicOr(base + (int64_t)(bx / 32 - HW + k / kRows) * stride + (by - H + k % kRows), m);
                lds[k] = 0;
            }
        }
        __syncthreads();
    }
}

__device__ inline bool long_ok(const CellFlags &f, int64_t n) {
    return f.n_long <= (unsigned long long)kLongCap && f.long_cells <= 4ull * (unsigned long long)n + (1ull << 22);
}

// The long segments, a wavefront to each, a row to a lane.  Where they are too
// many or too long for that to be cheap, none is marked, and a cell without a
// bit then says nothing (CellFlags::gaps).
__global__ __launch_bounds__(256) void k_cells_long(const double *__restrict__ obj, int64_t n, int level,
                                                    uint32_t *cells, CellFlags *flags,
                                                    const uint32_t *__restrict__ longs) {
    const CellFlags f = *flags;
    if (!long_ok(f, n)) {
        if (threadIdx.x == 0) flags->gaps = 1;
        return;
    }
    const int g = 256 << level;
    uint32_t *base = cells + cell_level_words(level) + cell_origin(level);
    const int64_t stride = cell_stride(level);
    const int64_t waves = (int64_t)gridDim.x * 4;
    for (int64_t k = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); k < (int64_t)f.n_long; k += waves) {
        const Line l = line_of(reinterpret_cast<const double4 *>(obj)[longs[k]], (double)g, g);
        for (int r = l.r0 + (int)(threadIdx.x & 63); r <= l.r1; r += 64) mark_row(l, r, g, stride, base);
    }
}

// Every second bit of v, packed into the lower half.
__device__ inline uint32_t even_bits(uint32_t v) {
    v &= 0x55555555u;
    v = (v | (v >> 1)) & 0x33333333u;
    v = (v | (v >> 2)) & 0x0f0f0f0fu;
    v = (v | (v >> 4)) & 0x00ff00ffu;
    return (v | (v >> 8)) & 0x0000ffffu;
}

// Level `level` from level + 1: a cell is occupied iff one of its four is.
// One thread per word (32 cells of a row).
__global__ __launch_bounds__(256) void k_cells_up(uint32_t *cells, int level) {
    const int g = 256 << level;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)(g >> 5) * g) return;
    const int xw = (int)(i >> (8 + level)), y = (int)(i & (g - 1));
    const uint32_t *fine = cells + cell_level_words(level + 1) + cell_origin(level + 1) +
                           2 * xw * cell_stride(level + 1) + 2 * y;
    const uint2 a = *reinterpret_cast<const uint2 *>(fine);
    const uint2 b = *reinterpret_cast<const uint2 *>(fine + cell_stride(level + 1));
    uint32_t lo = a.x | a.y, hi = b.x | b.y;
    lo |= lo >> 1;
    hi |= hi >> 1;
    cells[cell_level_words(level) + cell_origin(level) + xw * cell_stride(level) + y] =
        even_bits(lo) | (even_bits(hi) << 16);
}

// ------------------------------------------------------------ polygons
// Two bits per cell: `in`, the closed cell lies inside some polygon, and `near`,
// the cell may hold a point of one.  A polygon is drawn at the finest level at
// which its box spans at most kPolyCells cells, by one wavefront in LDS: the
// cells its edges come within kPolyEps of, and each row's parity of crossings
// left of the cells' centres.  A cell that no edge comes near has its centre's
// parity throughout.
constexpr double kPolyCells = 61.0;
constexpr double kPolyEps = 1e-6;  // cells

__device__ inline uint64_t columns64(int c0, int c1) { return (~0ull >> (63 - (c1 - c0))) << c0; }

__device__ inline void or64(uint32_t *w, uint64_t m) {
    if ((uint32_t)m) atomicOr(&w[0], (uint32_t)m);
    if ((uint32_t)(m >> 32)) atomicOr(&w[1], (uint32_t)(m >> 32));
}

__global__ __launch_bounds__(256) void k_poly_cells(const double4 *__restrict__ edges, const int64_t *__restrict__ first,
                                                    const double4 *__restrict__ boxes, int64_t npoly, int top,
                                                    uint32_t *in, uint32_t *near, CellFlags *flags) {
    __shared__ uint32_t lds[4][2][128];  // touched cells, parity: 64 rows of 64 cells
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t k = (int64_t)blockIdx.x * 4 + wv;
    if (k >= npoly) return;
    uint32_t *const touched = lds[wv][0], *const odd = lds[wv][1];
    double4 b = boxes[k];
    if (!((int)in_world(b.x) & (int)in_world(b.y) & (int)in_world(b.z) & (int)in_world(b.w))) {
        if (lane == 0) flags->outside = 1;
        return;
    }
    const double ext = fmax(b.z - b.x, b.w - b.y);
    int level = top;
    while (level > 0 && ldexp(ext, 8 + level) > kPolyCells) --level;
    const int g = 256 << level;
    const double G = (double)g;
    if (ext * G > kPolyCells) {
        if (lane == 0) flags->gaps = 1;
        return;
    }
    const int bx = cell_of(b.x * G, g) - 1, by = cell_of(b.y * G, g) - 1;
    for (int q = lane; q < 128; q += 64) touched[q] = odd[q] = 0;
    __builtin_amdgcn_wave_barrier();
    for (int64_t e = first[k] + lane; e < first[k + 1]; e += 64) {
        const double4 s = edges[e];
        const double x0 = s.x * G - bx, y0 = s.y * G - by, x1 = s.z * G - bx, y1 = s.w * G - by;
        const double ylo = fmin(y0, y1), yhi = fmax(y0, y1), xlo = fmin(x0, x1), xhi = fmax(x0, x1);
        const int r0 = max((int)floor(ylo - kPolyEps), 0), r1 = min((int)floor(yhi + kPolyEps), 63);
        const double slope = (x1 - x0) / (y1 - y0);  // not used where the ends share a row
        for (int r = r0; r <= r1; ++r) {
            double a = x0, c = x1;
            if (r0 != r1) {
                // x where the edge enters and leaves the row, within the edge
                a = x0 + (fmin(fmax((double)r - kPolyEps, ylo), yhi) - y0) * slope;
                c = x0 + (fmin(fmax((double)r + 1.0 + kPolyEps, ylo), yhi) - y0) * slope;
                if (!(yhi > ylo)) a = x0, c = x1;
                a = fmin(fmax(a, xlo), xhi);
                c = fmin(fmax(c, xlo), xhi);
            }
            const int c0 = max((int)floor(fmin(a, c) - kPolyEps), 0), c1 = min((int)floor(fmax(a, c) + kPolyEps), 63);
            if (c0 <= c1) or64(&touched[2 * r], columns64(c0, c1));
            const double yc = (double)r + 0.5;
            if ((y0 > yc) != (y1 > yc)) {
                const int from = (int)fmin(fmax(floor(x0 + (yc - y0) * slope - 0.5) + 1.0, 0.0), 64.0);
                if (from < 64) {
                    const uint64_t m = ~0ull << from;
                    if ((uint32_t)m) atomicXor(&odd[2 * r], (uint32_t)m);
                    atomicXor(&odd[2 * r + 1], (uint32_t)(m >> 32));
                }
            }
        }
    }
    __builtin_amdgcn_wave_barrier();
    // lane r writes row r; cells beyond the world's edge stay unmarked
    const int y = by + lane;
    if (y < 0 || y >= g) return;
    uint64_t world = bx < 0 ? ~1ull : ~0ull;
    if (g - bx < 64) world &= ~0ull >> (64 - (g - bx));
    const uint64_t t = ((uint64_t)touched[2 * lane + 1] << 32 | touched[2 * lane]) & world;
    const uint64_t i = ((uint64_t)odd[2 * lane + 1] << 32 | odd[2 * lane]) & world & ~t;
    const int64_t stride = cell_stride(level);
    const int xw = bx >> 5, sh = bx & 31;
    const int64_t at = cell_level_words(level) + cell_origin(level) + xw * stride + y;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        auto part = [&](uint64_t v) -> uint32_t {
            return q == 0 ? (uint32_t)(v << sh) : q == 1 ? (uint32_t)(v >> (32 - sh)) : sh ? (uint32_t)(v >> (64 - sh)) : 0u;
        };
        const uint32_t mi = part(i), mn = part(t | i);
        if (mn) mark(near + at + q * stride, mn);
        if (mi) mark(in + at + q * stride, mi);
    }
}

// Bit b of the low half of v doubled into bits 2b and 2b + 1.
__device__ inline uint32_t twice_bits(uint32_t v) {
    v &= 0xffffu;
    v = (v | (v << 8)) & 0x00ff00ffu;
    v = (v | (v << 4)) & 0x0f0f0f0fu;
    v = (v | (v << 2)) & 0x33333333u;
    v = (v | (v << 1)) & 0x55555555u;
    return v | (v << 1);
}

// What polygons drawn at coarser levels cover of level `level` (>= 1).
__global__ __launch_bounds__(256) void k_poly_down(uint32_t *in, uint32_t *near, int level) {
    const int g = 256 << level;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)(g >> 5) * g) return;
    const int xw = (int)(i >> (8 + level)), y = (int)(i & (g - 1));
    const int64_t from = cell_level_words(level - 1) + cell_origin(level - 1) + (xw >> 1) * cell_stride(level - 1) + (y >> 1);
    const int64_t to = cell_level_words(level) + cell_origin(level) + xw * cell_stride(level) + y;
    const int half = 16 * (xw & 1);
    const uint32_t a = twice_bits(in[from] >> half), b = twice_bits(near[from] >> half);
    if (a) in[to] |= a;
    if (b) near[to] |= b;
}

// Level `level` from the one below it: inside where all four cells are, near
// where one is.
__global__ __launch_bounds__(256) void k_poly_up(uint32_t *in, uint32_t *near, int level) {
    const int g = 256 << level;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)(g >> 5) * g) return;
    const int xw = (int)(i >> (8 + level)), y = (int)(i & (g - 1));
    const int64_t stride = cell_stride(level + 1);
    const int64_t from = cell_level_words(level + 1) + cell_origin(level + 1) + 2 * xw * stride + 2 * y;
    const int64_t to = cell_level_words(level) + cell_origin(level) + xw * cell_stride(level) + y;
    uint2 a = *reinterpret_cast<const uint2 *>(in + from), b = *reinterpret_cast<const uint2 *>(in + from + stride);
    const uint32_t al = a.x & a.y, bl = b.x & b.y;
    const uint32_t inside = even_bits(al & (al >> 1)) | even_bits(bl & (bl >> 1)) << 16;
    a = *reinterpret_cast<const uint2 *>(near + from), b = *reinterpret_cast<const uint2 *>(near + from + stride);
    const uint32_t an = a.x | a.y, bn = b.x | b.y;
    const uint32_t close = even_bits(an | (an >> 1)) | even_bits(bn | (bn >> 1)) << 16;
    if (inside) in[to] |= inside;
    if (close) near[to] |= close;
}

}  // namespace

int cell_top(int64_t n) {
    int top = -1;
    while (top < kCellTopMax && ldexp(1.0, 2 * (8 + top + 1)) <= kCellBitsPerObject * (double)n) ++top;
    return top;
}

size_t cell_long_bytes(int64_t n) { return sizeof(uint32_t) * (size_t)std::min(n, kLongCap); }

hipError_t build_poly_cells(const double *edges, const int64_t *first, const double *boxes, int64_t npoly, int top,
                            uint32_t *cells, CellFlags *flags, hipStream_t st) {
    const int64_t words = cell_level_words(top + 1);
    uint32_t *const in = cells, *const near = cells + words;
    hipError_t e = hipMemsetAsync(cells, 0, 2 * sizeof(uint32_t) * (size_t)words, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_poly_cells, dim3((uint32_t)((npoly + 3) / 4)), dim3(256), 0, st,
                       reinterpret_cast<const double4 *>(edges), first, reinterpret_cast<const double4 *>(boxes), npoly,
                       top, in, near, flags);
    for (int l = 1; l <= top; ++l)
        hipLaunchKernelGGL(k_poly_down, dim3((uint32_t)(256ll << (2 * l)) / 32), dim3(256), 0, st, in, near, l);
    for (int l = top - 1; l >= 0; --l)
        hipLaunchKernelGGL(k_poly_up, dim3((uint32_t)(256ll << (2 * l)) / 32), dim3(256), 0, st, in, near, l);
    return hipGetLastError();
}

hipError_t build_cells(const double *obj, int64_t n, int seg, int top, uint32_t *cells, CellFlags *flags,
                       uint32_t *longs, hipStream_t st) {
    hipError_t e = hipMemsetAsync(cells, 0, sizeof(uint32_t) * cell_level_words(top + 1), st);
    if (e != hipSuccess) return e;
    const dim3 grid((uint32_t)((n + kMarkChunk - 1) / kMarkChunk));
    if (seg) {
        hipLaunchKernelGGL(k_cells_mark<4>, grid, dim3(256), 0, st, obj, n, top, cells, flags, longs);
        hipLaunchKernelGGL(k_cells_long, dim3(1024), dim3(256), 0, st, obj, n, top, cells, flags, longs);
    } else {
        hipLaunchKernelGGL(k_cells_mark<2>, grid, dim3(256), 0, st, obj, n, top, cells, flags, longs);
    }
    for (int l = top - 1; l >= 0; --l)
        hipLaunchKernelGGL(k_cells_up, dim3((uint32_t)(256ll << (2 * l)) / 32), dim3(256), 0, st, cells, l);
    return hipGetLastError();
}

}  // namespace hv
