// Internal interfaces between the C ABI (hv_api.hip), the index build
// (hv_build.hip) and the query kernels (hv_query.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/hv.h"

namespace hv {

constexpr int kLeaf = 16;        // objects per leaf
constexpr int kFan = 16;         // children per inner node
constexpr int kEdgeChunk = 8;    // polygon edges per chunk box (filling)
constexpr int kChunkSuper = 8;   // chunk boxes per super-chunk box (filling)
constexpr int kFrontier = 256;   // most nodes in a tile's frontier
constexpr int kMaxLevels = 16;   // node levels (2e9 objects need 8)
constexpr int kMetaExtent = 2 * kMaxLevels, kMetaWords = kMetaExtent + 1;
constexpr int kLevelShift = 27;  // stack entry: level << 27 | node index
constexpr uint32_t kIdxMask = (1u << kLevelShift) - 1;
constexpr double kCullPad = 1e-5;  // px beyond r for every cull box

// Device view of an index, passed to kernels by value.
struct DevIndex {
    const double *obj;           // Hilbert order; 2 (points) or 4 (segments) doubles each
    const double4 *nodes;        // all levels, level 0 (leaves) first; (minX, minY, maxX, maxY)
    const double2 *rep;          // per node, same order: the first vertex of its first object
    const int64_t *meta;         // [0, kMaxLevels): level offsets; [kMaxLevels, 2*kMaxLevels): counts; [kMetaExtent]:
                                 // the bits of a double, the median over the objects of the larger side of their boxes
    int64_t n;
    int32_t levels;
    int32_t seg;                 // 0 points, 1 segments / edges
    const uint32_t *cells;       // occupancy cells, levels 0 .. cell_top (cell_top < 0: none)
    int32_t cell_top;
    int32_t cell_gaps;           // 1: a cell without a bit may still hold an object
    // polygon indexes only (filling): the tree above holds the polygons'
    // bounding boxes as diagonals, in sorted order
    const double *pedges;        // edges, 4 doubles each, polygon after polygon in sorted order
    const int64_t *pfirst;       // the polygon at sorted position k owns edges [pfirst[k], pfirst[k + 1])
    const float4 *pchunk;        // chunk c: a box holding edges [kEdgeChunk c, kEdgeChunk (c + 1))
    const float4 *psuper;        // super-chunk s: a box holding chunks [kChunkSuper s, kChunkSuper (s + 1))
};

// Occupancy cells (hv_cells.hip).  Level l is a grid of 2^(8 + l) x 2^(8 + l)
// cells over the world, stored by word columns: bit b of word (xw, y) is cell
// (32 xw + b, y), and a column's rows lie next to each other, so that a run of
// rows is one wide load.  kCellPad rows above and below and one column on
// either side are always zero, so that a look over the world's edge needs no
// test.
constexpr int kCellPad = 64;
constexpr int kCellTopMax = 9;             // 2^34 cells, 2 GiB
constexpr double kCellBitsPerObject = 32;  // the finest level has at most this many cells per object

__host__ __device__ constexpr int64_t cell_stride(int level) { return (int64_t(256) << level) + 2 * kCellPad; }
// Words of the levels below `level`: the offset of its first word.
__host__ __device__ constexpr int64_t cell_level_words(int level) {
    // a level has (8 * 2^l + 2) (256 * 2^l + 2 kCellPad) words
    return 2048 * (((int64_t(1) << (2 * level)) - 1) / 3) + (512 + 16 * kCellPad) * ((int64_t(1) << level) - 1) +
           4 * kCellPad * level;
}
// Word (0, 0) of a level, from the level's first word.
__host__ __device__ constexpr int64_t cell_origin(int level) { return cell_stride(level) + kCellPad; }

// What marking the cells found, in device memory.
struct CellFlags {
    int32_t bad;                    // a coordinate is not finite or out of range
    int32_t outside;                // an object lies outside [0, 1]^2: the cells are not used
    int32_t gaps;                   // long segments were left out
    int32_t pad;
    unsigned long long n_long, long_cells;
};

// The finest level for n objects, or -1 if they are too few.
int cell_top(int64_t n);
size_t cell_long_bytes(int64_t n);
// Marks the cells of n sorted objects and fills all levels.  flags starts at
// zero; longs: scratch of cell_long_bytes(n) (segments only).
hipError_t build_cells(const double *obj, int64_t n, int seg, int top, uint32_t *cells, CellFlags *flags,
                       uint32_t *longs, hipStream_t st);
// The same for npoly polygons (edges and boxes in sorted order): cells inside
// some polygon, then, cell_level_words(top + 1) words on, cells that may hold a
// point of one.
hipError_t build_poly_cells(const double *edges, const int64_t *first, const double *boxes, int64_t npoly, int top,
                            uint32_t *cells, CellFlags *flags, hipStream_t st);

// A request as the kernels see it: one tile of one index with its own
// radius / half-width.  `index` selects an entry of the batch's index table.
struct DevReq {
    int32_t z, x, y, index;
    double r;
};

struct BuildResult {
    int status;                  // HV_OK / HV_EINVAL / HV_ENOMEM / HV_EHIP
    const char *msg;
};

// Device memory for indexes and their builds.  Blocks given back are kept, up to
// kPoolBytes in all and half of that each (an index and its scratch), for the next
// request that they fit: loading 10M segments and drawing once took 43 ms with a
// hipMalloc and hipFree for every array and takes 1.1.  (One block more or less costs
// 0.1 and 0.35 ms: 13M segments 1.39 ms, 14M, whose index is not kept, 1.89, 40M
// 4.4.)  Beyond the bound the oldest are freed, and all of
// them before an allocation of the library fails (device_trim, which returns
// whether there were any).  device_release waits for the device, as hipFree does.
// Safe from several threads; a block stays on its device.
constexpr size_t kPoolBytes = size_t(1) << 30;
hipError_t device_acquire(void **p, size_t bytes, size_t *held);
void device_release(void *p, size_t held);
bool device_trim();

// Device arrays owned by one index (freed by free_index_arrays).
struct IndexArrays {
    void *block = nullptr;       // holds them all but the cells
    size_t block_bytes = 0;      // (up to twice what they take, where a kept block was reused)
    double *obj = nullptr;
    double4 *nodes = nullptr;
    double2 *rep = nullptr;      // per node: the first vertex of its first object
    uint32_t *order = nullptr;
    int64_t *meta = nullptr;     // device copy of level_off / level_cnt, and the objects' extent
    uint32_t *cells = nullptr;   // occupancy cells (a block), or NULL
    size_t cell_bytes = 0;
    int32_t cell_top = -1;
    int32_t cell_gaps = 0;
    int64_t n = 0;
    int32_t seg = 0;
    int32_t levels = 0;
    int32_t key_bits = 0;
    int64_t level_off[kMaxLevels] = {};
    int64_t level_cnt[kMaxLevels] = {};
    int64_t nodes_total = 0;
};

// Device arrays of a polygon index beyond its box tree (freed by
// free_poly_arrays).
struct PolyArrays {
    void *block = nullptr;       // holds them all
    size_t block_bytes = 0;
    double *edges = nullptr;     // projected, polygon after polygon in the tree's sorted order
    int64_t *first = nullptr;    // npoly + 1 offsets into edges, by sorted position
    float4 *chunks = nullptr;    // ceil(n_edges / kEdgeChunk) conservative float boxes
    float4 *supers = nullptr;    // ceil(chunks / kChunkSuper) unions of chunk boxes
    int64_t npoly = 0, n_edges = 0;
};

// Builds a polygon index: projects `edges` (device, n x 4 lon0, lat0, lon1,
// lat1, or normalised with HV_INPUT_MERC01 in flags; polygon p owns edges
// [first[p], first[p + 1]), `first` on the host), computes each polygon's
// bounding box, builds the Hilbert R-tree over those boxes (as diagonal
// segments), then stores the edges polygon after polygon in the tree's
// order, with a conservative box per kEdgeChunk edges.
BuildResult build_polygons(const double *edges, int64_t n, const int64_t *first, int64_t npoly, int flags,
                           hipStream_t stream, IndexArrays *tree, PolyArrays *poly);
void free_poly_arrays(PolyArrays *p);

// Builds the index on `stream` and synchronises.  `objects` is a device
// pointer; validation of coordinates happens on the device.  with_cells:
// mark the occupancy cells too (for distance masks).
BuildResult build_index(const double *objects, int kind_flags, int64_t n, hipStream_t stream,
                        IndexArrays *out, bool with_cells);
void free_index_arrays(IndexArrays *a);
void free_cells(IndexArrays *a);

struct LaunchShape {
    int block;        // 8 or 16
    int cand_cap;     // staged candidates per wave
    int waves;        // waves per workgroup
    int grid;         // workgroups of the persistent query kernel (0: fill the GPU)
    int region;       // 0: one wave per block; 32 or 64: one workgroup per region of that side
    int opl;          // region mode: objects loaded per lane at a leaf step (1, 2 or 4)
    int fill = 0;     // 1: polygon filling (region mode) instead of the distance masks
    int aa = 0;       // 1: anti-aliased values 0-4 (region mode, HV_AA_BYTES per request)
    int cull = kFrontier;  // frontier cap of the per-tile pass (cull depth)
};

// LDS bytes per workgroup for a shape and the deepest index of a batch.
size_t query_lds_bytes(const LaunchShape &s, int max_levels);

// Header of a batch, in device memory and staged from the host each launch,
// so that a captured graph's kernel arguments never change.
struct BatchHeader {
    int64_t n_req;      // live requests
    uint8_t *out;       // request k at out + k * 8192 (anti-aliased values: k * 65536)
    int32_t counter;    // tiles appended to the compacted list (0 when staged)
    int32_t ecounter;   // tiles with no data within r, listed for zero-filling (0 when staged)
    uint64_t t_start;   // wall clock when the batch started on the device
    int32_t leaf_tiles; // tiles for the object kernel: frontier at the leaves (0 when staged)
    int32_t node_tiles; // and above (0 when staged)
};

// Device addresses of one batch's workspace (a kernel argument).
struct DevBatch {
    BatchHeader *hdr;
    const DevIndex *ixs;
    const DevReq *reqs;
    const uint32_t *order;  // the requests by zoom, lowest first: the tile-frontier kernel's order
    uint32_t *frontier;  // per request: up to 256 frontier nodes
    int32_t *fmeta;      // per request: frontier size, frontier level, 64 bits of regions it reaches
    uint32_t *list;      // from the front: requests for the region kernel; from the back: leaf_tiles
    uint32_t *elist;     // from the front: requests whose tile has no data within r; from the back: node_tiles
    uint32_t *done;      // per request: parts finished
    uint64_t *ts;        // per request: wall clock at completion
};

// Device workspace of one batch of up to n_req requests over n_ix indexes.
// Its first staged_bytes() bytes (header, index table, requests) are copied
// from the host; the rest is written by the kernels.
struct Workspace {
    int64_t n_req;
    size_t hdr_off, table_off, req_off, order_off, frontier_off, fmeta_off, list_off, elist_off, done_off, ts_off,
        total;
    size_t staged_bytes() const { return frontier_off; }
};
Workspace workspace_layout(int64_t n_req, int n_ix);

// Fills the host part of a workspace: header, index table, requests, and
// their order by zoom (lowest first, stable), in which the tile-frontier
// kernel lists them for the query kernel, so that dense low-zoom tiles start
// first and the short high-zoom ones fill the end of the launch.
void stage_host(const Workspace &w, const DevIndex *ixs, int n_ix, const DevReq *reqs, int64_t n_req, uint8_t *out,
                unsigned char *host);

DevBatch device_batch(const Workspace &w, unsigned char *dws);

// Launches the tile-frontier and query kernels for a staged workspace `dws`
// (device) on `stream`; the grids cover w.n_req requests.  With `marks`
// (three events, or NULL) it records marks[0] before the frontier kernel,
// marks[1] between the two and marks[2] after the query kernel.
hipError_t launch_query(const Workspace &w, unsigned char *dws, int max_levels, const LaunchShape &s,
                        hipStream_t stream, hipEvent_t *marks = nullptr, bool strips = true);
// Whether launch_query's strips are worth their launch to a batch (true where the
// requests are not known yet).
bool strips_pay(const DevIndex *ixs, const DevReq *reqs, int64_t n_req);

// Batches that travel in the kernels' arguments: this many requests over this
// many indexes, in the default shape or filling (and no number of workgroups is
// asked for: their launches have one per piece of a tile).
constexpr int kFewRequests = 64, kFewIndexes = 4;
constexpr int kSelfRequests = 32;      // up to this many walk for their frontier in every workgroup
bool few_requests(const LaunchShape &s, int64_t n_req, int n_ix);
// Device bytes that launch_few needs at dws (0: none), and the launch itself
// (marks as for launch_query).
size_t few_bytes(const LaunchShape &s, int64_t n_req);
hipError_t launch_few(const DevIndex *ixs, int n_ix, const DevReq *reqs, int64_t n_req, uint8_t *out, unsigned char *dws,
                      int max_levels, const LaunchShape &s, hipStream_t st, hipEvent_t *marks);

// The object kernel (hv_objects.h): tiles with few objects in reach, in strips
// of whole pixel rows, a workgroup to a strip.  More
// strips spread a tile's objects over more workgroups, and each reads the
// frontier anew.
constexpr int kLeafStrips = 4;         // up to 4,096 objects in reach
constexpr int kNodeStrips = 16;        // up to 65,536, or 262,144
constexpr int kObjectUpper = 64;       // most level-2 nodes of a tile taken object by object
constexpr int kStripRows = 64;         // most rows of a strip
constexpr int64_t kObjectsGrid = 4096;

// Workgroups that fill the current device for a shape (occupancy x CUs).
int persistent_grid(const LaunchShape &s, int max_levels);

// Anti-aliased values of n requests (HV_AA_BYTES each at out) from child
// masks or one-pass values: map[k] >= 0 takes the 2 x 2 bit counts of the
// four 8192-byte masks at kids + 4 map[k] * 8192 (child (2x + a, 2y + b)
// at index 2b + a), map[k] < 0 copies request -1 - map[k] of `whole`.  map,
// kids, whole and out are device memory.
hipError_t launch_aa_assemble(const int32_t *map, int64_t n, const uint8_t *kids, const uint8_t *whole,
                              uint8_t *out, hipStream_t stream);

}  // namespace hv

// An index as the C ABI hands it out.
struct hv_index {
    hv::IndexArrays a;
    hv::PolyArrays p;   // polygon indexes only
    int kind = 0;
    int device = 0;     // -1 for an empty index (no device memory)
    double root[4] = {0, 0, 0, 0};
    double build_ms = 0;
};
