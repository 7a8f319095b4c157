// Internal declarations shared by the library's HIP sources (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <functional>
#include <string>

#include "../../include/lumiq.h"

namespace lq {

// Device image of a plenoctree.
//  child: [n_nodes][8] int32 (the descriptor's table, unchanged).
//  child_skip: the same tree with every data leaf whose stored density is
//         below sigma_min removed, and every node left without children
//         removed in turn (leaf indices unchanged).  The plain query marches
//         it: those leaves are never composited (Sec. 6.2, sigma_min), so it
//         visits the composited leaves with the same segments in fewer steps.
//  rows:  [n_leaves][row_elems] in the storage type: sigma, then the SH
//         coefficients of R, G, B (K each), zero padded so that a row is a
//         power-of-two number of bytes >= 64 (one row never straddles a
//         128-byte line when it is <= 128 bytes).
// Level of the dense top grid: for each cell of level kTopLevel the grid
// holds the node covering it (> 0) or, where the tree ends above that level
// in an empty node, minus the level of that node's cell.  One read replaces
// the first kTopLevel steps of a descent.  Trees of depth <= kTopLevel have
// no grid.
constexpr int kTopLevel = 4;
constexpr int kTopCells = 1 << (3 * kTopLevel);

// Brick tables of child_skip, marched by the plain query: finest cells in
// bricks of 8^3 (kBrickBits bits per axis), over a dense grid of
// (2^brick_top_bits(depth))^3 bricks.
//  brick_top[z][y][x]: kBrickFull | index of the brick in `bricks`, or, where
//         the brick holds no leaf, its empty extents;
//  bricks[brick][z & 7][y & 7][x & 7]: kBrickFull | leaf index, or the empty
//         extents of an empty cell.
// Empty extents: for each of the 8 ray octants f (bit a of f set: the ray
// moves down along axis a) the code in bits 3f..3f+2 is the largest size m of
// {1, 2, 3, 4, 6, 8, 12, 16} (brick_extent) such that the cube of m cells
// (brick_top: m bricks) that starts at the cell and reaches along the
// octant's directions holds no leaf; cells outside the grid count as empty.
// One entry thus says, for the cell a ray is in, either which leaf it is or
// how far the ray may go at once, in place of a descent from node to node.
// The tables take 2 KB per brick that holds a leaf, up to 4 GB at depth 10.  A
// tree that loads onto a card without room for them goes without: its plain
// queries march child_skip, to the same results.
constexpr int kBrickBits = 3;
constexpr int kBrickCells = 1 << (3 * kBrickBits);
constexpr uint32_t kBrickFull = 0x80000000u;
__host__ __device__ inline int brick_top_bits(int depth) { return depth > kBrickBits ? depth - kBrickBits : 0; }
// size of an extent code: 1, 2, 3, 4, 6, 8, 12, 16
__host__ __device__ constexpr int brick_extent(int code) { return ((2 | ((code + 1) & 1)) << ((code + 1) >> 1)) >> 1; }

struct DevTree {
    const int32_t *child;
    const int32_t *child_skip;
    const int32_t *top;        // [kTopCells] grid of `child`, or null
    const int32_t *top_skip;   // [kTopCells] grid of `child_skip`, or null
    const uint32_t *brick_top;   // null, like bricks, for a tree without brick tables
    const uint32_t *bricks;
    const void *rows;
    int32_t depth, sh_degree, K, storage;
    int32_t n_nodes, n_leaves, row_elems, pad;
    float l_max, sigma_min, alpha_max, pad2;
};

// Words of the ray counters of one query launch: one per accelerator die, each
// in a line of its own (see octree_kernels.h).
constexpr int kCounterStride = 32;
constexpr int kQueryCounters = 8 * kCounterStride;

struct QueryArgs {
    const float *o, *d;
    int64_t n;
    float *rgb, *alpha;
    int model;
    uint32_t flags;
    // trace outputs (nullptr when not tracing)
    uint32_t *count;
    uint64_t *hash;
    int32_t *term_idx;
    uint32_t *n_comp;
    uint32_t *n_steps;
    uint32_t *leaf_ids;
    int32_t max_ids;
    // ray i of the launch is index[i] of the arrays (null: i itself), and
    // the launch covers *n_dev rays when n_dev is set (n is then a bound)
    const int64_t *index;
    const unsigned long long *n_dev;
    // camera batch: when img_w > 0 the n = img_w * img_h rays are the pixels
    // of a row-major image and the waves take them up in 8 x 8 pixel tiles
    // (tile_order_pixel); excludes index
    uint32_t img_w, img_h;
    // kQueryCounters words for the launch's counters, or null: the launcher
    // then allocates them stream-ordered
    unsigned long long *counters;
};

// Pixel taken up at position v (< w h) of a camera batch's tile order, a
// bijection of [0, w h): whole 8 x 8 tiles first, tile by tile along each
// band of 8 rows (a tile row-major inside), then the pixels right of the
// last whole tile of each band, then the rows below the last whole band,
// both row-major.  A wave's 64 lanes thus take one tile: neighbouring
// pixels, whose rays cross mostly the same octree nodes.  w h < 2^32.
__host__ __device__ inline uint32_t tile_order_pixel(uint32_t v, uint32_t w, uint32_t h) {
    const uint32_t w8 = w & ~7u, h8 = h & ~7u;   // columns and rows of whole tiles
    const uint32_t n_tiled = h8 * w8;
    if (v < n_tiled) {                           // then w8 >= 8
        const uint32_t band = v / (8u * w8), j = v - band * (8u * w8);
        const uint32_t p = j & 63u;
        return (band * 8u + (p >> 3)) * w + (j >> 6) * 8u + (p & 7u);
    }
    v -= n_tiled;
    const uint32_t ws = w - w8, n_side = h8 * ws;
    if (v < n_side) {                            // then ws >= 1
        const uint32_t r = v / ws;
        return r * w + w8 + (v - r * ws);
    }
    return h8 * w + (v - n_side);
}

// launch the emission query; returns hipSuccess or the launch error
hipError_t launch_query(const DevTree &t, const QueryArgs &a, bool trace, hipStream_t s);
// several trees of one storage type and SH degree (2 or 3) in one launch;
// trees/offsets are device arrays; bricks: every tree has brick tables
hipError_t launch_query_multi(int storage, int sh_degree, const DevTree *trees, const int64_t *offsets,
                              int n_trees, bool bricks, const QueryArgs &a, hipStream_t s);

// Brick tables of the pruned child table (device memory) of a tree: one new
// allocation *buf of *bytes that holds both tables.  Synchronous.
hipError_t build_bricks(const int32_t *child_skip, int depth, uint32_t **buf, size_t *bytes, const uint32_t **brick_top,
                        const uint32_t **bricks);

// An octree on `device` (current) from its child tables in device memory (which
// it takes over) and its leaves' densities and coefficients in host or device
// memory (read during the call).  On failure the child tables are freed.
// Synchronous.
struct OctreeParts {
    int32_t max_depth, sh_degree, n_nodes, n_skip_nodes, n_leaves;
    float l_max, sigma_min, alpha_max;
    int32_t *child, *child_skip;
    const float *sigma, *sh;
    bool leaves_on_host;
    std::function<void()> make_room;   // gives device scratch back, called when an allocation fails; or empty
};
lq_status make_octree(const OctreeParts &p, int storage, int device, lq_octree **out);
// the scalars of a tree: LQ_OK, or the error a loader returns for them
lq_status check_octree_scalars(float l_max, float sigma_min, float alpha_max);

void set_error(const std::string &msg);

// a device array on `device` holding `bytes` from ptr on (else an error
// status, with the message set)
lq_status check_device_array(const void *ptr, size_t bytes, int device, const char *name);
// device of a tree
int octree_device(const lq_octree *t);

// emission query (default flags) over rays in the library's own device
// scratch (no pointer checks: the caller made the arrays): the rays listed
// in index[0 .. *n_dev) of o/d, writing rgb and alpha at those rays
lq_status query_scratch(const lq_octree *t, const float *o, const float *d, int64_t n_max, const int64_t *index,
                        const unsigned long long *n_dev, float *rgb, float *alpha, int model, hipStream_t s);

// emission query (linear model, default flags) of the rays listed in
// index[0 .. *n_dev) of origins/dirs, writing rgb at those rays
lq_status query_indexed(const lq_octree *tree, const float *o, const float *d, int64_t n_max,
                        const int64_t *index, const unsigned long long *n_dev, float *rgb, hipStream_t s);

}  // namespace lq
