// bricks.hip -- the brick tables the plain query marches (layout in
// lq_internal.h), built on the device from the pruned child table at load:
//   k_brick_mark    one thread per brick of the dense grid: the node that
//                   covers it, a bit per brick (rows along x), counts per
//                   block;
//   k_brick_scan    exclusive scan of the block counts (one block);
//   k_brick_number  the brick grid: index of each brick that holds a leaf;
//   k_brick_fill    one block per such brick: its cells' leaves and a
//                   512-bit occupancy mask;
//   k_top_extents, k_brick_extents  the empty extents, from the bit rows.
// Each pass streams its tables once; the extents take whole rows of cells as
// bits (row_codes).  All kernels of it: 0.12 ms for a depth-8 luminaire of 882k
// leaves, 0.31 ms at depth 9 (6.2M), 1.27 ms at depth 10 (46M).
#include <hip/hip_runtime.h>

#include "lq_internal.h"

namespace lq {
namespace {

constexpr int kMarkBlock = 256;
constexpr int kScanThreads = 1024;

// node that covers cell (x, y, z) of level `levels`, descending from `node`;
// a negative value (leaf) or 0 (empty) ends the descent
__device__ inline int32_t descend(const int32_t *child, int32_t node, int levels, int x, int y, int z) {
    for (int l = levels - 1; l >= 0; --l) {
        const int oct = ((x >> l) & 1) | (((y >> l) & 1) << 1) | (((z >> l) & 1) << 2);
        node = child[(uint32_t)node * 8u + (uint32_t)oct];
        if (node <= 0) return node;
    }
    return node;
}

// rows: [z][y][2] 64-bit words, bit x of a row set where the brick holds a leaf
__global__ __launch_bounds__(kMarkBlock) void k_brick_mark(const int32_t *child, int bits, int32_t *node,
                                                           unsigned long long *rows, uint32_t *counts) {
    __shared__ uint32_t s_n;
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    const uint32_t i = blockIdx.x * kMarkBlock + threadIdx.x, n = 1u << (3 * bits), m = (1u << bits) - 1u;
    bool full = false;
    if (i < n) {
        const int x = i & m, y = (i >> bits) & m, z = i >> (2 * bits);
        const int32_t c = bits ? descend(child, 0, bits, x, y, z) : 0;
        full = bits == 0 || c > 0;       // the single brick of a shallow tree always exists
        node[i] = full ? c : -1;
        if (full) atomicOr(rows + ((size_t)(i >> bits)) * 2 + (x >> 6), 1ull << (x & 63));
    }
    const unsigned long long b = __ballot(full);
    if ((threadIdx.x & 63) == 0) atomicAdd(&s_n, (uint32_t)__popcll(b));
    __syncthreads();
    if (threadIdx.x == 0) counts[blockIdx.x] = s_n;
}

// exclusive scan of n counts in place; the total in *total
__global__ __launch_bounds__(kScanThreads) void k_brick_scan(uint32_t *counts, uint32_t n, uint32_t *total) {
    __shared__ uint32_t s[kScanThreads];
    const uint32_t per = (n + kScanThreads - 1) / kScanThreads, a = min(n, threadIdx.x * per), b = min(n, a + per);
    uint32_t sum = 0;
    for (uint32_t i = a; i < b; ++i) sum += counts[i];
    s[threadIdx.x] = sum;
    __syncthreads();
    for (int off = 1; off < kScanThreads; off <<= 1) {
        const uint32_t v = threadIdx.x >= (unsigned)off ? s[threadIdx.x - off] : 0u;
        __syncthreads();
        s[threadIdx.x] += v;
        __syncthreads();
    }
    uint32_t run = s[threadIdx.x] - sum;
    for (uint32_t i = a; i < b; ++i) {
        const uint32_t c = counts[i];
        counts[i] = run;
        run += c;
    }
    if (threadIdx.x == kScanThreads - 1) *total = run;
}

// top[i] = kBrickFull | index, and brick_of[index] = i
__global__ __launch_bounds__(kMarkBlock) void k_brick_number(const int32_t *node, uint32_t n, const uint32_t *offsets,
                                                             uint32_t *top, uint32_t *brick_of) {
    __shared__ uint32_t s_wave[kMarkBlock / 64];
    const uint32_t i = blockIdx.x * kMarkBlock + threadIdx.x, lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
    const bool full = i < n && node[i] >= 0;
    const unsigned long long b = __ballot(full);
    if (lane == 0) s_wave[w] = (uint32_t)__popcll(b);
    __syncthreads();
    uint32_t pos = offsets[blockIdx.x];
    for (uint32_t j = 0; j < w; ++j) pos += s_wave[j];
    pos += (uint32_t)__popcll(lane ? b & (~0ull >> (64 - lane)) : 0ull);
    if (i < n) top[i] = full ? kBrickFull | pos : 0u;
    if (full) brick_of[pos] = i;
}

// cells of brick blockIdx.x, and its occupancy: occ[brick][z] bit 8 y + x
__global__ __launch_bounds__(kBrickCells) void k_brick_fill(const int32_t *child, const int32_t *node,
                                                            const uint32_t *brick_of, int depth, uint32_t *bricks,
                                                            unsigned long long *occ) {
    const int t = threadIdx.x, x = t & 7, y = (t >> 3) & 7, z = t >> 6;
    const int levels = depth < kBrickBits ? depth : kBrickBits, edge = 1 << levels;
    uint32_t e = 0;
    if (x < edge && y < edge && z < edge) {
        const int32_t c = descend(child, node[brick_of[blockIdx.x]], levels, x, y, z);
        if (c < 0) e = kBrickFull | (uint32_t)(-(int64_t)c - 1);
    }
    bricks[(size_t)blockIdx.x * kBrickCells + t] = e;
    const unsigned long long b = __ballot(e != 0);
    if ((t & 63) == 0) occ[(size_t)blockIdx.x * 8 + z] = b;
}

// The extents of all cells of a row (z, y), for one octant f, a bit per cell:
// the rows of the m x m square that the cubes of m cells cover are ORed, the
// cells along x ORed by shifts; a cell whose bit stays clear has an empty cube.
// The codes are counted in three bit planes (the cubes are nested).  A wave takes
// rows of one octant, so its loops are uniform.  Both extent kernels of a
// depth-8, 9 and 10 luminaire: 0.09, 0.25 and 1.01 ms; tested cell by cell, a lane
// per cell, the tables took 3.2, 9.7 and 42.7 ms.
struct Bits128 {
    unsigned long long lo, hi;
};
__device__ inline unsigned long long bits_or(unsigned long long a, unsigned long long b) { return a | b; }
__device__ inline unsigned long long bits_andn(unsigned long long a, unsigned long long b) { return a & ~b; }
__device__ inline unsigned long long bits_and(unsigned long long a, unsigned long long b) { return a & b; }
__device__ inline unsigned long long bits_xor(unsigned long long a, unsigned long long b) { return a ^ b; }
__device__ inline bool bits_any(unsigned long long a) { return a != 0; }
// toward bit 0 (up: away from it); 0 < n < 64
__device__ inline unsigned long long bits_shift(unsigned long long a, int n, bool up) { return up ? a << n : a >> n; }
__device__ inline Bits128 bits_or(Bits128 a, Bits128 b) { return {a.lo | b.lo, a.hi | b.hi}; }
__device__ inline Bits128 bits_andn(Bits128 a, Bits128 b) { return {a.lo & ~b.lo, a.hi & ~b.hi}; }
__device__ inline Bits128 bits_and(Bits128 a, Bits128 b) { return {a.lo & b.lo, a.hi & b.hi}; }
__device__ inline Bits128 bits_xor(Bits128 a, Bits128 b) { return {a.lo ^ b.lo, a.hi ^ b.hi}; }
__device__ inline bool bits_any(Bits128 a) { return (a.lo | a.hi) != 0; }
__device__ inline Bits128 bits_shift(Bits128 a, int n, bool up) {
    if (up) return {a.lo << n, (a.hi << n) | (a.lo >> (64 - n))};
    return {(a.lo >> n) | (a.hi << (64 - n)), a.hi >> n};
}

// planes[0..2]: the codes of the cells of `cells` in row (z, y); row(z, y)
// returns a row's occupied cells.
template <class B, class Row>
__device__ inline void row_codes(int f, int z, int y, B cells, Row row, B planes[3]) {
    const int sy = f & 2 ? -1 : 1, sz = f & 4 ? -1 : 1;
    B square = {}, open = cells;
    planes[0] = planes[1] = planes[2] = B{};
    int done = 0;
    for (int code = 1; code < 8; ++code) {
        const int m = brick_extent(code);
        for (int k = 0; k < m; ++k)
            for (int j = k < done ? done : 0; j < m; ++j) square = bits_or(square, row(z + sz * k, y + sy * j));
        done = m;
        B d = square;
        int w = 1;
        for (; 2 * w <= m; w *= 2) d = bits_or(d, bits_shift(d, w, f & 1));
        if (w < m) d = bits_or(d, bits_shift(d, m - w, f & 1));
        open = bits_andn(open, d);
        if (!__any(bits_any(open))) break;
        B carry = open;
        for (int b = 0; b < 3; ++b) {
            const B t = bits_and(planes[b], carry);
            planes[b] = bits_xor(planes[b], carry);
            carry = t;
        }
    }
}

// Block: 64 rows y of slice z (a wave per octant).
constexpr int kTopRows = 64;

__global__ __launch_bounds__(8 * kTopRows) void k_top_extents(const unsigned long long *rows, int bits,
                                                              uint32_t *top) {
    __shared__ unsigned long long s_plane[8][3][2][kTopRows];
    const int edge = 1 << bits, groups = (edge + kTopRows - 1) / kTopRows;
    const int z = (int)blockIdx.x / groups, y0 = ((int)blockIdx.x % groups) * kTopRows;
    {
        const int f = threadIdx.x / kTopRows, r = threadIdx.x % kTopRows;
        const Bits128 all = {~0ull, ~0ull};
        Bits128 planes[3];
        row_codes(f, z, y0 + r, all, [&](int zz, int yy) -> Bits128 {
            if (zz < 0 || zz >= edge || yy < 0 || yy >= edge) return Bits128{};
            const unsigned long long *w = rows + ((size_t)zz * edge + yy) * 2;
            return Bits128{w[0], w[1]};
        }, planes);
        for (int b = 0; b < 3; ++b) {
            s_plane[f][b][0][r] = planes[b].lo;
            s_plane[f][b][1][r] = planes[b].hi;
        }
    }
    __syncthreads();
    const int n = (edge - y0 < kTopRows ? edge - y0 : kTopRows) << bits;
    for (int t = threadIdx.x; t < n; t += 8 * kTopRows) {
        const int x = t & (edge - 1), r = t >> bits;
        const size_t i = ((size_t)z * edge + y0) * edge + t;
        if (top[i] & kBrickFull) continue;
        uint32_t e = 0;
        for (int f = 0; f < 8; ++f)
            for (int b = 0; b < 3; ++b)
                e |= (uint32_t)((s_plane[f][b][x >> 6][r] >> (x & 63)) & 1u) << (3 * f + b);
        top[i] = e;
    }
}

// The extents of a brick's cells look up to 15 cells beyond it: the rows of
// the 5^3 bricks around it, 40 bits each, are gathered in LDS first.
constexpr int kReach = 2;                              // bricks on each side
constexpr int kRows = (2 * kReach + 1) << kBrickBits;  // 40

__global__ __launch_bounds__(kBrickCells) void k_brick_extents(const uint32_t *top, int bits, const uint32_t *brick_of,
                                                               const unsigned long long *occ, uint32_t *bricks) {
    __shared__ unsigned long long s_row[kRows * kRows];
    __shared__ uint32_t s_code[8][64];
    const uint32_t i = brick_of[blockIdx.x], m = (1u << bits) - 1u;
    const int edge = 1 << bits, bx = i & m, by = (i >> bits) & m, bz = i >> (2 * bits);
    for (int r = threadIdx.x; r < kRows * kRows; r += kBrickCells) {
        const int zz = r / kRows, yy = r - zz * kRows;
        const int z = bz + (zz >> 3) - kReach, y = by + (yy >> 3) - kReach;
        unsigned long long v = 0;
        if (z >= 0 && z < edge && y >= 0 && y < edge)
            for (int k = 0; k <= 2 * kReach; ++k) {
                const int x = bx + k - kReach;
                if (x < 0 || x >= edge) continue;
                const uint32_t e = top[((uint32_t)z << (2 * bits)) | ((uint32_t)y << bits) | (uint32_t)x];
                if (e & kBrickFull)
                    v |= ((occ[(size_t)(e & ~kBrickFull) * 8 + (zz & 7)] >> (8 * (yy & 7))) & 0xFFull) << (8 * k);
            }
        s_row[r] = v;
    }
    __syncthreads();
    const int t = threadIdx.x, x = t & 7, y = (t >> 3) & 7, z = t >> 6, at = kReach << kBrickBits;
    {
        const int f = t >> 6, rz = (t >> 3) & 7, ry = t & 7;     // a wave per octant, a lane per row
        unsigned long long planes[3];
        row_codes(f, rz + at, ry + at, 0xFFull << at, [&](int zz, int yy) { return s_row[zz * kRows + yy]; }, planes);
        s_code[f][t & 63] =
            (uint32_t)(planes[0] >> at) | (uint32_t)(planes[1] >> at) << 8 | (uint32_t)(planes[2] >> at) << 16;
    }
    __syncthreads();
    const size_t j = (size_t)blockIdx.x * kBrickCells + t;
    if (bricks[j] & kBrickFull) return;
    uint32_t e = 0;
    for (int f = 0; f < 8; ++f) {
        const uint32_t c = s_code[f][z * 8 + y] >> x;
        e |= ((c & 1u) | (c >> 7 & 2u) | (c >> 14 & 4u)) << (3 * f);
    }
    bricks[j] = e;
}

__global__ void k_zero_words(unsigned long long *p, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

struct Scratch {
    void *p = nullptr;
    ~Scratch() { (void)hipFree(p); }
};

}  // namespace

hipError_t build_bricks(const int32_t *child_skip, int depth, uint32_t **buf, size_t *bytes, const uint32_t **brick_top,
                        const uint32_t **bricks) {
    *buf = nullptr;
    const int bits = brick_top_bits(depth);
    const uint32_t n = 1u << (3 * bits), blocks = (n + kMarkBlock - 1) / kMarkBlock;
    const size_t row_words = (size_t)2 << (2 * bits);
    // scratch: bit rows, node of each brick, block counts and their total
    Scratch a;
    hipError_t e = hipMalloc(&a.p, row_words * 8 + (size_t)n * 4 + ((size_t)blocks + 1) * 4);
    if (e != hipSuccess) return e;
    unsigned long long *rows = static_cast<unsigned long long *>(a.p);
    int32_t *node = reinterpret_cast<int32_t *>(rows + row_words);
    uint32_t *counts = reinterpret_cast<uint32_t *>(node + n);
    hipStream_t s = nullptr;
    hipLaunchKernelGGL(k_zero_words, dim3((unsigned)((row_words + 255) / 256)), dim3(256), 0, s, rows, row_words);
    hipLaunchKernelGGL(k_brick_mark, dim3(blocks), dim3(kMarkBlock), 0, s, child_skip, bits, node, rows, counts);
    hipLaunchKernelGGL(k_brick_scan, dim3(1), dim3(kScanThreads), 0, s, counts, blocks, counts + blocks);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    uint32_t total = 0;
    if ((e = hipMemcpy(&total, counts + blocks, 4, hipMemcpyDeviceToHost)) != hipSuccess) return e;
    // the tables, bricks first (2 KB each), and scratch of 68 bytes per brick
    *bytes = (size_t)total * kBrickCells * 4 + (size_t)n * 4;
    Scratch b;
    if ((e = hipMalloc((void **)buf, *bytes)) != hipSuccess) {
        *buf = nullptr;
        return e;
    }
    uint32_t *out = *buf, *top = out + (size_t)total * kBrickCells;
    e = hipMalloc(&b.p, (size_t)total * 68 + 8);
    if (e == hipSuccess) {
        unsigned long long *occ = static_cast<unsigned long long *>(b.p);
        uint32_t *brick_of = reinterpret_cast<uint32_t *>(occ + (size_t)total * 8);
        hipLaunchKernelGGL(k_brick_number, dim3(blocks), dim3(kMarkBlock), 0, s, node, n, counts, top, brick_of);
        if (total) {
            hipLaunchKernelGGL(k_brick_fill, dim3(total), dim3(kBrickCells), 0, s, child_skip, node, brick_of, depth,
                               out, occ);
            hipLaunchKernelGGL(k_brick_extents, dim3(total), dim3(kBrickCells), 0, s, top, bits, brick_of, occ, out);
        }
        const unsigned edge = 1u << bits;
        hipLaunchKernelGGL(k_top_extents, dim3(edge * ((edge + kTopRows - 1) / kTopRows)), dim3(8 * kTopRows), 0, s, rows,
                           bits, top);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipStreamSynchronize(s);
    }
    if (e != hipSuccess) {
        (void)hipFree(*buf);
        *buf = nullptr;
        return e;
    }
    *brick_top = top;
    *bricks = out;
    return hipSuccess;
}

}  // namespace lq
