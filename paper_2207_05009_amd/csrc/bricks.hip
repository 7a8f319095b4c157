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
// Each pass streams its tables once; the extents test cubes of growing size
// row by row (one 64-bit AND covers a row of the cube), which takes under a
// millisecond for a depth-9 luminaire of 3M leaves (16k bricks).
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

// Is the cube of m cells from (x, y, z) along octant f empty?  row(z, y)
// returns the bits of row (z, y) from bit x0 on, x0 the cube's lowest x.
template <class Row>
__device__ inline bool cube_empty(int f, int m, int x, int y, int z, Row row) {
    const int x0 = f & 1 ? x - m + 1 : x, y0 = f & 2 ? y - m + 1 : y, z0 = f & 4 ? z - m + 1 : z;
    const unsigned long long mask = (1ull << m) - 1ull;
    for (int k = 0; k < m; ++k)
        for (int j = 0; j < m; ++j)
            if (row(z0 + k, y0 + j, x0) & mask) return false;
    return true;
}

template <class Row>
__device__ inline uint32_t extents(int x, int y, int z, Row row) {
    uint32_t e = 0;
    for (int f = 0; f < 8; ++f) {
        int code = 0;
        while (code < 7 && cube_empty(f, brick_extent(code + 1), x, y, z, row)) ++code;   // the cubes are nested
        e |= (uint32_t)code << (3 * f);
    }
    return e;
}

// a row of up to 128 bits, from bit x0 on (bits outside it are 0)
__device__ inline unsigned long long row_bits(const unsigned long long *w, int x0) {
    if (x0 <= -64 || x0 >= 128) return 0ull;
    if (x0 < 0) return w[0] << -x0;
    if (x0 >= 64) return w[1] >> (x0 - 64);
    return x0 == 0 ? w[0] : (w[0] >> x0) | (w[1] << (64 - x0));
}

__global__ __launch_bounds__(kMarkBlock) void k_top_extents(const unsigned long long *rows, int bits, uint32_t *top) {
    const uint32_t i = blockIdx.x * kMarkBlock + threadIdx.x, m = (1u << bits) - 1u;
    if (i >= (1u << (3 * bits)) || (top[i] & kBrickFull)) return;
    const int edge = 1 << bits;
    top[i] = extents(i & m, (i >> bits) & m, i >> (2 * bits), [&](int z, int y, int x0) -> unsigned long long {
        if (z < 0 || z >= edge || y < 0 || y >= edge) return 0ull;
        return row_bits(rows + ((size_t)z * edge + y) * 2, x0);
    });
}

// The extents of a brick's cells look up to 15 cells beyond it: the rows of
// the 5^3 bricks around it, 40 bits each, are gathered in LDS first.
constexpr int kReach = 2;                              // bricks on each side
constexpr int kRows = (2 * kReach + 1) << kBrickBits;  // 40

__global__ __launch_bounds__(kBrickCells) void k_brick_extents(const uint32_t *top, int bits, const uint32_t *brick_of,
                                                               const unsigned long long *occ, uint32_t *bricks) {
    __shared__ unsigned long long s_row[kRows * kRows];
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
    const size_t j = (size_t)blockIdx.x * kBrickCells + t;
    if (bricks[j] & kBrickFull) return;
    bricks[j] = extents(x + at, y + at, z + at, [&](int zz, int yy, int x0) { return s_row[zz * kRows + yy] >> x0; });
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
        hipLaunchKernelGGL(k_top_extents, dim3(blocks), dim3(kMarkBlock), 0, s, rows, bits, top);
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
