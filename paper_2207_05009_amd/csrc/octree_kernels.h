// octree_kernels.h -- the emission-query kernels and their launchers,
// instantiated per storage type by octree_query_{f32,f16,bf16}.hip.
//
// Persistent waves: the grid holds as many 256-lane blocks as fit on the
// chip at once.  Every lane marches one ray at a time, one table entry per
// step (BrickMarcher in march.h; the validation variants one octree node per
// step, Marcher).  Every kStepsPerCheck steps the wave counts its busy lanes;
// when fewer than kRefillBelow still hold a ray, the idle lanes are refilled:
// each takes the wave's next position plus the number of idle lanes below it.
// Rays of very different lengths then do not leave most of a wave idle until
// its longest ray is done, while the per-ray set-up is paid for many lanes at
// once.
//
// A wave reserves positions in chunks from a ray counter, one atomic each.
// The counters lie kCounterStride words apart: with all of them in one
// 128-byte line, and an atomic per refill, these atomics (about 10 ns each,
// one after the other) were what bounded batches of short rays -- refilling
// more often made the launch slower.  Counters of their own lines and chunks
// of 128: 4.2M room rays, float16, 1.49 -> 1.02 ms, 3M rays over 12 trees
// 0.82 -> 0.55 ms.
//
// XCD-aware work split: the batch is cut into kXcds contiguous ranges, with a
// counter each.  Workgroups are dispatched to the accelerator dies round
// robin, so a wave of block b starts on range b % kXcds: the rays one die's
// L2 sees are neighbours in the batch (for a camera, a band of image rows),
// not every kXcds-th chunk (two ranges per die: camera 0.93 -> 1.03 ms).  A
// wave whose range is used up continues on the next ranges, so the tail stays
// balanced.
//
// Camera batches are split by position in their tile order instead
// (tile_order_pixel), in chunks of one 8 x 8 pixel tile, and a wave takes the
// next tile when it is done with the last: its lanes then march neighbouring
// pixels, cell by cell through mostly the same bricks and leaf rows.  Mixing
// the rest of one tile with rays of the next (refill below 16 busy lanes)
// costs more in cache lines than the idle lanes do: 0.93 -> 0.77 ms, and the
// exponential model with float16 rows alike.  The ranges too are whole tiles
// (range_begin): split at any position, seven of eight ranges of a 1283 x 721
// image had every chunk straddle two tiles (float16, degree 3: 0.300 -> 0.290 ms).
#pragma once

#include <algorithm>

#include "launch_shape.h"
#include "march.h"

namespace lq {
namespace {

constexpr int kBlock = 256;
constexpr int kRefillBelow = 40;     // refill when fewer lanes of a wave are busy
constexpr int kStepsPerCheck = 4;    // steps between refill checks
constexpr int kTileStepsPerCheck = 16;
constexpr int kXcds = 8;             // accelerator dies (XCDs) of an MI355X
constexpr int kRanges = kXcds;       // ray counters (contiguous ranges)
static_assert(kRanges * kCounterStride == kQueryCounters, "the counters of a launch");
constexpr uint32_t kAllRanges = (1u << kRanges) - 1u;   // every range used up
constexpr int kMaxTries = 8;         // refill attempts per check
// positions per reservation: a tile of a camera batch; otherwise kChunk, or
// half of it when the batch would leave a wave fewer than two such chunks
constexpr int kTile = 64;
constexpr int kChunk = 128;

__device__ inline uint64_t lanemask_lt() {
    const unsigned lane = __lane_id();
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// The radiance and opacity of a finished ray go out as non-temporal stores:
// lanes finish at different steps, so each store fills only part of a line,
// and without the hint those partial lines occupy L2 until evicted
// (incoherent batches: room f32 5.81 -> 5.74 ms, f16 5.37 -> 5.28 ms).
template <class M>
__device__ inline void write_ray(const QueryArgs &a, int64_t i, const M &m, bool trace) {
    RayOut r;
    m.result(r);
    if (a.rgb) {
        __builtin_nontemporal_store(r.rgb[0], a.rgb + 3 * i);
        __builtin_nontemporal_store(r.rgb[1], a.rgb + 3 * i + 1);
        __builtin_nontemporal_store(r.rgb[2], a.rgb + 3 * i + 2);
    }
    if (a.alpha) __builtin_nontemporal_store(r.alpha, a.alpha + i);
    if (trace) {
        a.count[i] = r.count;
        a.hash[i] = r.hash;
        a.term_idx[i] = r.term_idx;
        a.n_comp[i] = r.n_comp;
        if (a.n_steps) a.n_steps[i] = r.n_steps;
    }
}

// ORDER maps a position of the split to a ray: kOrderAny takes a.index, then
// the image tile order, then the position itself, whichever the arguments
// set; kOrderBatch only a.index or the position; kOrderTiles only the tile
// order.
enum { kOrderAny = 0, kOrderBatch = 1, kOrderTiles = 2 };

// How a lane walks its ray.  OctreeWalk: node by node through the octree
// (the validation variants, and trees without brick tables).  The block copies the tree's top grid into LDS,
// and each lane keeps its node path there.
template <int ST, int DEG, bool ACC64, bool TRACE_, bool SKIP, int MODEL>
struct OctreeWalk {
    using M = Marcher<ST, DEG, ACC64, TRACE_, SKIP, MODEL>;
    static constexpr bool TRACE = TRACE_;
    int32_t *path;
    const int32_t *top;
    __device__ void setup(const DevTree &t0) {
        __shared__ int32_t s_path[10 * kBlock];   // per-lane node path, [level][lane]
        __shared__ int32_t s_top[kTopCells];
        path = s_path + threadIdx.x;
        const int32_t *src = SKIP ? t0.top_skip : t0.top;
        top = src ? s_top : nullptr;
        if (src)
            for (int i = threadIdx.x; i < kTopCells; i += kBlock) s_top[i] = src[i];
        __syncthreads();
    }
    __device__ bool step(M &m, const DevTree &t, const QueryArgs &a, uint32_t *ids) {
        return m.step(t, a.model, a.flags, ids, TRACE ? a.max_ids : 0, path, kBlock, top);
    }
};

// The same over several trees: each ray reads its tree's grid from global
// memory.
template <int ST, int DEG, bool ACC64, bool SKIP>
struct MultiOctreeWalk {
    using M = Marcher<ST, DEG, ACC64, false, SKIP, -1>;
    static constexpr bool TRACE = false;
    int32_t *path;
    __device__ void setup(const DevTree &) {
        __shared__ int32_t s_path[10 * kBlock];
        path = s_path + threadIdx.x;
    }
    __device__ bool step(M &m, const DevTree &t, const QueryArgs &a, uint32_t *) {
        return m.step(t, a.model, a.flags, nullptr, 0, path, kBlock, SKIP ? t.top_skip : t.top);
    }
};

// BrickWalk: cell by cell through the brick tables (the plain queries).
template <int ST, int DEG, int MODEL>
struct BrickWalk {
    using M = BrickMarcher<ST, DEG, MODEL>;
    static constexpr bool TRACE = false;
    __device__ void setup(const DevTree &) {}
    __device__ bool step(M &m, const DevTree &t, const QueryArgs &a, uint32_t *) { return m.step(t, a.flags); }
};

// the persistent loop shared by all query kernels; tree_index(ray) finds the
// tree a ray queries (once, when a lane takes the ray) and tree_at(k) returns
// tree k.  Without counters (queue null) the launch has a lane for every ray
// and each lane takes the ray at its own position.
template <class Walk, int ORDER, class TreeIndex, class TreeAt>
__device__ inline void persistent_query(const QueryArgs &a, unsigned long long *queue, TreeIndex tree_index,
                                        TreeAt tree_at) {
    constexpr bool TRACE = Walk::TRACE;
    Walk walk;
    walk.setup(tree_at(0));
    constexpr bool tiles = ORDER == kOrderTiles;
    constexpr int refill_below = tiles ? 1 : kRefillBelow;
    constexpr int steps_per_check = tiles ? kTileStepsPerCheck : kStepsPerCheck;
    typename Walk::M m;
    int64_t ray = -1;            // ray held by this lane, -1 when idle
    int tk = 0;                  // tree of that ray
    uint32_t *ids = nullptr;
    int cur = (int)(blockIdx.x % kXcds);   // range this wave reserves from (wave-uniform)
    uint32_t used_up = 0;                  // ranges known to be exhausted (wave-uniform)
    int64_t pool = 0, pool_end = 0;        // positions reserved for this wave (wave-uniform)
    const int64_t n = a.n_dev ? (int64_t)*a.n_dev : a.n;
    const int chunk = tiles || n < (int64_t)gridDim.x * (kBlock / 64) * (2 * kChunk) ? kTile : kChunk;
    for (;;) {
        bool want = ray < 0 && (pool < pool_end || used_up != kAllRanges);
        uint64_t need = __ballot(want);
        const int busy = __popcll(__ballot(ray >= 0));
        if (__builtin_expect(need && busy < refill_below, 0)) {
            for (int tries = 0; need && tries < kMaxTries; ++tries) {
                int64_t pos = -1;    // position this lane takes up, if any
                if (queue) {
                    if (pool == pool_end) {    // reserve the next chunk
                        unsigned long long base = 0;
                        if (__lane_id() == 0) base = atomicAdd(queue + cur * kCounterStride, (unsigned long long)chunk);
                        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)base);
                        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
                        base = ((unsigned long long)hi << 32) | lo;
                        constexpr int unit = tiles ? kTile : 1;
                        const int64_t start = range_begin(cur, kRanges, n, unit);
                        const int64_t end = range_begin(cur + 1, kRanges, n, unit);
                        pool = std::min<int64_t>(start + (int64_t)base, end);
                        pool_end = std::min<int64_t>(pool + chunk, end);
                        if (pool_end == end) {   // this range is used up: the next reservation is from another
                            used_up |= 1u << cur;
                            for (int j = 1; j <= kRanges; ++j) {
                                const int c = (cur + j) % kRanges;
                                if (!(used_up & (1u << c))) { cur = c; break; }
                            }
                        }
                    }
                    const int64_t p = pool + __popcll(need & lanemask_lt());
                    if (want && p < pool_end) pos = p;
                    pool = std::min<int64_t>(pool + __popcll(need), pool_end);
                } else {
                    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
                    if (p < n) pos = p;
                    used_up = kAllRanges;
                }
                if (pos >= 0) {
                    int64_t idx = pos;
                    if constexpr (ORDER == kOrderTiles) {
                        idx = tile_order_pixel((uint32_t)pos, a.img_w, a.img_h);
                    } else {
                        if (a.index) idx = a.index[pos];
                        else if (ORDER == kOrderAny && a.img_w) idx = tile_order_pixel((uint32_t)pos, a.img_w, a.img_h);
                    }
                    ids = TRACE && a.max_ids > 0 ? a.leaf_ids + (size_t)idx * a.max_ids : nullptr;
                    tk = tree_index(idx);
                    if (m.init(tree_at(tk), a.o + 3 * idx, a.d + 3 * idx)) {
                        ray = idx;
                        want = false;
                    } else {
                        write_ray(a, idx, m, TRACE);   // no positive-length overlap: done
                    }
                }
                want = want && (pool < pool_end || used_up != kAllRanges);
                need = __ballot(want);
            }
        }
        if (__all(ray < 0) && pool == pool_end && used_up == kAllRanges) break;
        for (int k = 0; k < steps_per_check && ray >= 0; ++k) {
            if (__builtin_expect(walk.step(m, tree_at(tk), a, ids), 0)) {
                write_ray(a, ray, m, TRACE);
                ray = -1;
            }
        }
    }
}

// The validation kernels (traces, FP64 accumulation, every leaf composited) and
// the plain query of a tree without brick tables; the transmittance model and
// the ray order come from the arguments.
template <int ST, int DEG, bool ACC64, bool TRACE, bool SKIP>
__global__ __launch_bounds__(kBlock) void k_query(const DevTree t, const QueryArgs a,
                                                  unsigned long long *queue) {
    persistent_query<OctreeWalk<ST, DEG, ACC64, TRACE, SKIP, -1>, kOrderAny>(
        a, queue, [](int64_t) { return 0; }, [&](int) -> const DevTree & { return t; });
}

// Register budgets of the plain queries (float32 accumulation, no trace), in
// waves per SIMD: they wait on dependent loads, so as many waves as hold the
// leaf row and the (l+1)^2 basis values in registers, up to 16 bytes per lane
// of which the budget may move to scratch (float32, degree 2: camera 0.77 ms
// with four waves, 0.71 with five).  Beyond that spilling costs more than the
// wave gains (float16, degree 3: 0.28 ms with four waves, 0.61 with five).
template <int ST, int DEG>
constexpr int plain_waves_per_simd() {
    constexpr int K = (DEG + 1) * (DEG + 1);
    if (ST == LQ_F32) return K <= 9 ? 5 : 4;
    return K <= 4 ? 5 : (K <= 16 ? 4 : 3);
}

// without the sigma_min skip (LQ_NO_SIGMA_SKIP): the full table
template <int ST, int DEG>
constexpr int full_waves_per_simd() {
    constexpr int K = (DEG + 1) * (DEG + 1);
    constexpr int row_regs = ((1 + 3 * K) * Storage<ST>::bytes + 15) / 16 * 4;
    return row_regs + K <= 40 ? 5 : (row_regs + K <= 70 ? 4 : 3);
}

template <int ST, int DEG>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(full_waves_per_simd<ST, DEG>())))
void k_query_full(const DevTree t, const QueryArgs a, unsigned long long *queue) {
    persistent_query<OctreeWalk<ST, DEG, false, false, false, -1>, kOrderAny>(
        a, queue, [](int64_t) { return 0; }, [&](int) -> const DevTree & { return t; });
}

// the production query, in batch order or, with TILES, in the tile order of
// a camera batch
template <int ST, int DEG, int MODEL, bool TILES>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(plain_waves_per_simd<ST, DEG>())))
void k_query_plain(const DevTree t, const QueryArgs a, unsigned long long *queue) {
    persistent_query<BrickWalk<ST, DEG, MODEL>, TILES ? kOrderTiles : kOrderBatch>(
        a, queue, [](int64_t) { return 0; }, [&](int) -> const DevTree & { return t; });
}

// several trees: rays [offsets[k], offsets[k+1]) query trees[k]; the tree of
// a ray is found by binary search when a lane takes it.
struct TreeOfRay {
    const int64_t *offsets;
    int n_trees;
    __device__ int operator()(int64_t ray) const {
        int lo = 0, hi = n_trees;            // offsets[lo] <= ray < offsets[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (offsets[mid] <= ray) lo = mid;
            else hi = mid;
        }
        return lo;
    }
};

template <int ST, int DEG, bool ACC64, bool SKIP>
__global__ __launch_bounds__(kBlock) void k_query_multi(const DevTree *trees, const int64_t *offsets,
                                                        int n_trees, const QueryArgs a,
                                                        unsigned long long *queue) {
    persistent_query<MultiOctreeWalk<ST, DEG, ACC64, SKIP>, kOrderBatch>(
        a, queue, TreeOfRay{offsets, n_trees}, [&](int k) -> const DevTree & { return trees[k]; });
}

// the plain multi-tree kernels keep the default register budget: a lane's
// tree fields come from memory and need registers
template <int ST, int DEG, int MODEL>
__global__ __launch_bounds__(kBlock) void k_query_multi_plain(
    const DevTree *trees, const int64_t *offsets, int n_trees, const QueryArgs a, unsigned long long *queue) {
    persistent_query<BrickWalk<ST, DEG, MODEL>, kOrderBatch>(
        a, queue, TreeOfRay{offsets, n_trees}, [&](int k) -> const DevTree & { return trees[k]; });
}

__global__ void k_zero_u64(unsigned long long *p) { p[threadIdx.x * kCounterStride] = 0ull; }

// blocks of a kernel that the current device holds at once
int resident_blocks(const void *kern) {
    static ResidentBlocks known;
    int dev = 0;
    (void)hipGetDevice(&dev);
    return known.get(dev, kern, [&] {
        int per_cu = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kBlock, 0) != hipSuccess || per_cu < 1)
            per_cu = 1;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 1;
        (void)hipGetLastError();
        return per_cu * cus;
    });
}

// Launch over persistent blocks with ray counters.  kStatic: no counters when
// the batch fits the chip at once and its size is known on the host; each
// lane then takes one ray, without the counters' allocation, their clearing
// launch and the refill atomics (4,096 rays on a depth-6 tree: 84 -> 35 us
// with the brick march).  Batches of up to 64 K rays go out in one-wave
// blocks, which spread over more CUs.
template <bool kStatic, class Kern, class... Args>
hipError_t launch_persistent(Kern kern, const QueryArgs &a, unsigned long long *queue, hipStream_t s, Args... args) {
    const int64_t need_blocks = (a.n + kBlock - 1) / kBlock;
    const int64_t nb = std::min<int64_t>(need_blocks, resident_blocks(reinterpret_cast<const void *>(kern)));
    if (kStatic && nb == need_blocks && !a.n_dev) {
        const int block = a.n <= (int64_t)64 * 1024 ? 64 : kBlock;
        hipLaunchKernelGGL(kern, dim3((unsigned)((a.n + block - 1) / block)), dim3(block), 0, s, args...,
                           (unsigned long long *)nullptr);
        return hipGetLastError();
    }
    hipError_t e = hipSuccess;
    const bool own = !queue;
    if (own && (e = hipMallocAsync((void **)&queue, kQueryCounters * sizeof(unsigned long long), s)) != hipSuccess) return e;
    // cleared by a kernel (not a memset node), so the launch can be captured
    hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(kRanges), 0, s, queue);
    hipLaunchKernelGGL(kern, dim3((unsigned)nb), dim3(kBlock), 0, s, args..., queue);
    e = hipGetLastError();
    const hipError_t f = own ? hipFreeAsync(queue, s) : hipSuccess;
    return e != hipSuccess ? e : f;
}

template <int ST, int DEG, bool ACC64, bool TRACE, bool SKIP>
hipError_t launch_checked(const DevTree &t, const QueryArgs &a, hipStream_t s) {
    return launch_persistent<false>(k_query<ST, DEG, ACC64, TRACE, SKIP>, a, a.counters, s, t, a);
}

template <int ST, int DEG, int MODEL>
hipError_t launch_plain(const DevTree &t, const QueryArgs &a, hipStream_t s) {
    // the kernels of camera batches have the tile order built in
    return a.img_w ? launch_persistent<true>(k_query_plain<ST, DEG, MODEL, true>, a, a.counters, s, t, a)
                   : launch_persistent<true>(k_query_plain<ST, DEG, MODEL, false>, a, a.counters, s, t, a);
}

template <int ST, int DEG>
hipError_t launch_deg(const DevTree &t, const QueryArgs &a, bool trace, hipStream_t s) {
    // traces record every data leaf, so they march the full table; so do
    // queries that composite every leaf
    const bool acc64 = (a.flags & LQ_FP64_ACCUM) != 0;
    const bool full = trace || (a.flags & LQ_NO_SIGMA_SKIP) != 0;
    // a trace of the pruned table (the production query's work)
    if (trace && (a.flags & LQ_TRACE_PRUNED)) return launch_checked<ST, DEG, false, true, true>(t, a, s);
    if (trace) return acc64 ? launch_checked<ST, DEG, true, true, false>(t, a, s)
                            : launch_checked<ST, DEG, false, true, false>(t, a, s);
    if (full) return acc64 ? launch_checked<ST, DEG, true, false, false>(t, a, s)
                           : launch_persistent<false>(k_query_full<ST, DEG>, a, a.counters, s, t, a);
    if (acc64) return launch_checked<ST, DEG, true, false, true>(t, a, s);
    if (!t.bricks) return launch_checked<ST, DEG, false, false, true>(t, a, s);
    return a.model == LQ_EXP ? launch_plain<ST, DEG, LQ_EXP>(t, a, s) : launch_plain<ST, DEG, LQ_LINEAR>(t, a, s);
}

template <int ST>
hipError_t launch_st(const DevTree &t, const QueryArgs &a, bool trace, hipStream_t s) {
    switch (t.sh_degree) {
        case 0: return launch_deg<ST, 0>(t, a, trace, s);
        case 1: return launch_deg<ST, 1>(t, a, trace, s);
        case 2: return launch_deg<ST, 2>(t, a, trace, s);
        case 3: return launch_deg<ST, 3>(t, a, trace, s);
        case 4: return launch_deg<ST, 4>(t, a, trace, s);
    }
    return hipErrorInvalidValue;
}

template <int ST, int DEG>
hipError_t launch_multi_deg(const DevTree *trees, const int64_t *offsets, int n_trees, bool bricks,
                            const QueryArgs &a, hipStream_t s) {
    const bool acc64 = (a.flags & LQ_FP64_ACCUM) != 0;
    const bool full = (a.flags & LQ_NO_SIGMA_SKIP) != 0;
    const auto checked = [&](auto kern) {
        return launch_persistent<false>(kern, a, nullptr, s, trees, offsets, n_trees, a);
    };
    const auto plain = [&](auto kern) {
        return launch_persistent<true>(kern, a, nullptr, s, trees, offsets, n_trees, a);
    };
    if (full) return acc64 ? checked(k_query_multi<ST, DEG, true, false>) : checked(k_query_multi<ST, DEG, false, false>);
    if (acc64) return checked(k_query_multi<ST, DEG, true, true>);
    if (!bricks) return checked(k_query_multi<ST, DEG, false, true>);
    return a.model == LQ_EXP ? plain(k_query_multi_plain<ST, DEG, LQ_EXP>) : plain(k_query_multi_plain<ST, DEG, LQ_LINEAR>);
}

template <int ST>
hipError_t launch_multi_st(int deg, const DevTree *trees, const int64_t *offsets, int n_trees, bool bricks,
                           const QueryArgs &a, hipStream_t s) {
    switch (deg) {
        case 2: return launch_multi_deg<ST, 2>(trees, offsets, n_trees, bricks, a, s);
        case 3: return launch_multi_deg<ST, 3>(trees, offsets, n_trees, bricks, a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace
}  // namespace lq
