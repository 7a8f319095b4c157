// distill.hip -- plenoctree distillation from a continuous radiance field
// (Sec. 5, "Creating the plenoctree"): one density sample at the centre of
// every voxel of the finest grid, pruning of the voxels whose centre density
// is below a threshold (0.01 in the paper), the mean density and mean SH
// coefficients of a number of uniformly random positions inside every voxel
// kept (256 in the paper: averaging against aliasing at discontinuities),
// and the octree over the kept voxels with its empty octants collapsed
// bottom-up.
//
// The field (the stand-in for a trained radiance field) is a sum of
// Gaussian blobs in log-density, clamped, with thin spherical shells of
// constant density; its SH emission coefficients are blended by the
// normalised blob weights w_k (a softmax of -|x - c_k|^2 / (2 r_k^2)): the
// DC coefficient is logit(E_c / L_max) / Y_00 with E_c = sum_k w_k e_kc, the
// others sum_k w_k h_kcj (lq_field_desc in include/lumiq.h).
//
// Kernels, stream-ordered:
//   k_centre_bits     voxels in Morton order, words of 64: the centre test
//                     in FP64 (its decision is an integer), one 64-bit
//                     ballot word per 64 voxels, a count per chunk;
//   k_scan_counts     exclusive scan of the chunk counts (one block);
//   k_centre_compact  the Morton codes of the kept voxels, ascending;
//   k_distill<NB>     one lane per kept voxel: n_samples positions from
//                     Philox4x32-10 (counter = code, sample index, 0, 0;
//                     key = seed), the blob exponents in FP64, their
//                     exponentials and the per-sample sums in float32 with
//                     every blob's weight kept in registers (NB >= blobs,
//                     fully unrolled), shell membership as in FP64 (a
//                     decision), and the means.  The higher SH coefficients
//                     are linear in the weights, so their mean is
//                     sum_k mean(w_k) h_k: the lane averages the NB weights
//                     and combines them with h once at the end (the same
//                     value as averaging the per-sample coefficients, in
//                     other rounding);
//   tree build        per level, bottom-up: run heads of the parent codes,
//                     a scan for the parents' positions, their compaction;
//                     then the child table, breadth-first, Morton order
//                     within a level.
#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <type_traits>
#include <vector>

#include "lq_internal.h"
#include "storage.h"

namespace lq {
namespace {

constexpr int kMaxBlobs = 32;
constexpr int kMaxShells = 8;
constexpr int kThreads = 256;
constexpr int kCentreThreads = 1024;         // of k_centre_bits
constexpr int kWordsPerChunk = 256;          // 64-bit occupancy words per chunk (16,384 voxels)
constexpr int kScanBlock = 1024;

// The field as kernel arguments: float32 copies for the samples, FP64 for
// the decisions (centre occupancy, shell membership).
struct FieldArgs {
    int nb, ns, K, pad;
    float cx[kMaxBlobs], cy[kMaxBlobs], cz[kMaxBlobs], inv2r2[kMaxBlobs], amp[kMaxBlobs];
    float cxl[kMaxBlobs], cyl[kMaxBlobs], czl[kMaxBlobs];     // centre = float32 + lower part
    float er[kMaxBlobs], eg[kMaxBlobs], eb[kMaxBlobs];
    float sx[kMaxShells], sy[kMaxShells], sz[kMaxShells], sr[kMaxShells];
    float sxl[kMaxShells], syl[kMaxShells], szl[kMaxShells];
    float log_base, sigma_max, l_max, half_width, threshold, pad2[3];
    double dcx[kMaxBlobs], dcy[kMaxBlobs], dcz[kMaxBlobs], dinv2r2[kMaxBlobs], damp[kMaxBlobs];
    double dsx[kMaxShells], dsy[kMaxShells], dsz[kMaxShells], dsr[kMaxShells];
    double dhalf_width, dthreshold;   // density(centre) >= prune  <=>  S >= dthreshold
};
static_assert(sizeof(FieldArgs) < 4000, "kernel argument space");

__device__ inline uint32_t compact3(uint32_t v) {   // every third bit, from bit 0
    v &= 0x09249249u;
    v = (v | (v >> 2)) & 0x030C30C3u;
    v = (v | (v >> 4)) & 0x0300F00Fu;
    v = (v | (v >> 8)) & 0x030000FFu;
    v = (v | (v >> 16)) & 0x000003FFu;
    return v;
}

// Shell membership, decided as in FP64: a float32 distance first (centres
// as a float32 pair, so each difference is within 2 ulp of its own value;
// positions and centres within [-2, 2]: the distance is off by under
// 2e-6), and FP64 only when its margin to a shell boundary is below 1e-5.
__device__ inline bool in_shell_f64(const FieldArgs &f, int j, double x, double y, double z) {
    const double dx = x - f.dsx[j], dy = y - f.dsy[j], dz = z - f.dsz[j];
    const double dist = sqrt(dx * dx + dy * dy + dz * dz);
    return fabs(dist - f.dsr[j]) < f.dhalf_width;
}

__device__ inline bool in_one_shell(const FieldArgs &f, int j, float xf, float yf, float zf, double x, double y,
                                    double z) {
    const float dx = (xf - f.sx[j]) - f.sxl[j], dy = (yf - f.sy[j]) - f.syl[j], dz = (zf - f.sz[j]) - f.szl[j];
    const float dist = __builtin_amdgcn_sqrtf(fmaf(dz, dz, fmaf(dy, dy, dx * dx)));
    const float m = fabsf(dist - f.sr[j]) - f.half_width;
    return fabsf(m) > 1e-5f ? m < 0.0f : in_shell_f64(f, j, x, y, z);
}

__device__ inline bool in_shell(const FieldArgs &f, double x, double y, double z) {
    const float xf = (float)x, yf = (float)y, zf = (float)z;
    bool in = false;
    for (int j = 0; j < f.ns; ++j) in = in || in_one_shell(f, j, xf, yf, zf, x, y, z);
    return in;
}

__device__ inline bool centre_kept_f64(const FieldArgs &f, double x, double y, double z) {
    double S = 0.0;
    for (int k = 0; k < f.nb; ++k) {
        const double dx = x - f.dcx[k], dy = y - f.dcy[k], dz = z - f.dcz[k];
        const double d2 = dx * dx + dy * dy + dz * dz;
        S += f.damp[k] * exp(-d2 * f.dinv2r2[k]);
    }
    return S >= f.dthreshold;
}

// The centre test, decided as in FP64: S in float32 first, FP64 only when
// S_32 lies within 4e-3 of the threshold.  Bound: voxel centres are exact
// in float32 and blob centres are float32 pairs, so every difference, the
// squared distance and lw = -d^2 / (2 r^2) carry under 6 ulp of relative
// error, and exp2 one more: each term a g is off by under
// |a| (6 |lw| + 2) 2^-24 <= |a| (6 / e + 2) 2^-24 (g |lw| <= 1 / e), under
// 1.1e-4 for 32 blobs of |a| <= 12; the running sum adds under
// 32 2^-24 sum |a| g <= 7.4e-4.
__device__ inline bool centre_kept(const FieldArgs &f, double x, double y, double z) {
    if (in_shell(f, x, y, z)) return true;
    const float xf = (float)x, yf = (float)y, zf = (float)z;
    float S = 0.0f;
    for (int k = 0; k < f.nb; ++k) {
        const float dx = (xf - f.cx[k]) - f.cxl[k], dy = (yf - f.cy[k]) - f.cyl[k], dz = (zf - f.cz[k]) - f.czl[k];
        const float d2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
        S = fmaf(f.amp[k], __builtin_amdgcn_exp2f(-d2 * f.inv2r2[k] * 1.4426950408889634f), S);
    }
    const float m = S - f.threshold;
    if (fabsf(m) > 4e-3f) return m >= 0.0f;
    return centre_kept_f64(f, x, y, z);
}

// The centre test for all 64 centres of an occupancy word (a cube of 4^3
// voxels) at once: 0 none is kept, 1 all are, -1 undecided.  x, y, z: the
// cube's centre; h: the voxel size.  A centre's distance to a point differs
// from the cube centre's by at most 1.5 sqrt(3) h, and by 1e-5 more for
// rounding (distances up to 7 in float32); with the nearest and farthest
// distance in place of its own, every Gaussian is bounded, and so is S.  The
// margin is that of centre_kept, whose error bound holds for both sums.
__device__ inline int word_kept(const FieldArgs &f, float x, float y, float z, float h) {
    const float r = 2.5980763f * h + 1e-5f;
    bool shell = false;
    for (int j = 0; j < f.ns; ++j) {
        const float dx = (x - f.sx[j]) - f.sxl[j], dy = (y - f.sy[j]) - f.syl[j], dz = (z - f.sz[j]) - f.szl[j];
        const float d = __builtin_amdgcn_sqrtf(fmaf(dz, dz, fmaf(dy, dy, dx * dx)));
        shell = shell || fabsf(d - f.sr[j]) <= f.half_width + r;
    }
    float lo = 0.0f, hi = 0.0f;
    for (int k = 0; k < f.nb; ++k) {
        const float dx = (x - f.cx[k]) - f.cxl[k], dy = (y - f.cy[k]) - f.cyl[k], dz = (z - f.cz[k]) - f.czl[k];
        const float d = __builtin_amdgcn_sqrtf(fmaf(dz, dz, fmaf(dy, dy, dx * dx)));
        const float near = fmaxf(d - r, 0.0f), far = d + r;
        const float q = -f.inv2r2[k] * 1.4426950408889634f;
        const float g0 = __builtin_amdgcn_exp2f(far * far * q), g1 = __builtin_amdgcn_exp2f(near * near * q);
        lo = fmaf(f.amp[k], f.amp[k] > 0.0f ? g0 : g1, lo);
        hi = fmaf(f.amp[k], f.amp[k] > 0.0f ? g1 : g0, hi);
    }
    if (lo - f.threshold > 4e-3f) return 1;
    return !shell && hi - f.threshold < -4e-3f ? 0 : -1;
}

// Occupancy of the voxels [chunk * kWordsPerChunk * 64, ...) in Morton
// order: bits[word] bit l = voxel 64 word + l kept; counts[chunk] = kept.
//
// Bound by VALU issue: every blob's Gaussian at every centre.  Most words lie
// wholly inside or outside, which two Gaussians per blob and word tell
// (word_kept, a lane per word); the block's 16 waves share the words left, a
// lane per voxel: sixteen, since most blocks have none left and some nearly
// all.  256^3, 16 blobs, 4 shells: 62 us (90 us with four waves, 222 us with
// every centre tested).
__global__ __launch_bounds__(kCentreThreads) void k_centre_bits(const FieldArgs f, int depth, uint64_t n_vox,
                                                          unsigned long long *bits, uint32_t *counts) {
    __shared__ uint32_t s_cnt, s_open;
    __shared__ uint32_t s_list[kWordsPerChunk];
    if (threadIdx.x == 0) s_cnt = s_open = 0;
    __syncthreads();
    const double h = 2.0 / (double)(1 << depth);
    const uint64_t first = (uint64_t)blockIdx.x * kWordsPerChunk;
    {
        const uint64_t word = first + threadIdx.x;
        const uint32_t c = (uint32_t)(word * 64);
        if (threadIdx.x < kWordsPerChunk && word * 64 < n_vox) {
            int kept = -1;
            if (n_vox >= 64)
                kept = word_kept(f, (float)(-1.0 + ((double)compact3(c) + 2.0) * h),
                                 (float)(-1.0 + ((double)compact3(c >> 1) + 2.0) * h),
                                 (float)(-1.0 + ((double)compact3(c >> 2) + 2.0) * h), (float)h);
            if (kept < 0) {
                s_list[atomicAdd(&s_open, 1u)] = threadIdx.x;
            } else {
                bits[word] = kept ? ~0ull : 0ull;
                if (kept) atomicAdd(&s_cnt, 64u);
            }
        }
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const uint32_t open = s_open;
    uint32_t cnt = 0;
    for (uint32_t it = threadIdx.x >> 6; it < open; it += kCentreThreads / 64) {
        const uint64_t word = first + s_list[it];
        const uint64_t code = word * 64 + lane;
        bool kept = false;
        if (code < n_vox) {
            const uint32_t c = (uint32_t)code;
            const double x = -1.0 + ((double)compact3(c) + 0.5) * h;
            const double y = -1.0 + ((double)compact3(c >> 1) + 0.5) * h;
            const double z = -1.0 + ((double)compact3(c >> 2) + 0.5) * h;
            kept = centre_kept(f, x, y, z);
        }
        const unsigned long long m = __ballot(kept);
        if (lane == 0) bits[word] = m;
        cnt += (uint32_t)__popcll(m);
    }
    if (lane == 0) atomicAdd(&s_cnt, cnt);
    __syncthreads();
    if (threadIdx.x == 0) counts[blockIdx.x] = s_cnt;
}

// Exclusive scan of n counts by one block; total in *total.
__global__ __launch_bounds__(kScanBlock) void k_scan_counts(const uint32_t *counts, uint32_t n, uint32_t *offsets,
                                                            uint32_t *total) {
    __shared__ uint32_t s[kScanBlock];
    const uint32_t per = (n + kScanBlock - 1) / kScanBlock;
    const uint32_t a = threadIdx.x * per, b = min(n, a + per);
    uint32_t sum = 0;
    for (uint32_t i = a; i < b; ++i) sum += counts[i];
    s[threadIdx.x] = sum;
    __syncthreads();
    for (int off = 1; off < kScanBlock; off <<= 1) {   // Hillis-Steele, inclusive
        const uint32_t v = threadIdx.x >= (unsigned)off ? s[threadIdx.x - off] : 0u;
        __syncthreads();
        s[threadIdx.x] += v;
        __syncthreads();
    }
    uint32_t run = s[threadIdx.x] - sum;
    for (uint32_t i = a; i < b; ++i) {
        offsets[i] = run;
        run += counts[i];
    }
    if (threadIdx.x == kScanBlock - 1) *total = s[kScanBlock - 1];
}

// Codes of the kept voxels of a chunk at its offset, ascending.  Writes
// only below cap (the caller's capacity).
__global__ __launch_bounds__(kWordsPerChunk) void k_centre_compact(const unsigned long long *bits, uint64_t n_words,
                                                                   const uint32_t *offsets, uint32_t *codes,
                                                                   uint64_t cap) {
    __shared__ uint32_t s[kWordsPerChunk];
    const uint64_t word = (uint64_t)blockIdx.x * kWordsPerChunk + threadIdx.x;
    const unsigned long long m = word < n_words ? bits[word] : 0ull;
    const uint32_t c = (uint32_t)__popcll(m);
    s[threadIdx.x] = c;
    __syncthreads();
    for (int off = 1; off < kWordsPerChunk; off <<= 1) {
        const uint32_t v = threadIdx.x >= (unsigned)off ? s[threadIdx.x - off] : 0u;
        __syncthreads();
        s[threadIdx.x] += v;
        __syncthreads();
    }
    uint64_t pos = (uint64_t)offsets[blockIdx.x] + s[threadIdx.x] - c;
    unsigned long long r = m;
    while (r) {
        const int bit = __ffsll(r) - 1;
        r &= r - 1;
        if (pos < cap) codes[pos] = (uint32_t)(word * 64 + bit);
        ++pos;
    }
}

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC 2011): 10 rounds of two
// 32x32 -> 64-bit multiplications with the key bumped by the Weyl constants.
// Each product is one 64-bit multiply (a single v_mad_u64_u32).
template <int ROUNDS>
__device__ inline void philox4x32_rounds(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1,
                                         uint32_t out[4]) {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        c0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1, k0, 0x96);   // three-way xor
        c1 = (uint32_t)p1;
        c2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3, k1, 0x96);
        c3 = (uint32_t)p0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0;
    out[1] = c1;
    out[2] = c2;
    out[3] = c3;
}

// One lane per kept voxel i < n: the means over n_samples positions.
// sh_out[i][c][k]; hi [nb][3][K - 1] (device, FP64).
//
// Precision: the exponent t_k = -log2(e) |x - c_k|^2 / (2 r_k^2) is taken in
// FP64 (full rate on this chip, like float32 without packing): a softmax
// weight depends on the absolute error of t_k - max_j t_j, and at points far
// from every blob (|t| in the hundreds, on the shells) float32 would leave
// relative errors of 1e-4 in the weights.  exp2, log2 and the per-sample
// sums are float32; the sums over samples run in blocks of kBlock samples
// (float32 inside a block, FP64 across blocks), and the higher coefficients
// sum_k mean(w_k) h_k are formed in FP64 once per voxel.
//
// The kernel is bound by VALU issue (about four cycles per wave instruction,
// transcendentals sixteen), so what it does per sample is kept down:
//  - CENTRED: the exponents are taken relative to their maximum at the voxel's
//    centre, m, as a_k |x|^2 + b_k . x + (C_k - m): five FP64 instructions per
//    blob instead of nine (differences, square, scale, maximum over the blobs,
//    difference to it).  The host takes this form when no exponent changes by
//    more than 7.5 within half a voxel diagonal: the terms that count then stay
//    below 8, whose rounding to float32 (2^-22) is about exp2's own error, where
//    an exponent relative to the sample's maximum loses nothing in its largest
//    terms (two weights at a change of 62, one sample: off by 9.4e-7, 1.2e-7 in
//    the other form).  Neither does exp2 overflow, and the terms that cancel in
//    FP64 stay far below 1e5.  m is rounded to a whole number, so 2^m is exact.
//    Otherwise the maximum is each sample's own.
//  - Philox: of counter (code, j, 0, 0), round 1's products and one of round
//    2's depend on the voxel or on j alone: the former are taken once per
//    voxel, the latter are scalar.
//  - Only the shells that a voxel of the wave can touch are tested.
//  - PRODUCT: the logarithms of up to four samples' DC terms are taken of
//    their product (three roundings of 2^-24 instead of three logarithms'
//    errors); the host takes this form when the products stay within range and
//    no radiance is above L_max / 2.  Otherwise each term has its own logarithm,
//    and L_max - E, which would cancel, is summed from the blobs' L_max - e_k
//    (one blob at L_max (1 - 2^-10): DC off by 4e-4 in the first form).
// 256^3, 882k voxels kept, 256 samples, 16 blobs, 4 shells: 2.0 ms (2.95 ms
// with nine FP64 instructions per blob, all shells tested, a logarithm per
// sample and the radiance sums sunk below the shell loop); VALU busy 97 %.
// (Taking the exponents and the sums over the blobs to the matrix cores, a
// wave per voxel, was slower, 3.16 ms: FP64 and float32 MFMA take the cycles
// of the FMAs they replace, and no VALU work ran beside them.)
//
// rec: NB records of four doubles -- CENTRED: b_k and a_k, else the centre and
// a_k = -log2(e) / (2 r_k^2) --, NB constant terms C_k, then NB float4 records
// (amplitude, radiance) and NB of (0, L_max - radiance); those past nb are padded so that their terms vanish
// (exp2 of a huge negative argument is exactly 0).  The records are read
// inside the sample loop through an offset the compiler cannot prove constant
// (zero is 0), so they arrive by scalar loads from cache each sample instead
// of being held across the loop, where they would overflow the scalar
// register file; groups of four blobs are separated by scheduling barriers so
// that the loads are not all issued at once.
constexpr int kBlock = 16;
constexpr int kProduct = 4;   // DC terms per logarithm
constexpr double kCentredChange = 7.5;

template <int NB, bool CENTRED, bool PRODUCT>
__global__ __launch_bounds__(kThreads, NB == 8 ? 5 : NB == 16 ? 4 : 2) void k_distill(const FieldArgs f, const double *__restrict__ rec,
                                                      uint32_t zero, const double *hi, int depth, int n_samples,
                                                      uint32_t key0, uint32_t key1,
                                                      const uint32_t *codes, uint64_t n, float *sigma_out,
                                                      float *sh_out) {
    const uint64_t i0 = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
    const bool mine = i0 < n;
    const uint64_t i = mine ? i0 : n - 1;    // lanes past the end repeat the last voxel
    const uint32_t code = codes[i];
    const double hd = 2.0 / (double)(1 << depth);
    const double hd24 = hd * 0x1p-24;
    const double lox = -1.0 + (double)compact3(code) * hd;
    const double loy = -1.0 + (double)compact3(code >> 1) * hd;
    const double loz = -1.0 + (double)compact3(code >> 2) * hd;
    constexpr float kLog2e = 1.4426950408889634f;
    constexpr float kLn2InvY00 = 0.69314718055994531f * 3.5449077018110318f;
    const float log_base2 = f.log_base * kLog2e;
    const double cx = lox + 0.5 * hd, cy = loy + 0.5 * hd, cz = loz + 0.5 * hd;
    double m = -INFINITY;         // CENTRED: the largest exponent at the centre
    if constexpr (CENTRED) {
        const double c2 = fma(cz, cz, fma(cy, cy, cx * cx));
        const double4 *qa = reinterpret_cast<const double4 *>(rec);
        const double *qc = reinterpret_cast<const double *>(qa + NB);
        for (int k = 0; k < f.nb; ++k) {
            const double4 a = qa[k];
            m = fmax(m, fma(a.x, cx, fma(a.y, cy, fma(a.z, cz, fma(a.w, c2, qc[k])))));
        }
        m = rint(m);              // 2^m exact
    }
    float scale = __builtin_amdgcn_exp2f((float)m) * kLog2e;
    // shells that a voxel of this wave may touch: its centre within half a
    // diagonal (and a margin) of the shell
    uint32_t shells = 0;
    for (int j = 0; j < f.ns; ++j) {
        const double dx = cx - f.dsx[j], dy = cy - f.dsy[j], dz = cz - f.dsz[j];
        const double dist = sqrt(dx * dx + dy * dy + dz * dz);
        if (__any(fabs(dist - f.dsr[j]) < f.dhalf_width + 0.87 * hd + 1e-6)) shells |= 1u << j;
    }
    // Philox round 1 leaves (j ^ key0, 0, hi(p0) ^ key1, lo(p0))
    const uint64_t p0 = (uint64_t)0xD2511F53u * code;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * ((uint32_t)(p0 >> 32) ^ key1);
    double wsum[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) wsum[k] = 0.0;
    double sig_sum = 0.0, dc0_sum = 0.0, dc1_sum = 0.0, dc2_sum = 0.0;
    for (int j0 = 0; j0 < n_samples; j0 += kBlock) {
        const int j1 = min(n_samples, j0 + kBlock);
        float wb[NB];
#pragma unroll
        for (int k = 0; k < NB; ++k) wb[k] = 0.0f;
        float sig_acc = 0.0f, dc0 = 0.0f, dc1 = 0.0f, dc2 = 0.0f;
        float n0 = 1.0f, n1 = 1.0f, n2 = 1.0f, d0 = 1.0f, d1 = 1.0f, d2 = 1.0f;
        for (int j = j0; j < j1; ++j) {
            const uint32_t jz = (uint32_t)j & zero;   // 0, opaque to the compiler
            const double4 *qa = reinterpret_cast<const double4 *>(rec) + jz;
            const double *qc = reinterpret_cast<const double *>(qa + NB);
            const float4 *qb = reinterpret_cast<const float4 *>(qc + NB);
            uint32_t u[4];
            {
                const uint32_t k0 = key0 + jz, k1 = key1 + jz;
                const uint64_t q0 = (uint64_t)0xD2511F53u * ((uint32_t)j ^ k0);   // scalar
                philox4x32_rounds<8>((uint32_t)(p1 >> 32) ^ (k0 + 0x9E3779B9u), (uint32_t)p1,
                                     (uint32_t)(q0 >> 32) ^ (uint32_t)p0 ^ (k1 + 0xBB67AE85u), (uint32_t)q0,
                                     k0 + 2u * 0x9E3779B9u, k1 + 2u * 0xBB67AE85u, u);
            }
            // the position exactly in FP64 (cell + offset: 34 bits)
            const double x = fma((double)(u[0] >> 8), hd24, lox);
            const double y = fma((double)(u[1] >> 8), hd24, loy);
            const double z = fma((double)(u[2] >> 8), hd24, loz);
            // t_k = log2 of blob k's Gaussian, relative to m
            double t[CENTRED ? 4 : NB];
            if constexpr (!CENTRED) {
                m = -INFINITY;
#pragma unroll
                for (int g = 0; g < NB; g += 4) {
#pragma unroll
                    for (int k = g; k < g + 4; ++k) {
                        const double4 a = qa[k];
                        const double dx = x - a.x, dy = y - a.y, dz = z - a.z;
                        t[k] = fma(dz, dz, fma(dy, dy, dx * dx)) * a.w;
                        m = fmax(m, t[k]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                scale = __builtin_amdgcn_exp2f((float)m) * kLog2e;
            }
            const double x2 = fma(z, z, fma(y, y, x * x));
            float e[NB];
            float s = 0.0f, sa = 0.0f, e0 = 0.0f, e1 = 0.0f, e2 = 0.0f;
            float r0 = 0.0f, r1 = 0.0f, r2 = 0.0f;   // L_max - E, of !PRODUCT
#pragma unroll
            for (int g = 0; g < NB; g += 4) {
#pragma unroll
                for (int k = g; k < g + 4; ++k) {
                    const float4 b = qb[k];
                    if constexpr (CENTRED) {
                        const double4 a = qa[k];
                        const double tk = fma(a.x, x, fma(a.y, y, fma(a.z, z, fma(a.w, x2, qc[k] - m))));
                        e[k] = __builtin_amdgcn_exp2f((float)tk);
                    } else {
                        e[k] = __builtin_amdgcn_exp2f((float)(t[k] - m));
                    }
                    s += e[k];
                    sa = fmaf(b.x, e[k], sa);
                    e0 = fmaf(b.y, e[k], e0);
                    e1 = fmaf(b.z, e[k], e1);
                    e2 = fmaf(b.w, e[k], e2);
                    if constexpr (!PRODUCT) {
                        const float4 c = qb[NB + k];
                        r0 = fmaf(c.y, e[k], r0);
                        r1 = fmaf(c.z, e[k], r1);
                        r2 = fmaf(c.w, e[k], r2);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // the sums belong here: sunk below the shells, they would keep every
            // blob's record in scalar registers until then
            asm volatile("" : "+v"(s), "+v"(e0), "+v"(e1), "+v"(e2));
            const float inv = __builtin_amdgcn_rcpf(s);
#pragma unroll
            for (int k = 0; k < NB; ++k) wb[k] = fmaf(e[k], inv, wb[k]);
            // density: exp(log_base + sum_k a_k g_k), sum_k a_k g_k = 2^m sa
            float sg = fminf(__builtin_amdgcn_exp2f(fmaf(scale, sa, log_base2)), f.sigma_max);
            if (shells) {
                const float xf = (float)x, yf = (float)y, zf = (float)z;
                for (uint32_t rest = shells; rest; rest &= rest - 1)
                    if (in_one_shell(f, __builtin_ctz(rest), xf, yf, zf, x, y, z)) sg = f.sigma_max;
            }
            sig_acc += sg;
            // DC: logit(E / L_max) / Y_00 = ln(E / (L_max - E)) 2 sqrt(pi),
            // E = e_c / s
            if constexpr (PRODUCT) {
                // both through the same rounded 1 / s, which so cancels
                n0 *= e0 * inv, n1 *= e1 * inv, n2 *= e2 * inv;
                d0 *= fmaf(f.l_max, s, -e0) * inv, d1 *= fmaf(f.l_max, s, -e1) * inv, d2 *= fmaf(f.l_max, s, -e2) * inv;
                if ((j & (kProduct - 1)) == kProduct - 1 || j + 1 == j1) {
                    dc0 = fmaf(__builtin_amdgcn_logf(n0 * __builtin_amdgcn_rcpf(d0)), kLn2InvY00, dc0);
                    dc1 = fmaf(__builtin_amdgcn_logf(n1 * __builtin_amdgcn_rcpf(d1)), kLn2InvY00, dc1);
                    dc2 = fmaf(__builtin_amdgcn_logf(n2 * __builtin_amdgcn_rcpf(d2)), kLn2InvY00, dc2);
                    n0 = n1 = n2 = d0 = d1 = d2 = 1.0f;
                }
            } else {
                dc0 = fmaf(__builtin_amdgcn_logf(e0 * __builtin_amdgcn_rcpf(r0)), kLn2InvY00, dc0);
                dc1 = fmaf(__builtin_amdgcn_logf(e1 * __builtin_amdgcn_rcpf(r1)), kLn2InvY00, dc1);
                dc2 = fmaf(__builtin_amdgcn_logf(e2 * __builtin_amdgcn_rcpf(r2)), kLn2InvY00, dc2);
            }
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) wsum[k] += (double)wb[k];
        sig_sum += (double)sig_acc;
        dc0_sum += (double)dc0;
        dc1_sum += (double)dc1;
        dc2_sum += (double)dc2;
    }
    if (!mine) return;
    // no ceiling: ln(E / infinity), where inf * 0 has entered the sums of L_max - e_k
    if (!PRODUCT && isinf(f.l_max)) dc0_sum = dc1_sum = dc2_sum = -INFINITY;
    const double invn = 1.0 / (double)n_samples;
    sigma_out[i] = (float)(sig_sum * invn);
    const int K = f.K;
    float *row = sh_out + i * (uint64_t)(3 * K);
    row[0] = (float)(dc0_sum * invn);
    row[K] = (float)(dc1_sum * invn);
    row[2 * K] = (float)(dc2_sum * invn);
    for (int c = 0; c < 3; ++c)
        for (int j = 1; j < K; ++j) {
            double acc = 0.0;
#pragma unroll
            for (int k = 0; k < NB; ++k)
                if (k < f.nb) acc = fma(wsum[k], hi[(k * 3 + c) * (K - 1) + (j - 1)], acc);
            row[c * K + j] = (float)(acc * invn);
        }
}

// ---- octree build (bottom-up collapse) ---------------------------------
// generic exclusive scan of n uint32 values (n < 2^31): block sums, one
// block scanning them, per-block scans plus the block's offset
__global__ __launch_bounds__(kScanBlock) void k_block_sums(const uint32_t *v, uint64_t n, uint32_t *sums) {
    __shared__ uint32_t s[kScanBlock];
    const uint64_t i = (uint64_t)blockIdx.x * kScanBlock + threadIdx.x;
    s[threadIdx.x] = i < n ? v[i] : 0u;
    __syncthreads();
    for (int off = kScanBlock / 2; off > 0; off >>= 1) {
        if (threadIdx.x < (unsigned)off) s[threadIdx.x] += s[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = s[0];
}

__global__ __launch_bounds__(kScanBlock) void k_block_scan(const uint32_t *v, uint64_t n, const uint32_t *block_off,
                                                           uint32_t *out) {
    __shared__ uint32_t s[kScanBlock];
    const uint64_t i = (uint64_t)blockIdx.x * kScanBlock + threadIdx.x;
    const uint32_t x = i < n ? v[i] : 0u;
    s[threadIdx.x] = x;
    __syncthreads();
    for (int off = 1; off < kScanBlock; off <<= 1) {
        const uint32_t y = threadIdx.x >= (unsigned)off ? s[threadIdx.x - off] : 0u;
        __syncthreads();
        s[threadIdx.x] += y;
        __syncthreads();
    }
    if (i < n) out[i] = block_off[blockIdx.x] + s[threadIdx.x] - x;
}

// run heads of the parent codes of a sorted level
__global__ void k_parent_heads(const uint32_t *kids, uint64_t n, uint32_t *head) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) head[i] = (i == 0 || (kids[i] >> 3) != (kids[i - 1] >> 3)) ? 1u : 0u;
}

// parents[pos[i]] = kids[i] >> 3 at run heads; pidx[i] = the parent's position
__global__ void k_parent_compact(const uint32_t *kids, uint64_t n, const uint32_t *head, const uint32_t *pos,
                                 uint32_t *parents, uint32_t *pidx) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t p = pos[i] + head[i] - 1u;   // inclusive count of heads, minus one
    pidx[i] = p;
    if (head[i]) parents[p] = kids[i] >> 3;
}

// codes strictly ascending and below 8^depth?  (flag set on a violation)
__global__ void k_check_codes(const uint32_t *codes, uint64_t n, uint64_t limit, uint32_t *bad) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (codes[i] >= limit || (i > 0 && codes[i] <= codes[i - 1])) atomicOr(bad, 1u);
}

// leaves: the leaf index of each kid, for the leaves' level (null: a level of nodes)
__global__ void k_child_write(const uint32_t *kids, uint64_t n, const uint32_t *pidx, int32_t base_parent,
                              int32_t base_kids, const uint32_t *leaves, int32_t *child) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t v = leaves ? -(int32_t)(leaves[i] + 1u) : base_kids + (int32_t)i;
    child[(uint64_t)(base_parent + (int32_t)pidx[i]) * 8u + (kids[i] & 7u)] = v;
}

// leaves that the sigma_min skip keeps, compared as stored
__global__ void k_kept_leaves(const float *sigma, uint64_t n, int storage, float sigma_min, uint32_t *kept) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) kept[i] = as_stored(storage, sigma[i]) >= sigma_min ? 1u : 0u;
}

__global__ void k_compact_leaves(const uint32_t *codes, uint64_t n, const uint32_t *kept, const uint32_t *pos,
                                 uint32_t *out_codes, uint32_t *out_leaf) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n || !kept[i]) return;
    out_codes[pos[i]] = codes[i];
    out_leaf[pos[i]] = (uint32_t)i;
}

__global__ void k_iota(uint32_t *p, uint64_t n) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = (uint32_t)i;
}

__global__ void k_fill_i32(int32_t *p, uint64_t n, int32_t v) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

lq_status dfail(lq_status s, const std::string &m) {
    set_error(m);
    return s;
}
lq_status dhip(hipError_t e, const char *what) {
    return dfail(LQ_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

// Device scratch, freed by release() or at scope exit (hipFree waits for the
// device).  Arrays are cut from blocks of at least 16 MiB: an allocation
// per array (56 for a depth-8 tree) took longer than the kernels between them.
// reuse(mark()) gives up the arrays made in between and keeps their blocks for
// the next ones, which only later work of the same stream may write.
struct DevBufs {
    static constexpr size_t kBlockBytes = (size_t)16 << 20;
    struct Block {
        char *p;
        size_t bytes;
    };
    struct Place {
        size_t next = 0;      // the first block that no array has been cut from
        char *at = nullptr;
        size_t left = 0;
    };
    std::vector<Block> blocks;
    Place here;
    DevBufs() = default;
    DevBufs(const DevBufs &) = delete;
    ~DevBufs() { release(); }
    Place mark() const { return here; }
    void reuse(const Place &m) { here = m; }
    void release() {
        for (const Block &b : blocks) (void)hipFree(b.p);
        blocks.clear();
        here = Place();
    }
    template <class T>
    hipError_t alloc(T **out, size_t count) {
        const size_t bytes = (std::max<size_t>(count, 1) * sizeof(T) + 255) & ~(size_t)255;
        *out = nullptr;
        if (bytes > here.left) {
            while (here.next < blocks.size() && blocks[here.next].bytes < bytes) ++here.next;
            if (here.next == blocks.size()) {
                void *q = nullptr;
                const size_t block = std::max(bytes, kBlockBytes);
                const hipError_t e = hipMalloc(&q, block);
                if (e != hipSuccess) {
                    (void)hipGetLastError();
                    return e;
                }
                blocks.push_back({static_cast<char *>(q), block});
            }
            here.at = blocks[here.next].p;
            here.left = blocks[here.next].bytes;
            ++here.next;
        }
        *out = reinterpret_cast<T *>(here.at);
        here.at += bytes;
        here.left -= bytes;
        return hipSuccess;
    }
};

// exclusive scan of v[0..n) into out (device), total on the host
hipError_t scan_u32(const uint32_t *v, uint64_t n, uint32_t *out, uint32_t *total_host, DevBufs &b, hipStream_t s) {
    const uint64_t nb = (n + kScanBlock - 1) / kScanBlock;
    uint32_t *sums, *offs, *tot;
    hipError_t e;
    if ((e = b.alloc(&sums, nb)) != hipSuccess || (e = b.alloc(&offs, nb)) != hipSuccess ||
        (e = b.alloc(&tot, 1)) != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_block_sums, dim3((unsigned)nb), dim3(kScanBlock), 0, s, v, n, sums);
    hipLaunchKernelGGL(k_scan_counts, dim3(1), dim3(kScanBlock), 0, s, sums, (uint32_t)nb, offs, tot);
    hipLaunchKernelGGL(k_block_scan, dim3((unsigned)nb), dim3(kScanBlock), 0, s, v, n, offs, out);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = hipMemcpyAsync(total_host, tot, 4, hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
    return hipStreamSynchronize(s);
}

constexpr unsigned kBuildThreads = 256;
dim3 build_grid(uint64_t m) {
    return dim3((unsigned)std::max<uint64_t>(1, (m + kBuildThreads - 1) / kBuildThreads));
}

// Child table (hipMalloc, the caller's) of the tree whose leaves are n
// ascending codes with leaf indices leaf[0..n): levels bottom-up, then the
// slots, breadth-first, Morton order within a level.
lq_status build_child(int max_depth, const uint32_t *codes, const uint32_t *leaf, uint64_t n, DevBufs &b,
                      hipStream_t s, int32_t **child, int64_t *n_nodes_out) {
    hipError_t e;
    *child = nullptr;
    std::vector<const uint32_t *> level(max_depth + 1, nullptr);
    std::vector<uint32_t *> pidx(max_depth + 1, nullptr);
    std::vector<uint64_t> count(max_depth + 1, 0);
    level[max_depth] = codes;
    count[max_depth] = n;
    for (int l = max_depth - 1; l >= 0; --l) {
        const uint64_t m = count[l + 1];
        if (m == 0) continue;
        uint32_t *head, *pos, *par, *pi;
        if ((e = b.alloc(&head, m)) != hipSuccess || (e = b.alloc(&pos, m)) != hipSuccess ||
            (e = b.alloc(&par, m)) != hipSuccess || (e = b.alloc(&pi, m)) != hipSuccess)
            return dfail(LQ_ERR_OOM, "device scratch of the octree build");
        hipLaunchKernelGGL(k_parent_heads, build_grid(m), dim3(kBuildThreads), 0, s, level[l + 1], m, head);
        uint32_t total = 0;
        if ((e = scan_u32(head, m, pos, &total, b, s)) != hipSuccess) return dhip(e, "scanning a level");
        hipLaunchKernelGGL(k_parent_compact, build_grid(m), dim3(kBuildThreads), 0, s, level[l + 1], m, head, pos, par,
                           pi);
        level[l] = par;
        pidx[l + 1] = pi;
        count[l] = total;
    }
    // the root always exists (level 0 holds code 0 when any leaf exists)
    count[0] = 1;
    std::vector<int64_t> base(max_depth + 1, 0);
    int64_t n_nodes = 0;
    for (int l = 0; l < max_depth; ++l) {
        base[l] = n_nodes;
        n_nodes += (int64_t)count[l];
    }
    if (n_nodes >= (1 << 29)) return dfail(LQ_ERR_UNSUPPORTED, "too many nodes");
    const uint64_t slots = (uint64_t)n_nodes * 8;
    if (hipMalloc((void **)child, slots * 4) != hipSuccess) {
        (void)hipGetLastError();
        *child = nullptr;
        return dfail(LQ_ERR_OOM, "device child table");
    }
    hipLaunchKernelGGL(k_fill_i32, build_grid(slots), dim3(kBuildThreads), 0, s, *child, slots, 0);
    for (int l = 0; l < max_depth; ++l) {
        const uint64_t m = count[l + 1];
        if (m == 0 || !pidx[l + 1]) continue;
        hipLaunchKernelGGL(k_child_write, build_grid(m), dim3(kBuildThreads), 0, s, level[l + 1], m, pidx[l + 1],
                           (int32_t)base[l], (int32_t)base[l + 1], l + 1 == max_depth ? leaf : nullptr, *child);
    }
    if ((e = hipGetLastError()) != hipSuccess) {
        (void)hipFree(*child);
        *child = nullptr;
        return dhip(e, "launching the octree build");
    }
    *n_nodes_out = n_nodes;
    return LQ_OK;
}

lq_status field_args(const lq_field_desc *fd, int depth, float prune_sigma, FieldArgs &f) {
    if (!fd) return dfail(LQ_ERR_INVALID_ARG, "field is NULL");
    if (fd->n_blobs < 1 || fd->n_blobs > kMaxBlobs) return dfail(LQ_ERR_UNSUPPORTED, "n_blobs must be in [1, 32]");
    if (fd->n_shells < 0 || fd->n_shells > kMaxShells) return dfail(LQ_ERR_UNSUPPORTED, "n_shells must be in [0, 8]");
    if (fd->sh_degree < 0 || fd->sh_degree > 4) return dfail(LQ_ERR_UNSUPPORTED, "sh_degree must be in [0, 4]");
    if (depth < 1 || depth > 10) return dfail(LQ_ERR_INVALID_ARG, "max_depth must be in [1, 10]");
    if (!(prune_sigma > 0.0f) || !std::isfinite(prune_sigma)) return dfail(LQ_ERR_INVALID_ARG, "prune_sigma must be > 0");
    if (!fd->blobs || (fd->n_shells && !fd->shells)) return dfail(LQ_ERR_INVALID_ARG, "field arrays are NULL");
    const int K = (fd->sh_degree + 1) * (fd->sh_degree + 1);
    if (K > 1 && !fd->blob_sh) return dfail(LQ_ERR_INVALID_ARG, "blob_sh is NULL");
    if (!(fd->l_max > 0.0) || !(fd->sigma_max > 0.0) || !std::isfinite(fd->log_density_base) ||
        !(fd->shell_half_width >= 0.0))
        return dfail(LQ_ERR_INVALID_ARG, "bad field scalars");
    memset(&f, 0, sizeof(f));
    f.nb = fd->n_blobs;
    f.ns = fd->n_shells;
    f.K = K;
    for (int k = 0; k < f.nb; ++k) {
        const double *b = fd->blobs + 8 * k;
        if (!(b[3] >= 1e-3 && b[3] <= 4.0) || !std::isfinite(b[0] + b[1] + b[2] + b[4]) || std::fabs(b[0]) > 2.0 ||
            std::fabs(b[1]) > 2.0 || std::fabs(b[2]) > 2.0 || std::fabs(b[4]) > 12.0)
            return dfail(LQ_ERR_INVALID_ARG,
                         "a blob needs a centre in [-2, 2]^3, a radius in [1e-3, 4] and |amplitude| <= 12");
        for (int c = 0; c < 3; ++c)
            if (!(b[5 + c] > 0.0) || !(b[5 + c] < fd->l_max))
                return dfail(LQ_ERR_INVALID_ARG, "blob radiance must be in (0, l_max)");
        const double inv = 1.0 / (2.0 * b[3] * b[3]);
        f.dcx[k] = b[0];
        f.dcy[k] = b[1];
        f.dcz[k] = b[2];
        f.dinv2r2[k] = inv;
        f.damp[k] = b[4];
        f.cx[k] = (float)b[0];
        f.cy[k] = (float)b[1];
        f.cz[k] = (float)b[2];
        f.cxl[k] = (float)(b[0] - (double)f.cx[k]);
        f.cyl[k] = (float)(b[1] - (double)f.cy[k]);
        f.czl[k] = (float)(b[2] - (double)f.cz[k]);
        f.inv2r2[k] = (float)inv;
        f.amp[k] = (float)b[4];
        f.er[k] = (float)b[5];
        f.eg[k] = (float)b[6];
        f.eb[k] = (float)b[7];
    }
    for (int j = 0; j < f.ns; ++j) {
        for (int a = 0; a < 4; ++a)
            if (!std::isfinite(fd->shells[4 * j + a]) || std::fabs(fd->shells[4 * j + a]) > 2.0)
                return dfail(LQ_ERR_INVALID_ARG, "shell centres and radii must lie in [-2, 2]");
        f.dsx[j] = fd->shells[4 * j];
        f.dsy[j] = fd->shells[4 * j + 1];
        f.dsz[j] = fd->shells[4 * j + 2];
        f.dsr[j] = fd->shells[4 * j + 3];
        f.sx[j] = (float)f.dsx[j];
        f.sy[j] = (float)f.dsy[j];
        f.sz[j] = (float)f.dsz[j];
        f.sr[j] = (float)f.dsr[j];
        f.sxl[j] = (float)(f.dsx[j] - (double)f.sx[j]);
        f.syl[j] = (float)(f.dsy[j] - (double)f.sy[j]);
        f.szl[j] = (float)(f.dsz[j] - (double)f.sz[j]);
    }
    f.dhalf_width = fd->shell_half_width;
    f.half_width = (float)fd->shell_half_width;
    f.dthreshold = log((double)prune_sigma) - fd->log_density_base;
    f.threshold = (float)f.dthreshold;
    f.log_base = (float)fd->log_density_base;
    f.sigma_max = (float)fd->sigma_max;
    f.l_max = (float)fd->l_max;
    return LQ_OK;
}


// Largest change of a blob's exponent t = -log2(e) |x - c|^2 / (2 r^2) from a
// voxel's centre to any point of it, over the whole box.
double exponent_change(const FieldArgs &f, int depth) {
    const double half = 0.8660254037844387 * 2.0 / (double)(1 << depth);   // half a voxel's diagonal
    double worst = 0.0;
    for (int k = 0; k < f.nb; ++k) {
        // farthest point of the box from the blob's centre
        const double x = 1.0 + std::fabs(f.dcx[k]), y = 1.0 + std::fabs(f.dcy[k]), z = 1.0 + std::fabs(f.dcz[k]);
        const double far = std::sqrt(x * x + y * y + z * z);
        worst = std::max(worst, 1.4426950408889634 * f.dinv2r2[k] * half * (2.0 * far + half));
    }
    return worst;
}

// Whether products of four factors E, of four factors L_max - E and of their
// quotients stay within 2^-100 .. 2^100, and L_max - E cancels no more than a
// bit; E, a mean of the blobs' radiances, lies between them (quotients between
// 2^-24 and 1).
bool dc_products_in_range(const FieldArgs &f) {
    float lo = f.l_max, hi = 0.0f;
    for (int k = 0; k < f.nb; ++k) {
        lo = std::min({lo, f.er[k], f.eg[k], f.eb[k]});
        hi = std::max({hi, f.er[k], f.eg[k], f.eb[k]});
    }
    return lo > 0x1p-24f * std::max(1.0f, f.l_max) && f.l_max < 0x1p24f && f.l_max > 0x1p-23f && hi <= 0.5f * f.l_max;
}

// The sample loop's blob records (layout at k_distill), as bytes.  Those past
// nb: far outside the field with a huge falloff, or a constant term alone, so
// that their exp2 terms are exactly 0; their amplitude and radiance are 0.
std::vector<unsigned char> blob_records(const lq_field_desc *fd, const FieldArgs &f, int NB,
                                        bool centred) {
    std::vector<unsigned char> r((size_t)NB * 72, 0);
    for (int k = 0; k < NB; ++k) {
        double q[4] = {1000.0, 1000.0, 1000.0, -1e300}, c = -1e300;
        float w[4] = {0.0f, 0.0f, 0.0f, 0.0f}, v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (centred) q[0] = q[1] = q[2] = q[3] = 0.0;
        if (k < f.nb) {
            const double a = -f.dinv2r2[k] * 1.4426950408889634;
            const double s = centred ? -2.0 * a : 1.0;
            q[0] = s * f.dcx[k], q[1] = s * f.dcy[k], q[2] = s * f.dcz[k];
            q[3] = a;
            c = a * (f.dcx[k] * f.dcx[k] + f.dcy[k] * f.dcy[k] + f.dcz[k] * f.dcz[k]);
            w[0] = f.amp[k], w[1] = f.er[k], w[2] = f.eg[k], w[3] = f.eb[k];
            for (int c = 0; c < 3; ++c) v[1 + c] = (float)(fd->l_max - fd->blobs[8 * k + 5 + c]);
        }
        memcpy(r.data() + 32 * k, q, 32);
        memcpy(r.data() + 32 * NB + 8 * k, &c, 8);
        memcpy(r.data() + 40 * NB + 16 * k, w, 16);
        memcpy(r.data() + 56 * NB + 16 * k, v, 16);
    }
    return r;
}

}  // namespace
}  // namespace lq

using namespace lq;

extern "C" {

lq_status lq_distill_leaves(const lq_field_desc *field, int32_t max_depth, float prune_sigma, int32_t n_samples,
                            uint64_t seed, int device, int64_t capacity, uint32_t *codes, float *sigma, float *sh,
                            int64_t *n_leaves, void *hip_stream) {
    if (!n_leaves) return dfail(LQ_ERR_INVALID_ARG, "n_leaves is NULL");
    *n_leaves = 0;
    FieldArgs f;
    lq_status st = field_args(field, max_depth, prune_sigma, f);
    if (st != LQ_OK) return st;
    if (n_samples < 1 || n_samples > (1 << 20)) return dfail(LQ_ERR_INVALID_ARG, "n_samples must be in [1, 2^20]");
    if (capacity < 0) return dfail(LQ_ERR_INVALID_ARG, "capacity must be >= 0");
    hipError_t e = hipSetDevice(device);
    if (e != hipSuccess) return dhip(e, "hipSetDevice");
    const int K = f.K;
    if (capacity > 0) {
        if ((st = check_device_array(codes, (size_t)capacity * 4, device, "codes")) != LQ_OK) return st;
        if ((st = check_device_array(sigma, (size_t)capacity * 4, device, "sigma")) != LQ_OK) return st;
        if ((st = check_device_array(sh, (size_t)capacity * 12 * K, device, "sh")) != LQ_OK) return st;
    }
    hipStream_t s = (hipStream_t)hip_stream;
    const uint64_t n_vox = 1ull << (3 * max_depth);
    const uint64_t n_words = (n_vox + 63) / 64;
    const uint64_t n_chunks = (n_words + kWordsPerChunk - 1) / kWordsPerChunk;
    DevBufs b;
    unsigned long long *bits;
    uint32_t *counts, *offs, *tot;
    double *d_hi = nullptr;
    if ((e = b.alloc(&bits, n_words)) != hipSuccess || (e = b.alloc(&counts, n_chunks)) != hipSuccess ||
        (e = b.alloc(&offs, n_chunks)) != hipSuccess || (e = b.alloc(&tot, 1)) != hipSuccess)
        return dfail(LQ_ERR_OOM, "device scratch of the distillation");
    if (K > 1) {
        const size_t nh = (size_t)f.nb * 3 * (K - 1);
        if ((e = b.alloc(&d_hi, nh)) != hipSuccess) return dfail(LQ_ERR_OOM, "device copy of blob_sh");
        if ((e = hipMemcpy(d_hi, field->blob_sh, nh * 8, hipMemcpyHostToDevice)) != hipSuccess)
            return dhip(e, "copying blob_sh");
    }
    hipLaunchKernelGGL(k_centre_bits, dim3((unsigned)n_chunks), dim3(kCentreThreads), 0, s, f, max_depth, n_vox, bits,
                       counts);
    hipLaunchKernelGGL(k_scan_counts, dim3(1), dim3(kScanBlock), 0, s, counts, (uint32_t)n_chunks, offs, tot);
    if ((e = hipGetLastError()) != hipSuccess) return dhip(e, "launching the centre test");
    uint32_t total = 0;
    if ((e = hipMemcpyAsync(&total, tot, 4, hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipStreamSynchronize(s)) != hipSuccess)
        return dhip(e, "the centre test");
    *n_leaves = total;
    if (capacity == 0 || total == 0) return LQ_OK;
    if ((int64_t)total > capacity) return dfail(LQ_ERR_INVALID_ARG, "more kept voxels than capacity (n_leaves set)");
    hipLaunchKernelGGL(k_centre_compact, dim3((unsigned)n_chunks), dim3(kWordsPerChunk), 0, s, bits, n_words, offs,
                       codes, (uint64_t)capacity);
    const unsigned nb = (unsigned)((total + kThreads - 1) / kThreads);
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    const bool product = dc_products_in_range(f);
    const bool centred = product && exponent_change(f, max_depth) <= kCentredChange;
    const int NB = f.nb <= 8 ? 8 : f.nb <= 16 ? 16 : 32;
    std::vector<unsigned char> rec = blob_records(field, f, NB, centred);
    double *d_rec;
    if ((e = b.alloc(&d_rec, rec.size() / 8)) != hipSuccess) return dfail(LQ_ERR_OOM, "device copy of the blobs");
    if ((e = hipMemcpy(d_rec, rec.data(), rec.size(), hipMemcpyHostToDevice)) != hipSuccess)
        return dhip(e, "copying the blobs");
    const auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(nb), dim3(kThreads), 0, s, f, d_rec, 0u, d_hi, max_depth, n_samples, k0, k1,
                           codes, (uint64_t)total, sigma, sh);
    };
    const auto form = [&](auto nb_tag) {
        constexpr int N = decltype(nb_tag)::value;
        if (centred) launch(k_distill<N, true, true>);
        else if (product) launch(k_distill<N, false, true>);
        else launch(k_distill<N, false, false>);
    };
    if (NB == 8) form(std::integral_constant<int, 8>());
    else if (NB == 16) form(std::integral_constant<int, 16>());
    else form(std::integral_constant<int, 32>());
    if ((e = hipGetLastError()) != hipSuccess) return dhip(e, "launching the distillation");
    // the scratch above is freed on return: wait for its last use
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return dhip(e, "the distillation");
    return LQ_OK;
}

lq_status lq_octree_from_leaves(int32_t max_depth, int32_t sh_degree, const uint32_t *codes, const float *sigma,
                                const float *sh, int64_t n_leaves, float l_max, float sigma_min, float alpha_max,
                                int storage, int device, lq_octree **out) {
    if (!out) return dfail(LQ_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (max_depth < 1 || max_depth > 10) return dfail(LQ_ERR_INVALID_ARG, "max_depth must be in [1, 10]");
    if (sh_degree < 0 || sh_degree > 4) return dfail(LQ_ERR_INVALID_ARG, "sh_degree must be in [0, 4]");
    if (n_leaves < 0 || n_leaves > (int64_t)1 << 30) return dfail(LQ_ERR_INVALID_ARG, "n_leaves out of range");
    hipError_t e = hipSetDevice(device);
    if (e != hipSuccess) return dhip(e, "hipSetDevice");
    const int K = (sh_degree + 1) * (sh_degree + 1);
    lq_status st;
    if (n_leaves > 0) {
        if ((st = check_device_array(codes, (size_t)n_leaves * 4, device, "codes")) != LQ_OK) return st;
        if ((st = check_device_array(sigma, (size_t)n_leaves * 4, device, "sigma")) != LQ_OK) return st;
        if ((st = check_device_array(sh, (size_t)n_leaves * 12 * K, device, "sh")) != LQ_OK) return st;
    }
    (void)hipGetLastError();   // what an earlier call of the program left is not this call's
    hipStream_t s = nullptr;
    DevBufs b;
    const uint64_t n = (uint64_t)n_leaves;
    if (n > 0) {
        uint32_t *bad;
        if ((e = b.alloc(&bad, 1)) != hipSuccess) return dfail(LQ_ERR_OOM, "device scratch");
        uint32_t hbad = 0;
        if ((e = hipMemcpy(bad, &hbad, 4, hipMemcpyHostToDevice)) != hipSuccess) return dhip(e, "scratch");
        hipLaunchKernelGGL(k_check_codes, build_grid(n), dim3(kBuildThreads), 0, s, codes, n, 1ull << (3 * max_depth),
                           bad);
        if ((e = hipMemcpy(&hbad, bad, 4, hipMemcpyDeviceToHost)) != hipSuccess) return dhip(e, "checking codes");
        if (hbad) return dfail(LQ_ERR_FORMAT, "codes must be strictly ascending Morton codes below 8^max_depth");
    }
    if (storage != LQ_F32 && storage != LQ_F16 && storage != LQ_BF16)
        return dfail(LQ_ERR_INVALID_ARG, "storage must be LQ_F32, LQ_F16 or LQ_BF16");
    if ((st = check_octree_scalars(l_max, sigma_min, alpha_max)) != LQ_OK) return st;
    // the full table, and the one without the leaves below sigma_min: the
    // same build over the leaves kept
    uint32_t *leaf, *kept, *pos, *kept_codes, *kept_leaf;
    if ((e = b.alloc(&leaf, n)) != hipSuccess || (e = b.alloc(&kept, n)) != hipSuccess ||
        (e = b.alloc(&pos, n)) != hipSuccess || (e = b.alloc(&kept_codes, n)) != hipSuccess ||
        (e = b.alloc(&kept_leaf, n)) != hipSuccess)
        return dfail(LQ_ERR_OOM, "device scratch of the octree build");
    uint32_t n_kept = 0;
    if (n > 0) {
        hipLaunchKernelGGL(k_iota, build_grid(n), dim3(kBuildThreads), 0, s, leaf, n);
        hipLaunchKernelGGL(k_kept_leaves, build_grid(n), dim3(kBuildThreads), 0, s, sigma, n, storage, sigma_min, kept);
        if ((e = scan_u32(kept, n, pos, &n_kept, b, s)) != hipSuccess) return dhip(e, "scanning the leaves");
        hipLaunchKernelGGL(k_compact_leaves, build_grid(n), dim3(kBuildThreads), 0, s, codes, n, kept, pos, kept_codes,
                           kept_leaf);
    }
    OctreeParts p{};
    int64_t n_nodes = 0, n_skip = 0;
    const DevBufs::Place leaves = b.mark();
    if ((st = build_child(max_depth, codes, leaf, n, b, s, &p.child, &n_nodes)) != LQ_OK) return st;
    b.reuse(leaves);
    if ((st = build_child(max_depth, kept_codes, kept_leaf, n_kept, b, s, &p.child_skip, &n_skip)) != LQ_OK) {
        (void)hipFree(p.child);
        return st;
    }
    p.max_depth = max_depth;
    p.sh_degree = sh_degree;
    p.n_nodes = (int32_t)n_nodes;
    p.n_skip_nodes = (int32_t)n_skip;
    p.n_leaves = (int32_t)n;
    p.l_max = l_max;
    p.sigma_min = sigma_min;
    p.alpha_max = alpha_max;
    p.sigma = sigma;
    p.sh = sh;
    // on a full card the scratch goes first (giving it back each time costs 0.5 ms
    // of 2.4 for 882k leaves: allocations that follow frees wait)
    p.make_room = [&] { b.release(); };
    return make_octree(p, storage, device, out);
}

}  // extern "C"
