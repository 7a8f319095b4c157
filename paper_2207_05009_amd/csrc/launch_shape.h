// launch_shape.h -- how launches are sized (host arithmetic, plain C++).
#pragma once

#include <stdint.h>

#include <map>
#include <mutex>
#include <utility>

namespace lq {

// Blocks of kStreamThreads for a kernel that strides over n items.  A launch of
// 2^32 threads or more in a dimension is not refused: the count wraps and the
// rest of the items is left out.  The largest trees hold that many words (a
// float32 leaf of SH degree 4 has 128, so 2^25 leaves do): at most kStreamBlocks,
// each thread then taking several items.  All tables up to 2^30 words keep a
// thread per word.
constexpr unsigned kStreamThreads = 256;
constexpr unsigned kStreamBlocks = 1u << 22;
inline unsigned stream_blocks(uint64_t n) {
    const uint64_t blocks = n / kStreamThreads + (n % kStreamThreads != 0);
    return (unsigned)(blocks < 1 ? 1 : blocks > kStreamBlocks ? kStreamBlocks : blocks);
}

// Leaves per slice for work that goes through a tree's leaves with scratch of
// `bytes` per leaf, so that a large tree does not need as much again: 64 MiB, a
// few milliseconds of copying to the host, beside which a launch per slice does
// not count.
constexpr uint64_t kSliceBytes = (uint64_t)64 << 20;
inline uint64_t slice_leaves(uint64_t leaves, uint64_t bytes) {
    const uint64_t fit = kSliceBytes / bytes;
    return leaves < 1 ? 1 : fit < leaves ? fit : leaves;
}

// Blocks of a kernel that a device holds at once.  ask() finds them, once per
// device and kernel: kernels of one signature have register budgets of their own
// (a 3-wave kernel's blocks would leave a 5-wave one's launch under-filled).
class ResidentBlocks {
public:
    template <class Ask>
    int get(int device, const void *kernel, Ask ask) {
        std::lock_guard<std::mutex> lock(mu_);
        const auto key = std::make_pair(device, kernel);
        const auto it = known_.find(key);
        return it != known_.end() ? it->second : known_[key] = ask();
    }

private:
    std::mutex mu_;
    std::map<std::pair<int, const void *>, int> known_;
};

// First position of range x when a launch splits n positions into `ranges`
// (range x ends where x + 1 begins): multiples of `unit`, so that reservations
// of `unit` positions within a range start on them too.
constexpr int64_t range_begin(int x, int ranges, int64_t n, int64_t unit) {
    return x >= ranges ? n : n / unit * x / ranges * unit;
}

}  // namespace lq
