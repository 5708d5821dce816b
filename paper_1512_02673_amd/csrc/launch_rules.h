// How launches split their work: plain C++ on sizes, so the host checks run the
// same code.
#pragma once
#include <cstdint>

namespace coded {

// A range of `total` < 2^31 elements in chunks of `per` (a multiple of `unit`),
// about `want` of them, of at least 64 elements each.
struct Chunks {
    int64_t per, count;
};
constexpr Chunks split_chunks(int64_t total, int64_t want, int64_t unit) {
    const int64_t n = total > 1 ? total : 1, w = want > 1 ? want : 1;
    const int64_t even = ((n + w - 1) / w + unit - 1) / unit * unit;
    const int64_t per = even > 64 ? even : 64;
    return {per, (n + per - 1) / per};
}

// End of the chunk that starts at e0 < total (e0 + per may pass 2^31).
constexpr uint32_t chunk_end(uint32_t e0, uint32_t per, uint32_t total) {
    return e0 + (per < total - e0 ? per : total - e0);
}

// A launch counts the threads of each grid dimension modulo 2^32 and reports
// nothing: one of 2^32 or more would leave work undone.
constexpr bool grid_fits(int64_t blocks, int64_t threads) { return blocks <= ((int64_t(1) << 32) - 1) / threads; }

// Survivor sets per launch.  The sets of a larger batch take one chunk each, so
// a launch of 512-thread workgroups stays at half of what a grid takes.
constexpr int64_t kSetsPerLaunch = int64_t(1) << 22;

}  // namespace coded
