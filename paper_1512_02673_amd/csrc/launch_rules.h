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

// Chunks per survivor set where `resident` workgroups run at once and each
// repeats its set's elimination, worth about 384 elements of the work: the count
// that fills some number of rounds of them at the least cost.
constexpr int64_t chunks_per_set(int64_t total, int64_t sets, int64_t resident) {
    const int64_t least = (sets + resident - 1) / resident;
    int64_t best = 1, best_cost = -1;
    for (int64_t rounds = least; rounds < least + 8; ++rounds) {
        const int64_t c = rounds * resident / sets > 1 ? rounds * resident / sets : 1;
        const int64_t cost = rounds * (384 + (total + c - 1) / c);
        if (best_cost < 0 || cost < best_cost) {
            best = c;
            best_cost = cost;
        }
    }
    return best;
}

// End of the chunk that starts at e0 < total (e0 + per may pass 2^31).
constexpr uint32_t chunk_end(uint32_t e0, uint32_t per, uint32_t total) {
    return e0 + (per < total - e0 ? per : total - e0);
}

// A launch counts the threads of each grid dimension modulo 2^32 and reports
// nothing: one of 2^32 or more would leave work undone.
constexpr bool grid_fits(int64_t blocks, int64_t threads) { return blocks <= ((int64_t(1) << 32) - 1) / threads; }

// Tiles of the fp32 products with several columns, by the workgroups that come
// out, column tiles counted: a launch that fills the 256 compute units gains
// nothing from smaller tiles and reads A once more for every one of them.
enum class ColumnTiles {
    kLongK4,     // 16 rows x 4 columns, 256 k a chunk, every column in one launch
    kShort4,     // 16 rows x 4 columns, 128 k a chunk, every column in one launch
    kShort16,    // 16 rows x 16 columns, 128 k a chunk, every column in one launch
    kWide32,     // 32 rows x 32 columns, every column in one launch
    kStream,     // 16 rows x up to 8 columns, or launches of 32 rows x 32 columns
};
// blocks16, blocks32: workgroups of 16 and of 32 row slots for one column tile.
// Measured with (20,16), (32,24) and (4,2) codes, rows of 512 to 8192 elements:
// - up to 4 columns: one workgroup a compute unit, 256 k a chunk (220, 2048 and
//   8192 elements: 9.1 and 25.0 us against 10.2 and 30.5 streamed; 260: 11.3 and
//   31.9 against 10.7 and 34.1).
// - up to 8: two column tiles while they fit that ((20,16), 62 workgroups each:
//   8.7 and 23.6 us, streamed 11.1 and 36.9), in chunks of 128 k up to 384
//   workgroups (376: 11.4 and 36.3, streamed 11.9 and 39.2; 498: 15.9 and 51.3
//   against 13.1 and 44.4).
// - more columns: with 2048 elements 16 x 16 tiles take 8.2 us for every 256
//   workgroups; 32 x 32 tiles, all columns in one launch, 33 us up to 256
//   workgroups and 22 + 0.0625 each above (260: 38, 384: 46, 520: 55, 1176: 98);
//   the same in proportion with 512 and 8192.  Launches of 32 columns are slower
//   in every case past one (12000 rows, 64 columns 78 against 60).
constexpr ColumnTiles column_tiles(int64_t blocks16, int64_t blocks32, int64_t s) {
    const int64_t tiles4 = (s + 3) / 4;
    if (tiles4 > 65535) return ColumnTiles::kStream;
    if (s <= 4) return blocks16 <= 256 ? ColumnTiles::kLongK4 : ColumnTiles::kStream;
    if (s <= 8)
        return blocks16 * tiles4 <= 192   ? ColumnTiles::kLongK4
               : blocks16 * tiles4 <= 384 ? ColumnTiles::kShort4
                                          : ColumnTiles::kStream;
    const int64_t small = blocks16 * ((s + 15) / 16), wide = blocks32 * ((s + 31) / 32);
    if (s <= 16) return small <= 768 ? ColumnTiles::kShort16 : ColumnTiles::kStream;
    if (blocks16 > 768) return ColumnTiles::kStream;
    const bool quicker = wide <= 256 ? small <= 768 : 140 * ((small + 255) / 256) < 350 + wide;
    return quicker ? ColumnTiles::kShort16 : ColumnTiles::kWide32;
}

// Bytes of A and of the parity planes a code holds for it: `size` bytes an
// element, `parity_size` for a parity element of every plane.
constexpr int64_t operand_bytes(int64_t q, int64_t r, int64_t qb, int64_t parity_workers, int64_t size, int64_t parity_size) {
    return (q * size + parity_workers * qb * parity_size) * r;
}

// Loads of A and the planes: non-temporal when what a caller goes through before
// it returns to the same bytes (every worker's block, and every matrix of an
// iteration) does not fit the 256 MB memory-side cache, whatever part of it one
// launch reads; plain loads while it fits, where the next call finds it.
constexpr bool streams(int64_t bytes) { return bytes > (int64_t(256) << 20); }

// Survivor sets per launch.  The sets of a larger batch take one chunk each, so
// a launch of 512-thread workgroups stays at half of what a grid takes.
constexpr int64_t kSetsPerLaunch = int64_t(1) << 22;

}  // namespace coded
