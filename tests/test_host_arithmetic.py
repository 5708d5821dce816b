"""Index and size arithmetic that kernels and launches share, compiled for the host
from the library's own headers with the undefined-behaviour sanitizer and run."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1512_02673_amd", "csrc")


def run_host(tmp_path, source):
    """Compile a host program against csrc/ and run it; a failed check or undefined behaviour ends it with an error."""
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text("#include <cstdint>\n#include <cstdio>\n#include <cstdlib>\n#include <initializer_list>\n"
                   "#define CHECK(c, ...) do { if (!(c)) { std::printf(__VA_ARGS__); std::exit(1); } } while (0)\n" + source)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", f"-I{CSRC}",
                    str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr


def test_bits_below_every_position(tmp_path):
    """Every position of 0 .. 128 (128: the whole mask, the place of k in a code of 128 blocks)."""
    run_host(tmp_path, r"""
#include "survivor_mask.h"
int main() {
    const uint64_t masks[][2] = {{~0ull, ~0ull}, {0, 0}, {1, 1ull << 63}, {~0ull, 1}, {0x8000000000000001ull, ~0ull},
                                 {0x0123456789abcdefull, 0xfedcba9876543210ull}};
    for (const auto& m : masks)
        for (int i = 0; i <= 128; ++i) {
            int want = 0;
            for (int b = 0; b < i; ++b) want += (m[b / 64] >> (b % 64)) & 1;
            const int got = coded::bits_below(m[0], m[1], i);
            CHECK(got == want, "bits below %d: %d, not %d\n", i, got, want);
        }
}
""")


def test_chunks_cover_their_range(tmp_path):
    """Chunks meet end to end and end with the range, up to the longest one (2^31 - 1
    elements); the tile loops' steps of 256 past an end stay in 32 bits."""
    run_host(tmp_path, r"""
#include "launch_rules.h"
int main() {
    const int64_t totals[] = {1, 63, 64, 65, 4096, 32768 + 5, (1ll << 30) + 1, (1ll << 31) - 16384, (1ll << 31) - 2, (1ll << 31) - 1};
    const int64_t wants[] = {1, 2, 500, 512, 1024};
    const int64_t units[] = {16, 32};
    for (int64_t total : totals) for (int64_t want : wants) for (int64_t unit : units) {
        const auto c = coded::split_chunks(total, want, unit);
        CHECK(c.per % unit == 0 && c.per >= 64 && c.count <= want, "split of %lld\n", static_cast<long long>(total));
        int64_t at = 0;
        for (int64_t i = 0; i < c.count; ++i) {
            const uint32_t e0 = static_cast<uint32_t>(i) * static_cast<uint32_t>(c.per);
            CHECK(e0 == at && at < total, "chunk %lld of %lld starts at %u\n", static_cast<long long>(i), static_cast<long long>(total), e0);
            const uint32_t e1 = coded::chunk_end(e0, static_cast<uint32_t>(c.per), static_cast<uint32_t>(total));
            CHECK(e1 > e0 && e1 <= total, "chunk %lld of %lld ends at %u\n", static_cast<long long>(i), static_cast<long long>(total), e1);
            CHECK(static_cast<uint32_t>(e1 + 256 + 31) > e1, "tile steps past %u\n", e1);
            at = e1;
        }
        CHECK(at == total, "%lld of %lld covered\n", static_cast<long long>(at), static_cast<long long>(total));
    }
}
""")


def test_grids_stay_below_2_32_threads(tmp_path):
    """Launches of the largest part of a batch, and the limit itself."""
    run_host(tmp_path, r"""
#include "launch_rules.h"
int main() {
    for (int threads : {64, 256, 512, 1024}) {
        const int64_t most = ((1ll << 32) - 1) / threads;
        CHECK(coded::grid_fits(most, threads) && most * threads < (1ll << 32), "%d threads\n", threads);
        CHECK(!coded::grid_fits(most + 1, threads) && !coded::grid_fits(1ll << 62, threads), "%d threads\n", threads);
    }
    for (int64_t batch : {coded::kSetsPerLaunch, coded::kSetsPerLaunch - 1, int64_t(1000), int64_t(600), int64_t(1)})
        for (int64_t total : {int64_t(1), int64_t(1000), (int64_t(1) << 31) - 1})
            for (int64_t resident : {int64_t(256), int64_t(512)}) {
                const auto c = coded::split_chunks(total, (1024 + batch - 1) / batch, 16);
                CHECK(coded::grid_fits(c.count * batch, 512), "%lld sets of %lld\n", static_cast<long long>(batch), static_cast<long long>(total));
                const int64_t per_set = coded::chunks_per_set(total, batch, resident);
                const auto w = coded::split_chunks(total, per_set, 32);
                CHECK(per_set >= 1 && coded::grid_fits(w.count * batch, 512), "%lld wide sets of %lld\n", static_cast<long long>(batch), static_cast<long long>(total));
                // no round is left nearly empty while a set could be cut
                const int64_t blocks = per_set * batch, rounds = (blocks + resident - 1) / resident;
                CHECK(batch != 600 || total < 10000 || blocks * 10 >= rounds * resident * 9, "600 sets of %lld: %lld workgroups\n", static_cast<long long>(total), static_cast<long long>(blocks));
            }
}
""")


def test_column_tiles_count_the_columns(tmp_path):
    """The small tiles of the fp32 products re-read A once per column tile: they are for launches
    whose workgroups, column tiles counted, leave compute units idle."""
    run_host(tmp_path, r"""
#include "launch_rules.h"
using namespace coded;
int main() {
    const int codes[][2] = {{20, 16}, {4, 2}, {3, 2}, {64, 48}, {128, 96}, {10, 10}};
    for (const auto& c : codes) for (int64_t qb : {1, 8, 16, 17, 40, 80, 83, 125, 200, 250, 300, 333, 600, 1333, 1400, 5000, 100000})
        for (int64_t s : {2, 4, 5, 8, 9, 16, 17, 32, 33, 64, 96, 200, 1000, 300000}) {
            const int64_t k = c[1], p = c[0] - c[1];
            const int64_t rows = k * ((qb + 15) / 16) + p * ((qb + 7) / 8), rows32 = k * ((qb + 31) / 32) + p * ((qb + 15) / 16);
            const auto t = column_tiles(rows, rows32, s);
            const int64_t n4 = rows * ((s + 3) / 4), n16 = rows * ((s + 15) / 16);
            auto check = [&](bool ok) { CHECK(ok, "(%d,%d) qb %ld s %ld\n", c[0], c[1], (long)qb, (long)s); };
            if (t == ColumnTiles::kLongK4) check(s <= 8 && n4 <= 256);
            if (t == ColumnTiles::kShort4) check(s > 4 && s <= 8 && n4 <= 384);
            if (t == ColumnTiles::kShort16) check(s > 8 && (n16 <= 768 || (s > 16 && 35 * n16 <= 64 * (350 + rows32 * ((s + 31) / 32)))));
            if (t == ColumnTiles::kWide32) check(s > 16 && (s + 31) / 32 <= 65535);
            if (rows > 768) check(t == ColumnTiles::kStream);
            if (s > 8 && s <= 300 && n16 <= 768) check(t == ColumnTiles::kShort16);
        }
}
""")


def test_cache_policy_takes_the_whole_operands(tmp_path):
    """Every worker's block and plane counts, whichever of them a launch reads: one worker of
    65536 x 8192 reads 179 MB, the 16 of them 3.6 GB."""
    run_host(tmp_path, r"""
#include "launch_rules.h"
using namespace coded;
int main() {
    const int64_t qb = (65536 + 11) / 12;
    const int64_t all = operand_bytes(65536, 8192, qb, 4, 4, 8);
    CHECK(all == 65536ll * 8192 * 4 + 4 * qb * 8192 * 8 && streams(all), "%ld\n", (long)all);
    CHECK(qb * 8192 * 4 < (256ll << 20), "one worker alone would not stream\n");
    CHECK(operand_bytes(10, 7, 5, 2, 4, 6) == 10 * 7 * 4 + 2 * 5 * 7 * 6, "a bfloat16 lo plane\n");
    CHECK(operand_bytes(10, 7, 5, 0, 2, 4) == 10 * 7 * 2, "no parity workers\n");
    CHECK(!streams(256ll << 20) && streams((256ll << 20) + 1), "the cache's size\n");
}
""")
