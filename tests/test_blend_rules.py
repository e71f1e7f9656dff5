"""The host's choice of blend kernels by sizes (blend_rules.hpp), on the CPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = """
#include <stdio.h>
#include <string.h>
#include "blend_rules.hpp"
using namespace megs;
int main() {
    char kind[16];
    int tile;
    long long n_tiles, records, pairs;
    while (scanf("%15s %d %lld %lld %lld", kind, &tile, &n_tiles, &records, &pairs) == 5) {
        if (!strcmp(kind, "order")) {
            printf("%d\\n", (int)orders_tiles_fwd(tile, n_tiles, pairs));
            continue;
        }
        const BlendKind k = !strcmp(kind, "fwd") ? kBlendForward : !strcmp(kind, "imp") ? kBlendImportance : kBlendBackward;
        printf("%d\\n", (int)blends_by_sub_tile(k, tile, n_tiles, records, pairs));
    }
}
"""

CASES = [
    # one launch holds 2^32 threads, 64 of them for a sub-tile: seventeen views of 16384 x 16384 do not fit
    ("fwd", 16, 1 << 24, 10, 1 << 31, False), ("fwd", 16, (1 << 24) - 1, 10, 1 << 31, True),
    ("fwd", 32, 1 << 22, 10, 1 << 31, False), ("fwd", 32, 17 << 18, 10, 1 << 31, False), ("bwd", 32, 17 << 18, 1 << 30, 1 << 31, False),
    ("fwd", 32, (1 << 22) - 1, 10, 1 << 31, True),
    # small launches, and ordinary ones: a 979 x 546 and a 1080p view, eight of them
    ("bwd", 16, 2048, 3, 2048 * 3, True), ("imp", 32, 512, 3, 512 * 3, True), ("fwd", 32, 512, 1, 1, True),
    ("fwd", 16, 8160, 1_000_000, 2_000_000, True), ("bwd", 16, 8160, 1_000_000, 2_000_000, True),
    ("imp", 32, 4 * 920, 800_000, 1_500_000, True), ("bwd", 32, 8 * 2040, 8_000_000, 10_000_000, True),
    # short lists of 32 x 32 tiles
    ("fwd", 32, 16384, 5000, 16 * 16384 - 1, False), ("fwd", 32, 16384, 5000, 16 * 16384, True),
    ("imp", 32, 16384, 50_000, 100_000, False), ("fwd", 16, 65536, 256, 1000, True), ("bwd", 32, 16384, 50_000, 100_000, True),
    ("fwd", 32, 130_560, 50_000, 40 * 130_560 - 1, False), ("fwd", 32, 130_560, 50_000, 40 * 130_560, True),
    # few records that cover many sub-tiles
    ("bwd", 16, 8160, 3000, 200 * 3000 - 1, True), ("bwd", 16, 8160, 3000, 200 * 3000, False), ("fwd", 16, 8160, 3000, 200 * 3000, True),
    ("bwd", 32, 2040, 3000, 50 * 3000, False), ("bwd", 32, 2040, 8160, 200 * 8160, True), ("imp", 16, 8160, 3000, 200 * 3000, True),
    ("imp", 32, 2040, 3000, 50 * 3000 - 1, True), ("imp", 32, 2040, 3000, 50 * 3000, False),
    ("imp", 32, 16320, 24_000, 34 * 24_000, False), ("bwd", 32, 16320, 24_000, 34 * 24_000, True),
    ("fwd", 16, 1, 0, 0, True), ("bwd", 16, 100_000, 0, 0, False),
    # the forward's tile order: from 12,289 sub-tiles on, to 16,384 tiles of 16 x 16; of 32 x 32 beyond 65,536 with long lists
    ("order", 8, 20_000, 0, 1 << 20, False), ("order", 16, 3072, 0, 0, False), ("order", 16, 3073, 0, 0, True),
    ("order", 16, 16384, 0, 0, True), ("order", 16, 16385, 0, 1 << 30, False), ("order", 32, 768, 0, 0, False),
    ("order", 32, 769, 0, 0, True), ("order", 32, 65536, 0, 0, True), ("order", 32, 65537, 0, 8 * 65537 - 1, False),
    ("order", 32, 65537, 0, 8 * 65537, True),
]


def test_choice_by_sizes(tmp_path):
    src, exe = tmp_path / "rules.cpp", str(tmp_path / "rules")
    src.write_text(CODE)
    r = subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2509_07021_amd", "csrc"), str(src),
                        "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    text = "".join(" ".join(map(str, c[:5])) + "\n" for c in CASES)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=60).stdout.split()
    assert [(c, bool(int(o))) for c, o in zip(CASES, out)] == [(c, c[5]) for c in CASES] and len(out) == len(CASES)
