// blend_rules.hpp -- which of its kernels a blend runs, by sizes that the host knows before it launches. Host code
// only, without HIP.
#pragma once
#include <stdint.h>

namespace megs {

constexpr int64_t sub_tiles(int tile, int64_t n_tiles) { return n_tiles * (tile / 8) * (tile / 8); }

// Does a sub-tile blend (unless persistent) run its tiles by list length, given memory for the order? The limits
// are measured where the order is made (with_order, blend.hip).
constexpr int64_t kOrderItemsFwd = 12288, kOrderTilesFwd16 = 16384;
constexpr int64_t kOrderItemsBwd = 8192, kOrderTilesBwd = 65536;
constexpr bool orders_tiles_fwd(int tile, int64_t n_tiles) {
    return tile > 8 && (tile == 32 || n_tiles <= kOrderTilesFwd16) && sub_tiles(tile, n_tiles) > kOrderItemsFwd;
}
// `pairs` is the pair table's capacity. Above 65,536 tiles, where most of them are empty or nearly, the waves only pay
// for looking up the order: a 16384 x 16384 image in 32 x 32 tiles with 0.04 / 0.7 pairs a tile 1.56 and 2.45 / 2.07 and
// 2.59 ms without and with it.
constexpr bool orders_tiles_fwd(int tile, int64_t n_tiles, int64_t pairs) {
    return orders_tiles_fwd(tile, n_tiles) && (n_tiles <= 65536 || pairs >= 8 * n_tiles);
}
constexpr bool orders_tiles_bwd(int tile, int64_t n_tiles) {
    return tile > 8 && n_tiles <= kOrderTilesBwd && sub_tiles(tile, n_tiles) > kOrderItemsBwd;
}

// Does a launch with waves = 0 (the library's choice) of 16 x 16 or 32 x 32 tiles blend per sub-tile? The per-tile
// kernels give the same images, bit for bit, and take their place where they are faster, or where the sub-tiles are
// more than one launch can hold (2^32 threads). `pairs` is the pair table's capacity. Measured (waves = 4 and
// sub-tiles, us):
//  - Forward of 32 x 32 tiles with short lists: sixteen waves start for each tile instead of four, and a
//    launch of hundreds of thousands of them is bound by that. 4096 x 4096 with 0.1 / 11 / 17 / 67 pairs a tile 53 and
//    135 / 162 and 196 / 182 and 189 / 856 and 674; 16 x 4K with 8 / 18 / 41 pairs 926 and 1395 / 1230 and 1459 / 3665 and
//    3382; 1080p with 0.2 / 5 pairs 13 and 26 / 30 and 28. (16 x 16 tiles: 1080p with 0.1 / 2 / 8 pairs 16 and 28 / 22 and
//    29 / 51 and 34, 16 x 4K with 0.1 pairs 1320 and 870: sub-tiles throughout, since a scene of few pairs may hold
//    them all in a few long lists, which the per-tile kernels take several times as long for.)
//  - Backward of few records that each cover many sub-tiles: every sub-tile's sums go to the same few addresses, one
//    atomic after the other, where a tile's workgroup adds its waves' sums first. 100 records over a 979 x 546 image
//    108 and 331, 300 over 1080p 348 and 1063 (16 x 16), 3,000 over 1080p that cover 370 tiles of 32 x 32 each 476 and 688,
//    34 each 528 and 246; 20,000 records that cover 63 each 430 and 225.
//  - Importance with 32 x 32 tiles: the same of its one sum (300 records over 979 x 546 528 and 1121, 3,000 over 1080p
//    that cover 193 tiles 814 and 1095; of eight 1080p views at 34 tiles 941 and 1964, of one 340 and 248).
enum BlendKind { kBlendForward, kBlendImportance, kBlendBackward };
constexpr int64_t kSubTileLaunch = (int64_t)1 << 26;  // sub-tiles, one wave64 each, below 2^32 threads
constexpr bool blends_by_sub_tile(BlendKind kind, int tile, int64_t n_tiles, int64_t records, int64_t pairs) {
    const int64_t items = sub_tiles(tile, n_tiles), per_tile = items / (n_tiles > 0 ? n_tiles : 1);
    if (items >= kSubTileLaunch) return false;
    if (items <= 8192) return true;  // small launches: sub-tiles win, or lose a few us
    const int64_t sparse = items / 16384 < 40 ? items / 16384 : 40;
    if (kind != kBlendBackward && tile == 32 && pairs < sparse * n_tiles) return false;
    const int64_t cover = kind == kBlendImportance && items > 65536 ? 200 : 800;  // sub-tiles a record covers
    const bool crowded = records < items / 4 && per_tile * pairs >= cover * records;
    return !(crowded && (kind == kBlendBackward || (kind == kBlendImportance && tile == 32)));
}

}  // namespace megs
