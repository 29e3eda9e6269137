// Tiles of the grouped expert kernels: their heights and how many a launch may have.  Plain host code, no HIP.
#pragma once
#include <stdint.h>

namespace kmoe {

constexpr int kRowBlk = 32;        // rows (tokens) per MFMA block
constexpr int kTileLg = 3, kTileBlks = 1 << kTileLg;     // row blocks per tile (256 rows), at most
constexpr int kShortLg = 1, kShortBlks = 1 << kShortLg;  // the same for small batch groups (see short_tiles)

// Tiles of two row blocks instead of eight: such a tile's accumulators and activation stages leave
// room for two workgroups per compute unit, so that one streams weights while the other starts or
// stores, and the last round of workgroups costs half as much; but a workgroup's weight ring is half
// as deep, and an expert of more than 64 rows is several tiles that share its weights through L2.
//
// Layer times, tall / short, over rows per expert r (even routing unless stated):
//   bf16, no shared experts: 16 x 4096 x 14336: r 1 634 / 685 us, r 48 916 / 956, r 64 954 / 1340;
//     64 x 2048 x 1408: r 4 230 / 233, r 48 254 / 262, r 64 272 / 331: never short.
//   bf16, shared experts (a row per token: the tallest of an uneven launch), 64 + 2 x 2048 x 1408: 16
//     tokens 172 / 178 us, 170 256 / 253, 341 288 / 285, 512 (r 48) 312 / 293, 682 (r 64) 362 / 342, 2048 463 / 714;
//     skewed routing 128 tokens 261 / 255, 256 296 / 286, 512 376 / 330; 64 + 2 x 5120 x 1536: 341 tokens 673 /
//     661, 512 761 / 690, 682 818 / 959; 160 + 2 x 2048 x 1408: 106 tokens 536 / 562, 853 (r 32) 669 / 673, 1280 (r
//     48) 765 / 692, 2560 (r 96) 873 / 1055; 16 experts (4096 x 1792, top-4, 1 shared, skewed): 128 tokens 192 /
//     207, 192 211 / 222: short from 256 tokens and 32 experts to r 48.
//   4-bit (two workgroups overlap dequantisation and MFMAs), no shared experts: 8 x 4096 x 14336: r 1 218 /
//     176 us, r 16 288 / 226, r 48 301 / 291, r 64 336 / 403; 128 x 4096 x 1536: r 16 509 / 389, r 48 578 / 553, r 64
//     667 / 712; 64 x 2048 x 1408: r 48 161 / 174, r 64 186 / 198: short to r 48.
//     Shared experts: up to r 64 short tiles are the faster ones by 3 to 48 % (4, 8, 16, 24, 32, 64, 96, 128 and 256
//     experts, one to four shared): 8 + 1 x 4096 x 14336 r 64 664 / 574, 8 + 2 870 / 719, 8 + 4 x 4096 x 4096 354 / 326.
//     Beyond, an expert is two short tiles.  With 16 experts and more the shared tiles end a tall launch all the
//     same: 16 + 1 x 4096 x 4096 r 72 415 / 397, r 96 517 / 455; 32 + 2 x 2048 x 2048 r 80 260 / 246; 64 + 2 x 2048 x
//     1408 r 72 319 / 294, r 96 377 / 303 (skewed routing +26 to +45 %), r 128 399 / 365, r 160 425 / 435; 128 + 1 x
//     4096 x 1536 r 80 1356 / 1240, r 96 1555 / 1352; 160 + 2 x 2048 x 1408 r 96 839 / 732; worst: 64 + 1 x 5120 x 1536 r
//     80 600 / 685 (2048 x 1408 266 / 280, skewed +22 to +38 %), 24 + 1 x 4096 x 4096 r 72 -6 %.  With fewer experts a
//     shared expert of more than 256 tokens is cut evenly and tall tiles win on even routing: 8 + 1 x 4096 x 14336 r
//     72 584 / 646, r 96 714 / 690; 8 + 2 r 72 656 / 818, r 96 828 / 920; 8 + 4 x 4096 x 4096 r 88 313 / 415; 12 + 1 x 4096 x
//     8192 r 88 -18 % (skewed 8 + 1 +7 to +16 %): short to r 96 from 16 experts, to r 64 with fewer.
//     Launches below a workgroup per compute unit gain nothing: 16 x 2048 x 1408 (176): r 16 63 / 65, r 48 68 / 75;
//     16 x 1024 x 512 (68) r 16 66 / 85: short from 256 workgroups.
inline int64_t most_short_rows(int E, int S, bool q4) { return (q4 && S > 0 ? (E >= 16 ? 96ll : 64ll) : 48ll) * E; }
inline bool short_tiles(int64_t n_tokens, int k, int E, int S, int f, bool q4) {
    const int64_t A = n_tokens * k;
    if (A > most_short_rows(E, S, q4)) return false;
    if (!q4) return S > 0 && E >= 32 && n_tokens >= 256;
    const int64_t rows = (int64_t)kTileBlks * kRowBlk, tiles = (A < E ? A : E) + S * ((n_tokens + rows - 1) / rows);
    return tiles * ((f / 16 + 7) / 8) >= 256;
}

// Capacity of the tile tables for a context (either tile height its weights may take).
inline int max_tiles_for(int max_rowblks, int E, int S, int max_tokens, bool q4) {
    auto tiles = [&](int rowblks, int tokens, int blks) {
        return rowblks / blks + E + S * ((tokens + blks * kRowBlk - 1) / (blks * kRowBlk) + 1) + 1;
    };
    const int short_rows = (int)most_short_rows(E, S, q4), short_rowblks = short_rows / kRowBlk + 1 + E;
    const int tall = tiles(max_rowblks, max_tokens, kTileBlks);
    const int low = tiles(max_rowblks < short_rowblks ? max_rowblks : short_rowblks,
                          max_tokens < short_rows ? max_tokens : short_rows, kShortBlks);
    return tall > low ? tall : low;
}

}  // namespace kmoe
