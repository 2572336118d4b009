// How a batch-1 launch of a few projections is cut into ranges of 16-row tiles, and which launches are (goq_gemv_short.hip).  Plain
// C++ on its own, so that ranges and choices can be checked without a device.
#pragma once
#include <stdint.h>
#include "goq_layout.h"

constexpr int GOQ_SHORT_WGS = 256;           // workgroups: one per CU
constexpr int GOQ_SHORT_GN = 128;            // macro-blocks of the deepest layer: its digits fit into LDS
constexpr int GOQ_SHORT_TILES = 64;          // tiles of a workgroup: its sums fit into LDS

// Tile at which the launch is cut after `at` of its (tile, macro-block) slices, in a problem of gn macro-blocks whose first
// tile is `first` and before which there are `before` slices: at the tile boundary that lies nearest.
GOQ_HD int goq_short_cut(int at, int before, int first, int gn) { return first + (at - before + gn / 2) / gn; }

// slices of the launch before workgroup k, of each = total / GOQ_SHORT_WGS, rest = total % GOQ_SHORT_WGS
GOQ_HD int goq_short_share(int k, int each, int rest) { return k * each + (k < rest ? k : rest); }

struct GoqRows {
    int out, gn;
};

// Does a launch that the streaming kernel would take (more than 512 tiles or 24576 slices) go to ranges of tiles?
//
// The kernel's time grows with the slices of its fullest workgroup, which are whole tiles, the streaming kernel's with those of
// all and with the parts that a row group is put together from.  117 launches were timed in either kernel (3.6 to 110 thousand slices, all types; ns):
//     ranges of tiles   5100 + 45 (W4: 61) per slice of the fullest workgroup + 500 per layer with another depth than the one before
//     streaming         6000 + 39 (W4: 59; with int8 4 % more) per slice / 256 + 90 per part, W3 and W4 with up to 256 units 6200 + 41 and 6400 + 35
// by which the choice loses 0.7 % on average against the better kernel, and gains 8.1 % against streaming (us, streaming / ranges of tiles: 11008 x 4096 W3/A16
// 11.5 / 9.1, two of them W4/A8 18.3 / 16.9; three of 4096 x 4096 W3/A16 11.9 / 9.6; 8192 x 8192 W3/A16 13.5 / 11.3, W4/A16 15.5 / 13.6; 22555 x 1024 W3/A8 8.8 / 7.0).  The ones it
// leaves are those whose tiles do not divide by 256 workgroups (9000 x 14336, W3/A16 17.0 / 20.8, three tiles where 2.2 would do) and large ones
// (7B block 23.1 / 25.8), whose cost per slice decides: the streaming kernel reads digits and block scales once for four slices.
inline bool goq_short(int bw, bool int8, int n, const GoqRows *p)
{
    int64_t slices = 0, tiles = 0, units = 0;
    int deepest = 0, least = 0x7fffffff, changes = 0;
    for (int i = 0; i < n; ++i) {
        const int64_t t = ((int64_t)p[i].out + 15) / 16;
        tiles += t;
        slices += t * p[i].gn;
        units += (p[i].out + 511) / 512 * (int64_t)p[i].gn;
        deepest = p[i].gn > deepest ? p[i].gn : deepest;
        least = p[i].gn < least ? p[i].gn : least;
        changes += i && p[i].gn != p[i - 1].gn ? 1 : 0;
    }
    if (deepest > GOQ_SHORT_GN || slices > 1 << 19 || (tiles <= 512 && slices <= 24576)) return false;
    const int total = (int)slices, share = (total + GOQ_SHORT_WGS - 1) / GOQ_SHORT_WGS;
    if (share / least + 4 > GOQ_SHORT_TILES) return false;
    int fullest = 0;
    for (int i = 0; i < n; ++i) {
        const int s = (share + p[i].gn - 1) / p[i].gn * p[i].gn;
        fullest = s > fullest ? s : fullest;
    }
    const int ranges = 5100 + (bw == 3 ? 45 : 61) * fullest + 500 * changes;
    if (units <= 256) return ranges < (bw == 3 ? 6200 + 41 * share : 6400 + 35 * share);
    const int parts = units > 512 ? (int)(deepest * 512 / units) : deepest;
    const int streaming = 6000 + (bw == 3 ? 39 : 59) * share + 90 * parts;
    return ranges < (bw == 4 && int8 ? streaming + streaming / 25 : streaming);
}
