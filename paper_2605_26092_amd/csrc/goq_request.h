// What the tile kernel of goq_gemm requests of X for one slab: a buffer window and the byte offsets of
// its pieces in that window.  Kept apart from the kernel so that the host can check the arithmetic.
//
// A piece is 16 bytes of one token's slab.  The window begins at the slab's first byte of the tile's first
// token and ends with the last token of the tile that exists; past the last slab it is empty.  All
// of a piece's offset is per-lane: that is the operand that the range check of a raw buffer load
// counts on every target (the scalar offset is excluded from it by the intrinsic's definition), so a
// token or a slab that does not exist is out of the window, reads as zeros and touches no memory.
#pragma once
#include <stdint.h>
#include "goq_layout.h"

struct GoqWindow {
    uint32_t begin;      // bytes from the tile's first token in X
    uint32_t records;    // bytes
};

// Bytes that a tile's tokens span: rows = tokens of X from the tile's first one on, line = bytes of a token (<= 2^25)
GOQ_HD uint32_t goq_tile_bytes(int rows, int tile_rows, uint32_t line) { return (uint32_t)(rows < tile_rows ? rows : tile_rows) * line; }

GOQ_HD GoqWindow goq_slab_window(uint32_t tile_bytes, int g, int gn, int slab)
{
    const uint32_t at = (uint32_t)(g * slab);
    return GoqWindow{at, g < gn ? tile_bytes - at : 0u};
}

// byte offset in the window of piece `piece` of the tile's token `row`
GOQ_HD uint32_t goq_piece_offset(int row, int piece, uint32_t line) { return (uint32_t)row * line + (uint32_t)piece * 16u; }
