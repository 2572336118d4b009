// Host check of the requests of goq_gemm's tile kernel (goq_request.h): every tile, slab and piece of layers with
// ragged token counts and the largest rows, under the range check of a raw buffer load as it is defined: a load
// is in range if its PER-LANE offset lies inside the window; a scalar offset would not be looked at.
//   - a piece of a token and a slab that exist lies in the window, and at its own place of X;
//   - any other piece is out of the window;
//   - the window lies inside X.
#include <cstdio>
#include "../paper_2605_26092_amd/csrc/goq_request.h"

static long long checked = 0;

static int check(int64_t tokens, int64_t in, int xb, int tm)
{
    const uint32_t line = (uint32_t)(in * xb);
    const int gn = (int)(in / GOQ_N), slab = GOQ_N * xb, per_row = slab / 16;
    const int64_t total = tokens * (int64_t)line;
    for (int64_t m0 = 0; m0 < tokens; m0 += tm) {
        if (m0 > 2 * tm && m0 + 2 * tm < tokens) continue;       // inner tiles are alike
        const uint32_t bytes = goq_tile_bytes((int)(tokens - m0), tm, line);
        for (int g = 0; g < gn + 2; ++g) {                       // the pipeline asks for two slabs past the end
            if (g > 3 && g < gn - 2) continue;
            const GoqWindow win = goq_slab_window(bytes, g, gn, slab);
            const int64_t begin = m0 * (int64_t)line + win.begin;
            if (win.records && begin + (int64_t)win.records > total) return printf("window past X\n"), 1;
            for (int row = 0; row < tm; ++row)
                for (int piece = 0; piece < per_row; ++piece) {
                    const uint32_t off = goq_piece_offset(row, piece, line);
                    const bool wanted = m0 + row < tokens && g < gn;
                    const bool in_range = (uint64_t)off + 16 <= win.records, touches = off < win.records;
                    if (wanted && !in_range) return printf("a piece is cut off\n"), 1;
                    if (!wanted && touches) return printf("a piece that does not exist is in range\n"), 1;
                    if (wanted && begin + off != (m0 + row) * (int64_t)line + (int64_t)g * slab + piece * 16) return printf("wrong place\n"), 1;
                    ++checked;
                }
        }
    }
    return 0;
}

int main()
{
    const int64_t tokens[] = {33, 40, 63, 64, 65, 97, 203, 1025, 16777216}, ins[] = {128, 256, 384, 4096, 11008, 16777216};
    for (int64_t t : tokens)
        for (int64_t in : ins)
            for (int xb = 1; xb <= 2; ++xb)
                for (int tm = 32; tm <= (xb == 1 ? 128 : 64); tm *= 2)
                    if (check(t, in, xb, tm)) return printf("tokens %lld in %lld bytes %d tile %d\n", (long long)t, (long long)in, xb, tm), 1;
    printf("requests in range: ok (%lld pieces)\n", checked);
    return 0;
}
