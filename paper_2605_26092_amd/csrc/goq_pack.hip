// goq_pack / goq_unpack: canonical arrays <-> packed device layout (see goq_layout.h).  Unpacking is a
// test hook: one thread per (row, macro-block).
#include <hip/hip_runtime.h>
#include "goq_layout.h"
#include "goq_internal.h"
#include "goq_gemm_rules.h"

namespace {

// Packing moves 1.8 (bw = 3) or 1.9 bytes per weight and computes next to nothing, so it is laid out
// for memory: a workgroup takes a row block of 64 rows and one macro-block, thread
// (row, h) the 32 codes of chunk h.  The four threads of a row read 128 consecutive bytes of codes, a wavefront
// writes 256-byte runs of each chunk.  Of a line of patterns, signs or coefficients a workgroup uses an eighth and less, so neighbours along the
// row belong on one XCD, whose L2 then reads the line once: every XCD takes a range of workgroups instead of every eighth.  (us, 4096 x 11008, bw = 3 / 4, one box:
// eight macro-blocks per workgroup and no ranges 24.7 / 24.7, two 23.1 / 22.5, two and ranges 19.0 / 18.5, one and ranges 18.6 / 18.3; 1500 x 1024 6.4, 5.0, 5.1, 5.0;
// with one thread per (row, macro-block) reading single bytes 220.)
// WIDE: the codes are 16-byte, pattern and signs 4-byte aligned; else they are read byte by byte.
template <bool WIDE>
__device__ __forceinline__ uint4 load16(const uint8_t *p)
{
    if constexpr (WIDE) return *reinterpret_cast<const uint4 *>(p);
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = p[4 * i] | (uint32_t)p[4 * i + 1] << 8 | (uint32_t)p[4 * i + 2] << 16 | (uint32_t)p[4 * i + 3] << 24;
    return make_uint4(w[0], w[1], w[2], w[3]);
}
template <bool WIDE>
__device__ __forceinline__ uint32_t load4(const uint8_t *p)
{
    if constexpr (WIDE) return *reinterpret_cast<const uint32_t *>(p);
    return p[0] | (uint32_t)p[1] << 8 | (uint32_t)p[2] << 16 | (uint32_t)p[3] << 24;
}

template <int BW, bool WIDE>
__global__ __launch_bounds__(256) void pack_kernel(int64_t out, int64_t in, int units,
                                                   const uint8_t *__restrict__ codes,
                                                   const uint8_t *__restrict__ pattern,
                                                   const uint8_t *__restrict__ signs,
                                                   const uint16_t *__restrict__ c1,
                                                   const uint16_t *__restrict__ c2,
                                                   uint32_t *__restrict__ packed)
{
    constexpr int CH = (BW == 3) ? 4 : 5;
    const int gn = (int)(in / GOQ_N);
    const int r = threadIdx.x >> 2, h = threadIdx.x & 3;
    for (int unit = (int)blockIdx.x; unit < units; unit += (int)gridDim.x) {
        const int at = goq_xcd_tile(unit, units);
        const int R = at / gn, g = at % gn;
        const int64_t row = (int64_t)R * GOQ_ROWS + r;

        // padding rows: zero codes, pattern 0, signs 0, zero coefficients
        uint32_t c[8], pat = 0, sg = 0, cw = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) c[k] = (uint32_t)goq_zero_code(BW) * 0x01010101u;
        if (row < out) {
            const int64_t k0 = row * in + (int64_t)g * GOQ_N + 32 * h;
            const uint4 a = load16<WIDE>(codes + k0), b = load16<WIDE>(codes + k0 + 16);
            c[0] = a.x; c[1] = a.y; c[2] = a.z; c[3] = a.w; c[4] = b.x; c[5] = b.y; c[6] = b.z; c[7] = b.w;
            pat = load4<WIDE>(pattern + k0 / GOQ_G);
            sg = load4<WIDE>(signs + k0 / GOQ_G);
            cw = (uint32_t)c1[row * gn + g] | ((uint32_t)c2[row * gn + g] << 16);
        }
        uint32_t d[4], meta = ((cw >> (8 * h)) & 0xffu) << 24;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t s = (pat >> (8 * q)) & 3u, e = (sg >> (8 * q)) & 15u;
            if constexpr (BW == 3) {
                d[q] = (c[2 * q] & 0x07070707u) | ((c[2 * q + 1] & 0x07070707u) << 3) | s << 6 | (e & 3u) << 14 |
                       (e >> 2) << 22 | ((cw >> (30 - 2 * (4 * h + q))) & 3u) << 30;
            } else {
                d[q] = (c[2 * q] & 0x0f0f0f0fu) | ((c[2 * q + 1] & 0x0f0f0f0fu) << 4);
                meta |= (s | e << 2) << (6 * q);
            }
        }
        *reinterpret_cast<uint4 *>(packed + goq_quad_index(CH, gn, R, g, h, r)) = make_uint4(d[0], d[1], d[2], d[3]);
        if constexpr (BW == 4) packed[goq_quad_index(CH, gn, R, g, 4, r) + h] = meta;
    }
}

template <int BW>
__global__ __launch_bounds__(256) void unpack_kernel(int64_t out, int64_t in,
                                                     const uint32_t *__restrict__ packed,
                                                     uint8_t *__restrict__ codes,
                                                     uint8_t *__restrict__ pattern,
                                                     uint8_t *__restrict__ signs,
                                                     uint16_t *__restrict__ c1,
                                                     uint16_t *__restrict__ c2)
{
    constexpr int CH = (BW == 3) ? 4 : 5;
    const int64_t gn = in / GOQ_N;
    const int64_t rows = goq_row_blocks(out) * GOQ_ROWS;
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (tid >= rows * gn) return;
    const int64_t g = tid / rows % gn;
    const int64_t row = tid % rows;
    if (row >= out) return;
    const int64_t R = row / GOQ_ROWS;
    const int r = (int)(row % GOQ_ROWS);

    uint8_t *cp = codes + row * in + g * GOQ_N;
    uint8_t *pp = pattern + (row * in + g * GOQ_N) / GOQ_G;
    uint8_t *sp = signs + (row * in + g * GOQ_N) / GOQ_G;
    uint32_t cw = 0;
    uint4 meta = make_uint4(0, 0, 0, 0);
    if (BW == 4) meta = *reinterpret_cast<const uint4 *>(packed + goq_quad_index(CH, gn, R, g, 4, r));
    for (int h = 0; h < 4; ++h) {
        const uint4 v = *reinterpret_cast<const uint4 *>(packed + goq_quad_index(CH, gn, R, g, h, r));
        const uint32_t d[4] = {v.x, v.y, v.z, v.w};
        for (int q = 0; q < 4; ++q) {
            const int m = 4 * h + q;
            const uint32_t w = d[q];
            for (int j = 0; j < 4; ++j) {
                const uint32_t b = (w >> (8 * j)) & 0xffu;
                if (BW == 3) {
                    cp[8 * m + j] = (uint8_t)(b & 7u);
                    cp[8 * m + j + 4] = (uint8_t)((b >> 3) & 7u);
                } else {
                    cp[8 * m + j] = (uint8_t)(b & 15u);
                    cp[8 * m + j + 4] = (uint8_t)(b >> 4);
                }
            }
            if (BW == 3) {
                pp[m] = (uint8_t)((w >> 6) & 3u);
                sp[m] = (uint8_t)(((w >> 14) & 3u) | (((w >> 22) & 3u) << 2));
                cw = (cw << 2) | (w >> 30);
            } else {
                const uint32_t md = h == 0 ? meta.x : h == 1 ? meta.y : h == 2 ? meta.z : meta.w;
                const uint32_t v = (md >> (6 * q)) & 63u;
                pp[m] = (uint8_t)(v & 3u);
                sp[m] = (uint8_t)(v >> 2);
            }
        }
    }
    if (BW == 4) cw = (meta.x >> 24) | ((meta.y >> 24) << 8) | ((meta.z >> 24) << 16) | ((meta.w >> 24) << 24);
    c1[row * gn + g] = (uint16_t)(cw & 0xffffu);
    c2[row * gn + g] = (uint16_t)(cw >> 16);
}

}  // namespace

int goq_launch_pack(hipStream_t st, int bw, int64_t out, int64_t in, const uint8_t *codes,
                    const uint8_t *pattern, const uint8_t *signs, const uint16_t *c1,
                    const uint16_t *c2, void *packed)
{
    const int64_t units = goq_row_blocks(out) * (in / GOQ_N);
    const int64_t grid = units < 1 << 22 ? units : 1 << 22;      // (a launch has less than 2^32 threads)
    if (units > 0x7fffffff - grid) return goq_set_error(GOQ_ESHAPE, "goq_pack: layer too large for one launch");
    const bool wide = ((uintptr_t)codes & 15) == 0 && (((uintptr_t)pattern | (uintptr_t)signs) & 3) == 0;
    const auto kernel = bw == 3 ? (wide ? pack_kernel<3, true> : pack_kernel<3, false>)
                                : (wide ? pack_kernel<4, true> : pack_kernel<4, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(256), 0, st, out, in, (int)units, codes, pattern, signs, c1, c2,
                       (uint32_t *)packed);
    return goq_check_launch("goq_pack");
}

int goq_launch_unpack(hipStream_t st, int bw, int64_t out, int64_t in, const void *packed,
                      uint8_t *codes, uint8_t *pattern, uint8_t *signs, uint16_t *c1, uint16_t *c2)
{
    const int64_t n = goq_row_blocks(out) * GOQ_ROWS * (in / GOQ_N);
    const unsigned grid = (unsigned)((n + 255) / 256);
    if (bw == 3)
        hipLaunchKernelGGL(unpack_kernel<3>, dim3(grid), dim3(256), 0, st, out, in,
                           (const uint32_t *)packed, codes, pattern, signs, c1, c2);
    else
        hipLaunchKernelGGL(unpack_kernel<4>, dim3(grid), dim3(256), 0, st, out, in,
                           (const uint32_t *)packed, codes, pattern, signs, c1, c2);
    return goq_check_launch("goq_unpack");
}
