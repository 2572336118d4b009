// goq_ref_coefficients: the REF-mode (activation-aware) block coefficients on the device
// (Sec. 3.4, Eq. 3).  The bases b1, b2 stay those of the canonical arrays; for every output channel
// o and macro-block g, with the M calibration rows X_q = X[:, 128 g .. 128 g + 127],
//     Y = X_q w,   A = [X_q b1, X_q b2],   c* = (A^T A + lambda I)^-1 A^T Y.
//
// A^T A and A^T Y are quadratic forms of the slab's Gram matrix S_g = X_q^T X_q (128 x 128), which
// all output channels share:
//     A^T A = [b1 b2]^T S_g [b1 b2],   A^T Y = [b1 b2]^T S_g w,
// so the tokens are reduced once per macro-block (kernel 1) instead of once per output channel, and
// kernel 2 needs, per (o, g), products with the upper triangle of S_g and five dot products.  Both are
// fp64 contractions and run on v_mfma_f64_16x16x4: it has the rate of the vector ALU (one 16 x 16 x 4
// product in 64 cycles) but takes one operand register pair per 16 fused multiply-adds of a lane, so that
// loads, conversions and address arithmetic hide behind it, which bound the same sums on the vector ALU
// (4096 x 4096, 512 tokens: Gram matrices 120 us, solve 272 us; now 16 and 127).  Everything is fp64 with
// fixed summation orders (tokens ascending, in one or two parts by the layer's size; columns, then rows of a 16-row tile, then tiles), so the result is a pure function of
// the inputs.  It differs from a token-by-token evaluation of Eq. 3 only by fp64 rounding, far below
// the fp16 quantum of the stored coefficients.
//
// Operand layout of the instruction: A lane l holds A[l % 16][l / 16], B lane l holds
// B[l / 16][l % 16], element v of D is D[4 v + l / 16][l % 16].
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>
#include "goq_layout.h"
#include "goq_decode.h"
#include "goq_internal.h"
#include "goq_f64.h"

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int RT = 256;                  // threads per workgroup of the solve kernel: four wavefronts
constexpr int TT = 64;                   // tokens per LDS tile of the Gram kernel
constexpr int XP = GOQ_N + 16;           // floats per LDS row: the four tokens of an operand in different banks
constexpr int OB = 64;                   // output channels per workgroup of the solve kernel, 16 per wavefront
constexpr int TILES = 36;                // 16 x 16 tiles of S_g on and above the diagonal
constexpr int H = 4;                     // row tiles of M^T that the solve kernel takes at a time

__device__ __forceinline__ f64x4 mfma(double a, double b, f64x4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
__device__ __forceinline__ double half_to_double(_Float16 h) { return (double)(float)h; }

// ---- kernel 1: S_g = X_q^T X_q.  Workgroup (g, y): wavefront w owns tile 4 y + w of the upper triangle
// over all tokens (or its part of them), so that 32 macro-blocks already fill the chip with one tile per SIMD.  What is stored is M_g: the tiles on the
// diagonal as they are, those above it twice (exact), nothing below.  A tile of 64 tokens takes 1.3 us where its products
// take 0.43; what takes the rest has not been found (four tiles of X in flight instead of one, two or four accumulators in turn: no faster).
// PARTS: of the tokens, each with four wavefronts of the workgroup and an LDS tile of its own.  Two where there is a tile for either and at most two
// workgroups per CU, so that wavefronts cover each other's waits (both kernels, us, one part / two: 512 tokens, 4096 x 4096 140.7 / 139.6, 4096 x 11008, 774 workgroups, 358.8 /
// 361.4; 4096 tokens, 768 x 768 93.2 / 82.7; 64 tokens, 2304 x 768 23.0 / 23.8).
template <int PARTS>
__global__ __launch_bounds__(256 * PARTS) void gram_kernel(const uint16_t *__restrict__ X, int tokens, int64_t in,
                                                  double *__restrict__ M)
{
    __shared__ __attribute__((aligned(16))) float staged[PARTS][TT][XP];
    const int g = blockIdx.x;
    const int part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), tid = threadIdx.x & 255, lane = tid & 63;
    float (&xt)[TT][XP] = staged[part];
    const int n = lane & 15, k = lane >> 4;
    const int tile = __builtin_amdgcn_readfirstlane(blockIdx.y * 4 + (tid >> 6));
    int ti = 0;
    while ((ti + 1) * (ti + 2) / 2 <= tile) ++ti;
    const int tj = tile - ti * (ti + 1) / 2;
    // 64 tokens x 128 halfs = 1024 pieces of 16 bytes, four per thread (rows past the end: the last one, which becomes zeros in LDS)
    const uint16_t *rows = X + (int64_t)g * GOQ_N + (tid & 15) * 8;
    f16x8 v[4];
    auto load = [&](int64_t t0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const f16x8 *>(rows + min(t0 + 16 * i + (tid >> 4), (int64_t)tokens - 1) * in);
    };
    // operands of four products, and the next four's on their way
    float f[2][2][4];
    double d[2][4];
    auto read = [&](int t, float (&o)[2][4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            o[0][i] = xt[t + 4 * i + k][16 * tj + n];
            o[1][i] = xt[t + 4 * i + k][16 * ti + n];
        }
    };
    load(part * TT);
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int64_t first = 0; first < tokens; first += PARTS * TT) {
        const int64_t t0 = first + part * TT;                  // (a part without tokens adds zeros)
        __syncthreads();                                       // the previous tile has been used
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float *o = &xt[16 * i + (tid >> 4)][(tid & 15) * 8];
            const f16x8 x = t0 + 16 * i + (tid >> 4) < tokens ? v[i] : f16x8{};
            *reinterpret_cast<f32x4 *>(o) = f32x4{(float)x[0], (float)x[1], (float)x[2], (float)x[3]};
            *reinterpret_cast<f32x4 *>(o + 4) = f32x4{(float)x[4], (float)x[5], (float)x[6], (float)x[7]};
        }
        __syncthreads();
        load(t0 + PARTS * TT);
        read(0, f[0]);
#pragma unroll
        for (int b = 0; b < TT / 16; ++b) {
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int i = 0; i < 4; ++i) d[c][i] = (double)f[b & 1][c][i];
            if (b + 1 < TT / 16) read(16 * (b + 1), f[(b + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);                 // (left alone, the reads move behind the products)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc = mfma(d[0][i], d[1][i], acc);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (PARTS == 2) {
        __syncthreads();
        f64x4 *sums = reinterpret_cast<f64x4 *>(staged[0]);
        if (part) sums[tid] = acc;
        __syncthreads();
        if (part) return;
        acc += sums[tid];
    }
    double *Mg = M + (int64_t)g * GOQ_N * GOQ_N + (16 * tj + k) * GOQ_N + 16 * ti + n;
    const double scale = ti == tj ? 1.0 : 2.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) Mg[4 * e * GOQ_N] = scale * acc[e];
}

// ---- kernel 2: per (g, block of OB output channels).  With M = D + 2 U (diagonal tiles of S and twice those above) and any a, b
//     a^T S b = (a^T M b + b^T M a) / 2,
// so the five dot products need M^T b1, M^T b2 and M^T w: 3 x 36 tile products instead of the 2 x 64 of S b1 and S b2.  A wavefront forms
// them for its 16 output channels (columns of B), H 16-row tiles of M^T at a time (column j of M^T is the contiguous row j of M, from L2, two steps of four in flight),
// and adds their share of the dot products per lane; the four lanes of a channel are added in order and the 2 x 2 system is solved.  b1, b2 and w are
// staged as fp16, which holds them exactly.  Bound by the fp64 matrix rate (4096 x 4096, 512 tokens, both kernels, us: both products with S 158.4, H = 2 at
// three wavefronts per SIMD 145.8, H = 4 142.1 with six registers spilled, at two without 140.9; states staged as the upper halves of doubles, so
// that a shift converts them, 143.4; the last but one with dot products per row tile, as now, 140.9 .. 141.2).  Error of the unrounded pairs against extended
// precision, rms over 256 to 700 channels, six sets of inputs: with S 6.5e-16 .. 7.7e-16, now 4.9e-16 .. 6.3e-16 (dot products as one chain of additions, two sets, up to 8.5e-16).
template <int BW>
__global__ __launch_bounds__(RT, 2) void ref_solve_kernel(const uint16_t *__restrict__ w, const uint8_t *__restrict__ codes,
                                                       const uint8_t *__restrict__ pattern, const uint8_t *__restrict__ signs,
                                                       const double *__restrict__ M, int64_t out, int64_t in, double lambda,
                                                       double *__restrict__ craw, uint16_t *__restrict__ c1,
                                                       uint16_t *__restrict__ c2)
{
    // (rows of 130 halfs: the 16 channels of an operand read fall into different banks)
    constexpr int VP = GOQ_N + 2;
    __shared__ __attribute__((aligned(16))) _Float16 vb1[OB][VP], vb2[OB][VP], vw[OB][VP];
    __shared__ __attribute__((aligned(16))) uint4 xtab[64];                 // exchange table
    const int tid = threadIdx.x;
    const int g = blockIdx.x;
    const int64_t o0 = (int64_t)blockIdx.y * OB;
    const int64_t gn = in / GOQ_N;

    if (tid < 64) xtab[tid] = goq_exchange_entry<0x80u>(tid);
    __syncthreads();
    // stage b1, b2 (Theorem 1 exchange from pattern and pair signs) and w of the OB channels: a
    // micro-block at a time, as fp16 high bytes until they are written
    const bool wide = ((uintptr_t)w & 15) == 0;
#pragma unroll
    for (int it = tid; it < OB * 16; it += RT) {
        const int oo = it >> 4, m = it & 15;
        const int64_t o = min(o0 + oo, out - 1);               // channels past the end repeat the last one
        const int64_t k0 = o * in + (int64_t)g * GOQ_N + m * GOQ_G;
        const uint2 cw = *reinterpret_cast<const uint2 *>(codes + k0);
        const uint32_t v = (pattern[k0 / GOQ_G] & 3u) | ((signs[k0 / GOQ_G] & 15u) << 2);
        uint32_t wd[4];
        if (wide) {
            const uint4 t = *reinterpret_cast<const uint4 *>(w + k0);
            wd[0] = t.x; wd[1] = t.y; wd[2] = t.z; wd[3] = t.w;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) wd[i] = w[k0 + 2 * i] | (uint32_t)w[k0 + 2 * i + 1] << 16;
        }
        // the dword of the packed layout without its metadata
        const uint32_t d = BW == 3 ? (cw.x & 0x07070707u) | ((cw.y & 0x07070707u) << 3)
                                   : (cw.x & 0x0f0f0f0fu) | ((cw.y & 0x0f0f0f0fu) << 4);
        uint32_t lo, hi;
        goq_decode_bytes<BW, 0>(d, lo, hi);
        const uint4 e = xtab[v];
        const uint32_t xlo = goq_perm(hi, lo, e.x) ^ e.z, xhi = goq_perm(hi, lo, e.y) ^ e.w;
        uint32_t *p1 = reinterpret_cast<uint32_t *>(&vb1[oo][m * GOQ_G]);
        uint32_t *p2 = reinterpret_cast<uint32_t *>(&vb2[oo][m * GOQ_G]);
        uint32_t *pw = reinterpret_cast<uint32_t *>(&vw[oo][m * GOQ_G]);
        p1[0] = goq_widen01(lo); p1[1] = goq_widen23(lo); p1[2] = goq_widen01(hi); p1[3] = goq_widen23(hi);
        p2[0] = goq_widen01(xlo); p2[1] = goq_widen23(xlo); p2[2] = goq_widen01(xhi); p2[3] = goq_widen23(xhi);
#pragma unroll
        for (int i = 0; i < 4; ++i) pw[i] = wd[i];
    }
    __syncthreads();

    const int lane = tid & 63, n = lane & 15, k = lane >> 4;
    const int oo = (tid >> 6) * 16 + n;                        // this lane's channel
    const double *Mg = M + (int64_t)g * GOQ_N * GOQ_N + k * GOQ_N + n;
    double q[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int p = 0; p < 8 / H; ++p) {
        f64x4 u[H][3];
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int c = 0; c < 3; ++c) u[h][c] = f64x4{0.0, 0.0, 0.0, 0.0};
        const double *rows = Mg + 16 * H * p;
        auto load = [&](int t, double (&a)[H]) {               // columns 4 t .. 4 t + 3 (below the diagonal: not used)
#pragma unroll
            for (int h = 0; h < H; ++h) a[h] = rows[4 * t * GOQ_N + 16 * h];
        };
        auto products = [&](int t, const double (&a)[H], auto first) {   // for row tiles first .. H - 1
            const double b[3] = {half_to_double(vb1[oo][4 * t + k]), half_to_double(vb2[oo][4 * t + k]), half_to_double(vw[oo][4 * t + k])};
#pragma unroll
            for (int h = first; h < H; ++h)
#pragma unroll
                for (int c = 0; c < 3; ++c) u[h][c] = mfma(a[h], b[c], u[h][c]);
        };
        double a[2][H];
        load(0, a[0]);
        load(1, a[1]);
        const int square = 4 * H * p;                          // steps that all row tiles have; then one column of tiles at a time ends
        for (int t = 0; t < square; t += 2)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                products(t + i, a[i], std::integral_constant<int, 0>());
                load(t + i + 2, a[i]);
            }
        auto triangle = [&](auto first) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                products(square + 4 * first + i, a[i % 2], first);
                if (first < H - 1 || i < 2) load(square + 4 * first + i + 2, a[i % 2]);
            }
        };
        triangle(std::integral_constant<int, 0>());
        triangle(std::integral_constant<int, 1>());
        if constexpr (H == 4) {
            triangle(std::integral_constant<int, 2>());
            triangle(std::integral_constant<int, 3>());
        }
#pragma unroll
        for (int h = 0; h < H; ++h) {
            double s[5] = {0.0, 0.0, 0.0, 0.0, 0.0};           // of a row tile: short chains of roundings
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int r = 16 * (H * p + h) + 4 * e + k;
                const double b1 = half_to_double(vb1[oo][r]), b2 = half_to_double(vb2[oo][r]), wr = half_to_double(vw[oo][r]);
                const double u1 = u[h][0][e], u2 = u[h][1][e], uw = u[h][2][e];
                s[0] = fma(b1, u1, s[0]);
                s[1] = fma(b1, u2, fma(b2, u1, s[1]));
                s[2] = fma(b2, u2, s[2]);
                s[3] = fma(b1, uw, fma(wr, u1, s[3]));
                s[4] = fma(b2, uw, fma(wr, u2, s[4]));
            }
#pragma unroll
            for (int c = 0; c < 5; ++c) q[c] += s[c];
        }
    }
    q[1] *= 0.5; q[3] *= 0.5; q[4] *= 0.5;
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        q[c] += __shfl_xor(q[c], 16);
        q[c] += __shfl_xor(q[c], 32);
    }
    if (k == 0 && o0 + oo < out) {
        const double a11 = q[0] + lambda, a22 = q[2] + lambda, a12 = q[1];
        const double det = a11 * a22 - a12 * a12;
        double s1 = 0.0, s2 = 0.0;
        if (det != 0.0) {                                       // det = 0 only without a ridge, dependent columns
            s1 = (a22 * q[3] - a12 * q[4]) / det;
            s2 = (a11 * q[4] - a12 * q[3]) / det;
        }
        const int64_t idx = (o0 + oo) * gn + g;
        if (craw) { craw[2 * idx] = s1; craw[2 * idx + 1] = s2; }
        c1[idx] = (uint16_t)double_to_half_bits(s1);
        c2[idx] = (uint16_t)double_to_half_bits(s2);
    }
}

}  // namespace

int goq_launch_ref(hipStream_t st, int bw, int64_t tokens, int64_t out, int64_t in, const uint16_t *w,
                   const uint8_t *codes, const uint8_t *pattern, const uint8_t *signs, const uint16_t *X,
                   double lambda, void *workspace, double *craw, uint16_t *c1, uint16_t *c2)
{
    const int64_t gn = in / GOQ_N;
    const int64_t ob = (out + OB - 1) / OB;
    if (gn > 0x7fffffff || ob > 65535 || tokens > 0x7fffffff)
        return goq_set_error(GOQ_ESHAPE, "goq_ref_coefficients: layer too large for one launch");
    double *M = reinterpret_cast<double *>(workspace);
    if (tokens > TT && gn * (TILES / 4) <= 512)
        hipLaunchKernelGGL(gram_kernel<2>, dim3((unsigned)gn, TILES / 4), dim3(512), 0, st, X, (int)tokens, in, M);
    else
        hipLaunchKernelGGL(gram_kernel<1>, dim3((unsigned)gn, TILES / 4), dim3(256), 0, st, X, (int)tokens, in, M);
    int rc = goq_check_launch("goq_ref_coefficients");
    if (rc) return rc;
    if (bw == 3)
        hipLaunchKernelGGL(ref_solve_kernel<3>, dim3((unsigned)gn, (unsigned)ob), dim3(RT), 0, st, w, codes, pattern, signs,
                           M, out, in, lambda, craw, c1, c2);
    else
        hipLaunchKernelGGL(ref_solve_kernel<4>, dim3((unsigned)gn, (unsigned)ob), dim3(RT), 0, st, w, codes, pattern, signs,
                           M, out, in, lambda, craw, c1, c2);
    return goq_check_launch("goq_ref_coefficients");
}
