// goq_ref_coefficients: the REF-mode (activation-aware) block coefficients on the device
// (Sec. 3.4, Eq. 3).  The bases b1, b2 stay those of the canonical arrays; for every output channel
// o and macro-block g, with the M calibration rows X_q = X[:, 128 g .. 128 g + 127],
//     Y = X_q w,   A = [X_q b1, X_q b2],   c* = (A^T A + lambda I)^-1 A^T Y.
//
// A^T A and A^T Y are quadratic forms of the slab's Gram matrix S_g = X_q^T X_q (128 x 128), which
// all output channels share:
//     A^T A = [b1 b2]^T S_g [b1 b2],   A^T Y = [b1 b2]^T S_g w,
// so the tokens are reduced once per macro-block (kernel 1) instead of once per output channel, and
// kernel 2 needs, per (o, g), the two products S_g b1 and S_g b2 and five dot products.  Both are
// fp64 contractions and run on v_mfma_f64_16x16x4: it has the rate of the vector ALU (one 16 x 16 x 4
// product in 64 cycles) but takes one operand register pair per 16 fused multiply-adds of a lane, so that
// loads, conversions and address arithmetic hide behind it, which bound the same sums on the vector ALU
// (4096 x 4096, 512 tokens: Gram matrices 120 us, solve 272 us; now 16 and 141).  Everything is fp64 with
// fixed summation orders (tokens ascending; columns, then rows), so the result is a pure function of
// the inputs.  It differs from a token-by-token evaluation of Eq. 3 only by fp64 rounding, far below
// the fp16 quantum of the stored coefficients.
//
// Operand layout of the instruction: A lane l holds A[l % 16][l / 16], B lane l holds
// B[l / 16][l % 16], element v of D is D[4 v + l / 16][l % 16].
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "goq_layout.h"
#include "goq_decode.h"
#include "goq_internal.h"
#include "goq_f64.h"

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int RT = 256;                  // threads per workgroup (both kernels): four wavefronts
constexpr int TT = 64;                   // tokens per LDS tile of the Gram kernel
constexpr int XP = GOQ_N + 16;           // halfs per LDS row: the four tokens of an operand in different banks
constexpr int OB = 64;                   // output channels per workgroup of the solve kernel, 16 per wavefront
constexpr int TILES = 36;                // 16 x 16 tiles of S_g on and below the diagonal

__device__ __forceinline__ f64x4 mfma(double a, double b, f64x4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
__device__ __forceinline__ double half_to_double(_Float16 h) { return (double)(float)h; }

// ---- kernel 1: S_g = X_q^T X_q.  Workgroup (g, y): wavefront w owns tile 4 y + w of the lower triangle
// over all tokens, so that 32 macro-blocks already fill the chip with one tile per SIMD; the tile's
// mirror image is stored beside it.
__global__ __launch_bounds__(RT) void gram_kernel(const uint16_t *__restrict__ X, int tokens, int64_t in,
                                                  double *__restrict__ S)
{
    __shared__ __attribute__((aligned(16))) _Float16 xt[TT][XP];
    const int g = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int n = lane & 15, k = lane >> 4;
    const int tile = __builtin_amdgcn_readfirstlane(blockIdx.y * 4 + (tid >> 6));
    int ti = 0;
    while ((ti + 1) * (ti + 2) / 2 <= tile) ++ti;
    const int tj = tile - ti * (ti + 1) / 2;
    // 64 tokens x 128 halfs = 1024 pieces of 16 bytes, four per thread; rows past the end are zero
    auto load = [&](int t0, uint4 (&v)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int t = t0 + 16 * i + (tid >> 4);
            v[i] = make_uint4(0, 0, 0, 0);
            if (t < tokens) v[i] = *reinterpret_cast<const uint4 *>(X + (int64_t)t * in + (int64_t)g * GOQ_N + (tid & 15) * 8);
        }
    };
    uint4 v[4];
    load(0, v);
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int t0 = 0; t0 < tokens; t0 += TT) {
        __syncthreads();                                       // the previous tile has been used
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<uint4 *>(&xt[16 * i + (tid >> 4)][(tid & 15) * 8]) = v[i];
        __syncthreads();
        if (t0 + TT < tokens) load(t0 + TT, v);
#pragma unroll
        for (int t = 0; t < TT; t += 4)
            acc = mfma(half_to_double(xt[t + k][16 * ti + n]), half_to_double(xt[t + k][16 * tj + n]), acc);
    }
    double *Sg = S + (int64_t)g * GOQ_N * GOQ_N;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = 16 * ti + 4 * e + k, j = 16 * tj + n;
        Sg[i * GOQ_N + j] = acc[e];
        if (ti != tj) Sg[j * GOQ_N + i] = acc[e];
    }
}

// ---- kernel 2: per (g, block of OB output channels).  A wavefront forms u1 = S_g b1 and u2 = S_g b2 of
// its 16 output channels (columns of B), all 128 rows: eight 16-row tiles and two bases of
// accumulators, one read of a row of S_g (symmetric: column j is read as the contiguous row j, from
// L2, the next four rows in flight) for all of them.  Then its share of the five dot products per lane, the four
// lanes of a channel are added in order and the 2 x 2 system is solved.  b1, b2 and w are staged as
// fp16, which holds them exactly.
template <int BW>
__global__ __launch_bounds__(RT, 2) void ref_solve_kernel(const uint16_t *__restrict__ w, const uint8_t *__restrict__ codes,
                                                       const uint8_t *__restrict__ pattern, const uint8_t *__restrict__ signs,
                                                       const double *__restrict__ S, int64_t out, int64_t in, double lambda,
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
    const double *Sg = S + (int64_t)g * GOQ_N * GOQ_N + k * GOQ_N + n;
    f64x4 u1[8], u2[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) { u1[i] = f64x4{0.0, 0.0, 0.0, 0.0}; u2[i] = f64x4{0.0, 0.0, 0.0, 0.0}; }
    // rows 4 t + k of S_g, column 16 i + n
    auto load = [&](int t, double (&a)[8]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) a[i] = Sg[4 * t * GOQ_N + 16 * i];
    };
    auto products = [&](int t, const double (&a)[8]) {
        const double b1 = half_to_double(vb1[oo][4 * t + k]), b2 = half_to_double(vb2[oo][4 * t + k]);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            u1[i] = mfma(a[i], b1, u1[i]);
            u2[i] = mfma(a[i], b2, u2[i]);
        }
    };
    double a0[8], a1[8];
    load(0, a0);
    for (int t = 0; t < 30; t += 2) {
        load(t + 1, a1);
        products(t, a0);
        load(t + 2, a0);
        products(t + 1, a1);
    }
    load(31, a1);
    products(30, a0);
    products(31, a1);

    double q[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int r = 16 * i + 4 * e + k;
            const double b1 = half_to_double(vb1[oo][r]), b2 = half_to_double(vb2[oo][r]), wr = half_to_double(vw[oo][r]);
            q[0] = fma(b1, u1[i][e], q[0]);
            q[1] = fma(b2, u1[i][e], q[1]);
            q[2] = fma(b2, u2[i][e], q[2]);
            q[3] = fma(wr, u1[i][e], q[3]);
            q[4] = fma(wr, u2[i][e], q[4]);
        }
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
    double *S = reinterpret_cast<double *>(workspace);
    hipLaunchKernelGGL(gram_kernel, dim3((unsigned)gn, TILES / 4), dim3(RT), 0, st, X, (int)tokens, in, S);
    int rc = goq_check_launch("goq_ref_coefficients");
    if (rc) return rc;
    if (bw == 3)
        hipLaunchKernelGGL(ref_solve_kernel<3>, dim3((unsigned)gn, (unsigned)ob), dim3(RT), 0, st, w, codes, pattern, signs,
                           S, out, in, lambda, craw, c1, c2);
    else
        hipLaunchKernelGGL(ref_solve_kernel<4>, dim3((unsigned)gn, (unsigned)ob), dim3(RT), 0, st, w, codes, pattern, signs,
                           S, out, in, lambda, craw, c1, c2);
    return goq_check_launch("goq_ref_coefficients");
}
