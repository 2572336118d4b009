// goq_quantize: the data-free GEO-mode quantizer on the device (Sec. 3.2 - 3.4): fp16 weights of a
// layer [out][in] -> canonical arrays (codes, pattern, signs, c1, c2).
//
// One LANE per micro-block of 8 weights, one ROW of 16 lanes per macro-block of 128 weights, four
// macro-blocks per wavefront.  Everything that belongs to a micro-block -- nearest states, the 16
// cross terms of the four exchange patterns, scores, argmax, pair signs, the exchange itself -- is
// lane-local and lives in registers; what belongs to the macro-block -- the norm s_norm and the
// sums of Eq. 1 and Eq. 2 -- is reduced across the 16 lanes of a row with data-parallel-primitive
// (DPP) moves, which stay inside a row by construction.  No LDS, no barriers.  It is bound by
// vector-ALU issue (391 instructions per micro-block, 76 % of the SIMD cycles), so the arithmetic is laid out around what is
// exact and need not be computed twice:
//
//   products    A lattice state is a signed power of two, so every product with a state is exact
//               in fp64.
//   sums        <w, b1> and <w, b2> (Eq. 1, Eq. 2) are sums of multiples of 2^-31 below 2^23: every
//               partial sum is exactly representable in fp64 whatever the order (always for
//               bw = 3; for bw = 4 unless |<w, b>| reaches 2^22, i.e. more than 64 weights of the
//               block at the fp16 maximum), so the reduction tree is free.  ||b1||^2 = ||b2||^2 is a
//               multiple of 2^-14 of at most 128: exact in fp32.
//   nearest     Q(v), v = w / s_norm (Sec. 3.2), is decided without the division: |v| lies above
//               the midpoint 0.75 * 2^-k of the states 2^-k and 2^-(k+1) exactly when
//               |w| > 0.75 * 2^-k * s_norm, and above the midpoint to zero, 2^-(emin+1), when
//               |w| > 2^-(emin+1) * s_norm.  The thresholds fall with k, so the exponent of the
//               nearest state is the NUMBER of thresholds |w| does not exceed, and that number is
//               a difference of fp32 exponent fields (see the loop); an exact tie goes to the
//               smaller magnitude.
//   cross terms The method's cross term of a pair is t = x_i r_j - x_j r_i with the residual
//               r = w - c b1, c = <w,b1> / ||b1||^2 (Eq. 1, Sec. 3.3), x = b1.  The c terms cancel:
//               in real arithmetic t = u = x_i w_j - x_j w_i, and u is EXACT in fp64 (a multiple of
//               2^-31 below 2^18).  A sequential fp64 evaluation rounds r and t, which moves t by less
//               than 2^-50 s_norm; it has the sign of u, because a nonzero u is at least 2^-31 (and where
//               u = 0 the states and weights of the pair are proportional by a power of two, or
//               zero, and so are the rounded residuals: t = 0).  So eta = sgn(u) (+1 at zero), the
//               scores A_s = sum |t| equal the exact U_s = sum |u| within 2^-46 s_norm, and s* =
//               argmax U_s unless two scores lie closer than that.  Only then (equal scores, a few per
//               million of real micro-blocks) the wavefront evaluates residuals and t as the method
//               writes them, to let their roundings decide as the sequential evaluation does
//               (ties: smallest s).  The pair's share of <w, b2> under the Theorem 1 exchange
//               (b2_i = -eta x_j for the lower index, +eta x_i for the upper one) is eta u = |u|:
//               U_s* is <w, b2> of the micro-block.
//
// The results are a pure function of the weights and equal those of a sequential fp64 evaluation
// of the same formulas bit for bit under the condition on the sums stated above.
// Measured, 11008 x 4096, bw = 3: 64 us (with states and signs by compare and select 77 us, with residuals and
// cross terms of every micro-block in fp64 98 us).  No gain: the next group's weights requested one iteration
// ahead (65 us), a finer or coarser grid (64 - 66 us); six wavefronts per SIMD spill (122 us).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "goq_layout.h"
#include "goq_internal.h"
#include "goq_f64.h"

namespace {

constexpr int QW = 4;                        // wavefronts per workgroup
constexpr int ROWS = 4;                      // macro-blocks (rows of 16 lanes) per wavefront

// ---- DPP moves inside a row of 16 lanes -------------------------------------------------------
// quad_perm [a, b, c, d]: lane 4 m + i reads lane 4 m + (a, b, c, d)[i]
constexpr int QUAD_SWAP1 = 1 | (0 << 2) | (3 << 4) | (2 << 6);      // i xor 1
constexpr int QUAD_SWAP2 = 2 | (3 << 2) | (0 << 4) | (1 << 6);      // i xor 2
constexpr int ROW_HALF_MIRROR = 0x141;                              // i -> 7 - i within 8 lanes
constexpr int ROW_MIRROR = 0x140;                                   // i -> 15 - i within 16 lanes

template <int CTRL>
__device__ __forceinline__ uint32_t dpp32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double dpp_double(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint64_t m = ((uint64_t)dpp32<CTRL>((uint32_t)(u >> 32)) << 32) | dpp32<CTRL>((uint32_t)u);
    return __builtin_bit_cast(double, m);
}
// After the four steps every lane of a row holds the row's result: the partners are i xor 1,
// i xor 2 (a quad holds one value), 7 - i (a group of eight does), 15 - i.
__device__ __forceinline__ double row_sum(double v)
{
    v += dpp_double<QUAD_SWAP1>(v);
    v += dpp_double<QUAD_SWAP2>(v);
    v += dpp_double<ROW_HALF_MIRROR>(v);
    v += dpp_double<ROW_MIRROR>(v);
    return v;
}
template <int CTRL>
__device__ __forceinline__ float dpp_float(float v) { return __uint_as_float(dpp32<CTRL>(__float_as_uint(v))); }
__device__ __forceinline__ float row_sum(float v)
{
    v += dpp_float<QUAD_SWAP1>(v);
    v += dpp_float<QUAD_SWAP2>(v);
    v += dpp_float<ROW_HALF_MIRROR>(v);
    v += dpp_float<ROW_MIRROR>(v);
    return v;
}
__device__ __forceinline__ uint32_t row_max(uint32_t v)
{
    v = max(v, dpp32<QUAD_SWAP1>(v));
    v = max(v, dpp32<QUAD_SWAP2>(v));
    v = max(v, dpp32<ROW_HALF_MIRROR>(v));
    v = max(v, dpp32<ROW_MIRROR>(v));
    return v;
}

// lower index of the p-th pair of pattern s, pairs in ascending lower index
__device__ __forceinline__ constexpr int pair_lower(int s, int p)
{
    return s == 1 ? 2 * p : s == 4 ? p : ((p & 1) | ((p >> 1) << 2));
}

// Pattern and signs of a micro-block as Sec. 3.3 writes them: residuals r = w - c x, cross terms and
// scores in fp64 in pair order; sets s - 1 and the sign bits.
__device__ __forceinline__ void choose_by_residual(const double (&wv)[8], const double (&x)[8], double c,
                                                   uint32_t &best, uint32_t &best_signs)
{
    double r[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = wv[i] - c * x[i];
    double bestA = -1.0;
#pragma unroll
    for (int s = 1; s <= 4; ++s) {
        double A = 0.0;
        uint32_t sg = 0;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int i = pair_lower(s, p), j = i ^ s;
            const double t = x[i] * r[j] - x[j] * r[i];
            A = (p == 0) ? fabs(t) : A + fabs(t);
            sg |= (t < 0.0 ? 1u : 0u) << p;
        }
        const bool better = A > bestA;                               // ties: the smaller s stays
        bestA = better ? A : bestA;
        best = better ? (uint32_t)(s - 1) : best;
        best_signs = better ? sg : best_signs;
    }
}

template <int BW>
__global__ __launch_bounds__(64 * QW) void quantize_kernel(const uint4 *__restrict__ w, int64_t nblocks,
                                                           uint2 *__restrict__ codes, uint8_t *__restrict__ pattern,
                                                           uint8_t *__restrict__ signs, uint16_t *__restrict__ c1,
                                                           uint16_t *__restrict__ c2)
{
    constexpr int E = 1 << (BW - 1);
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int row = lane >> 4, m = lane & 15;        // macro-block of the wavefront, micro-block of the macro-block
    const int64_t groups = (nblocks + ROWS - 1) / ROWS;

    for (int64_t grp = (int64_t)blockIdx.x * QW + wave; grp < groups; grp += (int64_t)gridDim.x * QW) {
        const int64_t mb_raw = grp * ROWS + row;
        const bool valid = mb_raw < nblocks;         // rows past the end repeat the last macro-block, store nothing
        const int64_t mb = valid ? mb_raw : nblocks - 1;
        const uint4 q = w[mb * 16 + m];
        const uint32_t pk[4] = {q.x, q.y, q.z, q.w};

        // macro-block normalisation s_norm = ||w||_inf: magnitude bits order like magnitudes
        uint32_t amax = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) amax = max(amax, max(pk[i] & 0x7fffu, (pk[i] >> 16) & 0x7fffu));
        amax = row_max(amax);
        const bool zero_block = amax == 0;           // nothing to represent: zero codes, c1 = c2 = 0
        const float sn = (float)__builtin_bit_cast(_Float16, (unsigned short)amax);

        // nearest states.  Thresholds common to both signs: 0.75 2^-k s_norm, k = 0 .. E-3; then a
        // negative weight has the state 2^-(E-1) (midpoints 0.75 2^-(E-2) s_norm and, to zero,
        // 2^-E s_norm), a positive one ends at 2^-(E-2) (midpoint to zero 2^-(E-1) s_norm).
        const int T075 = (int)__float_as_uint(0.75f * sn);
        const int Tzero = zero_block ? 0x7f000000 : (int)__float_as_uint(sn) - ((E - 1) << 23);
        double wv[8], x[8];
        int codes_lo = 0, codes_hi = 0;                              // minus the codes, byte i
        double s1 = 0.0, n1 = 0.0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float wf = (float)__builtin_bit_cast(_Float16, (unsigned short)(pk[i >> 1] >> (16 * (i & 1))));
            wv[i] = (double)wf;
            const uint32_t bits = __float_as_uint(wf);
            const int neg = (int)bits >> 31;                         // -1 for a negative weight
            // Number of thresholds |w| does not exceed.  |w| (11 significant bits) and 0.75 s_norm
            // (13) are exact in fp32 and order like their bits, and a factor 2^k is k units of the
            // exponent field: |w| 2^k <= 0.75 s_norm  <=>  A + (k << 23) <= T.  That holds for
            // k = 0 .. (T - A) >> 23 when T >= A and for no k otherwise; a negative weight has E - 1
            // such thresholds, a positive one E - 2, and below the midpoint to zero it is zero.
            // ne is minus that number (-((T - A) >> 23) - 1 = (A - T - 1) >> 23): the state's exponent,
            // which goes into the exponent field and the code by shift-and-add.
            const int A = (int)(bits & 0x7fffffffu);
            int ne;
            asm("v_med3_i32 %0, %1, 0, %2" : "=v"(ne) : "v"((A - T075 - 1) >> 23), "v"(neg - (E - 2)));
            const bool is_zero = A <= Tzero + (neg << 23);
            int nc = is_zero ? 1 - E : (neg << (BW - 1)) + ne;       // minus the code
            asm("" : "+v"(nc));                                      // keeps the shift below out of the selection
            if (i < 4) codes_lo += nc << (8 * i);
            else codes_hi += nc << (8 * (i - 4));
            // b1_i = +-2^ne assembled from sign and exponent field (low word zero); a zero keeps the
            // weight's sign, so that x_i w_j and x_j w_i share a sign for every pair
            const int mag = is_zero ? 0 : (ne << 20) + (1023 << 20);
            x[i] = __hiloint2double((int)((uint32_t)mag | (bits & 0x80000000u)), 0);
            s1 = fma(wv[i], x[i], s1);                              // a weight and its state share the sign
            n1 = fma(x[i], x[i], n1);
        }
        const uint32_t code_lo = (uint32_t)-codes_lo, code_hi = (uint32_t)-codes_hi;
        if (valid) codes[mb * 16 + m] = make_uint2(code_lo, code_hi);
        const double S1 = row_sum(s1);
        const double N1 = (double)row_sum((float)n1);    // > 0 unless the block is zero: the largest weight maps to +-1

        // the four patterns: exact cross terms, scores and sign bits.  u is never -0 (the difference of
        // two equal numbers is +0, of two zeros of one sign too), so its sign bit says u < 0.
        double U[4];
        uint32_t sg[4];
#pragma unroll
        for (int s = 1; s <= 4; ++s) {
            double sum = 0.0;
            uint32_t bit = 0;
#pragma unroll
            for (int p = 3; p >= 0; --p) {
                const int i = pair_lower(s, p), j = i ^ s;
                const double u = fma(x[i], wv[j], -(x[j] * wv[i]));
                sum += fabs(u);
                bit = __builtin_amdgcn_alignbit(bit, (uint32_t)__double2hiint(u), 31);    // 2 bit + sign of u
            }
            U[s - 1] = sum;
            sg[s - 1] = bit;
        }
        const double top = fmax(fmax(U[0], U[1]), fmax(U[2], U[3]));
        const double limit = fma((double)sn, -0x1p-44, top);
        const bool k0 = U[0] >= limit, k1 = U[1] >= limit, k2 = U[2] >= limit, k3 = U[3] >= limit;
        uint32_t best = k0 ? 0u : k1 ? 1u : k2 ? 2u : 3u;
        uint32_t best_signs = k0 ? sg[0] : k1 ? sg[1] : k2 ? sg[2] : sg[3];
        // scores too close to tell without their roundings (all zero: the first pattern, no signs)
        const bool close = ((k0 && (k1 || k2 || k3)) || (k1 && (k2 || k3)) || (k2 && k3)) && top > 0.0;
        if (__any(close)) {
            uint32_t b = 0, bs = 0;
            choose_by_residual(wv, x, S1 / N1, b, bs);
            if (close) { best = b; best_signs = bs; }
        }
        if (valid) {
            pattern[mb * 16 + m] = (uint8_t)best;
            signs[mb * 16 + m] = (uint8_t)best_signs;
        }
        // <w, b2> of the chosen pattern, and the GEO coefficients, Eq. 2 (the normal equations are
        // diagonal: <b1, b2> = 0): lane 0 of the row divides for c1, lane 1 for c2
        double d = best == 0 ? U[0] : best == 1 ? U[1] : best == 2 ? U[2] : U[3];
        const double S2 = row_sum(d);
        if (valid && m < 2) {
            const double c = zero_block ? 0.0 : (m == 0 ? S1 : S2) / N1;
            (m == 0 ? c1 : c2)[mb] = (uint16_t)double_to_half_bits(c);
        }
    }
}

}  // namespace

int goq_launch_quantize(hipStream_t st, int bw, int64_t out, int64_t in, const uint16_t *w, uint8_t *codes,
                        uint8_t *pattern, uint8_t *signs, uint16_t *c1, uint16_t *c2)
{
    const int64_t nblocks = out * (in / GOQ_N);
    int64_t grid = (nblocks + QW * ROWS - 1) / (QW * ROWS);
    if (grid > 256 * 32) grid = 256 * 32;            // every wavefront walks its share of the row groups
    if (bw == 3)
        hipLaunchKernelGGL(quantize_kernel<3>, dim3((unsigned)grid), dim3(64 * QW), 0, st, (const uint4 *)w, nblocks,
                           (uint2 *)codes, pattern, signs, c1, c2);
    else
        hipLaunchKernelGGL(quantize_kernel<4>, dim3((unsigned)grid), dim3(64 * QW), 0, st, (const uint4 *)w, nblocks,
                           (uint2 *)codes, pattern, signs, c1, c2);
    return goq_check_launch("goq_quantize");
}
