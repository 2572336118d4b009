// goq_quantize: the data-free GEO-mode quantizer on the device (Sec. 3.2 - 3.4): fp16 weights of a
// layer [out][in] -> canonical arrays (codes, pattern, signs, c1, c2).
//
// One LANE per micro-block of 8 weights, one ROW of 16 lanes per macro-block of 128 weights, four
// macro-blocks per wavefront and step.  Everything that belongs to a micro-block -- nearest states, the 16
// cross terms of the four exchange patterns, scores, argmax, pair signs, the exchange itself -- is
// lane-local and lives in registers; what belongs to the macro-block -- the norm s_norm and the
// sums of Eq. 1 and Eq. 2 -- is reduced across the 16 lanes of a row with data-parallel-primitive
// (DPP) moves, which stay inside a row by construction.  No LDS, no barriers.
//
// The outputs are those of a sequential fp64 evaluation, bit for bit, but fp64 is only used where fp32 cannot vouch for
// them: on this chip v_fma_f32, v_add_f32 and the like take 2.4 cycles, fp64 operations and most others more than 4.
//
//   products    A lattice state is a signed power of two, so every product with a state is exact, in
//               fp32 too (11 significant bits).  ||b1||^2 = ||b2||^2 is a multiple of 2^-14 of at most 128: exact in fp32.
//   nearest     Q(v), v = w / s_norm (Sec. 3.2), is decided without the division: |v| lies above
//               the midpoint 0.75 * 2^-k of the states 2^-k and 2^-(k+1) exactly when
//               |w| > 0.75 * 2^-k * s_norm, and above the midpoint to zero, 2^-(emin+1), when
//               |w| > 2^-(emin+1) * s_norm.  The thresholds fall with k, so the exponent of the
//               nearest state is the NUMBER of thresholds |w| does not exceed, and that number is
//               a difference of fp32 exponent fields (nearest_states); an exact tie goes to the
//               smaller magnitude.
//   cross terms The method's cross term of a pair is t = x_i r_j - x_j r_i with the residual
//               r = w - c b1, c = <w,b1> / ||b1||^2 (Eq. 1, Sec. 3.3), x = b1.  The c terms cancel:
//               in real arithmetic t = u = x_i w_j - x_j w_i.  One fused operation rounds u once, so its sign is right
//               (u is a multiple of 2^-31: nothing underflows).  A sequential fp64 evaluation rounds r and t, which moves t by less
//               than 2^-50 s_norm; it has the sign of u, because a nonzero u is at least 2^-31 (and where
//               u = 0 the states and weights of the pair are proportional by a power of two, or
//               zero, and so are the rounded residuals: t = 0).  So eta = sgn(u) (+1 at zero).
//   pattern     The scores A_s = sum |t| equal U_s = sum |u| within 2^-46 s_norm, and a U_s in fp32 has three roundings at most: s* =
//               argmax U_s unless a second score lies within 2^-20 of the largest (and 2^-43 s_norm).  Then -- 0.4 % of the micro-blocks of normal
//               weights for bw = 3, 0.1 % for bw = 4, nearly all of them equal scores -- the wavefront evaluates residuals and t as the method
//               writes them in fp64, to let their roundings decide as the sequential evaluation does
//               (ties: smallest s).  The pair's share of <w, b2> under the Theorem 1 exchange
//               (b2_i = -eta x_j for the lower index, +eta x_i for the upper one) is eta u = |u|:
//               U_s* is <w, b2> of the micro-block.
//   sums        <w, b1> and <w, b2> are sums of terms of one sign, so every rounding on the way is at most 2^-24 of the
//               result.  Longest way, from weight to quotient (the quotient itself counts as two): bw = 3, where a lane's sum of w x
//               has 21 bits and u 19, eight roundings; bw = 4 ten.  The fp16 coefficient is the rounded quotient unless that lies within
//               as many last places of a midpoint of two fp16 numbers (or outside their normal range): then (0.25 % of the coefficients) both sums are taken
//               in fp64, where they are exact -- multiples of 2^-31 below 2^23; always for bw = 3, for bw = 4 unless |<w, b>| reaches 2^22,
//               i.e. more than 64 weights of the block at the fp16 maximum -- and divided and rounded there.
//
// Bound now by both, vector-ALU issue (about 255 instructions per micro-block, some 840 cycles) and memory (3.3 bytes per weight).  Measured, 4096 x 11008
// (us, all sums and cross terms in fp64, 391 instructions, a byte or two per lane and store / this): bw = 3 63.6 / 46.9, bw = 4 58.2 / 42.5; 4096 x 4096 bw = 3
// 25.9 / 20.8.  Of the rest, the fp64 evaluation of close scores takes 6 us for bw = 3.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>
#include "goq_layout.h"
#include "goq_internal.h"

namespace {

constexpr int QW = 4;                        // wavefronts per workgroup
constexpr int PER_CU = 24;                   // workgroups per CU: four or five at a time, the rest evens out what close scores cost
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

// Pattern of a micro-block (s - 1) as Sec. 3.3 writes it: residuals r = w - c x, cross terms and scores in fp64 in pair order.
__device__ __forceinline__ uint32_t choose_by_residual(const float (&wf)[8], const float (&x)[8], double c)
{
    double r[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = fma(-c, (double)x[i], (double)wf[i]);       // (c x is exact)
    double bestA = -1.0;
    uint32_t best = 0;
#pragma unroll
    for (int s = 1; s <= 4; ++s) {
        double A = 0.0;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int i = pair_lower(s, p), j = i ^ s;
            const double t = fma((double)x[i], r[j], -((double)x[j] * r[i]));      // (the products are exact)
            A = (p == 0) ? fabs(t) : A + fabs(t);
        }
        const bool better = A > bestA;                               // ties: the smaller s stays
        bestA = better ? A : bestA;
        best = better ? (uint32_t)(s - 1) : best;
        __builtin_amdgcn_sched_barrier(0);                           // (one pattern after the other: registers)
    }
    return best;
}

// The score of pattern best + 1 in fp64 (exact): the micro-block's share of <w, b2>.  (All four patterns: a branch per pattern
// would be four of them, one after the other.)
__device__ __forceinline__ double exact_score(const float (&wf)[8], const float (&x)[8], uint32_t best)
{
    double got = 0.0;
#pragma unroll
    for (int s = 1; s <= 4; ++s) {
        double sum = 0.0;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int i = pair_lower(s, p), j = i ^ s;
            sum += fabs(fma((double)x[i], (double)wf[j], -((double)x[j] * (double)wf[i])));
        }
        got = best == (uint32_t)(s - 1) ? sum : got;
        __builtin_amdgcn_sched_barrier(0);
    }
    return got;
}

// c >= 0, rounded once to fp16: cut off to fp32 with the last place set where anything was cut off, then rounded.
__device__ __forceinline__ uint32_t half_bits(double c)
{
    const float f = (float)c;
    const double back = (double)f;
    uint32_t bits = __float_as_uint(f) - (back > c ? 1u : 0u);
    bits |= back != c ? 1u : 0u;
    return __half_as_ushort(__float2half(__uint_as_float(bits)));
}

// What a lane has of one macro-block: its eight weights, their states and the macro-block's norm.
struct States {
    float wf[8], x[8], sn;
    // What is computed from here on is not computed before (a conversion that two branches share is otherwise moved out of both).
    __device__ __forceinline__ void stay()
    {
#pragma unroll
        for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(wf[i]), "+v"(x[i]));
    }
};

// Nearest states.  Thresholds common to both signs: 0.75 2^-k s_norm, k = 0 .. E-3; then a
// negative weight has the state 2^-(E-1) (midpoints 0.75 2^-(E-2) s_norm and, to zero,
// 2^-E s_norm), a positive one ends at 2^-(E-2) (midpoint to zero 2^-(E-1) s_norm).
//
// |w| (11 significant bits) and 0.75 s_norm (13) are exact in fp32 and order like their bits, and a
// factor 2^k is k units of the exponent field.  With A the bits of |w| and T those of 0.75 s_norm the
// number of thresholds that |w| does not exceed is minus the floor of (A - T - 1) / 2^23, and the state is 2^ to that
// floor: the exponent field of A - T - 1 + bits(1), cut off below at the sign's smallest state (never above 1, because
// |w| <= s_norm).
template <int BW>
__device__ __forceinline__ void nearest_states(const uint4 &q, States &v)
{
    constexpr int E = 1 << (BW - 1);
    const uint32_t pk[4] = {q.x, q.y, q.z, q.w};
    uint32_t amax = 0;                               // s_norm = ||w||_inf: magnitude bits order like magnitudes
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        v.wf[i] = (float)__builtin_bit_cast(_Float16, (unsigned short)(pk[i >> 1] >> (16 * (i & 1))));
        asm("" : "+v"(v.wf[i]));                     // (its sign is taken from here, not from the half it came from)
        amax = max(amax, __float_as_uint(v.wf[i]) & 0x7fffffffu);
    }
    amax = row_max(amax);
    v.sn = __uint_as_float(amax);
    uint32_t T1 = __float_as_uint(0.75f * v.sn) + 1u - 0x3f800000u;
    asm("" : "+v"(T1));
    const int Tzero = amax == 0 ? 0x7f000000 : (int)amax - ((E - 1) << 23);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t bits = __float_as_uint(v.wf[i]);
        const uint32_t A = bits & 0x7fffffffu;
        const uint32_t one = (bits >> 8) & 0x00800000u;          // a negative weight: one more exponent
        const int state = max((int)((A - T1) & 0xff800000u), (int)(((127 - (E - 2)) << 23) - one));
        // (a zero keeps the weight's sign, so that x_i w_j and x_j w_i share a sign for every pair)
        const uint32_t mag = (int)(A + one) <= Tzero ? 0u : (uint32_t)state;
        v.x[i] = __uint_as_float(mag | (bits & 0x80000000u));
    }
}

// G: groups of four macro-blocks per round of a wavefront, 1 or 2
template <int BW, int G>
__global__ __launch_bounds__(64 * QW) void quantize_kernel(const uint4 *__restrict__ w, int64_t nblocks,
                                                      uint2 *__restrict__ codes, uint8_t *__restrict__ pattern,
                                                      uint8_t *__restrict__ signs, uint16_t *__restrict__ c1,
                                                      uint16_t *__restrict__ c2)
{
    constexpr int E = 1 << (BW - 1);
    constexpr uint32_t MARGIN = BW == 3 ? 9 : 11;   // fp32 last places a coefficient may be off (see above), and one to spare
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane >> 4, m = lane & 15;        // macro-block of the wavefront, micro-block of the macro-block
    const int64_t groups = (nblocks + ROWS - 1) / ROWS;
    const int64_t stride = (int64_t)gridDim.x * QW * G;

    // Group grp: its first macro-block (uniform), and this lane's from there.  Rows past the end repeat the last macro-block (and store it again),
    // so that every request and store is unconditional and the compiler's wait for the next weights leaves the stores alone.
    struct Place {
        int64_t base;
        uint32_t at;
    };
    auto place_of = [&](int64_t grp) {
        const int64_t base = min(grp * ROWS, nblocks - 1);
        return Place{base, (uint32_t)min(row, (int)min(nblocks - 1 - base, (int64_t)(ROWS - 1)))};
    };
    auto request = [&](int64_t grp) {
        const Place p = place_of(grp);
        return *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(w + p.base * 16) + (p.at * 16 + m) * 16);
    };
    // What lane r of a quad stores for two groups of its row: r & 1: patterns and c1, or signs and c2; r >> 1: of which group.
    const int r = m & 3;
    uint8_t *const choices = (r & 1 ? signs : pattern) + (m & ~3);
    uint16_t *const cs = r & 1 ? c2 : c1;
    const uint32_t take1 = r & 1 ? 0x03070105u : 0x06020400u, take2 = r & 2 ? 0x03020706u : 0x05040100u;

    int64_t grp = ((int64_t)blockIdx.x * QW + wave) * G;
    if (grp >= groups) return;
    uint4 next = request(grp);
    // (waited for here: were it still on its way when the loop is entered, the wait inside would be for everything, the
    // last round's stores included)
    asm volatile("" : "+v"(next.x), "+v"(next.y), "+v"(next.z), "+v"(next.w));
    for (; grp < groups; grp += stride) {
        uint32_t choice = 0, coefficient[2];         // pattern and signs of either group, a byte each; c1 (even lanes) or c2
#pragma unroll
        for (int h = 0; h < G; ++h) {
            const Place p = place_of(grp + h);
            States v;
            nearest_states<BW>(next, v);
            next = request(h + 1 < G ? grp + 1 : grp + stride);
            const float (&wf)[8] = v.wf;
            const float (&x)[8] = v.x;

            // Codes, four at a time: the high byte of a state as fp16 is sign << 7 | (15 - e) << 2, of a zero the sign only (e = 15,
            // whose low bits are those of the zero code; it loses the sign).
            uint32_t code[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const uint32_t a = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(x[4 * k], x[4 * k + 1]));
                const uint32_t b = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(x[4 * k + 2], x[4 * k + 3]));
                const uint32_t t = __builtin_amdgcn_perm(b, a, 0x07050301u) ^ 0x3c3c3c3cu;
                code[k] = ((t >> 2) & ((E - 1) * 0x01010101u)) | ((t & ~(t << 2) & 0x80808080u) >> (8 - BW));
            }
            *reinterpret_cast<uint2 *>(reinterpret_cast<char *>(codes + p.base * 16) + (p.at * 16 + m) * 8) = make_uint2(code[0], code[1]);

            float s1[2], n1 = x[0] * x[0];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                s1[k] = wf[4 * k] * x[4 * k];
#pragma unroll
                for (int i = 1; i < 4; ++i) s1[k] = fmaf(wf[4 * k + i], x[4 * k + i], s1[k]);
            }
#pragma unroll
            for (int i = 1; i < 8; ++i) n1 = fmaf(x[i], x[i], n1);
            const float S1 = row_sum(s1[0] + s1[1]);
            const float N1 = row_sum(n1);                    // exact; > 0 unless the block is zero
            auto block_sum1 = [&] {                          // S1 without rounding
                double e = 0.0;
                if constexpr (BW == 3) e = (double)(s1[0] + s1[1]);
                else
#pragma unroll
                    for (int i = 0; i < 8; ++i) e = fma((double)wf[i], (double)x[i], e);
                return row_sum(e);
            };

            // the four patterns: cross terms, scores and sign bits
            float U[4];
            uint32_t sg[4];
#pragma unroll
            for (int s = 1; s <= 4; ++s) {
                float u[4];
                uint32_t bit = 0;
#pragma unroll
                for (int p = 3; p >= 0; --p) {
                    const int i = pair_lower(s, p), j = i ^ s;
                    u[p] = fmaf(x[i], wf[j], -(x[j] * wf[i]));
                    bit = __builtin_amdgcn_alignbit(bit, __float_as_uint(u[p]), 31);    // 2 bit + sign of u
                }
                U[s - 1] = (fabsf(u[0]) + fabsf(u[1])) + (fabsf(u[2]) + fabsf(u[3]));
                asm volatile("" : "+v"(bit));                   // (here: kept for later, the cross terms take sixteen registers)
                sg[s - 1] = bit;
            }
            const float top = fmaxf(fmaxf(U[0], U[1]), fmaxf(U[2], U[3]));
            const float limit = fmaf(v.sn, -0x1p-43f, fmaf(top, -0x1p-20f, top));
            bool k0 = U[0] >= limit, k1 = U[1] >= limit, k2 = U[2] >= limit, k3 = U[3] >= limit;
            float d = top;
            // scores too close to tell without their roundings (all zero: the first pattern, no signs)
            const uint64_t b0 = __ballot(k0), b1 = __ballot(k1), b2 = __ballot(k2), b3 = __ballot(k3);
            const uint64_t tied = ((b0 & b1) | (b2 & b3) | ((b0 | b1) & (b2 | b3))) & __ballot(top > 0.f);
            if (tied) {
                const bool close = (tied >> lane) & 1;
                v.stay();
                const uint32_t b = choose_by_residual(wf, x, block_sum1() / (double)N1);
                k0 = close ? b == 0 : k0;
                k1 = close ? b == 1 : k1;
                k2 = close ? b == 2 : k2;
                d = close ? (b == 0 ? U[0] : b == 1 ? U[1] : b == 2 ? U[2] : U[3]) : top;
            }
            const bool low = k0 || k1;
            const uint32_t best = low ? (k0 ? 0u : 1u) : (k2 ? 2u : 3u);
            const uint32_t best_signs = low ? (k0 ? sg[0] : sg[1]) : (k2 ? sg[2] : sg[3]);
            choice |= (best | best_signs << 8) << (16 * h);

            // <w, b2> of the chosen pattern, and the GEO coefficients, Eq. 2 (the normal equations are
            // diagonal: <b1, b2> = 0)
            const float S2 = row_sum(d);
            const float S = m & 1 ? S2 : S1;
            const float rn = __builtin_amdgcn_rcpf(N1);
            float cf = S * rn;
            cf = fmaf(fmaf(-cf, N1, S), rn, cf);
            cf = S == 0.f ? 0.f : cf;
            coefficient[h] = __half_as_ushort(__float2half(cf));
            const uint32_t cb = __float_as_uint(cf);
            const bool near = (((cb + (MARGIN - 0x1000)) & 0x1fffu) <= 2 * MARGIN) | (cb - 0x38800000u >= 0x477f0000u - 0x38800000u);
            if (__any(near & (S != 0.f))) {
                v.stay();
                const double E1 = block_sum1(), E2 = row_sum(exact_score(wf, x, best));
                coefficient[h] = v.sn == 0.f ? 0u : half_bits((m & 1 ? E2 : E1) / (double)N1);
            }
        }
        if constexpr (G == 1) {
            choice |= choice << 16;
            coefficient[1] = coefficient[0];
        }
        // the four bytes of the four lanes of a quad change places: lane r gets byte r of each
        choice = __builtin_amdgcn_perm(dpp32<QUAD_SWAP1>(choice), choice, take1);
        choice = __builtin_amdgcn_perm(dpp32<QUAD_SWAP2>(choice), choice, take2);
        const Place p = place_of(grp);
        const uint32_t at = min((uint32_t)(row + ROWS * (G - 1) * (r >> 1)), (uint32_t)min(nblocks - 1 - p.base, (int64_t)(G * ROWS - 1)));
        __builtin_memcpy(choices + p.base * 16 + at * 16, &choice, 4);
        cs[p.base + at] = (uint16_t)(r & 2 ? coefficient[1] : coefficient[0]);
    }
}

}  // namespace

int goq_launch_quantize(hipStream_t st, int bw, int64_t out, int64_t in, const uint16_t *w, uint8_t *codes,
                        uint8_t *pattern, uint8_t *signs, uint16_t *c1, uint16_t *c2)
{
    const int64_t nblocks = out * (in / GOQ_N);
    // Two groups per round share the stores of patterns, signs and coefficients (4096 x 11008, bw = 3: 47.7 -> 46.9 us), one
    // where wavefronts are few (1500 x 1024: 6.4 -> 6.1).  Every wavefront has the same number of rounds, but for the last workgroup.
    const int64_t groups = (nblocks + ROWS - 1) / ROWS;
    const bool pairs = groups > 6144;
    const int64_t work = (groups + (pairs ? 1 : 0)) / (pairs ? 2 : 1);              // rounds of all wavefronts
    const int64_t most = (work + 256 * PER_CU * QW - 1) / (256 * PER_CU * QW);      // of one
    const unsigned grid = (unsigned)((work + most * QW - 1) / (most * QW));
    const auto kernel = bw == 3 ? (pairs ? quantize_kernel<3, 2> : quantize_kernel<3, 1>) : (pairs ? quantize_kernel<4, 2> : quantize_kernel<4, 1>);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(64 * QW), 0, st, (const uint4 *)w, nblocks, (uint2 *)codes, pattern, signs, c1, c2);
    return goq_check_launch("goq_quantize");
}
