// goq_gemm / goq_gemm_batch for up to 32 tokens (batched decode, verification of draft tokens; the line to the
// tile kernel is drawn in goq_gemm_rules.h), and
// goq_gemv / goq_gemv_batch of small layers as one token: Y[tokens][out] = X[tokens][in] * W^T (Eq. 4).
//
// What bounds it: the packed weights are read once for a handful of tokens, so the floor is the
// weight stream; the work per weight that has to hide behind it is the decode on the vector ALU
// (about 20 instructions per dword of 8 weights, widening to fp16 included).  The tile kernel of
// many tokens (64 tokens x 128 outputs, one workgroup walks the whole depth) starts out / 128
// workgroups: 32 for a 4096-wide layer, an eighth of the chip, one slab at a time.
//
// Split: a workgroup owns 16 RT output rows and all tokens; its eight wavefronts take
// the macro-blocks round-robin (wavefront w: slabs w, w + 8, ..), so a 4096 x 4096 layer is 256
// workgroups with four slabs per wavefront, and the eight partial tiles meet in LDS in a fixed
// order: no scratch memory, no atomics, one launch.  More rows per workgroup (RT) share one fetch of
// the activations, which is what limits large launches (64 bytes per CU and cycle).
//   B operand (weights): v_mfma_f32_16x16x32_f16, lane (c = l % 16, q = l / 16) holds the quad
//       (chunk q, row c) of the packed layout, micro-block 4 q + t in k-step t.
//   A operand (activations): lane (token = l % 16, q) holds the same k, 32 q + 8 t .. + 7: the 32
//       consecutive activations of its token that its quad multiplies.  They are read straight
//       from global memory (every workgroup reads all of X, which L2 holds), so nothing is
//       staged and no barrier stands before the final sum.
// Measured against the tile kernel (one launch, us, weights of three copies in turn): 4096 x 4096, 5 tokens,
// W4/A16: 38.2 -> 4.8; the seven matrices of a LLaMA-2-7B block, 16 tokens, W3/A16: 105 -> 32.4.
// (Tried: activations through LDS in whole rows, 36 us for the block; micro-block 4 t + q per lane, so that
// lanes of a load lie side by side but weights come in dwords: 52 us; four wavefronts: no gain.)
// Integer activations are widened to fp16 in registers; int8 values and powers of two down to 2^-7
// are exact in fp16 and a slab sum needs at most 22 bits, so the fp32 slab sums P1, P2 are exact.
// The coefficient pair is applied once per slab in fp32, as everywhere in this library.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include "goq_layout.h"
#include "goq_decode.h"
#include "goq_activations.h"
#include "goq_internal.h"
#include "goq_gemm_rules.h"

namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) unsigned char *gbytes;
typedef const __attribute__((address_space(1))) uint32_t *gptr;
typedef const __attribute__((address_space(1))) u32x2 *gptr2;
typedef const __attribute__((address_space(1))) u32x4 *gptr4;

constexpr int WAVES = 8;
constexpr int NT = WAVES * 64;
constexpr int VC = 16;                    // copies of the exchange table (lane l reads copy l % 16: no bank conflicts)
constexpr int VS = VC * 16;               // bytes from one entry to the next

struct SmallArgs {
    const uint32_t *packed;
    const void *X;
    const float *sx;
    void *Y;
    int32_t *partials;
    int tokens, out, gn, ytype;
};
// workgroups first[i] .. first[i + 1] - 1 own problem i (unused problems start at INT_MAX)
struct SmallBatch {
    int first[GOQ_MAX_BATCH];
    SmallArgs p[GOQ_MAX_BATCH];
};

// What a lane holds of one slab: per row tile its quad (and for bw = 4 the metadata dword), per
// token tile its 32 activations as they lie in memory.
template <int BW, int ACT, int MT, int RT>
struct Slab {
    static constexpr int XW = ACT == GOQ_A16 ? 16 : ACT == GOQ_A8 ? 8 : ACT == GOQ_A4 ? 4 : ACT == GOQ_A6 ? 6 : 3;   // dwords
    u32x4 q[RT];
    uint32_t md[BW == 4 ? RT : 1];
    uint32_t x[MT][XW];
};

__device__ __forceinline__ f16x8 widen8(uint32_t lo, uint32_t hi)
{
    const u32x4 v = {goq_widen01(lo), goq_widen23(lo), goq_widen01(hi), goq_widen23(hi)};
    return __builtin_bit_cast(f16x8, v);
}

// the 32 activations of a lane as four k-steps of eight fp16
template <int ACT, int XW>
__device__ __forceinline__ void as_half(const uint32_t (&x)[XW], f16x8 (&A)[4])
{
    uint32_t h[16];
    if constexpr (ACT == GOQ_A16) {
#pragma unroll
        for (int i = 0; i < 16; ++i) h[i] = x[i];
    } else if constexpr (ACT == GOQ_A8) {
#pragma unroll
        for (int i = 0; i < 8; ++i) goq_widen_i8(x[i], h[2 * i], h[2 * i + 1]);
    } else if constexpr (ACT == GOQ_A4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t b0, b1;
            goq_unpack_i4(x[i], b0, b1);
            goq_widen_i8(b0, h[4 * i], h[4 * i + 1]);
            goq_widen_i8(b1, h[4 * i + 2], h[4 * i + 3]);
        }
    } else if constexpr (ACT == GOQ_A6) {
#pragma unroll
        for (int i = 0; i < 8; ++i) goq_widen_i8(goq_unpack_i6(goq_bits24(x, i)), h[2 * i], h[2 * i + 1]);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t b0, b1;
            goq_unpack_i3(goq_bits24(x, i), b0, b1);
            goq_widen_i8(b0, h[4 * i], h[4 * i + 1]);
            goq_widen_i8(b1, h[4 * i + 2], h[4 * i + 3]);
        }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const u32x4 v = {h[4 * t], h[4 * t + 1], h[4 * t + 2], h[4 * t + 3]};
        A[t] = __builtin_bit_cast(f16x8, v);
    }
}

// rows: which of problem a's groups of 16 RT rows
template <int BW, int ACT, int MT, int RT, bool PART>
__device__ __forceinline__ void few_tokens(const SmallArgs &a, int rows)
{
    constexpr int CH = (BW == 3) ? 4 : 5;
    constexpr int XROW = goq_block_bytes<ACT>();
    using SlabT = Slab<BW, ACT, MT, RT>;
    __shared__ __attribute__((aligned(256))) unsigned char vtab[64 * VS];
    __shared__ __attribute__((aligned(16))) float red[WAVES][MT * RT][256];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, q = lane >> 4;

    const int rt0 = rows * RT;                                      // first 16-row tile; RT divides 4: one row block
    const int gn = a.gn;

    // rows: lane (c, q) reads chunk q of row 16 (rt0 + r) % 64 + c (rows past `out` lie in the padding)
    gptr wbase = (gptr)a.packed + (int64_t)(rt0 >> 2) * gn * (CH * GOQ_ROWS * 4);
    const uint32_t wrow = (uint32_t)((rt0 & 3) * 16 + c) * 4;
    // tokens: rows past the end repeat the last one, their results are not stored
    uint32_t xoff[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) xoff[m] = (uint32_t)(min(16 * m + c, a.tokens - 1) * gn) * XROW + q * (XROW / 4);
    gbytes xbase = (gbytes)a.X;

    auto load = [&](int g, SlabT &s) {
        gptr base = wbase + (int64_t)g * (CH * GOQ_ROWS * 4);
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            s.q[r] = __builtin_nontemporal_load((gptr4)(base + (q * (GOQ_ROWS * 4) + wrow + 64 * r)));
            if constexpr (BW == 4) s.md[r] = __builtin_nontemporal_load(base + (4 * (GOQ_ROWS * 4) + wrow + 64 * r + q));
        }
        gbytes xg = xbase + (int64_t)g * XROW;
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            // (One row tile, W4 with int3 and W3 with int8: the order of the requests is kept.  Left alone the compiler puts some of them behind half of
            // this slab's matrix instructions, or behind the wait for all of this slab; us, 17 to 31 tokens: W4/A3 2133 x 2048 and 342 x 2048 6.4 / 6.15,
            // 3026 x 1664 6.6 / 6.4; W3/A8 4734 x 2816 8.5 / 8.4, 5865 x 10112 20.3 / 20.2.  Two row tiles lose by it, W4/A3 11862 x 1536 11.7 / 12.0; W4 with
            // int8 needs 130 registers for it, so that no two workgroups fit a CU.)
            if constexpr ((BW == 4 ? ACT == GOQ_A3 : ACT == GOQ_A8) && MT == 2 && RT == 1) asm volatile("" ::: "memory");
            if constexpr (SlabT::XW % 4 == 0) {
#pragma unroll
                for (int i = 0; i < SlabT::XW / 4; ++i) {
                    const u32x4 v = *(gptr4)(xg + (xoff[m] + 16 * i));
                    s.x[m][4 * i] = v.x; s.x[m][4 * i + 1] = v.y; s.x[m][4 * i + 2] = v.z; s.x[m][4 * i + 3] = v.w;
                }
            } else if constexpr (SlabT::XW == 6) {
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const u32x2 v = *(gptr2)(xg + (xoff[m] + 8 * i));
                    s.x[m][2 * i] = v.x; s.x[m][2 * i + 1] = v.y;
                }
            } else {
#pragma unroll
                for (int i = 0; i < 3; ++i) s.x[m][i] = *(gptr)(xg + (xoff[m] + 4 * i));
            }
        }
    };

    SlabT bufA, bufB;
    if (wave < gn) load(wave, bufA);
    goq_write_exchange_table<0x80u, VC, WAVES>(vtab, wave, lane);
    __syncthreads();
    const uint32_t vt = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)vtab + (lane % VC) * 16;

    f32x4 acc[RT][MT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[r][m] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto compute = [&](const SlabT &s, int g) {
        f16x8 A[MT][4];
#pragma unroll
        for (int m = 0; m < MT; ++m) as_half<ACT>(s.x[m], A[m]);
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const uint32_t dw[4] = {s.q[r].x, s.q[r].y, s.q[r].z, s.q[r].w};
            // exchange-table entries of the four micro-blocks, requested before the decode
            u32x4 ev[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                uint32_t at;
                if constexpr (BW == 3) at = __builtin_amdgcn_udot4(dw[t] & 0x00C0C0C0u, 0x00100401u * (VS / 64), vt, false);
                else at = vt + ((s.md[r] >> (6 * t)) & 63u) * VS;
                ev[t] = *reinterpret_cast<const __attribute__((address_space(3))) u32x4 *>(at);
            }
            // the row's coefficient word: each of its four lanes holds one byte of it
            uint32_t cw;
            if constexpr (BW == 3) {
                cw = dw[0] >> 30;
#pragma unroll
                for (int t = 1; t < 4; ++t) cw = __builtin_amdgcn_alignbit(cw, dw[t], 30);
                cw <<= 8 * (3 - q);
            } else {
                cw = (s.md[r] >> 24) << (8 * q);
            }
            {
                const auto u = __builtin_amdgcn_permlane32_swap(cw, cw, false, false);
                cw = u[0] | u[1];
                const auto v = __builtin_amdgcn_permlane16_swap(cw, cw, false, false);
                cw = v[0] | v[1];
            }
            f32x4 P1[MT], P2[MT];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                uint32_t lo, hi;
                goq_decode_bytes<BW, 0>(dw[t], lo, hi);
                const f16x8 B1 = widen8(lo, hi);
                const f16x8 B2 = widen8(goq_perm(hi, lo, ev[t].x) ^ ev[t].z, goq_perm(hi, lo, ev[t].y) ^ ev[t].w);
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
                    P1[m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[m][t], B1, t ? P1[m] : z, 0, 0, 0);
                    P2[m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[m][t], B2, t ? P2[m] : z, 0, 0, 0);
                }
            }
            const float c1 = __half2float(__ushort_as_half((unsigned short)(cw & 0xffffu)));
            const float c2 = __half2float(__ushort_as_half((unsigned short)(cw >> 16)));
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[r][m][v] = fmaf(c2, P2[m][v], fmaf(c1, P1[m][v], acc[r][m][v]));
            if constexpr (PART) {
                // exact int32 slab partials [tokens][out][in/128][2] (verification output)
                if (a.partials) {
                    constexpr float UNIT = (float)(1 << ((1 << (BW - 1)) - 1));
                    const int row = 16 * (rt0 + r) + c;
#pragma unroll
                    for (int m = 0; m < MT; ++m)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int token = 16 * m + 4 * q + v;
                            if (token < a.tokens && row < a.out)
                                *reinterpret_cast<int2 *>(a.partials + (((int64_t)token * a.out + row) * gn + g) * 2) =
                                    make_int2((int)(P1[m][v] * UNIT), (int)(P2[m][v] * UNIT));
                        }
                }
            }
        }
    };
    // ping-pong: the next slab's loads are in flight while this one is computed; the last slab is
    // peeled so that every load in the loop is unconditional (exact wait counts)
    if (wave < gn) {
        int g = wave;
        while (true) {
            if (g + WAVES >= gn) { compute(bufA, g); break; }
            load(g + WAVES, bufB);
            compute(bufA, g);
            g += WAVES;
            if (g + WAVES >= gn) { compute(bufB, g); break; }
            load(g + WAVES, bufA);
            compute(bufB, g);
            g += WAVES;
        }
    }

    // H6: the eight partial tiles, added in wavefront order.  Register v of a 16 x 16 tile: token
    // 4 q + v, output row c.  Element (token, row) of tile (r, m) lies at red[..][m RT + r][token * 16 + row].
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[wave][m * RT + r][(4 * q + v) * 16 + c] = acc[r][m][v];
    __syncthreads();
    for (int i = tid; i < MT * RT * 256; i += NT) {
        const int tile = i >> 8, e = i & 255;
        const int token = 16 * (tile / RT) + (e >> 4);
        const int row = 16 * (rt0 + tile % RT) + (e & 15);
        float y = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) y += red[w][tile][e];
        if (token >= a.tokens || row >= a.out) continue;
        if constexpr (ACT != GOQ_A16) y *= a.sx[token];
        const int64_t at = (int64_t)token * a.out + row;
        if (a.ytype == GOQ_F32) reinterpret_cast<float *>(a.Y)[at] = y;
        else reinterpret_cast<__half *>(a.Y)[at] = __float2half(y);
    }
}

// int8, two token tiles: two to four wavefronts per SIMD.  Without the upper bound the compiler takes the instances with one row tile below 100
// registers, for five wavefronts that no workgroup of eight can use, and moves the next slab's loads behind the matrix instructions of this one
// (us, 18 tokens, W3/A8, W4/A8: 4096 x 11008 14.4, 16.8 -> 12.7, 13.9; three of 2048 x 5120 12.4, 14.1 -> 11.8, 13.1).  The other types stay
// above 110 registers by themselves; bounded, int6 gains 5 % on deep layers and loses as much on others (768 x 3072, 32 tokens 7.3 -> 7.6).
template <int BW, int ACT, int MT, int RT, bool PART>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(MT == 2 || PART ? 2 : 4, MT == 2 && ACT == GOQ_A8 ? 4 : 8)))
void gemm_small_kernel(SmallBatch batch)
{
    int pi = 0;
#pragma unroll
    for (int i = 1; i < GOQ_MAX_BATCH; ++i) pi += ((int)blockIdx.x >= batch.first[i]) ? 1 : 0;
    pi = __builtin_amdgcn_readfirstlane(pi);
    few_tokens<BW, ACT, MT, RT, PART>(batch.p[pi], (int)blockIdx.x - batch.first[pi]);
}

// One problem, one row tile per workgroup: the launches that last a few microseconds.  The problem's fields are arguments of their own, so
// that they arrive in scalar registers with the wavefront (-amdgpu-kernarg-preload-count) and its first loads wait for no other; from a
// SmallBatch they come by two scalar loads, one after the other (us, batch / single: 4096 x 4096, one token, W3/A16 4.5 / 4.0; 5 tokens,
// W4/A16 5.5 / 4.9; 4096 x 11008, one token 8.6 / 8.0).
template <int BW, int ACT>
__global__ __launch_bounds__(NT, 4)
void gemm_small_single_kernel(const uint32_t *packed, const void *X, const float *sx, void *Y, int tokens, int out, int gn, int ytype)
{
    const SmallArgs a{packed, X, sx, Y, nullptr, tokens, out, gn, ytype};
    few_tokens<BW, ACT, 1, 1, false>(a, (int)blockIdx.x);
}

// alone: LDS that nothing uses keeps a second workgroup off the CU (goq_alone_on_cu)
template <int BW, int ACT, int MT, int RT>
int launch(hipStream_t st, const SmallBatch &b, int grid, bool part, bool alone, const char *what)
{
    constexpr unsigned SPARE = 57 * 1024;
    static_assert(2 * (64 * VS + WAVES * MT * RT * 1024 + SPARE) > 160 * 1024, "two workgroups do not fit");
    if constexpr (MT == 1 && RT == 1) {
        if (b.first[1] == 0x7fffffff && !part) {
            const SmallArgs &a = b.p[0];
            hipLaunchKernelGGL((gemm_small_single_kernel<BW, ACT>), dim3((unsigned)grid), dim3(NT), 0, st, a.packed, a.X, a.sx, a.Y, a.tokens, a.out,
                               a.gn, a.ytype);
            return goq_check_launch(what);
        }
    }
    if (ACT != GOQ_A16 && part)
        hipLaunchKernelGGL((gemm_small_kernel<BW, ACT, MT, RT, ACT != GOQ_A16>), dim3((unsigned)grid), dim3(NT), 0, st, b);
    else
        hipLaunchKernelGGL((gemm_small_kernel<BW, ACT, MT, RT, false>), dim3((unsigned)grid), dim3(NT), alone ? SPARE : 0, st, b);
    return goq_check_launch(what);
}

template <int BW, int ACT>
int launch_tiles(hipStream_t st, const SmallBatch &b, int grid, int mt, int rt, bool part, bool alone, const char *what)
{
    if (mt == 2) return rt == 1 ? launch<BW, ACT, 2, 1>(st, b, grid, part, alone, what) : launch<BW, ACT, 2, 2>(st, b, grid, part, alone, what);
    if constexpr (BW == 3)
        if (rt == 4) return launch<BW, ACT, 1, 4>(st, b, grid, part, alone, what);
    return rt == 1 ? launch<BW, ACT, 1, 1>(st, b, grid, part, alone, what) : launch<BW, ACT, 1, 2>(st, b, grid, part, alone, what);
}

template <int BW>
int launch_act(hipStream_t st, int act, const SmallBatch &b, int grid, int mt, int rt, bool part, bool alone, const char *what)
{
    if (act == GOQ_A16) return launch_tiles<BW, GOQ_A16>(st, b, grid, mt, rt, part, alone, what);
    if (act == GOQ_A8) return launch_tiles<BW, GOQ_A8>(st, b, grid, mt, rt, part, alone, what);
    if (act == GOQ_A4) return launch_tiles<BW, GOQ_A4>(st, b, grid, mt, rt, part, alone, what);
    if (act == GOQ_A6) return launch_tiles<BW, GOQ_A6>(st, b, grid, mt, rt, part, alone, what);
    return launch_tiles<BW, GOQ_A3>(st, b, grid, mt, rt, part, alone, what);
}

}  // namespace

int goq_launch_gemm_small(hipStream_t st, int bw, int act, int n, const goq_gemm_desc *descs, int row_tiles, const char *what)
{
    int64_t tiles16 = 0, most = 0;
    bool part = false;
    for (int i = 0; i < n; ++i) {
        tiles16 += (descs[i].out + 15) / 16;
        most = descs[i].tokens > most ? descs[i].tokens : most;
        part = part || descs[i].partials;
    }
    // Row tiles per workgroup: one until the chip is full (two workgroups per CU), then two; four
    // for launches of many row tiles, with 16 tokens and bw = 3 (the 7B block, 16 tokens: 2656 row
    // tiles, RT = 1, 2, 4: 54.8, 37.9, 34.7 us; bw = 4 and two token tiles have no registers for four).
    // (Neither choice changes a result: a row's sums are the same in every tile.)
    const int mt = most > 16 ? 2 : 1;
    const int rt = row_tiles ? row_tiles : tiles16 <= 512 ? 1 : mt == 2 || bw == 4 || tiles16 <= 2048 ? 2 : 4;
    GoqTileProblem p[GOQ_MAX_BATCH];
    for (int i = 0; i < n; ++i) p[i] = GoqTileProblem{(int)descs[i].tokens, (int)descs[i].out, (int)(descs[i].in / GOQ_N)};
    const bool alone = mt == 2 && rt == 1 && goq_alone_on_cu(act == GOQ_A16, n, p);
    // the problems with the deepest rows first: the launch should end with short ones
    int order[GOQ_MAX_BATCH];
    for (int i = 0; i < n; ++i) {
        int j = i;
        for (; j > 0 && descs[order[j - 1]].in < descs[i].in; --j) order[j] = order[j - 1];
        order[j] = i;
    }
    SmallBatch b;
    int64_t grid = 0;
    for (int i = 0; i < GOQ_MAX_BATCH; ++i) {
        if (i >= n) { b.first[i] = 0x7fffffff; b.p[i] = b.p[0]; continue; }
        const goq_gemm_desc &d = descs[order[i]];
        b.first[i] = (int)grid;
        SmallArgs &a = b.p[i];
        grid += (d.out + 16 * rt - 1) / (16 * rt);               // out <= 2^24: the sum stays below 2^24
        a.packed = (const uint32_t *)d.packed;
        a.X = d.X;
        a.sx = d.sx;
        a.Y = d.Y;
        a.partials = d.partials;
        a.tokens = (int)d.tokens;
        a.out = (int)d.out;
        a.gn = (int)(d.in / GOQ_N);
        a.ytype = d.ytype;
    }
    return bw == 3 ? launch_act<3>(st, act, b, (int)grid, mt, rt, part, alone, what)
                   : launch_act<4>(st, act, b, (int)grid, mt, rt, part, alone, what);
}
