// Integer activations on their way to matrix operands: unpacking of the packed storage types
// (GOQ_A4, GOQ_A6, GOQ_A3) to bytes, and widening of int8 to fp16 (exact).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "goq_decode.h"
#include "../../include/goq.h"

// bytes of a macro-block of activations
template <int ACT>
constexpr int goq_block_bytes() { return ACT == GOQ_A16 ? 256 : ACT == GOQ_A8 ? 128 : ACT == GOQ_A4 ? 64 : ACT == GOQ_A6 ? 96 : 48; }

// four int8 -> two registers of two fp16, without a conversion instruction: 0x6400 | u is the
// fp16 number 1024 + u
__device__ __forceinline__ void goq_widen_i8(uint32_t d, uint32_t &h0, uint32_t &h1)
{
    const goq_half2 off = {(_Float16)1152.f, (_Float16)1152.f};
    const uint32_t u = d ^ 0x80808080u;                        // x + 128
    h0 = __builtin_bit_cast(uint32_t, __builtin_bit_cast(goq_half2, goq_perm(0x64646464u, u, 0x04010400u)) - off);
    h1 = __builtin_bit_cast(uint32_t, __builtin_bit_cast(goq_half2, goq_perm(0x64646464u, u, 0x04030402u)) - off);
}

// eight int4 (element i in nibble i) -> two registers of four int8
__device__ __forceinline__ void goq_unpack_i4(uint32_t d, uint32_t &b0, uint32_t &b1)
{
    auto sext = [](uint32_t v) {      // per byte: low nibble, two's complement -> int8
        return ((((v ^ 0x08080808u) | 0x80808080u) - 0x08080808u) ^ 0x80808080u);
    };
    const uint32_t ev = sext(d & 0x0F0F0F0Fu);                 // elements 0, 2, 4, 6
    const uint32_t od = sext((d >> 4) & 0x0F0F0F0Fu);          // elements 1, 3, 5, 7
    b0 = goq_perm(od, ev, 0x05010400u);                        // elements 0, 1, 2, 3
    b1 = goq_perm(od, ev, 0x07030602u);                        // elements 4, 5, 6, 7
}

// four int6 (24 bits, element i in bits 6 i .. 6 i + 5) -> one register of four int8
__device__ __forceinline__ uint32_t goq_unpack_i6(uint32_t v)
{
    const uint32_t b = (v & 0x3Fu) | ((v << 2) & 0x3F00u) | ((v << 4) & 0x3F0000u) | ((v << 6) & 0x3F000000u);
    return ((((b ^ 0x20202020u) | 0x80808080u) - 0x20202020u) ^ 0x80808080u);   // per byte: 6 -> 8 bits, signed
}

// eight int3 (24 bits, element i in bits 3 i .. 3 i + 2) -> two registers of four int8
__device__ __forceinline__ void goq_unpack_i3(uint32_t v, uint32_t &b0, uint32_t &b1)
{
    auto spread = [](uint32_t t) {
        const uint32_t b = (t & 0x7u) | ((t << 5) & 0x700u) | ((t << 10) & 0x70000u) | ((t << 15) & 0x7000000u);
        return ((((b ^ 0x04040404u) | 0x80808080u) - 0x04040404u) ^ 0x80808080u);   // per byte: 3 -> 8 bits, signed
    };
    b0 = spread(v);
    b1 = spread(v >> 12);
}

// eight int4 / int3 as eight 8-bit floats (E5M2), elements 0..3 in b0 and 4..7 in b1: 0..7 are
// 00 3C 40 42 44 45 46 47, negative numbers have the sign bit, -8 is C8
__device__ __forceinline__ void goq_e5m2_i4(uint32_t d, uint32_t &b0, uint32_t &b1)
{
    // both halves are looked up by the low three bits, then picked by the sign bit (selector byte i = i
    // or 4 + i)
    auto four = [](uint32_t n, uint32_t pick) {
        const uint32_t e = n & 0x07070707u;
        return goq_perm(goq_perm(0xBCC0C2C4u, 0xC5C6C7C8u, e), goq_perm(0x47464544u, 0x42403C00u, e), pick | 0x03020100u);
    };
    const uint32_t ev = four(d, (d >> 1) & 0x04040404u);           // elements 0, 2, 4, 6
    const uint32_t od = four(d >> 4, (d >> 5) & 0x04040404u);      // elements 1, 3, 5, 7
    b0 = goq_perm(od, ev, 0x05010400u);
    b1 = goq_perm(od, ev, 0x07030602u);
}
__device__ __forceinline__ void goq_e5m2_i3(uint32_t v, uint32_t &b0, uint32_t &b1)
{
    auto four = [](uint32_t t) {
        const uint32_t e = (t & 0x7u) | ((t << 5) & 0x700u) | ((t << 10) & 0x70000u) | ((t << 15) & 0x7000000u);
        return goq_perm(0xBCC0C2C4u, 0x42403C00u, e);
    };
    b0 = four(v);
    b1 = four(v >> 12);
}

// the j-th group of 24 bits of a little-endian bit string of dwords
template <int NW>
__device__ __forceinline__ uint32_t goq_bits24(const uint32_t (&w)[NW], int j)
{
    const int dwi = (24 * j) >> 5, sh = (24 * j) & 31;
    return sh == 0 ? w[dwi] : sh == 8 ? (w[dwi] >> 8) : __builtin_amdgcn_alignbit(w[dwi + 1], w[dwi], sh);
}
