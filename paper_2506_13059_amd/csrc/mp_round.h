// Roundings to bf16 of the k-means means, as plain functions, so that they can be checked on the host.
#pragma once
#include <stdint.h>

namespace mp {

// fp64 -> bf16 with ONE rounding (nearest even).  The double is first truncated to fp32 with a
// sticky bit in the last place (round to odd), which makes the second rounding exact.  Values
// whose magnitude is below 2^-126 go to signed zero; overflow goes to infinity.
constexpr uint16_t f64_to_bf16_rne(double v)
{
    uint64_t b = __builtin_bit_cast(uint64_t, v);
    uint32_t sign = (uint32_t)(b >> 63) << 31;
    int32_t e = (int32_t)((b >> 52) & 0x7ff);
    uint64_t man = b & 0xfffffffffffffull;
    if (e == 0x7ff) {                                   // inf / nan
        uint32_t x = sign | 0x7f800000u | (man ? 0x400000u : 0u);
        return (uint16_t)(x >> 16);
    }
    int32_t fe = e - 1023 + 127;
    if (fe <= 0) return (uint16_t)(sign >> 16);         // below the fp32 normal range (incl. zero)
    if (fe >= 255) return (uint16_t)((sign | 0x7f800000u) >> 16);
    uint32_t m23 = (uint32_t)(man >> 29);
    uint32_t sticky = (man & ((1ull << 29) - 1)) ? 1u : 0u;
    uint32_t x = sign | ((uint32_t)fe << 23) | m23 | sticky;
    uint32_t lsb = (x >> 16) & 1u;
    uint32_t mag = (x & 0x7fffffffu) + 0x7fffu + lsb;   // may carry into the exponent: correct
    if (mag >= 0x7f800000u) mag = 0x7f800000u;
    return (uint16_t)((sign | mag) >> 16);
}

// bf16 of the quotient a / den (a whole number above 0, inv = 1 / den in fp64), as f64_to_bf16_rne(a / den) has it, without
// the division (some twenty instructions) wherever that cannot matter.  a * inv is within three units of the last place of the
// rounded quotient, and both round to the same bf16 value unless a number half way between two of them (the lower 45 bits
// of the mantissa: a one and zeros) or the end of the normal range is that near.
constexpr uint16_t quotient_to_bf16(double a, double den, double inv)
{
    double q = a * inv;
    const uint64_t b = __builtin_bit_cast(uint64_t, q);
    const uint32_t low = (uint32_t)b, e = (uint32_t)(b >> 52) & 0x7ffu;
    const bool half_way = (((uint32_t)(b >> 32) & 0x1fffu) == 0x1000u && low < 16u) || (((uint32_t)(b >> 32) & 0x1fffu) == 0xfffu && low > 0xfffffff0u);
    if (half_way || e - 900u > 245u) q = a / den;            // (exponents 2^-123 .. 2^122 are the ordinary case)
    return f64_to_bf16_rne(q);
}

}  // namespace mp
