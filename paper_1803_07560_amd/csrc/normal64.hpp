// The double-precision functions of the samplers that draw Gaussian numbers:
// logarithm, sine and cosine of a Philox word, roots.  Plain C++ on clang/GCC
// builtins, so the same arithmetic compiles for the GPU and for a host check;
// the includer sets BFI_HD (e.g. __device__).
//
// The arguments are narrow -- a word's uniform (x + 1/2) 2^-32, a radius, a sum
// of squares -- so nothing here scales, reduces or tests for what cannot occur,
// and small tables replace most of each series (Tang, "Table-driven
// implementation of the logarithm function in IEEE floating-point arithmetic",
// ACM TOMS 16 (1990); the same idea for the circle).  Tables of 64 pairs, from
// 60-digit decimal arithmetic, rounded to double.  Largest and mean error against
// long double, in units in the last place of the result: logarithm 1.52 and
// 0.37, roots 0.50 and 0.99 (reciprocal), 0.25 and 0.28; sine and cosine, in
// units of 2^-53, 0.64 and 0.1.
#pragma once

#include <cstdint>

#ifndef BFI_HD
#define BFI_HD
#define BFI_DATA
#else
#define BFI_DATA static __device__  // the tables too are the device's
#endif

namespace bfi {
namespace nrm {

// Interval i of [0x1.6p-1, 0x1.6p+0) is cut by the top bits of the significand
// from 0x1.6p-1 on: {1/c rounded, -2 ln c} for a c inside it (the middle, but 1
// in the interval below 1, where the logarithm must vanish with its argument).
BFI_DATA constexpr double kLog[64][2] = {
    {0x1.724287f46debcp+0, 0x1.79e26687cfb3dp-1}, {0x1.6e1f76b4337c7p+0, 0x1.6e60ee6af1973p-1},
    {0x1.6a13cd1537290p+0, 0x1.630030b3aac48p-1}, {0x1.661ec6a5122f9p+0, 0x1.57bf753c8d1fbp-1},
    {0x1.623fa77016240p+0, 0x1.4c9e09e172c3dp-1}, {0x1.5e75bb8d015e7p+0, 0x1.419b423d5e8c6p-1},
    {0x1.5ac056b015ac0p+0, 0x1.36b6776be1116p-1}, {0x1.571ed3c506b3ap+0, 0x1.2bef07cdc9355p-1},
    {0x1.5390948f40febp+0, 0x1.214456d0eb8d5p-1}, {0x1.5015015015015p+0, 0x1.16b5ccbacfb73p-1},
    {0x1.4cab88725af6ep+0, 0x1.0c42d676162e2p-1}, {0x1.49539e3b2d067p+0, 0x1.01eae5626c691p-1},
    {0x1.460cbc7f5cf9ap+0, 0x1.ef5ade4dcffe5p-2}, {0x1.42d6625d51f87p+0, 0x1.db13db0d48941p-2},
    {0x1.3fb013fb013fbp+0, 0x1.c6ffbc6f00f71p-2}, {0x1.3c995a47babe7p+0, 0x1.b31d8575bce3bp-2},
    {0x1.3991c2c187f63p+0, 0x1.9f6c407089663p-2}, {0x1.3698df3de0748p+0, 0x1.8beafeb38fe8fp-2},
    {0x1.33ae45b57bcb2p+0, 0x1.7898d85444c74p-2}, {0x1.30d190130d190p+0, 0x1.6574ebe8c1339p-2},
    {0x1.2e025c04b8097p+0, 0x1.527e5e4a1b58dp-2}, {0x1.2b404ad012b40p+0, 0x1.3fb45a59928cap-2},
    {0x1.288b01288b013p+0, 0x1.2d1610c86813dp-2}, {0x1.25e22708092f1p+0, 0x1.1aa2b7e23f729p-2},
    {0x1.23456789abcdfp+0, 0x1.08598b59e3a07p-2}, {0x1.20b470c67c0d9p+0, 0x1.ec739830a1126p-3},
    {0x1.1e2ef3b3fb874p+0, 0x1.c885801bc4b20p-3}, {0x1.1bb4a4046ed29p+0, 0x1.a4e7640b1bc38p-3},
    {0x1.19453808ca29cp+0, 0x1.8197e2f40e3f0p-3}, {0x1.16e0689427379p+0, 0x1.5e95a4d9791cdp-3},
    {0x1.1485f0e0acd3bp+0, 0x1.3bdf5a7d1ee5ep-3}, {0x1.12358e75d3033p+0, 0x1.1973bd1465561p-3},
    {0x1.0fef010fef011p+0, 0x1.eea31c006b87cp-4}, {0x1.0db20a88f4696p+0, 0x1.aaef2d0fb1108p-4},
    {0x1.0b7e6ec259dc8p+0, 0x1.67c94f2d4bb65p-4}, {0x1.0953f39010954p+0, 0x1.252f32f8d1840p-4},
    {0x1.073260a47f7c6p+0, 0x1.c63d2ec14aad7p-5}, {0x1.05197f7d73404p+0, 0x1.432a925980cbcp-5},
    {0x1.03091b51f5e1ap+0, 0x1.82448a388a283p-6}, {0x1.0000000000000p+0, 0x0.0p+0},
    {0x1.fc07f01fc07f0p-1, -0x1.fe02a6b106799p-7}, {0x1.f44659e4a4271p-1, -0x1.7b91b07d5b126p-5},
    {0x1.ecc07b301ecc0p-1, -0x1.39e87b9febd68p-4}, {0x1.e573ac901e574p-1, -0x1.b42dd711971b9p-4},
    {0x1.de5d6e3f8868ap-1, -0x1.16536eea37ae3p-3}, {0x1.d77b654b82c34p-1, -0x1.51b073f06183cp-3},
    {0x1.d0cb58f6ec074p-1, -0x1.8c345d6319b23p-3}, {0x1.ca4b3055ee191p-1, -0x1.c5e548f5bc743p-3},
    {0x1.c3f8f01c3f8f0p-1, -0x1.fec9131dbeabcp-3}, {0x1.bdd2b899406f7p-1, -0x1.1b72ad52f67a2p-2},
    {0x1.b7d6c3dda338bp-1, -0x1.371fc201e8f75p-2}, {0x1.b2036406c80d9p-1, -0x1.526e5e3a1b438p-2},
    {0x1.ac5701ac5701bp-1, -0x1.6d60fe719d21bp-2}, {0x1.a6d01a6d01a6dp-1, -0x1.87fa06520c911p-2},
    {0x1.a16d3f97a4b02p-1, -0x1.a23bc1fe2b561p-2}, {0x1.9c2d14ee4a102p-1, -0x1.bc286742d8cd4p-2},
    {0x1.970e4f80cb872p-1, -0x1.d5c216b4fbb94p-2}, {0x1.920fb49d0e229p-1, -0x1.ef0adcbdc5935p-2},
    {0x1.8d3018d3018d3p-1, -0x1.0402594b4d041p-1}, {0x1.886e5f0abb04ap-1, -0x1.1058bf9ae4ad4p-1},
    {0x1.83c977ab2beddp-1, -0x1.1c898c16999fbp-1}, {0x1.7f405fd017f40p-1, -0x1.2895a13de86a4p-1},
    {0x1.7ad2208e0ecc3p-1, -0x1.347dd9a987d56p-1}, {0x1.767dce434a9b1p-1, -0x1.404308686a7e4p-1},
};

// {cos, sin} of i/64 turn.
BFI_DATA constexpr double kTurn[64][2] = {
    {0x1.0000000000000p+0, 0x0.0p+0}, {0x1.fd88da3d12526p-1, 0x1.917a6bc29b42cp-4},
    {0x1.f6297cff75cb0p-1, 0x1.8f8b83c69a60bp-3}, {0x1.e9f4156c62ddap-1, 0x1.294062ed59f06p-2},
    {0x1.d906bcf328d46p-1, 0x1.87de2a6aea963p-2}, {0x1.c38b2f180bdb1p-1, 0x1.e2b5d3806f63bp-2},
    {0x1.a9b66290ea1a3p-1, 0x1.1c73b39ae68c8p-1}, {0x1.8bc806b151741p-1, 0x1.44cf325091dd6p-1},
    {0x1.6a09e667f3bcdp-1, 0x1.6a09e667f3bcdp-1}, {0x1.44cf325091dd6p-1, 0x1.8bc806b151741p-1},
    {0x1.1c73b39ae68c8p-1, 0x1.a9b66290ea1a3p-1}, {0x1.e2b5d3806f63bp-2, 0x1.c38b2f180bdb1p-1},
    {0x1.87de2a6aea963p-2, 0x1.d906bcf328d46p-1}, {0x1.294062ed59f06p-2, 0x1.e9f4156c62ddap-1},
    {0x1.8f8b83c69a60bp-3, 0x1.f6297cff75cb0p-1}, {0x1.917a6bc29b42cp-4, 0x1.fd88da3d12526p-1},
    {0x0.0p+0, 0x1.0000000000000p+0}, {-0x1.917a6bc29b42cp-4, 0x1.fd88da3d12526p-1},
    {-0x1.8f8b83c69a60bp-3, 0x1.f6297cff75cb0p-1}, {-0x1.294062ed59f06p-2, 0x1.e9f4156c62ddap-1},
    {-0x1.87de2a6aea963p-2, 0x1.d906bcf328d46p-1}, {-0x1.e2b5d3806f63bp-2, 0x1.c38b2f180bdb1p-1},
    {-0x1.1c73b39ae68c8p-1, 0x1.a9b66290ea1a3p-1}, {-0x1.44cf325091dd6p-1, 0x1.8bc806b151741p-1},
    {-0x1.6a09e667f3bcdp-1, 0x1.6a09e667f3bcdp-1}, {-0x1.8bc806b151741p-1, 0x1.44cf325091dd6p-1},
    {-0x1.a9b66290ea1a3p-1, 0x1.1c73b39ae68c8p-1}, {-0x1.c38b2f180bdb1p-1, 0x1.e2b5d3806f63bp-2},
    {-0x1.d906bcf328d46p-1, 0x1.87de2a6aea963p-2}, {-0x1.e9f4156c62ddap-1, 0x1.294062ed59f06p-2},
    {-0x1.f6297cff75cb0p-1, 0x1.8f8b83c69a60bp-3}, {-0x1.fd88da3d12526p-1, 0x1.917a6bc29b42cp-4},
    {-0x1.0000000000000p+0, 0x0.0p+0}, {-0x1.fd88da3d12526p-1, -0x1.917a6bc29b42cp-4},
    {-0x1.f6297cff75cb0p-1, -0x1.8f8b83c69a60bp-3}, {-0x1.e9f4156c62ddap-1, -0x1.294062ed59f06p-2},
    {-0x1.d906bcf328d46p-1, -0x1.87de2a6aea963p-2}, {-0x1.c38b2f180bdb1p-1, -0x1.e2b5d3806f63bp-2},
    {-0x1.a9b66290ea1a3p-1, -0x1.1c73b39ae68c8p-1}, {-0x1.8bc806b151741p-1, -0x1.44cf325091dd6p-1},
    {-0x1.6a09e667f3bcdp-1, -0x1.6a09e667f3bcdp-1}, {-0x1.44cf325091dd6p-1, -0x1.8bc806b151741p-1},
    {-0x1.1c73b39ae68c8p-1, -0x1.a9b66290ea1a3p-1}, {-0x1.e2b5d3806f63bp-2, -0x1.c38b2f180bdb1p-1},
    {-0x1.87de2a6aea963p-2, -0x1.d906bcf328d46p-1}, {-0x1.294062ed59f06p-2, -0x1.e9f4156c62ddap-1},
    {-0x1.8f8b83c69a60bp-3, -0x1.f6297cff75cb0p-1}, {-0x1.917a6bc29b42cp-4, -0x1.fd88da3d12526p-1},
    {0x0.0p+0, -0x1.0000000000000p+0}, {0x1.917a6bc29b42cp-4, -0x1.fd88da3d12526p-1},
    {0x1.8f8b83c69a60bp-3, -0x1.f6297cff75cb0p-1}, {0x1.294062ed59f06p-2, -0x1.e9f4156c62ddap-1},
    {0x1.87de2a6aea963p-2, -0x1.d906bcf328d46p-1}, {0x1.e2b5d3806f63bp-2, -0x1.c38b2f180bdb1p-1},
    {0x1.1c73b39ae68c8p-1, -0x1.a9b66290ea1a3p-1}, {0x1.44cf325091dd6p-1, -0x1.8bc806b151741p-1},
    {0x1.6a09e667f3bcdp-1, -0x1.6a09e667f3bcdp-1}, {0x1.8bc806b151741p-1, -0x1.44cf325091dd6p-1},
    {0x1.a9b66290ea1a3p-1, -0x1.1c73b39ae68c8p-1}, {0x1.c38b2f180bdb1p-1, -0x1.e2b5d3806f63bp-2},
    {0x1.d906bcf328d46p-1, -0x1.87de2a6aea963p-2}, {0x1.e9f4156c62ddap-1, -0x1.294062ed59f06p-2},
    {0x1.f6297cff75cb0p-1, -0x1.8f8b83c69a60bp-3}, {0x1.fd88da3d12526p-1, -0x1.917a6bc29b42cp-4},
};

constexpr uint32_t kLogBase = 0x3FE60000u;  // upper word of 0x1.6p-1

BFI_HD inline uint32_t upper(double x)
{
    return static_cast<uint32_t>(__builtin_bit_cast(uint64_t, x) >> 32);
}
BFI_HD inline double with_upper(double x, uint32_t hi)
{
    const uint64_t low = __builtin_bit_cast(uint64_t, x) & 0xFFFFFFFFull;
    return __builtin_bit_cast(double, static_cast<uint64_t>(hi) << 32 | low);
}

// -2 ln(y 2^-scale) for normal y > 0.  y = m 2^k with m in [0x1.6p-1, 0x1.6p+0);
// r = m/c - 1 in one rounding, |r| < 2^-7; ln(1 + r) to r^8 / 8.
template <int SCALE>
BFI_HD inline double minus_2log(double y, const double (*table)[2])
{
    const uint32_t t = upper(y) - (kLogBase + (static_cast<uint32_t>(SCALE) << 20));
    const double *row = table[(t >> 14) & 63u];
    const double m = with_upper(y, (t & 0xFFFFFu) + kLogBase);
    const double k = static_cast<double>(static_cast<int32_t>(t) >> 20);
    const double r = __builtin_fma(m, row[0], -1.0);
    // -2 ln(1 + r) = r (-2 + r - 2/3 r^2 + 1/2 r^3 - 2/5 r^4 + 1/3 r^5 - 2/7 r^6
    //                   + 1/4 r^7)
    double q = __builtin_fma(r, 0.25, -2.0 / 7.0);
    q = __builtin_fma(q, r, 1.0 / 3.0);
    q = __builtin_fma(q, r, -0.4);
    q = __builtin_fma(q, r, 0.5);
    q = __builtin_fma(q, r, -2.0 / 3.0);
    q = __builtin_fma(q, r, 1.0);
    q = __builtin_fma(q, r, -2.0);
    constexpr double kMinus2Ln2 = -0x1.62e42fefa39efp+0;
    return __builtin_fma(q, r, __builtin_fma(k, kMinus2Ln2, row[1]));
}

// Cosine and sine of the angle (x + 1/2) 2^-32 turn: the nearest 64th of a turn
// from the table, rotated by the rest, |d| <= pi/64.
BFI_HD inline void turn(uint32_t x, const double (*table)[2], double *cosine, double *sine)
{
    const uint32_t y = x + (1u << 25);  // wraps with the turn
    const double *row = table[y >> 26];
    // d = ((y mod 2^26) - 2^25 + 1/2) 2 pi 2^-32
    const double d = __builtin_fma(static_cast<double>(y & 0x3FFFFFFu), 0x1.921fb54442d18p-30,
                                   -0x1.921fb4dfbae43p-5);
    const double d2 = d * d;
    double ps = __builtin_fma(d2, -1.0 / 5040.0, 1.0 / 120.0);
    ps = __builtin_fma(ps, d2, -1.0 / 6.0);
    const double s = __builtin_fma(d * d2, ps, d);
    double pc = __builtin_fma(d2, 1.0 / 40320.0, -1.0 / 720.0);
    pc = __builtin_fma(pc, d2, 1.0 / 24.0);
    pc = __builtin_fma(pc, d2, -0.5);
    const double c1 = d2 * pc;  // cos d - 1
    *cosine = __builtin_fma(-row[1], s, __builtin_fma(row[0], c1, row[0]));
    *sine = __builtin_fma(row[0], s, __builtin_fma(row[1], c1, row[1]));
}

// Square root of a (normal, 2^-1000 < a < 2^1000) from y, its reciprocal root to
// 20 bits and more: Goldschmidt's coupled iteration for sqrt(a) and 1/(2 sqrt(a)),
// then a correction by the exact residual a - g^2.
BFI_HD inline double root(double a, double y)
{
    double g = a * y, h = 0.5 * y;
    double e = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, e, g);
    h = __builtin_fma(h, e, h);
    e = __builtin_fma(-g, g, a);
    return __builtin_fma(e, h, g);
}

// Reciprocal square root of a from y as above: one step of third order,
// y (1 + e/2 + 3/8 e^2), e = 1 - a y^2.
BFI_HD inline double reciprocal_root(double a, double y)
{
    const double e = __builtin_fma(-(a * y), y, 1.0);
    return __builtin_fma(y * e, __builtin_fma(e, 0.375, 0.5), y);
}

// Reciprocal of b from z, its value to 20 bits and more: z (1 + e + e^2),
// e = 1 - b z.
BFI_HD inline double reciprocal(double b, double z)
{
    const double e = __builtin_fma(-b, z, 1.0);
    return __builtin_fma(z, __builtin_fma(e, e, e), z);
}

}  // namespace nrm
}  // namespace bfi
