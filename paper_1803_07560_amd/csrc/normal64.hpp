// The double-precision functions of the samplers that draw Gaussian numbers:
// logarithm, sine and cosine of a Philox word, roots, the radius' power.  Plain
// C++ on clang/GCC builtins, so the same arithmetic compiles for the GPU and for
// a host check; the includer sets BFI_HD (e.g. __device__).
//
// The arguments are narrow -- a word's uniform (x + 1/2) 2^-32, a radius, a sum
// of squares -- so nothing here scales, reduces or tests for what cannot occur,
// and small tables replace most of each series (Tang, "Table-driven
// implementation of the logarithm function in IEEE floating-point arithmetic",
// ACM TOMS 16 (1990); the same idea for the circle), at arguments whose values
// happen to lie next to a double (Gal and Bachelis, "An accurate elementary
// mathematical library for the IEEE floating point standard", ACM TOMS 17 (1991);
// found with 113-bit arithmetic).  Each result is one rounded sum of a leading
// part without error and a small rest, so that none is further off than the
// device library's.  Largest and mean error in units in the last place of the
// result, 4 million arguments against long double, these and the library's on the
// GPU: logarithm of a word 0.631 and 0.250 (library 0.635 and 0.252), sine and
// cosine 0.752 and 0.251 (0.874 and 0.257), power 1/D for D = 3 .. 32 0.63 and 0.25
// (3.7 and 0.30 at D = 3, else up to 2.0 and 0.27), x / sqrt(a) the same two
// roundings (1.5 and 0.35), square root 0.50, reciprocal square root 0.99.
#pragma once

#include <cstdint>

#ifndef BFI_HD
#define BFI_HD
#define BFI_DATA
#else
#define BFI_DATA static __device__  // the tables too are the device's
#endif

#include "exp64.hpp"

namespace bfi {
namespace nrm {

// Interval i of [0x1.6p-1, 0x1.6p+0) is cut by the top bits of the significand
// from 0x1.6p-1 on: {-2/c, -2 ln c} for a c inside it, near the middle (but 1 in
// the two intervals below 1: there the logarithm vanishes with its argument, and
// elsewhere it is at least four times its rest).  -2/c has 28 bits (29 just below
// 1), so that its product with a word's 33, less 2, is exact; of these c the one
// was taken whose -2 ln c lies next to a multiple of 2^-46 (within 2^-61; 2^-65 just
// below 1), which adds up exactly with multiples of ln 2.
BFI_DATA constexpr double kLog[128][2] = {
    {-0x1.7411472p+1, 0x1.7edf121952b8p-1}, {-0x1.71944f6p+1, 0x1.7800208daf38p-1},
    {-0x1.6f2dde8p+1, 0x1.715421f94abp-1}, {-0x1.6c30a3p+1, 0x1.68f54bc3962p-1},
    {-0x1.6b25c7p+1, 0x1.6605e2ec46fp-1}, {-0x1.684336cp+1, 0x1.5ddaf9c3af3p-1},
    {-0x1.67b06eep+1, 0x1.5c397016d7p-1}, {-0x1.6538e1ap+1, 0x1.552d47092688p-1},
    {-0x1.633010cp+1, 0x1.4f540ee7603p-1}, {-0x1.6071118p+1, 0x1.476174704c38p-1},
    {-0x1.5f040dp+1, 0x1.433ac3e14418p-1}, {-0x1.5df7e86p+1, 0x1.402b5b26bbap-1},
    {-0x1.5bcfe96p+1, 0x1.39d73b30af8p-1}, {-0x1.596aeaap+1, 0x1.32c442a3847p-1},
    {-0x1.586d0f2p+1, 0x1.2fd29c5ac75p-1}, {-0x1.561c5cap+1, 0x1.28ea8922fa5p-1},
    {-0x1.53d201ap+1, 0x1.220990b7eep-1}, {-0x1.534bfcp+1, 0x1.207565d93de8p-1},
    {-0x1.518ec2cp+1, 0x1.1b3241263da8p-1}, {-0x1.4ef4a5ep+1, 0x1.1345bc5f811p-1},
    {-0x1.4e3dc8cp+1, 0x1.11161a2a5a9p-1}, {-0x1.4c3eb4ap+1, 0x1.0af3a39bcep-1},
    {-0x1.49b63p+1, 0x1.031d34cd9c08p-1}, {-0x1.4832a86p+1, 0x1.fccdbbb028bp-2},
    {-0x1.4635c6ap+1, 0x1.f05c95b3061p-2}, {-0x1.4503ea4p+1, 0x1.e8d8d0bc23ep-2},
    {-0x1.4317d0ap+1, 0x1.dcb2c479f4dp-2}, {-0x1.421efb6p+1, 0x1.d6871abeb42p-2},
    {-0x1.4076da6p+1, 0x1.cbf79826bcp-2}, {-0x1.3f40d82p+1, 0x1.c436a8e68b2p-2},
    {-0x1.3d1595cp+1, 0x1.b64088a557bp-2}, {-0x1.3b96b72p+1, 0x1.ac91c936036p-2},
    {-0x1.3a81828p+1, 0x1.a587c758016p-2}, {-0x1.393b516p+1, 0x1.9d375e0b4d2p-2},
    {-0x1.37d3be2p+1, 0x1.940312bc6dap-2}, {-0x1.35f2e1ep+1, 0x1.87a35b3249ep-2},
    {-0x1.3474d7cp+1, 0x1.7dc0ea9f038p-2}, {-0x1.32db248p+1, 0x1.7319a04055cp-2},
    {-0x1.31bf9dcp+1, 0x1.6bb1e882e04p-2}, {-0x1.30130dp+1, 0x1.60735a995fp-2},
    {-0x1.2e3ac08p+1, 0x1.53fca3fea16p-2}, {-0x1.2d3c6a2p+1, 0x1.4d3e554d9fcp-2},
    {-0x1.2bb50fap+1, 0x1.42d2e187646p-2}, {-0x1.2a4ebe6p+1, 0x1.393ca4a6dd9p-2},
    {-0x1.29c1338p+1, 0x1.356fff07fd6p-2}, {-0x1.28073c4p+1, 0x1.29873e76acap-2},
    {-0x1.26a5efep+1, 0x1.1ff551d4004p-2}, {-0x1.24b806p+1, 0x1.1281011a8acp-2},
    {-0x1.2359a08p+1, 0x1.08e7b6ee806p-2}, {-0x1.22ff47ap+1, 0x1.066c3f92d94p-2},
    {-0x1.21e53aap+1, 0x1.fd4ee3a53e8p-3}, {-0x1.1f9db7cp+1, 0x1.dcf9bd80c78p-3},
    {-0x1.1eb8fd6p+1, 0x1.d03b4eaa0b4p-3}, {-0x1.1d62dbep+1, 0x1.bd185789fc4p-3},
    {-0x1.1c2a478p+1, 0x1.ab886c94f8p-3}, {-0x1.1af7778p+1, 0x1.9a38a129fp-3},
    {-0x1.199f6b4p+1, 0x1.86b89a56d1ep-3}, {-0x1.18c12f8p+1, 0x1.7a1362d624cp-3},
    {-0x1.172723ep+1, 0x1.62a4001b18p-3}, {-0x1.164463cp+1, 0x1.559f9bfd402p-3},
    {-0x1.15588a6p+1, 0x1.480a3a9d21p-3}, {-0x1.144fd88p+1, 0x1.38bdc2fa90cp-3},
    {-0x1.126e6f2p+1, 0x1.1cc500f135cp-3}, {-0x1.120fe0cp+1, 0x1.1740c399c88p-3},
    {-0x1.10c41eap+1, 0x1.03d6b3fc5c8p-3}, {-0x1.0f846bap+1, 0x1.e215d052768p-4},
    {-0x1.0dd6154p+1, 0x1.af35a967438p-4}, {-0x1.0ce32dcp+1, 0x1.925a4c1f178p-4},
    {-0x1.0c38d06p+1, 0x1.7e0d7bb5c5cp-4}, {-0x1.0af32a2p+1, 0x1.571be175a78p-4},
    {-0x1.09a823bp+1, 0x1.2f54e4c9808p-4}, {-0x1.09206d5p+1, 0x1.1ef7c774ad4p-4},
    {-0x1.078d474p+1, 0x1.dc53f1c9e58p-5}, {-0x1.06cf40ap+1, 0x1.ae1e1a8c4f8p-5},
    {-0x1.0578bc6p+1, 0x1.5a7e7dfd84p-5}, {-0x1.04c9851p+1, 0x1.2f8ceec566p-5},
    {-0x1.03a098bp+1, 0x1.cd0a221af6p-6}, {-0x1.02f541bp+1, 0x1.78751f757p-6}, {-0x1p+1, 0x0p+0},
    {-0x1p+1, 0x0p+0}, {-0x1.fe2f7cep+0, -0x1.d15656af3cp-8}, {-0x1.f9e894ap+0, -0x1.88314b2c0ap-6},
    {-0x1.f62a632p+0, -0x1.3dc363b0b58p-5}, {-0x1.f269b5ap+0, -0x1.b8a8d311cc8p-5},
    {-0x1.ee8c964p+0, -0x1.1c15244b738p-4}, {-0x1.eaa6ea4p+0, -0x1.5ce49e078a8p-4},
    {-0x1.e7851a4p+0, -0x1.915ab606d08p-4}, {-0x1.e3c8a9ap+0, -0x1.d060111a9p-4},
    {-0x1.dfdac14p+0, -0x1.09976ae26p-3}, {-0x1.dc8c4dep+0, -0x1.25e9a93da04p-3},
    {-0x1.d90408p+0, -0x1.4462f7a9a46p-3}, {-0x1.d59f47ap+0, -0x1.61e0e3a8f16p-3},
    {-0x1.d2385c4p+0, -0x1.7fa89ceb27ap-3}, {-0x1.cf24014p+0, -0x1.9acdb96876cp-3},
    {-0x1.cbee60cp+0, -0x1.b74975998eap-3}, {-0x1.c87db34p+0, -0x1.d609f90761ep-3},
    {-0x1.c57597cp+0, -0x1.f1550d61372p-3}, {-0x1.c256feap+0, -0x1.06cdc5835acp-2},
    {-0x1.bf57cc4p+0, -0x1.147a6531b77p-2}, {-0x1.bc1759p+0, -0x1.236b63e378bp-2},
    {-0x1.b96da86p+0, -0x1.2fbc943ebebp-2}, {-0x1.b682f88p+0, -0x1.3d50514ecap-2},
    {-0x1.b3615a6p+0, -0x1.4bfd9429fddp-2}, {-0x1.b082422p+0, -0x1.598ade667b9p-2},
    {-0x1.ad8b656p+0, -0x1.67a0938a65ep-2}, {-0x1.ab1f86ep+0, -0x1.733460148c9p-2},
    {-0x1.a83adcap+0, -0x1.811fd9c222bp-2}, {-0x1.a59fa54p+0, -0x1.8dbed1d7e04p-2},
    {-0x1.a2d186ap+0, -0x1.9b6aadcbc9ap-2}, {-0x1.a0445a2p+0, -0x1.a7ee6ecd3adp-2},
    {-0x1.9da7b0ap+0, -0x1.b4d28f9879bp-2}, {-0x1.9ac7ff6p+0, -0x1.c319aca93ecp-2},
    {-0x1.987142p+0, -0x1.cecb4b7d728p-2}, {-0x1.95f56e2p+0, -0x1.db492d15fbfp-2},
    {-0x1.932938p+0, -0x1.e972dc96a4fp-2}, {-0x1.910215ep+0, -0x1.f46a0a9c5c5p-2},
    {-0x1.8e5e6b4p+0, -0x1.00f814d5cep-1}, {-0x1.8be41a8p+0, -0x1.075bab782338p-1},
    {-0x1.89bedfap+0, -0x1.0cec27b4895p-1}, {-0x1.874cb62p+0, -0x1.134dabdb0a2p-1},
    {-0x1.851b30ap+0, -0x1.190f4324441p-1}, {-0x1.8297378p+0, -0x1.1fb37d85309p-1},
    {-0x1.8082b06p+0, -0x1.2539db53bba8p-1}, {-0x1.7e1b90ep+0, -0x1.2ba5259c62ep-1},
    {-0x1.7c0042p+0, -0x1.314e6c42ff3p-1}, {-0x1.79c0ab6p+0, -0x1.376215b702bp-1},
    {-0x1.779df5ap+0, -0x1.3d304b4e17e8p-1}, {-0x1.755250ap+0, -0x1.43773c16ac18p-1},
};

// Cell i is the words from (i - 1/2) 2^26 on, row i {cos, sin} of an angle of it,
// near the middle, and how many words from the cell's start that angle is: of
// these the one was taken whose cosine and sine are next to a double (within 0.002
// of its last place).  A cell next to an axis takes the axis, so that a cosine or
// sine is never the difference of two numbers of its own size.
struct TurnTable {
    double row[64][2];
    int32_t from[64];
};
BFI_DATA constexpr TurnTable kTurn = {{
    {0x1p+0, 0x0p+0}, {0x1p+0, 0x0p+0}, {0x1.f63308ccbfae7p-1, 0x1.8ecb5c751be71p-3},
    {0x1.ea0226e0b06c3p-1, 0x1.28e3924c2c2f3p-2}, {0x1.d90426aefaa98p-1, 0x1.87eaa7e39ee93p-2},
    {0x1.c383a5dc8a9bfp-1, 0x1.e2d2051f832f1p-2}, {0x1.a9a0f94389ab4p-1, 0x1.1c93bc580f5afp-1},
    {0x1.8bb04ea9dabf9p-1, 0x1.44ec16f3dab1dp-1}, {0x1.6a19556588e16p-1, 0x1.69fa76c1e992p-1},
    {0x1.44ec16f3dab1dp-1, 0x1.8bb04ea9dabf9p-1}, {0x1.1c93bc580f5afp-1, 0x1.a9a0f94389ab4p-1},
    {0x1.e2d2051f832f1p-2, 0x1.c383a5dc8a9bfp-1}, {0x1.87eaa7e39ee93p-2, 0x1.d90426aefaa98p-1},
    {0x1.28e3924c2c2f3p-2, 0x1.ea0226e0b06c3p-1}, {0x1.8ecb5c751be71p-3, 0x1.f63308ccbfae7p-1},
    {0x0p+0, 0x1p+0}, {0x0p+0, 0x1p+0}, {0x0p+0, 0x1p+0},
    {-0x1.8ecb5c751be71p-3, 0x1.f63308ccbfae7p-1}, {-0x1.28e3924c2c2f3p-2, 0x1.ea0226e0b06c3p-1},
    {-0x1.87eaa7e39ee93p-2, 0x1.d90426aefaa98p-1}, {-0x1.e2d2051f832f1p-2, 0x1.c383a5dc8a9bfp-1},
    {-0x1.1c93bc580f5afp-1, 0x1.a9a0f94389ab4p-1}, {-0x1.44ec16f3dab1dp-1, 0x1.8bb04ea9dabf9p-1},
    {-0x1.69fa76c1e992p-1, 0x1.6a19556588e16p-1}, {-0x1.8bb04ea9dabf9p-1, 0x1.44ec16f3dab1dp-1},
    {-0x1.a9a0f94389ab4p-1, 0x1.1c93bc580f5afp-1}, {-0x1.c383a5dc8a9bfp-1, 0x1.e2d2051f832f1p-2},
    {-0x1.d90426aefaa98p-1, 0x1.87eaa7e39ee93p-2}, {-0x1.ea0226e0b06c3p-1, 0x1.28e3924c2c2f3p-2},
    {-0x1.f63308ccbfae7p-1, 0x1.8ecb5c751be71p-3}, {-0x1p+0, 0x0p+0}, {-0x1p+0, 0x0p+0},
    {-0x1p+0, 0x0p+0}, {-0x1.f63308ccbfae7p-1, -0x1.8ecb5c751be71p-3},
    {-0x1.ea0226e0b06c3p-1, -0x1.28e3924c2c2f3p-2}, {-0x1.d90426aefaa98p-1, -0x1.87eaa7e39ee93p-2},
    {-0x1.c383a5dc8a9bfp-1, -0x1.e2d2051f832f1p-2}, {-0x1.a9a0f94389ab4p-1, -0x1.1c93bc580f5afp-1},
    {-0x1.8bb04ea9dabf9p-1, -0x1.44ec16f3dab1dp-1}, {-0x1.6a19556588e16p-1, -0x1.69fa76c1e992p-1},
    {-0x1.44ec16f3dab1dp-1, -0x1.8bb04ea9dabf9p-1}, {-0x1.1c93bc580f5afp-1, -0x1.a9a0f94389ab4p-1},
    {-0x1.e2d2051f832f1p-2, -0x1.c383a5dc8a9bfp-1}, {-0x1.87eaa7e39ee93p-2, -0x1.d90426aefaa98p-1},
    {-0x1.28e3924c2c2f3p-2, -0x1.ea0226e0b06c3p-1}, {-0x1.8ecb5c751be71p-3, -0x1.f63308ccbfae7p-1},
    {0x0p+0, -0x1p+0}, {0x0p+0, -0x1p+0}, {0x0p+0, -0x1p+0},
    {0x1.8ecb5c751be71p-3, -0x1.f63308ccbfae7p-1}, {0x1.28e3924c2c2f3p-2, -0x1.ea0226e0b06c3p-1},
    {0x1.87eaa7e39ee93p-2, -0x1.d90426aefaa98p-1}, {0x1.e2d2051f832f1p-2, -0x1.c383a5dc8a9bfp-1},
    {0x1.1c93bc580f5afp-1, -0x1.a9a0f94389ab4p-1}, {0x1.44ec16f3dab1dp-1, -0x1.8bb04ea9dabf9p-1},
    {0x1.69fa76c1e992p-1, -0x1.6a19556588e16p-1}, {0x1.8bb04ea9dabf9p-1, -0x1.44ec16f3dab1dp-1},
    {0x1.a9a0f94389ab4p-1, -0x1.1c93bc580f5afp-1}, {0x1.c383a5dc8a9bfp-1, -0x1.e2d2051f832f1p-2},
    {0x1.d90426aefaa98p-1, -0x1.87eaa7e39ee93p-2}, {0x1.ea0226e0b06c3p-1, -0x1.28e3924c2c2f3p-2},
    {0x1.f63308ccbfae7p-1, -0x1.8ecb5c751be71p-3}, {0x1p+0, 0x0p+0},
}, {
    33554432, -33554432, 33299004, 33301532, 33589685, 33637796, 33755378, 33749385, 33440594,
    33359479, 33353486, 33471068, 33519179, 33807332, 33809860, 100663296, 33554432, -33554432,
    33299004, 33301532, 33589685, 33637796, 33755378, 33749385, 33440594, 33359479, 33353486,
    33471068, 33519179, 33807332, 33809860, 100663296, 33554432, -33554432, 33299004, 33301532,
    33589685, 33637796, 33755378, 33749385, 33440594, 33359479, 33353486, 33471068, 33519179,
    33807332, 33809860, 100663296, 33554432, -33554432, 33299004, 33301532, 33589685, 33637796,
    33755378, 33749385, 33440594, 33359479, 33353486, 33471068, 33519179, 33807332, 33809860,
    100663296,
}};

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

// -2 ln(y 2^-SCALE) for normal y > 0, as the exact k (-2 ln 2) - 2 ln c and the
// rest w, in that order.  y = m 2^k with m in [0x1.6p-1, 0x1.6p+0); r = -2 (m/c - 1),
// exact where y has 33 bits; -2 ln(1 - r/2) = r + r^2 (1/4 + r/12 + ..), the series
// fitted over |r| <= 2^-6 (the intervals below 1; 2^-57 of the result there).
template <int SCALE>
BFI_HD inline void minus_2log_parts(double y, const double (*table)[2], double &h, double &w)
{
    const uint32_t t = upper(y) - (kLogBase + (static_cast<uint32_t>(SCALE) << 20));
    const double *row = table[(t >> 13) & 127u];
    const double m = with_upper(y, (t & 0xFFFFFu) + kLogBase);
    const double k = static_cast<double>(static_cast<int32_t>(t) >> 20);
    const double r = __builtin_fma(m, row[0], 2.0);
    // -2 ln 2 as a multiple of 2^-46 and the rest
    constexpr double kHi = -0x1.62e42fefa3a00p+0, kLo = 0x1.0ca86c3898d00p-48;
    h = __builtin_fma(k, kHi, row[1]);
    double q = __builtin_fma(r, 0x1.24979e8d8acaep-9, 0x1.555b556aef384p-8);
    q = __builtin_fma(q, r, 0x1.999999919973cp-7);
    q = __builtin_fma(q, r, 0x1.fffffff6ffd66p-6);
    q = __builtin_fma(q, r, 0x1.5555555555564p-4);
    q = __builtin_fma(q, r, 0x1.0000000000008p-2);
    w = __builtin_fma(r * r, q, __builtin_fma(k, kLo, r));
}
template <int SCALE>
BFI_HD inline double minus_2log(double y, const double (*table)[2])
{
    double h, w;
    minus_2log_parts<SCALE>(y, table, h, w);
    return h + w;
}

// Cosine and sine of the angle (x + 1/2) 2^-32 turn: the table's angle rotated by
// the rest, n steps of 2 pi 2^-32 (n exact, up to 3 pi/64 next to an axis), whose
// sine and cosine - 1 are odd and even polynomials in n (Chebyshev fits, off by
// less than 2^-59 of the sine and 2^-56): the sine ends on n times the step
// itself, so it keeps its last bit however small it is.
BFI_HD inline void turn(uint32_t x, const TurnTable &table, double *cosine, double *sine)
{
    const uint32_t y = x + (1u << 25);  // wraps with the turn
    const double a = table.row[y >> 26][0], b = table.row[y >> 26][1];
    const double n =
        static_cast<double>(static_cast<int32_t>(y & 0x3FFFFFFu) - table.from[y >> 26]) + 0.5;
    const double n2 = n * n;
    double q = __builtin_fma(n2, 0x1.50562f667484fp-283, -0x1.32d2cb66c06cdp-218);
    q = __builtin_fma(q, n2, 0x1.466bc6774fe06p-154);
    q = __builtin_fma(q, n2, -0x1.4abbce625be51p-91);
    q = __builtin_fma(q, n2, 0x1.1a62633145c07p-84);
    const double s = __builtin_fma(n, 0x1.921fb54442d18p-30, n * q);
    double c = __builtin_fma(n2, 0x1.e1b977f3fea9cp-251, -0x1.55d3c54492b52p-186);
    c = __builtin_fma(c, n2, 0x1.03c1f081a2c28p-122);
    c = __builtin_fma(c, n2, -0x1.3bd3cc9be45d9p-60);
    c *= n2;  // cos - 1
    *cosine = a + __builtin_fma(-b, s, a * c);
    *sine = b + __builtin_fma(a, s, b * c);
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

// x / sqrt(a), y as above: the rounded root divides, as a quotient corrected by
// its exact residual.
BFI_HD inline double over_root(double x, double a, double y)
{
    const double g = root(a, y), i = reciprocal_root(a, y), q = x * i;
    return __builtin_fma(__builtin_fma(-q, g, x), i, q);
}

// Reciprocal of b from z, its value to 20 bits and more: z (1 + e + e^2),
// e = 1 - b z.
BFI_HD inline double reciprocal(double b, double z)
{
    const double e = __builtin_fma(-b, z, 1.0);
    return __builtin_fma(z, __builtin_fma(e, e, e), z);
}

// y^(1/D) for 2^-64 < y <= 1, D >= 3: e^(ln y / D), both the logarithm and its
// share of 1/D as sums (the quotient reaches 15, where a rounding is 16 of the
// result).  e^p as in exp_weight, with the reduced argument and 1 + r as sums.
template <int D, class Fma>
BFI_HD inline double root_of_degree(double y, const double (*table)[2], const Fma &fma = Fma())
{
    double h, w;
    minus_2log_parts<0>(y, table, h, w);
    const double l = h + w, ll = (h - l) + w;
    constexpr double c = -0.5 / D;
    const double cl = __builtin_fma(c, static_cast<double>(D), 0.5) * (-1.0 / D);  // -1/2D - c
    const double p = l * c;
    const double pl = __builtin_fma(ll, c, __builtin_fma(l, cl, __builtin_fma(l, c, -p)));
    const double k = __builtin_rint(p * expk::kInvLn2);
    const double r = __builtin_fma(-k, expk::kLn2Hi, p);
    const double rl = __builtin_fma(-k, expk::kLn2Lo, pl);
    double q = fma.coef(11);
    for (int j = 10; j >= 0; --j)
        q = fma.step(q, r, fma.coef(j));
    const double u = 1.0 + r;
    const double low = __builtin_fma(r * r, q, (1.0 - u) + r);
    return __builtin_ldexp(u + __builtin_fma(u + low, rl, low), static_cast<int>(k));
}

}  // namespace nrm
}  // namespace bfi
