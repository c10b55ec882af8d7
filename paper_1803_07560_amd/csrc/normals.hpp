// Standard normals from Philox words on the device (Box-Muller), shared by the
// samplers that draw Gaussian numbers: the Gaussian-proposal sampler and the
// sampler in spherical coordinates.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.hpp"
#include "normal64.hpp"

namespace bfi {
namespace dev {

// The tables of the double-precision functions, copied to LDS once per block: a
// lane's two reads per pair of normals are 16 bytes each at an address of its
// own, which LDS serves beside the vector instructions.  With the library's log,
// sincospi, pow, exp and log1p in their place (and the whole of Philox for every
// block) 2^24 evaluations of 10x2 by the spherical sampler in FP64, pilot and
// main pass, took 1.50 ms; with these 0.70 ms.  The errors of Z, C(r) and their
// error bars against 64-bit sums over 80 inputs are those of before (medians
// 1e-16 .. 2e-15).
struct NormalTables {
    alignas(16) double log[64][2];
    alignas(16) double turn[64][2];
    __device__ __forceinline__ void load(uint32_t tid, uint32_t block)
    {
        for (uint32_t i = tid; i < 64; i += block) {
            log[i][0] = nrm::kLog[i][0];
            log[i][1] = nrm::kLog[i][1];
            turn[i][0] = nrm::kTurn[i][0];
            turn[i][1] = nrm::kTurn[i][1];
        }
    }
};
// The single-precision form has no tables.
struct NoTables {
    __device__ __forceinline__ void load(uint32_t, uint32_t) {}
};

// Box-Muller: a standard normal pair from two words, u = (x + 1/2) 2^-32,
// radius sqrt(-2 ln u1), angle 2 pi u2.
__device__ __forceinline__ void box_muller(uint32_t x1, uint32_t x2, const NormalTables &tab,
                                           double &zc, double &zs)
{
    const double l = nrm::minus_2log<32>(static_cast<double>(x1) + 0.5, tab.log);
    const double r = nrm::root(l, __builtin_amdgcn_rsq(l));
    double s, c;
    nrm::turn(x2, tab.turn, &c, &s);
    zc = r * c;
    zs = r * s;
}
// FP32: hardware log2, square root and sine/cosine (whose argument is in
// turns, so the angle 2 pi u2 is u2 itself)
__device__ __forceinline__ void box_muller(uint32_t x1, uint32_t x2, const NoTables &, float &zc,
                                           float &zs)
{
    const float u1 = __fmaf_rn(static_cast<float>(x1), 0x1p-32f, 0x1p-33f);
    const float u2 = __fmaf_rn(static_cast<float>(x2), 0x1p-32f, 0x1p-33f);
    constexpr float kMinus2Ln2 = -1.38629436111989061883f;
    const float r = __builtin_amdgcn_sqrtf(kMinus2Ln2 * __builtin_amdgcn_logf(u1));
    zc = r * __builtin_amdgcn_cosf(u2);
    zs = r * __builtin_amdgcn_sinf(u2);
}

}  // namespace dev
}  // namespace bfi
