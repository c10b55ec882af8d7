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
// lane's reads per pair of normals are 16, 16 and 4 bytes at addresses of its own,
// which LDS serves beside the vector instructions.  What bounds the samplers is
// instruction issue, in these functions above all.  2^24 evaluations of 10x2 in
// FP64: spherical sampler, pilot and main pass, 0.63 ms; Gaussian proposal, 64
// streams, 0.72 ms.  With the library's log, sincospi, pow, exp and log1p in their
// place (and the whole of Philox for every block) they took 1.50 and 1.74 ms; with
// shorter forms of up to twice the library's errors, 0.59 and 0.69 ms.
struct NormalTables {
    alignas(16) double log[128][2];
    alignas(16) nrm::TurnTable turn;
    __device__ __forceinline__ void load(uint32_t tid, uint32_t block)
    {
        for (uint32_t i = tid; i < 128; i += block) {
            log[i][0] = nrm::kLog[i][0];
            log[i][1] = nrm::kLog[i][1];
        }
        for (uint32_t i = tid; i < 64; i += block) {
            turn.row[i][0] = nrm::kTurn.row[i][0];
            turn.row[i][1] = nrm::kTurn.row[i][1];
            turn.from[i] = nrm::kTurn.from[i];
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
