// How far launches reach.  HIP takes fewer than 2^32 threads per dimension of a
// launch, so kernels of several threads per subvolume, leaf or entry end before
// the counts do: a merge then takes fewer wavefronts a subvolume (its sums do not
// depend on them), leaf kernels run over slices.  Plain C++.
#pragma once

#include <cstdint>

namespace bfi {

constexpr uint64_t kMaxThreads = 0xFFFFFFFFull;

// Wavefronts per subvolume for a launch over `subvolumes`: as wanted (1, 4 or 16)
// where such a launch exists, else fewer.
constexpr int fitting_waves(uint64_t subvolumes, int wanted)
{
    while (wanted > 1 && subvolumes * 64 * static_cast<uint64_t>(wanted) > kMaxThreads)
        wanted /= 4;
    return wanted;
}

// Leaves of a launch of one thread each, in blocks of up to 1024.
constexpr uint64_t kMaxLeaves = kMaxThreads / 1024 * 1024;
// Entries and leaves of one launch of 64 and of 32 threads each (the latter beside
// one more thread per leaf).
constexpr uint32_t kFoldSlice = 1u << 25, kChoiceSlice = 1u << 26;

// f(first, n) over consecutive slices of `count`, until one returns an error
// (anything but Ok).
template <class Status, class F>
Status for_slices(uint32_t count, uint32_t slice, Status ok, F &&f)
{
    for (uint32_t first = 0; first < count;) {
        const uint32_t n = count - first < slice ? count - first : slice;
        const Status s = f(first, n);
        if (s != ok)
            return s;
        first += n;
    }
    return ok;
}

}  // namespace bfi
