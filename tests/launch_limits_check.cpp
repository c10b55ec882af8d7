// Host check of launch_limits.h at the counts where a launch of several threads
// each would pass 2^32 threads.  Exit status 0: every launch fits and the slices
// cover each entry once.
#include <cstdio>
#include <cstdint>
#include <initializer_list>

#include "launch_limits.h"

using namespace bfi;

static int bad = 0;
static void expect(bool ok, const char *what, uint64_t at)
{
    if (!ok) {
        std::printf("%s at %llu\n", what, static_cast<unsigned long long>(at));
        ++bad;
    }
}

// Slices of `count` entries, `per` threads each, in 256-thread blocks beside `more`
// threads per entry of the whole list.
static void slices(uint32_t count, uint32_t slice, uint64_t per, uint64_t more)
{
    uint64_t next = 0;
    const int status = for_slices(count, slice, 0, [&](uint32_t first, uint32_t n) {
        expect(first == next && n > 0, "slices not consecutive", count);
        next = uint64_t(first) + n;
        const uint64_t block = 256, each = block / per;
        // whole blocks but for the last slice: no entry in two launches
        expect(next == count || n % each == 0, "slice ends inside a block", count);
        uint64_t threads = (n + each - 1) / each * block;
        if (count <= slice)
            threads += more * ((uint64_t(count) + block - 1) / block * block);
        expect(threads <= kMaxThreads, "launch too long", count);
        // the last thread's entry, in the kernels' 32 bits
        const uint32_t last_block = static_cast<uint32_t>(threads / block - 1);
        if (count > slice)
            expect(first + last_block * static_cast<uint32_t>(each) +
                           static_cast<uint32_t>(each) - 1 >= next - 1,
                   "index wraps", count);
        return 0;
    });
    expect(status == 0 && next == count, "entries left out", count);
}

int main()
{
    for (int wanted : {1, 4, 16}) {
        for (uint64_t k = 0; k <= 26; ++k)
            for (int64_t off : {-1, 0, 1}) {
                const uint64_t n = (uint64_t(1) << k) + off;
                const int got = fitting_waves(n, wanted);
                expect(got == 1 || n * 64 * got <= kMaxThreads, "merge too long", n);
                expect(got == wanted || n * 64 * got * 4 > kMaxThreads, "too few wavefronts", n);
            }
    }
    for (uint64_t base : {uint64_t(1), uint64_t(1000), uint64_t(1) << 25, uint64_t(1) << 26,
                          uint64_t(1) << 27, uint64_t(3) << 26, uint64_t(1) << 31, kMaxLeaves})
        for (int64_t off : {-9, -1, 0, 1, 7}) {
            if (static_cast<int64_t>(base) + off < 1 || base + off > kMaxLeaves)
                continue;
            slices(static_cast<uint32_t>(base + off), kFoldSlice, 64, 0);
            slices(static_cast<uint32_t>(base + off), kChoiceSlice, 32, 1);
        }
    // an error ends the slices
    int calls = 0;
    expect(for_slices(5 * kFoldSlice, kFoldSlice, 0,
                      [&](uint32_t, uint32_t) { return ++calls == 2 ? 7 : 0; }) == 7 && calls == 2,
           "error not handed on", 0);
    expect((kMaxLeaves + 1023) / 1024 * 1024 <= kMaxThreads, "leaf launches", kMaxLeaves);
    return bad != 0;
}
