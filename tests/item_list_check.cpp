// Host check of the work-item lists (list_items, ItemCount of runtime.h), linked
// with the library: no device call.  Exit status 0: every list is right.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <random>
#include <vector>

#include "runtime.h"

using namespace bfi;

static int bad = 0;
static void expect(bool ok, const char *what)
{
    if (!ok) {
        std::printf("%s\n", what);
        ++bad;
    }
}

static double seconds(const std::chrono::steady_clock::time_point &t)
{
    return std::chrono::duration<double>(std::chrono::steady_clock::now() - t).count();
}

static void check(uint64_t chunk, const std::vector<uint64_t> &n)
{
    const int rec_len = 7;
    const ItemCount count(chunk);
    uint64_t total = 0;
    for (uint64_t x : n) {
        expect(count(x) == x / chunk + (x % chunk != 0), "ItemCount");
        total += x / chunk + (x % chunk != 0);
    }
    std::vector<WorkItem> items(total + 1);
    std::vector<uint32_t> first(n.size() + 1);
    const WorkItem guard{nullptr, nullptr, 7, 7, 7};
    items[total] = guard;
    EvalParams params;
    auto *rec = reinterpret_cast<double *>(uintptr_t(1) << 20);
    list_items(chunk, n.data(), n.size(), &params, rec, rec_len, first.data(), items.data());
    expect(items[total].start == 7 && items[total].rec == nullptr, "written past the end");
    expect(first[n.size()] == total, "item count");
    // order: whole items, then rests falling by 64ths
    uint64_t last = 64;
    std::vector<int> taken(total, 0);
    for (uint64_t i = 0; i < total; ++i) {
        const WorkItem &w = items[i];
        const uint64_t c = w.count * uint64_t(64) / chunk;
        expect(w.count > 0 && w.count <= chunk && c <= last, "order");
        last = c;
        const uint64_t slot = (w.rec - rec) / rec_len;
        expect(w.params == &params && w.sub < n.size() && slot >= first[w.sub] &&
                   slot < first[w.sub + 1],
               "record slot");
        expect(w.start == (slot - first[w.sub]) * chunk, "start");
        expect(w.count == std::min(chunk, n[w.sub] - w.start), "count");
        expect(slot < total && taken[slot]++ == 0, "slot taken twice");
    }
}

int main()
{
    std::mt19937_64 gen(4);
    for (uint64_t chunk : {uint64_t(1), uint64_t(2), uint64_t(63), uint64_t(64), uint64_t(65),
                           uint64_t(256), uint64_t(16384), uint64_t(1) << 28}) {
        std::vector<uint64_t> n;
        for (uint64_t k : {1, 2, 3, 5})
            for (int64_t off : {-1, 0, 1})
                if (k * chunk + off > 0)
                    n.push_back(k * chunk + off);
        check(chunk, n);
        check(chunk, {chunk * 3 + 1});
        n.clear();
        for (int i = 0; i < 3000; ++i)
            n.push_back(1 + gen() % (4 * chunk));
        check(chunk, n);
    }
    const ItemCount big(0x7FFFFF00ull);
    for (uint64_t k : {uint64_t(1), uint64_t(1000), uint64_t(100000)})
        for (int64_t off : {-1, 0, 1}) {
            const uint64_t n = k * 0x7FFFFF00ull + off;
            expect(big(n) == n / 0x7FFFFF00ull + (n % 0x7FFFFF00ull != 0), "ItemCount of long items");
        }
    // a long ragged list costs a pass, well below a sort of its rests (the best of
    // five of both: a sort takes about ten times as long)
    std::vector<uint64_t> n(1000000);
    for (uint64_t &x : n)
        x = 1000 + gen() % 10000;
    std::vector<WorkItem> items(n.size());
    std::vector<uint32_t> first(n.size() + 1);
    double list = 1e9, sort = 1e9;
    for (int k = 0; k < 5; ++k) {
        auto t = std::chrono::steady_clock::now();
        list_items(16384, n.data(), n.size(), nullptr, nullptr, 7, first.data(), items.data());
        list = std::min(list, seconds(t));
        std::vector<WorkItem> copy(n.size());
        for (size_t s = 0; s < n.size(); ++s)
            copy[s] = WorkItem{nullptr, nullptr, 0, uint32_t(s), uint32_t(n[s])};
        t = std::chrono::steady_clock::now();
        std::stable_sort(copy.begin(), copy.end(),
                         [](const WorkItem &a, const WorkItem &b) { return a.count > b.count; });
        sort = std::min(sort, seconds(t));
    }
    std::printf("10^6 rests: listed in %.1f ms, a sort alone %.1f ms\n", list * 1e3, sort * 1e3);
    expect(list < 0.5 * sort, "long list slow");
    return bad != 0;
}
