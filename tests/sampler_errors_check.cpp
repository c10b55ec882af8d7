// Host check of the samplers' double-precision functions (normal64.hpp) over all
// their arguments: the same IEEE operations compiled for the host, against long
// double.  Prints one line per function: name, largest error in units in the
// last place of the result (however small the result), its mean.  The hardware's
// approximate reciprocal root is stood in for by the exact one with a relative
// error of up to 2^-22 put on it.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <random>
#include <string>

#include "normal64.hpp"

using namespace bfi;
using namespace bfi::nrm;

struct Worst {
    double most = 0.0, sum = 0.0;
    long n = 0;
    void add(double got, long double want)
    {
        int e;
        (void)std::frexp(static_cast<double>(fabsl(want)), &e);
        const double off = static_cast<double>(fabsl(static_cast<long double>(got) - want)) *
                           std::ldexp(1.0, 53 - e);
        most = std::isnan(off) ? INFINITY : std::fmax(most, off);
        sum += off;
        ++n;
    }
    void tell(const std::string &name) const
    {
        std::printf("%s %.4f %.4f\n", name.c_str(), most, sum / n);
    }
};

// A word: the ends, both sides of every 64th of the range, random ones.
static uint32_t word(long i, std::mt19937_64 &gen)
{
    if (i < 64)
        return static_cast<uint32_t>(i);
    if (i < 128)
        return 0xFFFFFFFFu - static_cast<uint32_t>(i - 64);
    if (i < 128 + 64 * 64)
        return static_cast<uint32_t>((i - 128) / 64 * 0x4000000u + (i - 128) % 64 - 32u);
    return static_cast<uint32_t>(gen());
}

template <int D>
static void radius(std::mt19937_64 &gen)
{
    Worst inner, shells;
    std::uniform_real_distribution<double> part(0.0, 1.0);
    for (long i = 0; i < 500000; ++i) {
        const double v = std::fma(static_cast<double>(word(i, gen)), 0x1p-32, 0x1p-33);
        inner.add(root_of_degree<D, BuiltinFma>(v, kLog), powl(v, 1.0L / D));
        const double t = part(gen), y = std::fma(v, 1.0 - t, t);
        shells.add(root_of_degree<D, BuiltinFma>(y, kLog), powl(y, 1.0L / D));
    }
    inner.tell("inner" + std::to_string(D));
    shells.tell("shell" + std::to_string(D));
}

int main()
{
    const long double pi = 3.14159265358979323846264338327950288L;
    std::mt19937_64 gen(20261205);
    std::uniform_real_distribution<double> off(-0x1p-22, 0x1p-22), wide(-50.0, 50.0);
    Worst log_w, cos_w, sin_w, over_w;
    for (long i = 0; i < 4000000; ++i) {
        const uint32_t x = word(i, gen);
        const double half = static_cast<double>(x) + 0.5;
        log_w.add(minus_2log<32>(half, kLog), -2.0L * logl(static_cast<long double>(half) * 0x1p-32L));
        double c, s;
        turn(x, kTurn, &c, &s);
        // the angle within an eighth of a turn of an axis, exactly
        const uint32_t q = (x + 0x20000000u) >> 30;
        const long double a =
            (static_cast<long double>(static_cast<int32_t>(x - (q << 30))) + 0.5L) * 2.0L * pi * 0x1p-32L;
        const long double ca = cosl(a), sa = sinl(a);
        cos_w.add(c, q == 0 ? ca : q == 1 ? -sa : q == 2 ? -ca : sa);
        sin_w.add(s, q == 0 ? sa : q == 1 ? ca : q == 2 ? -sa : -ca);
        const double v = std::exp(wide(gen)), b = std::exp(wide(gen));
        const long double rv = 1.0L / sqrtl(static_cast<long double>(v));
        over_w.add(over_root(b, v, static_cast<double>(rv) * (1.0 + off(gen))), b * rv);
    }
    log_w.tell("log");
    cos_w.tell("cos");
    sin_w.tell("sin");
    over_w.tell("over_root");
    radius<3>(gen);
    radius<4>(gen);
    radius<6>(gen);
    radius<8>(gen);
    radius<15>(gen);
    radius<16>(gen);
    radius<20>(gen);
    radius<32>(gen);
    return 0;
}
