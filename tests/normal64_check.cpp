// Host check of the samplers' double-precision functions (normal64.hpp): the
// same IEEE operations compiled for the host, against long double.  Prints one
// line per function: name, largest error in units in the last place of the
// result, its mean.  The hardware's approximate reciprocals are stood in for by
// exact ones with a relative error of up to 2^-22 put on them.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>

#include "normal64.hpp"

using namespace bfi::nrm;

struct Worst {
    double most = 0.0, sum = 0.0;
    long n = 0;
    // floor: the size below which an error counts against this size's unit
    void add(double got, long double want, double floor = 0.0)
    {
        const double w = std::max(std::fabs(static_cast<double>(want)), floor);
        const double ulp = std::nextafter(w, INFINITY) - w;
        const double e = static_cast<double>(std::fabs(static_cast<long double>(got) - want)) / ulp;
        most = std::isnan(e) ? INFINITY : std::max(most, e);
        sum += e;
        ++n;
    }
    void tell(const char *name) const { std::printf("%s %.4f %.4f\n", name, most, sum / n); }
};

int main()
{
    const long double pi = 3.14159265358979323846264338327950288L;
    std::mt19937_64 gen(20261205);
    std::uniform_real_distribution<double> off(-0x1p-22, 0x1p-22), logy(-22.0, 0.0), wide(-50.0, 50.0);
    Worst log_w, log_y, cos_w, sin_w, root_w, rroot_w, rec_w;
    auto word = [&](long i) -> uint32_t {
        // the ends, the neighbours of every 64th, and random words
        if (i < 64)
            return static_cast<uint32_t>(i);
        if (i < 128)
            return 0xFFFFFFFFu - static_cast<uint32_t>(i - 64);
        if (i < 128 + 64 * 64)
            return static_cast<uint32_t>((i - 128) / 64 * 0x2000000u + (i - 128) % 64 - 32u);
        return static_cast<uint32_t>(gen());
    };
    for (long i = 0; i < 2000000; ++i) {
        const uint32_t x = word(i);
        const double half = static_cast<double>(x) + 0.5;
        log_w.add(minus_2log<32>(half, kLog), -2.0L * logl(static_cast<long double>(half) * 0x1p-32L));
        const double y = std::exp(logy(gen));
        log_y.add(minus_2log<0>(y, kLog), -2.0L * logl(static_cast<long double>(y)));
        double c, s;
        turn(x, kTurn, &c, &s);
        // the angle within an eighth of a turn of an axis, exactly
        const uint32_t q = (x + 0x20000000u) >> 30;
        const long double a =
            (static_cast<long double>(static_cast<int32_t>(x - (q << 30))) + 0.5L) * 2.0L * pi * 0x1p-32L;
        const long double ca = cosl(a), sa = sinl(a);
        const long double wc = q == 0 ? ca : q == 1 ? -sa : q == 2 ? -ca : sa;
        const long double ws = q == 0 ? sa : q == 1 ? ca : q == 2 ? -sa : -ca;
        // (a normal is the radius times either: errors count against 1/8 where
        // the sine or cosine is smaller)
        cos_w.add(c, wc, 0.125);
        sin_w.add(s, ws, 0.125);
        const double v = std::exp(wide(gen)), b = std::exp(wide(gen));
        const long double rv = 1.0L / sqrtl(static_cast<long double>(v));
        const double seed = static_cast<double>(rv) * (1.0 + off(gen));
        root_w.add(root(v, seed), sqrtl(static_cast<long double>(v)));
        rroot_w.add(reciprocal_root(v, seed), rv);
        rec_w.add(reciprocal(b, 1.0 / b * (1.0 + off(gen))), 1.0L / static_cast<long double>(b));
    }
    log_w.tell("log_word");
    log_y.tell("log");
    cos_w.tell("cos");
    sin_w.tell("sin");
    root_w.tell("root");
    rroot_w.tell("rroot");
    rec_w.tell("reciprocal");
    return 0;
}
