// Divisions by a product and a shift (kernels.hpp) against the machine's, on the host.
#include <cstdio>
#include <cstdlib>

#include "kernels.hpp"

using namespace strait;

static unsigned long long state = 1;
static unsigned next_random() {
    state = state * 6364136223846793005ULL + 1442695040888963407ULL;
    return (unsigned)(state >> 33);                        // 31 bits
}
static long long checked = 0;
static void check(long long d) {
    const Divisor by = divisor(d);
    auto one = [&](long long n) {
        if (n < 0 || n > 0x7fffffffLL) return;
        ++checked;
        const int q = divide((int)n, by);
        if (q != n / d) {
            printf("%lld / %lld: %d, not %lld\n", n, d, q, n / d);
            exit(1);
        }
    };
    for (long long k = 0; k < 64; ++k) { one(k); one(0x7fffffffLL - k); }
    for (long long m = 1; m <= 16 && d <= 0x7fffffffLL; ++m)     // on both sides of multiples: the first, the last, and some
        for (long long e = -1; e <= 1; ++e) { one(m * d + e); one((0x7fffffffLL / d - m + 1) * d + e); }
    for (int k = 0; k < 64; ++k) {
        one(next_random());
        for (long long e = -1; e <= 1; ++e) one(next_random() / d * d + e);
    }
}

int main() {
    for (long long d = 1; d <= 70000; ++d) check(d);
    for (int s = 1; s < 63; ++s)
        for (long long e = -3; e <= 3; ++e)
            if ((1LL << s) + e > 0) check((1LL << s) + e);  // from 2^31 on, larger than any number divided: 0
    for (int k = 0; k < 200000; ++k) { check((next_random() >> (next_random() % 31)) + 1LL); }
    check(0x7fffffffLL);
    check(0x7fffffffffffffffLL);
    printf("%lld quotients\n", checked);
    return 0;
}
