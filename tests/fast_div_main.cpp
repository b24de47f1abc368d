// Exits with 1 where quot() differs from the division: the edges of every divisor's multiples, and spread values.
#include "lotts_common.h"
#include <cstdio>

int main() {
    const long long top = 0x7fffffff;
    unsigned long long rnd = 12345;
    auto next = [&] { return (rnd = rnd * 6364136223846793005ULL + 1442695040888963407ULL) >> 33; };  // 31 bits
    auto check = [&](long long d) {
        const lotts::FastDiv f = lotts::fast_div((unsigned)d);
        auto one = [&](long long x) {
            if (x < 0 || x > top || lotts::quot((int)x, f) == (int)(x / d)) return true;
            printf("%lld / %lld: %d\n", x, d, lotts::quot((int)x, f));
            return false;
        };
        bool ok = one(0) && one(top) && one(top / d * d) && one(top / d * d - 1);
        for (int i = 0; i < 50; ++i) {
            const long long q = next() % (top / d + 1);
            ok = ok && one(q * d) && one(q * d - 1) && one(q * d + d - 1) && one((long long)next());
        }
        return ok;
    };
    for (long long d = 1; d <= 20000; ++d)
        if (!check(d)) return 1;
    for (int l = 1; l < 31; ++l)
        for (long long d = (1LL << l) - 3; d <= (1LL << l) + 3; ++d)
            if (d > 0 && !check(d)) return 1;
    for (int i = 0; i < 20000; ++i)
        if (!check((long long)next() % top + 1)) return 1;
    return check(top) ? 0 : 1;
}
