// Host driver of the index walks of the kernels (csrc/fsg_internal.hpp) at the
// largest arc index a graph may have: every position of a row is visited once,
// none outside it, and every share of a row lies inside it.
#include <cstdio>
#include <vector>

#include "fsg_internal.hpp"

using namespace fsg;

struct Outside {};

static int fail(const char *what, long long a, long long b, long long c)
{
    std::printf("FAIL %s: %lld %lld %lld\n", what, a, b, c);
    return 1;
}

int main()
{
    const int64_t end = ((int64_t)1 << 31) - 256;  // one past the last arc
    for (int64_t deg : {1, 255, 256, 1023, 1024, 1025, 4095, 4097, 9000})
        for (int S : {1, 4, 64, 128, 256, 1024}) {
            const int64_t e0 = end - deg;
            std::vector<int> seen((size_t)deg, 0), some((size_t)deg, 0);
            long long calls = 0;
            auto visit = [&](std::vector<int> &m, uint32_t e) {
                const int64_t i = (int64_t)(int32_t)e - e0;  // as an int32 index
                if (i < 0 || i >= deg || ++calls > 8 * deg + 8 * S) throw Outside();
                ++m[(size_t)i];
            };
            try {
                for (int s = 0; s < S; ++s) {
                    calls = 0;
                    walk_arcs((uint32_t)e0 + (uint32_t)s, (uint32_t)end, (uint32_t)S,
                              [&](uint32_t e) {
                                  for (int j = 0; j < 4; ++j) visit(seen, e + (uint32_t)(j * S));
                              },
                              [&](uint32_t e) { visit(seen, e); });
                    calls = 0;
                    any_arcs((uint32_t)e0 + (uint32_t)s, (uint32_t)end, (uint32_t)S,
                             [&](uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
                                 for (uint32_t e : {a, b, c, d}) visit(some, e);
                                 return false;
                             });
                }
            } catch (const Outside &) {
                return fail("walk outside the row", deg, S, 0);
            }
            for (int64_t i = 0; i < deg; ++i)
                if (seen[(size_t)i] != 1 || some[(size_t)i] < 1) return fail("position", deg, S, i);
        }
    for (int64_t deg : {(int64_t)257, (int64_t)100000, end - 1, end})
        for (int groups : {16, 32}) {  // as the aggregations cut a wide row
            const int per = (((int)deg + groups - 1) / groups + 15) & ~15;
            int64_t next = 0;
            for (int i = 0; i < groups; ++i) {
                int lo = 0, hi = 0;
                share_of((int)deg, per, i, lo, hi);
                if (lo < 0 || hi < lo || hi > deg || (lo < hi && lo != next)) return fail("share", deg, groups, i);
                if (lo < hi) next = hi;
            }
            if (next != deg) return fail("shares", deg, groups, next);
        }
    std::printf("index walks ok\n");
    return 0;
}
