// Whole-tile splits of staged calls over random layers, token counts and workspaces: every tile of the call belongs to one
// workgroup and round, the tiles cover the outputs and their weight words fit the room.  Host only; prints the first violation.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "skl_split.h"

#define CHECK(c)                                                                                                             \
    do {                                                                                                                     \
        if (!(c)) {                                                                                                          \
            printf("out %u, blocks %u, tokens %u, room %llu: cb %u, %s\n", out, nb, tokens, (unsigned long long)room, cb, #c); \
            return 1;                                                                                                        \
        }                                                                                                                    \
    } while (0)

int main()
{
    uint64_t s = 88172645463325252ull, seen[12] = {};
    auto rnd = [&](uint32_t lo, uint32_t hi) { s ^= s << 13; s ^= s >> 7; s ^= s << 17; return lo + (uint32_t)(s % (hi - lo + 1)); };
    for (uint32_t n = 0; n < 20000; ++n) {
        const uint32_t out = rnd(0, 3) ? rnd(1, 12000) : rnd(1, 60000), nb = rnd(1, 200), tokens = rnd(129, 4200);
        const uint64_t room = rnd(0, 3) ? ~0ull : (uint64_t)rnd(1, 60000) << rnd(0, 14);
        G3Split sp{};
        const uint32_t cb = skl_make_wide_split(out, nb, tokens, room, sp);
        CHECK(cb == 0 || cb == 4 || cb == 6 || cb == 7 || cb == 8 || cb == 10 || cb == 11);
        ++seen[cb];
        if (!cb) continue;
        CHECK((uint64_t)sp.n_col * nb * cb * 4096 <= room);
        CHECK(sp.n_col * cb * 32 >= out && (sp.n_col - 1) * cb * 32 < out);
        CHECK(sp.m_tiles * 256 >= tokens && (sp.m_tiles - 1) * 256 < tokens);
        std::vector<uint8_t> done((size_t)sp.n_col * sp.m_tiles, 0);
        for (uint32_t x = 0; x < 8; ++x)
            for (uint32_t wg = 0; wg < 32; ++wg)
                for (uint32_t k = wg; k < sp.tiles_of(x); k += 32) {        // as the kernel walks them
                    uint32_t tm, tn;
                    sp.tile_of(x, k, tm, tn);
                    CHECK(tm < sp.m_tiles && tn < sp.n_col && !done[(size_t)tn * sp.m_tiles + tm]);
                    done[(size_t)tn * sp.m_tiles + tm] = 1;
                }
        for (uint8_t d : done) CHECK(d);
    }
    for (uint32_t cb : {0u, 4u, 6u, 7u, 8u, 10u, 11u})
        if (seen[cb] < 20) {
            printf("width %u chosen %llu times only\n", cb, (unsigned long long)seen[cb]);
            return 1;
        }
    return 0;
}
