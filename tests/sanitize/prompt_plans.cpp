// Plans of one-pass prompts over random layers, token counts and workspaces: what the kernels rely on.  Host only; prints
// the first violation.
#include <cstdio>
#include <cstdlib>

#include "skl_split.h"

#define CHECK(c)                                                                                                         \
    do {                                                                                                                 \
        if (!(c)) {                                                                                                      \
            printf("out %u, blocks %u, tokens %u, room %llu: %s\n", L.out, L.n_blocks, tokens, (unsigned long long)room, #c); \
            return 1;                                                                                                    \
        }                                                                                                                \
    } while (0)

int main()
{
    uint64_t s = 88172645463325252ull, planned = 0, refused = 0;
    auto rnd = [&](uint32_t lo, uint32_t hi) { s ^= s << 13; s ^= s >> 7; s ^= s << 17; return lo + (uint32_t)(s % (hi - lo + 1)); };
    for (uint32_t n = 0; n < 200000; ++n) {
        const uint32_t out = rnd(0, 3) ? rnd(1, 2000) : rnd(1, 60000), tokens = rnd(1, SKL_PROMPT_MAX_TOKENS), n_blocks = rnd(1, rnd(0, 1) ? 12 : 900);
        const uint32_t nb = 1u << rnd(0, 3);                    // words per block
        const PromptLayer L{out, rnd(1, 8), n_blocks, (n_blocks * nb + 7) / 8, n_blocks * ((nb + 3) / 4), 1000ull * rnd(1, 65) * n_blocks};
        const uint64_t room = (uint64_t)rnd(1, 60000) << rnd(0, 14);
        const PromptPlan p = skl_make_prompt_plan(L, tokens, room);
        if (!p.P) {
            ++refused;
            continue;
        }
        ++planned;
        CHECK(p.rb == 2 || p.rb == 4 || p.rb == 6 || p.rb == 8);
        CHECK(p.nw >= 1 && p.nw <= (p.rb >= 6 ? 8u : 12u));
        CHECK(p.P <= n_blocks);                                 // no empty group: group g is blocks [g n / P, (g + 1) n / P)
        for (uint32_t g = 0; g < p.P; ++g) CHECK(g * n_blocks / p.P < (g + 1) * n_blocks / p.P);
        CHECK(p.T * p.nw * 32 >= out && (p.T - 1) * p.nw * 32 < out);
        CHECK(p.M * p.rb * 16 >= tokens && (p.M - 1) * p.rb * 16 < tokens);
        CHECK(p.M > 1 ? p.rows == p.rb : p.rows == (tokens + 15) / 16 && p.rows <= p.rb);
        CHECK(p.pack_bytes == (uint64_t)p.M * 8 * L.kb * p.rb * 256 && p.pack_bytes % 256 == 0);
        CHECK(p.part_bytes == (uint64_t)p.M * p.T * p.P * p.rows * 2 * p.nw * 1024);
        CHECK(p.pack_bytes + p.part_bytes <= room);
    }
    printf("%llu planned, %llu refused\n", (unsigned long long)planned, (unsigned long long)refused);
    return planned > 1000 && refused > 1000 ? 0 : 1;
}
