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
    uint64_t s = 88172645463325252ull, planned = 0, refused = 0, bounded = 0;
    auto rnd = [&](uint32_t lo, uint32_t hi) { s ^= s << 13; s ^= s >> 7; s ^= s << 17; return lo + (uint32_t)(s % (hi - lo + 1)); };
    for (uint32_t n = 0; n < 200000; ++n) {
        const uint32_t out = rnd(0, 3) ? rnd(1, 2000) : rnd(1, 60000), tokens = rnd(1, SKL_PROMPT_MAX_TOKENS), n_blocks = rnd(1, rnd(0, 1) ? 12 : 900);
        const uint32_t nb = 1u << rnd(0, 3);                    // words per block
        const PromptLayer L{out, rnd(1, 8), n_blocks, (n_blocks * nb + 7) / 8, n_blocks * ((nb + 3) / 4), 1000ull * rnd(1, 65) * n_blocks};
        const uint64_t room = (uint64_t)rnd(1, 60000) << rnd(0, 14);
        // as many groups as some split has chains, up to more than there are blocks; or whatever the model likes best
        const Rounding any{HUGE_VAL, HUGE_VAL};
        Rounding most = skl_chain_rounding(n_blocks, L.kb, rnd(1, std::min(n_blocks, 80u)), 0, false);
        if (rnd(0, 1)) most.wide = HUGE_VAL;
        if (!rnd(0, 3)) most.like *= 0.5;
        if (!rnd(0, 2)) most = any;
        const PromptPlan p = skl_make_prompt_plan(L, tokens, room, most);
        if (!p.P) {
            ++refused;
            continue;
        }
        const Rounding own = skl_prompt_rounding(n_blocks, L.kb, p.P);
        CHECK(own.within(most));

        bounded += skl_make_prompt_plan(L, tokens, room, any).P != p.P;
        ++planned;
        CHECK(p.rb == 2 || p.rb == 4 || p.rb == 6 || p.rb == 8);
        CHECK(p.nw >= 3 && p.nw <= (p.rb >= 6 ? 8u : 12u));
        CHECK(p.P <= n_blocks);                                 // no empty group: group g is blocks [g n / P, (g + 1) n / P)
        for (uint32_t g = 0; g < p.P; ++g) CHECK(g * n_blocks / p.P < (g + 1) * n_blocks / p.P);
        CHECK(p.T * p.nw * 32 >= out && (p.T - 1) * p.nw * 32 < out);
        CHECK(p.M * p.rb * 16 >= tokens && (p.M - 1) * p.rb * 16 < tokens);
        CHECK(p.M > 1 ? p.rows == p.rb : p.rows == (tokens + 15) / 16 && p.rows <= p.rb);
        CHECK(p.pack_bytes == (uint64_t)p.M * 8 * L.kb * p.rb * 256 && p.pack_bytes % 256 == 0);
        CHECK(p.part_bytes == (uint64_t)p.M * p.T * p.P * p.rows * 2 * p.nw * 1024);
        CHECK(p.pack_bytes + p.part_bytes <= room);
    }
    // no groups: a bound that the roundings of no number of groups keep
    {
        const uint32_t out = 4096, tokens = 100, n_blocks = 64;
        const uint64_t room = 1ull << 30;
        const PromptLayer L{out, 4, n_blocks, 64, 128, 64000ull * 64};
        CHECK(!skl_make_prompt_plan(L, tokens, room, Rounding{0.5, HUGE_VAL}).P);
        CHECK(!skl_make_prompt_plan(L, tokens, room, Rounding{HUGE_VAL, 5.0}).P);
    }
    printf("%llu planned (%llu by the bound), %llu refused\n", (unsigned long long)planned, (unsigned long long)bounded, (unsigned long long)refused);
    return planned > 1000 && refused > 1000 && bounded > 1000 ? 0 : 1;
}
