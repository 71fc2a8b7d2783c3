// Whole-tile splits of staged calls over random layers, token counts and workspaces: every tile of the call belongs to one
// workgroup and round, the tiles cover the outputs, their weight words and first chains fit the room, and the float32 sums
// are rounded no more than those of the shared tiles they replace; segments of the rebuild launch.  Host only; prints the first violation.
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

// The roundings of one output, a quarter each: a matrix instruction rounds its sum once per eight channels, an addition of
// chains the sum so far.  Sizes are fractions of the result: of all channels alike, or (wide) of the narrow ones alone, whose
// own roundings are the smaller part there; an addition behind the last block then counts 14.75 more, 9.75 for the tail's own
// chain.  `join`: the last chain is not added but takes up the sum of those before it.
static double roundings(const std::vector<uint32_t> &chains, uint32_t nb, bool wide, bool join = false, bool tail = false)
{
    double sum = 0, so_far = 0;
    for (size_t i = 0; i < chains.size(); ++i) {
        const bool last = i + 1 == chains.size(), joins = join && last;
        if (!(wide && tail && last))
            for (uint32_t k = 1; k <= 8 * chains[i]; ++k) sum += ((joins ? so_far : 0) + k / 8.0) / nb / 4;
        so_far += chains[i];
        if (i && !joins) sum += so_far / nb / 4;
    }
    if (wide && chains.size() > 1 && !join) sum += tail ? 9.75 : 14.75;
    return sum;
}

// The mean over the outputs of the shared-tile split, by walking it as the kernel does.
static double shared_roundings(const G3Split &sp, bool wide)
{
    std::vector<std::vector<uint32_t>> tiles(sp.T);
    for (uint32_t x = 0; x < 8; ++x)
        for (uint32_t wg = 0; wg < sp.gx; ++wg) {
            uint32_t round = 0, u = sp.share_begin(x, wg);
            G3Split::Seg sg;
            while (sp.next(x, wg, round, u, sg)) {
                uint32_t tm, tn;
                sp.tile_of(x, sg.k, tm, tn);
                tiles[(size_t)tn * sp.m_tiles + tm].push_back(sg.k1 - sg.k0);
            }
        }
    double sum = 0;
    for (const auto &t : tiles) sum += roundings(t, sp.nb, wide);
    return sum / sp.T;
}

int main()
{
    uint64_t s = 88172645463325252ull, seen[12] = {}, divided[12] = {};
    auto rnd = [&](uint32_t lo, uint32_t hi) { s ^= s << 13; s ^= s >> 7; s ^= s << 17; return lo + (uint32_t)(s % (hi - lo + 1)); };
    for (uint32_t n = 0; n < 8000; ++n) {
        const uint32_t out = rnd(0, 3) ? rnd(1, 12000) : rnd(1, 60000), nb = rnd(1, 200), tokens = rnd(129, 4200);
        const uint64_t room = rnd(0, 3) ? ~0ull : (uint64_t)rnd(1, 60000) << rnd(0, 14);
        const uint32_t tail = std::min(rnd(0, 3), nb - 1);
        const WideSplit w = skl_make_wide_split(out, nb, tokens, room, tail);
        const G3Split &sp = w.sp;
        const uint32_t cb = w.cb;
        CHECK(cb == 0 || cb == 4 || cb == 6 || cb == 7 || cb == 8 || cb == 10 || cb == 11);
        ++seen[cb];
        if (!cb) continue;
        CHECK((uint64_t)sp.n_col * nb * cb * 4096 + skl_wide_part_bytes(w) <= room);
        CHECK(w.chains >= 1 && w.chains <= w.body && (w.chains > 1 || w.body < nb) == (w.split > 0));
        CHECK(w.split ? w.body == (cb <= SW_HELD_CB ? nb - tail : nb) : w.body == nb);
        CHECK(cb <= SW_HELD_CB ? w.split == 0 || w.split == cb : w.split <= cb && w.chains <= 2);
        CHECK(skl_wide_part_bytes(w) == (cb <= SW_HELD_CB ? 0ull : 256ull * 8 * w.split * 4 * 64 * 16));
        std::vector<uint32_t> chains;
        for (uint32_t i = 0; i < w.chains; ++i) chains.push_back((i + 1) * w.body / w.chains - i * w.body / w.chains);
        if (w.body < nb) chains.push_back(nb - w.body);
        const G3Split shared = skl_make_split(out, nb, tokens, true);
        for (const bool wide : {false, true}) {
            if (wide && !tail) continue;
            const double one = roundings({nb}, nb, wide);
            double more = 0;
            if (cb <= SW_HELD_CB || !w.split)
                more = roundings(chains, nb, wide, w.body < nb && w.join, w.body < nb);
            else
                for (uint32_t c = 0; c < w.split; ++c)
                    for (uint32_t wg = 0; wg < 32; ++wg) {
                        const uint32_t end = skl_first_chain_end(nb, w.split, c, wg);
                        CHECK(end >= 1 && end < nb && (c == 0 || end >= skl_first_chain_end(nb, w.split, c - 1, wg)));
                        more += roundings({end, nb - end}, nb, wide) / (32 * w.split);
                    }
            const uint32_t many = w.split ? w.split : cb;
            // (the planner counts a chain of l blocks as l^2, here it is l^2 + l / 8, and the ends of chains on the mean)
            CHECK((many * more + (cb - many) * one) / cb <= shared_roundings(shared, wide) + 0.4);
        }
        divided[cb] += w.split > 0;
        // the rebuild launch: every segment has outputs; and 131 blocks of 8192 outputs don't start a second round for six of them
        const uint32_t cols = (out + 255) / 256, seg = skl_rebuild_segments(nb, 8 * nb, 65536ull * nb, cols);
        CHECK(seg >= 1 && seg <= cols);
        CHECK(skl_rebuild_segments(131, 8 * 131, 65536ull * 131, 32) == 3);
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
    for (uint32_t cb : {4u, 6u, 7u, 8u, 10u, 11u})
        if (divided[cb] < 20 || (cb == 4 && seen[cb] - divided[cb] < 20)) {
            printf("width %u in several chains %llu of %llu times\n", cb, (unsigned long long)divided[cb], (unsigned long long)seen[cb]);
            return 1;
        }
    return 0;
}
