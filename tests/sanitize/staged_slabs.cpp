// Walks the slabs of staged prefill calls as the launcher does and checks, for every slab, that each block of each of its
// output tiles is multiplied exactly once and that the partial tiles stay inside the room the workspace has for them,
// without overlap and in share order.  Host only; prints the first violation.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "skl_split.h"

#define CHECK(c)                                                                                                    \
    do {                                                                                                            \
        if (!(c)) {                                                                                                 \
            printf("out %u, blocks %u, tokens %u, slab at column %u: %s\n", out, kb, tokens, tile0, #c);            \
            exit(1);                                                                                                \
        }                                                                                                           \
    } while (0)

static uint64_t calls, slabs_of_two;

template <class Split>
static void check_slab(const Split &sp, uint32_t gx, uint32_t mt, bool parts_allowed, uint32_t width, uint64_t room, uint32_t out, uint32_t kb, uint32_t tokens, uint32_t tile0)
{
    const uint32_t m_tiles = (tokens + mt - 1) / mt;
    std::vector<uint32_t> next((size_t)width * m_tiles, 0);             // blocks of the tile covered so far
    std::vector<size_t> slot((size_t)width * m_tiles, SIZE_MAX);        // slot of the tile's last partial
    std::vector<uint8_t> used;
    for (uint32_t wg = 0; wg < gx; ++wg)
        for (uint32_t x = 0; x < 8; ++x) {                              // (the order of the short-prompt shares)
            if (sp.empty(x, wg)) continue;
            uint32_t round = 0, u_next = sp.share_begin(x, wg);
            G3Split::Seg sg;
            while (sp.next(x, wg, round, u_next, sg)) {
                uint32_t tm, tn;
                sp.tile_of(x, sg.k, tm, tn);
                CHECK(tm < m_tiles && tn < width && sg.k0 < sg.k1 && sg.k1 <= kb);
                uint32_t &at = next[(size_t)tn * m_tiles + tm];
                CHECK(sg.k0 == at);
                at = sg.k1;
                if (sg.whole) {
                    CHECK(sg.k0 == 0 && sg.k1 == kb);
                    continue;
                }
                CHECK(parts_allowed);
                CHECK((sg.part_slot + 1) * mt * GM3_NT <= room);
                if (used.size() <= sg.part_slot) used.resize(sg.part_slot + 1, 0);
                CHECK(!used[sg.part_slot]);
                used[sg.part_slot] = 1;
                size_t &last = slot[(size_t)tn * m_tiles + tm];
                CHECK(last == SIZE_MAX ? sg.k0 == 0 : sg.part_slot == last + 1);
                last = sg.part_slot;
            }
        }
    for (uint32_t v : next) CHECK(v == kb);
}

static void check_call(uint32_t out, uint32_t kb, uint32_t tokens)
{
    const uint32_t n_col = (out + GM3_NT - 1) / GM3_NT, cols = skl_staged_slab_cols(out, kb, tokens);
    const uint64_t room = skl_staged_part_floats(out, kb, tokens);
    uint32_t tile0 = 0;
    CHECK(cols >= 1 && cols <= n_col);
    ++calls;
    if (cols < n_col) ++slabs_of_two;
    for (; tile0 < n_col; tile0 += cols) {
        const uint32_t width = std::min(cols, n_col - tile0);
        if (tokens <= SKL_SHORT_TOKENS) {
            const ShortSplit sp = skl_make_short_split(width * GM3_NT, kb);
            CHECK(sp.T == width && sp.P >= 1 && (sp.P == 1 || sp.P * 4 <= kb));
            check_slab(sp, (sp.T * sp.P + 7) / 8, skl_short_mt(tokens), sp.P > 1, width, room, out, kb, tokens, tile0);
        } else {
            const G3Split sp = skl_make_split(width * GM3_NT, kb, tokens, true);
            check_slab(sp, sp.gx, sp.mt, !sp.single, width, room, out, kb, tokens, tile0);
        }
    }
}

int main()
{
    for (uint32_t tokens : {1u, 64u, 65u, 128u, 129u, 600u})
        for (uint32_t kb : {1u, 3u, 4u, 7u, 8u, 9u, 31u, 64u, 173u, 448u})
            for (uint32_t n_col = 1; n_col <= 300; n_col += n_col < 140 ? 1 : 13) check_call(n_col * 256 - (n_col % 3) * 85, kb, tokens);
    // several slabs, a narrower last one
    for (uint32_t tokens : {1u, 128u, 2048u})
        for (uint32_t kb : {64u, 448u, 1024u, 4096u})
            for (uint32_t n_col : {257u, 263u, 300u, 511u, 700u}) check_call(n_col * 256 - 1, kb, tokens);
    printf("%llu calls, %llu in several slabs\n", (unsigned long long)calls, (unsigned long long)slabs_of_two);
    return slabs_of_two ? 0 : 1;
}
