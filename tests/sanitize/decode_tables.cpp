// LDS areas of decode plans over layers of small and large tables: the copy of a block's table (whole chunks of 1 KiB) ends
// before what lies behind the table area, and everything fits a CU.  Host only; prints the first violation.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "skl_internal.h"

#define CHECK(c)                                                                                          \
    do {                                                                                                  \
        if (!(c)) {                                                                                       \
            printf("%u x %u, d = %u, K = %u, wide %u: table area %u, %s\n", in, out, d, K, wide, L.tab_bytes, #c); \
            return 1;                                                                                     \
        }                                                                                                 \
    } while (0)

int main()
{
    uint32_t planned = 0, small_alone = 0, small_beside = 0;
    const uint32_t ones[8] = {1, 3, 5, 7, 9, 11, 13, 15};
    for (uint32_t in : {24u, 520u, 8192u, 32768u, 65536u})
        for (uint32_t out : {64u, 333u, 4096u, 28672u})
            for (uint32_t d : {1u, 2u, 4u, 7u})
                for (uint32_t K : {1u, 2u, 4u, 9u, 300u})
                    for (uint32_t wide : {0u, 8000u}) {   // one channel in 64 this wide
                        if ((uint64_t)in * d * K > 4000000u || (uint64_t)in * out > 2200000000ull) continue;
                        std::vector<uint32_t> width(in, K);
                        for (uint32_t j = 0; wide && j < in; j += 64) width[j] = wide;
                        uint64_t n = 0;
                        for (uint32_t w : width) n += (uint64_t)w * d;
                        if (n > 20000000u) continue;
                        const std::vector<uint16_t> states(n, 0);
                        skl_desc_t D{};
                        D.struct_size = sizeof D;
                        D.in_features = in; D.out_features = out; D.tile_in = 1; D.tile_out = out; D.d = d;
                        D.hash_a = D.hash_c = ones;
                        D.group_width = width.data();
                        D.states = states.data(); D.n_states = n;
                        skl_plan P;
                        if (skl_make_plan(&D, &P) != SKL_OK) continue;
                        const skl_layer &L = P.L;
                        if (L.path != 1) continue;
                        ++planned;
                        for (const skl_group_info &g : P.ginfo)
                            for (uint32_t b = g.b_lo; b < g.b_hi; ++b) {
                                const uint32_t padded = std::max(1024u, d * P.bmeta[b].K * P.bmeta[b].rs * 16);
                                const uint32_t unpadded = (d * P.bmeta[b].K * P.bmeta[b].nb + 63) / 64 * 1024;
                                CHECK((g.flags & 2 ? SKL_PBUF_DIST : 0) + padded <= L.tab_bytes);
                                CHECK(!(g.flags & 2) || padded <= SKL_PBUF_DIST);
                                CHECK((g.flags & 1 ? SKL_PBUF_DIST : 0) + unpadded <= L.ptab_bytes);
                                if (padded == 1024) (g.flags & 2 ? small_beside : small_alone) += 1;
                            }
                        // as the launches size it: batched, sixteen rows of activations; one row, sums, state-row addresses, activations
                        CHECK(L.tab_bytes + 32ull * ((L.max_group_chan / 8 | 1) * 8) <= SKL_LDS_HARD_BYTES);
                        CHECK(L.ptab_bytes + 4096ull * (L.decode_upw + d) + 2ull * (L.max_group_chan + 64) <= SKL_LDS_HARD_BYTES);
                    }
    printf("%u layers; small tables: %u with one buffer, %u with two\n", planned, small_alone, small_beside);
    return planned > 200 && small_alone > 1000 && small_beside > 1000 ? 0 : 1;
}
