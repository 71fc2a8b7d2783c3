// The way of staged calls of more than 128 tokens: for every triple of 64-channel blocks, outputs and tokens on the command
// line a line of the kind (shared, half or whole), the width of whole tiles in 32 outputs, the chains of sums and the measure
// of rounding of the shared split.  Host only.
#include <cstdio>
#include <cstdlib>

#include "skl_split.h"

int main(int argc, char **argv)
{
    for (int i = 1; i + 2 < argc; i += 3) {
        const uint32_t nb = atoi(argv[i]), out = atoi(argv[i + 1]), tokens = atoi(argv[i + 2]);
        const uint64_t room = skl_staged_part_floats(out, nb, tokens) * 4 + (uint64_t)skl_staged_slab_cols(out, nb, tokens) * nb * SG_SLOT_BYTES;
        const G3Split sp = skl_make_split(out, nb, tokens, true);
        const WideSplit w = skl_make_wide_split(out, nb, tokens, room);
        printf("%s %u %u %.9g\n", w.cb ? "whole" : sp.single ? "half" : "shared", w.cb, w.chains, skl_split_chain(sp));
    }
}
