// The way of staged calls of more than 128 tokens: for every four of 64-channel blocks, outputs, tokens and tail on the command
// line a line of the kind (shared, half or whole), the width of whole tiles in 32 outputs, the chains of sums in them and the measure
// of rounding of the shared split.  Host only.
#include <cstdio>
#include <cstdlib>

#include "skl_split.h"

int main(int argc, char **argv)
{
    for (int i = 1; i + 3 < argc; i += 4) {
        const uint32_t nb = atoi(argv[i]), out = atoi(argv[i + 1]), tokens = atoi(argv[i + 2]), tail = atoi(argv[i + 3]);
        const G3Split sp = skl_make_split(out, nb, tokens, true);
        const WideSplit w = skl_staged_product(out, nb, tokens, tail);
        printf("%s %u %u %.9g\n", w.cb ? "whole" : sp.single ? "half" : "shared", w.cb, w.split ? w.chains + (w.body < nb && !w.join) : 1, skl_split_rounding(sp, nb).like);
    }
}
