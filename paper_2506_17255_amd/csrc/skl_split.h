// Work split of the 256 x 256-tile prefill kernels: which workgroup multiplies which blocks of which output
// tile.  One routine for the kernels, their launchers and the host-side diagnostic (plain C++: also compiled
// by the host compiler alone).
#pragma once

#include <math.h>
#include <stdint.h>
#include <algorithm>

#ifndef __HIPCC__
#ifndef __host__
#define __host__
#endif
#ifndef __device__
#define __device__
#endif
#endif

#define GM_MT 256            // tokens per workgroup tile
#define GM3_NT 256           // outputs per workgroup tile

// Work split of the 256 x 256-tile kernels.  Workgroup ids go round the 8 XCDs (each with its own L2), so
// XCD x runs the workgroups blockIdx.x % 8 == x, gx of them.  Tiles are dealt to the XCDs in units of mu
// token tiles of one output-tile column (mu divides the number of token tiles): unit
// u = tile_n * (m_tiles / mu) + token-tile group belongs to XCD u % 8.
//   mu = 1 (fused kernel: every workgroup streams the same tables, only the activations differ by tile):
//           tile t = tile_n * m_tiles + tile_m belongs to XCD t % 8, so with eight or more token tiles an
//           XCD keeps one token tile's activations in its L2;
//   mu > 1 (staged kernel: both operands come from memory): the workgroups of an XCD that run side by
//           side share weight words as well as activation words; the largest mu that still balances the
//           XCDs is taken (whole columns at best: 8 + 4 distinct operand streams for 32 workgroups at
//           2048 tokens instead of 1 + 32).
// An XCD's tiles are dealt out in rounds of gx whole tiles, and the blocks of the tiles left over after
// the last whole round are cut into equal contiguous shares, one per workgroup, so that every workgroup
// multiplies the same number of blocks (within one).  A share of a leftover tile leaves a float32 partial
// in the workspace; the fix-up kernel adds a tile's partials in workgroup order, which keeps the result
// independent of timing.
struct G3Split {
    uint32_t T, m_tiles, nb, gx;        // tiles, token tiles, blocks per tile, workgroups per XCD
    uint32_t l_max, p_cap;              // workspace slots: [xcd][l_max leftover tiles][p_cap parts]
    uint32_t mu, n_col;                 // token tiles per dealing unit; output tile columns
    uint32_t mt;                        // tokens per tile: GM_MT, or GM_MT / 2 in the single-round mode below
    uint32_t single;                    // every workgroup takes at most one whole tile: no leftovers, no partials
    __host__ __device__ uint32_t tiles_of(uint32_t x) const
    {
        const uint32_t U = n_col * (m_tiles / mu);
        return U > x ? mu * ((U - x + 7) / 8) : 0;
    }
    // the k-th tile of XCD x
    __host__ __device__ void tile_of(uint32_t x, uint32_t k, uint32_t &tile_m, uint32_t &tile_n) const
    {
        const uint32_t n_mg = m_tiles / mu, u = x + 8 * (k / mu);
        tile_n = u / n_mg;
        tile_m = (u % n_mg) * mu + k % mu;
    }
    __host__ __device__ uint32_t rounds(uint32_t x) const { return single ? 1 : tiles_of(x) / gx; }
    __host__ __device__ uint32_t left(uint32_t x) const { return single ? 0 : tiles_of(x) - rounds(x) * gx; }
    __host__ __device__ uint32_t units(uint32_t x) const { return left(x) * nb; }
    // workgroups that take a share of the leftover units: every share holds at least one unit
    __host__ __device__ uint32_t sharers(uint32_t x) const { const uint32_t u = units(x); return u < gx ? u : gx; }
    __host__ __device__ uint32_t share_begin(uint32_t x, uint32_t j) const
    {
        const uint32_t g = sharers(x);
        return j >= g ? units(x) : (uint32_t)(((uint64_t)j * units(x)) / g);
    }
    // the workgroup whose share holds unit v
    __host__ __device__ uint32_t owner(uint32_t x, uint32_t v) const
    {
        return (uint32_t)((((uint64_t)v + 1) * sharers(x) - 1) / units(x));
    }
    __host__ __device__ uint32_t parts(uint32_t x, uint32_t l) const { return owner(x, (l + 1) * nb - 1) - owner(x, l * nb) + 1; }
    __host__ __device__ size_t slot(uint32_t x, uint32_t l, uint32_t part) const { return ((size_t)x * l_max + l) * p_cap + part; }
    __host__ __device__ bool empty(uint32_t x, uint32_t wg) const { return rounds(x) == 0 && share_begin(x, wg) >= share_begin(x, wg + 1); }
    // next segment of workgroup wg of XCD x: blocks [k0, k1) of the XCD's k-th tile.  round and u_next
    // carry the position (start: 0 and share_begin(x, wg)); false when the workgroup is done.
    struct Seg { uint32_t k, k0, k1, whole; size_t part_slot; };
    __host__ __device__ bool next(uint32_t x, uint32_t wg, uint32_t &round, uint32_t &u_next, Seg &sg) const
    {
        const uint32_t n_rounds = rounds(x), u_end = share_begin(x, wg + 1);
        sg.part_slot = 0;
        if (round < n_rounds) {
            if (single && wg >= tiles_of(x)) return false;
            sg.k = wg + round * gx; sg.k0 = 0; sg.k1 = nb; sg.whole = 1;
            ++round;
            return true;
        }
        if (u_next >= u_end) return false;
        const uint32_t l = u_next / nb;
        sg.k0 = u_next - l * nb;
        sg.k1 = sg.k0 + (u_end - u_next) < nb ? sg.k0 + (u_end - u_next) : nb;
        sg.k = n_rounds * gx + l;
        // a share of the leftover tiles always leaves a partial, also when it happens to cover a whole
        // tile: the fix-up pass stores every leftover tile from its slots
        sg.whole = 0;
        sg.part_slot = slot(x, l, wg - owner(x, l * nb));
        u_next += sg.k1 - sg.k0;
        return true;
    }
};
#define G3_SLOT_FLOATS 65536u           // one 256 x 256 partial

// Short prompts: staged calls of at most SKL_SHORT_TOKENS tokens are one token tile of 64 or 128 tokens.
#define SKL_SHORT_TOKENS 128u
static inline uint32_t skl_short_mt(uint32_t tokens) { return tokens <= 64 ? 64 : 128; }

// Work split of the short-prompt product (one token tile): an output tile's 64-channel blocks are cut into P equal
// contiguous shares, one workgroup each.  Every weight word is read by exactly one workgroup, so nothing is gained from
// keeping a tile on one XCD.  P > 1: every share leaves a float32 partial in slot [tile][share], added up in share order.
struct ShortSplit {
    uint32_t T, nb, P;                  // output tiles, blocks per tile, shares per tile
    __host__ __device__ bool empty(uint32_t xcd, uint32_t wg) const { return wg * 8 + xcd >= T * P; }
    __host__ __device__ uint32_t share_begin(uint32_t, uint32_t) const { return 0; }
    __host__ __device__ void tile_of(uint32_t, uint32_t k, uint32_t &tile_m, uint32_t &tile_n) const { tile_m = 0; tile_n = k; }
    // a workgroup's only segment
    __host__ __device__ bool next(uint32_t xcd, uint32_t wg, uint32_t &round, uint32_t &, G3Split::Seg &sg) const
    {
        if (round++) return false;
        const uint32_t w = wg * 8 + xcd, part = w % P;
        sg.k = w / P;
        sg.k0 = part * nb / P;
        sg.k1 = (part + 1) * nb / P;
        sg.whole = P == 1;
        sg.part_slot = w;
        return true;
    }
};

// The fewest equal shares per tile that make 128 workgroups, but shares of at least four blocks.  More shares stream the
// weights no faster and write more partials (while the split was chosen, 4096 x 11008, 100 tokens, whole call by
// workgroups: 43 75.5 us, 86 60.7, 129 55.4, 172 56.2, 215 58.5; 4096 x 4096: 64 38.2, 128 33.9, 256 40.8); shares that
// ran on into the next tile, 62 us, added a partial and a second start-up to most workgroups.  (65 to 127 tiles need two
// shares each, up to 254 workgroups: one share would leave half the chip without work.)
static inline ShortSplit skl_make_short_split(uint32_t out, uint32_t nb)
{
    ShortSplit sp;
    sp.T = (out + GM3_NT - 1) / GM3_NT;
    sp.nb = nb;
    sp.P = std::max(1u, std::min((127 + sp.T) / sp.T, nb / 4));
    return sp;
}

// The split of a call: nb blocks per tile, 256 CUs = 32 workgroups per XCD (fewer when the busiest XCD's
// share of the work is under four blocks per workgroup).  grouped: deal tiles in units of several token
// tiles of one column -- the largest unit (halving from a whole column) whose busiest XCD is within 3 %
// of the best.
static inline G3Split skl_make_split(uint32_t out, uint32_t nb, uint32_t tokens, bool grouped)
{
    G3Split sp;
    sp.n_col = (out + GM3_NT - 1) / GM3_NT;
    sp.nb = nb;
    auto most = [&]() { uint32_t m = 0; for (uint32_t x = 0; x < 8; ++x) m = std::max(m, sp.tiles_of(x)); return m; };
    auto deal = [&](uint32_t mt) {
        sp.mt = mt;
        sp.m_tiles = (tokens + mt - 1) / mt;
        sp.T = sp.m_tiles * sp.n_col;
        sp.mu = 1;
        if (grouped) {
            const uint32_t best = (sp.T + 7) / 8;               // tiles of the busiest XCD when dealt one by one
            for (uint32_t mu = sp.m_tiles; mu >= 1; mu /= 2) {
                if (sp.m_tiles % mu) continue;
                sp.mu = mu;
                if (most() * 100 <= best * 103) break;
            }
        }
    };
    sp.single = 0;
    sp.gx = 1; sp.l_max = 0; sp.p_cap = 0;
    // Staged kernel, calls whose tiles of half the height (128 tokens: 32 per wavefront instead of 64) fill
    // at least seven eighths of the CUs exactly once: every workgroup multiplies one whole such tile.  With
    // full-height tiles these calls have fewer tiles than CUs, so that every tile would be shared by two
    // workgroups, written as float32 partials and passed through the fix-up.  (A block of a half-height
    // tile takes 0.55 of the time of a full-height one, measured; below 225 tiles sharing is faster.)
    if (grouped) {
        const uint32_t t_half = ((tokens + GM_MT / 2 - 1) / (GM_MT / 2)) * sp.n_col;
        if (t_half > 224 && t_half <= 256) {
            deal(GM_MT / 2);
            if (most() <= 32) {
                sp.single = 1;
                sp.gx = 32;
                return sp;
            }
        }
    }
    deal(GM_MT);
    sp.gx = (uint32_t)std::min<uint64_t>(32, std::max<uint64_t>(1, (uint64_t)most() * nb / 4));
    for (uint32_t x = 0; x < 8; ++x) {
        if (x && sp.left(x) == sp.left(x - 1)) continue;        // (neighbours mostly share alike)
        sp.l_max = std::max(sp.l_max, sp.left(x));
        for (uint32_t l = 0; l < sp.left(x); ++l) sp.p_cap = std::max(sp.p_cap, sp.parts(x, l));
    }
    return sp;
}

// ---- staged calls: slabs and partial tiles ----
#define SG_SLOT_BYTES 32768u            // weight words of one 64-channel block of an output tile (64 channels x 256 outputs)

// Output-tile columns per slab.  The weight words of a slab (kb x 32 KiB per column) are rebuilt, multiplied and released
// before the next slab is touched; up to 1 GiB of weight words the layer is one slab (measured on the 8192 x 28672 layer:
// four slabs of 134 MB cost 8 % -- every slab stages all tables again -- and the product kernel gained nothing from
// finding its words in the memory-side cache).  Slabs are whole rounds of the product kernel (32 columns x 8 token tiles =
// one tile per workgroup at 2048 tokens): about 512 MiB, but never less than one round, which with one token tile is 256
// columns (2 GiB for a layer of 16384 channels).
static inline uint32_t skl_staged_slab_cols(uint32_t out, uint32_t kb, uint32_t tokens)
{
    const uint32_t n_col = (out + GM3_NT - 1) / GM3_NT, m_tiles = (tokens + GM_MT - 1) / GM_MT;
    const uint64_t col_bytes = (uint64_t)kb * SG_SLOT_BYTES;
    if (n_col * col_bytes <= (1ull << 30)) return n_col;
    const uint32_t round_cols = std::max(1u, 256 / std::max(1u, m_tiles));      // columns of one tile per workgroup
    const uint32_t cols = round_cols * (uint32_t)std::max<uint64_t>(1, (512ull << 20) / (round_cols * col_bytes));
    return std::min(n_col, cols);
}

// Room for the partial tiles of a staged call: the most of any slab (the last one may be narrower, and its tiles be cut
// into more shares).
static inline uint64_t skl_staged_part_floats(uint32_t out, uint32_t kb, uint32_t tokens)
{
    const uint32_t n_col = (out + GM3_NT - 1) / GM3_NT, cols = skl_staged_slab_cols(out, kb, tokens);
    uint64_t most = 0;
    for (const uint32_t width : {cols, n_col % cols}) {
        if (!width) continue;
        if (tokens <= SKL_SHORT_TOKENS) {
            const ShortSplit sp = skl_make_short_split(width * GM3_NT, kb);
            if (sp.P > 1) most = std::max(most, (uint64_t)sp.T * sp.P * skl_short_mt(tokens) * GM3_NT);
        } else {
            const G3Split sp = skl_make_split(width * GM3_NT, kb, tokens, true);
            most = std::max(most, (uint64_t)sp.l_max * 8 * sp.p_cap * G3_SLOT_FLOATS);
        }
    }
    return most;
}

// Output segments per channel block in the rebuild launch, one workgroup each: two, or those that take least by rounds of
// 256 workgroups, each of which stages its table (3.7 us for 64 KiB) and rebuilds words of 256 outputs (84 us per 1024).
// Whole calls by segments, 17 tokens (the one chosen in brackets): 4096 x 11008 (67 blocks) 1 53.5, 2 41.7, [3] 40.2, 4 44.0
// us; 8192 x 8192 (131) 1 55.4, 2 59.1, [3] 51.9, 4 54.5; 2048 x 5632 (33) 4 26.1, 6 25.5, [7] 24.8, 8 25.2; 1024 x 8192 (17),
// 33 tokens, 8 24.9, 12 23.1, [15] 23.2, 16 25.5; 4096 x 11008 with 4-bit states (two-word blocks) 1 61.3, [2] 59.6, 4 63.7.
// Long prompts, whose activation workgroups fill the chip beside, hardly differ: 4096 x 11008, 2048 tokens, 2 180.4, [3] 179.9,
// 8 183.5; 8192 x 8192, 513 tokens, 2 131.9, [3] 127.3.
static inline uint32_t skl_rebuild_segments(uint32_t n_blocks, uint32_t n_words, uint64_t table_bytes, uint32_t cols)
{
    const double stage = 3.7 / 65536 * table_bytes / n_blocks, rebuild = 84.0 / 1024 * n_words / n_blocks * cols;
    uint32_t best = 1;
    double least = HUGE_VAL;
    for (uint32_t n = std::min(cols, 2u); n <= std::min(cols, 32u); ++n) {
        const double t = (double)(((uint64_t)n_blocks * n + 255) / 256) * (stage + rebuild / n);
        if (t < least) {
            least = t;
            best = n;
        }
    }
    return best;
}

// ---- rounding of float32 sums ----
// The variance of an output's rounding errors for a way of adding up its products, in units of four roundings of the result
// (a matrix instruction rounds its sums once per eight channels, as the errors of layers of all sizes show): a chain over a
// fraction f of nb blocks counts nb f^2, adding a chain to the sum of those before it a quarter of the fraction reached.
//   like:  all channels contribute alike (channels of equal width);
//   wide:  wide channels, which come last, carry the result (where the layer has such): measured with one percent of them,
//          the others are 1/40 of its variance.  In units of theirs an addition behind the last block, which rounds the whole
//          result, counts 15, and 10 where the last blocks are a chain of their own (their products then meet no sum of
//          others in the matrix cores).
// Roots of `like` are within 4 % of the errors measured on channels of equal width.
struct Rounding {
    double like, wide;
    bool within(const Rounding &o) const { return like <= o.like * (1 + 1e-9) && wide <= o.wide * (1 + 1e-9); }
};
#define SKL_LAST_ADDITION 14.75         // further weight of an addition behind the last block
#define SKL_LAST_OF_TAIL 9.75

// The mean over the outputs of a split, whose blocks hold the channels of nb (64-channel) blocks.
static inline Rounding skl_split_rounding(const G3Split &sp, double nb)
{
    const double unit = 1.0 / sp.nb;
    Rounding total{}, shared{};
    for (uint32_t x = 0; x < 8; ++x) {
        const uint32_t left = sp.left(x);
        if (!x || left != sp.left(x - 1)) {
            shared = Rounding{};
            for (uint32_t j = 0; left && j < sp.sharers(x); ++j)
                for (uint32_t u = sp.share_begin(x, j), end = sp.share_begin(x, j + 1); u < end;) {
                    const uint32_t k = u % sp.nb, n = std::min(end - u, sp.nb - k);
                    shared.like += nb * (n * unit) * (n * unit) + (k ? 0.25 * (k + n) * unit : 0);
                    if (k && k + n == sp.nb) shared.wide += SKL_LAST_ADDITION;
                    u += n;
                }
        }
        total.like += (double)(sp.tiles_of(x) - left) * nb + shared.like;
        total.wide += shared.wide;
    }
    return {total.like / sp.T, (total.like + total.wide) / sp.T};
}
// n equal chains in a row over all but the last `tail` of `blocks` blocks, which hold the channels of nb.  The last ones are a
// chain of their own or (join) go into the sum of the others: behind the last addition, but each of their products rounds it
// (where wide channels carry the result, those roundings are theirs in any case).
static inline Rounding skl_chain_rounding(uint32_t blocks, double nb, uint32_t n, uint32_t tail, bool join)
{
    const uint32_t body = blocks - tail, l = body / n, longer = body % n;       // chain i: blocks [i body / n, (i + 1) body / n)
    const double unit = 1.0 / blocks, squares = (double)longer * (2 * l + 1) + (double)n * l * l;
    const double ends = n > 1 ? 0.5 * ((double)(body - 1) * (n - 1)) + body - l : 0;        // of the chains behind the first
    const double chains = nb * squares * unit * unit + 0.25 * ends * unit, own = tail && !join ? 0.25 : 0;
    return {chains + own + nb * tail * ((join ? 2.0 * body : 0.0) + tail) * unit * unit,
            chains + own + (tail ? (join ? 0 : SKL_LAST_OF_TAIL) : n > 1 ? SKL_LAST_ADDITION : 0)};
}
// n equal chains whose sums are added up without roundings but the last (one pass).
static inline Rounding skl_prompt_rounding(uint32_t blocks, double nb, uint32_t n)
{
    const uint32_t l = blocks / n, longer = blocks % n;
    const double like = nb * ((double)longer * (2 * l + 1) + (double)n * l * l) / ((double)blocks * blocks) + (n > 1 ? 0.25 : 0);
    return {like, like + (n > 1 ? SKL_LAST_ADDITION : 0)};
}

// Whole tiles of another width instead: 256 tokens x 32 * cb outputs, one tile after another per workgroup (the k-th of XCD
// x by workgroup k % 32), no partial tiles, no fix-up.  An output of a shared tile is the sum of several chains of products,
// one of a whole tile would be a single chain with up to three times the rounding error (4096 x 2048, 600 tokens, channels
// of equal width: 1.4e-7 in eleven chains, 4.1e-7 in one).  So the first `split` of a wavefront's cb columns of outputs
// go through `chains` chains, one after the other, as many as keep both measures above at those of the shared tiles.
// Where those are whole as well, one chain does.
struct WideSplit {
    G3Split sp;
    uint32_t cb, chains, split;         // cb 0: shared tiles
    uint32_t body, join;                // blocks that the chains divide; the rest goes into their sum (join) or is one more
    double us;                          // estimated time of the product
};
#define SW_HELD_CB 6u                   // up to this width the sums of the earlier chains are held in registers
// Bytes of workspace for the first chains of `split` columns, wider tiles: 256 workgroups x 8 wavefronts x 4 KiB each.
static inline uint64_t skl_wide_part_bytes(const WideSplit &w) { return w.cb > SW_HELD_CB ? (uint64_t)w.split << 23 : 0; }

// Blocks of the first chain of column c of `split` through memory, in workgroup wg of an XCD: around the middle, but not all at
// the same time (4096 x 11008, 2048 tokens, 42 MB in one go cost the call 5 us more).
__host__ __device__ static inline uint32_t skl_first_chain_end(uint32_t nb, uint32_t split, uint32_t c, uint32_t wg)
{
    const int end = (int)(nb - split) / 2 + (int)c + ((int)(wg & 7) - 3) * (int)nb / 64;
    return end < 1 ? 1 : end < (int)nb ? end : nb - 1;
}

// cb is 0 where the split above is estimated to be no slower, or weight words and first chains do not fit `room`.
// The estimates of the product, in us: a 64-channel block of a 256 x 256 tile on every CU takes 1.52 (f[cb] per such area;
// narrow tiles read more operand words from LDS per product), 2.2 in a share of a tile; a round of tiles 5 to 8 more for its
// start and its stores; a partial tile 0.05 to write and read; a further chain 0.16 per column held in registers, 1 per
// column and 2 per round through memory; a round that leaves CUs idle runs at a higher clock.
// Whole calls, shared tiles / whole ones by cb, in one chain, then as they run (2048 tokens unless said): 4096 x 11008 224 /
// 4 188, 6 182, 8 198, 11 171, 180 us; 4096 x 4096 81 / 4 76; 2048 x 5632, 1500 tokens, 76 / 6 51, 57; 1024 x 2048 42 / 4 27, 29;
// 3000 x 7001, 1024 tokens, 95 / 4 61, 62; 8192 x 28672 845 / 4 900, 6 829, 8 835, 10 803, 811, 11 834; 4096 x 11008, 777
// tokens, 164 / 6 102, 105; 8192 x 3000, 1300 tokens, 137 / 4 110, 112; 4096 x 2048, 600 tokens, 49 / 4 53, 61 in twelve chains.
// tail: last blocks, those that hold the wide channels of the layer (0: it has none).
static inline WideSplit skl_make_wide_split(uint32_t out, uint32_t nb, uint32_t tokens, uint64_t room, uint32_t tail)
{
    const G3Split old = skl_make_split(out, nb, tokens, true);
    Rounding most = skl_split_rounding(old, nb);
    if (!tail) most.wide = HUGE_VAL;
    double whole = 0, shared = 0;
    uint32_t slots = 0, rounds = 1, of_x = 0;
    for (uint32_t x = 0; x < 8; ++x) {
        whole = std::max(whole, old.rounds(x) * nb * (old.mt < GM_MT ? 0.6 : 1.0));
        shared = std::max(shared, (double)old.units(x) / old.gx);
        rounds = std::max(rounds, old.rounds(x));
        if (!x || old.left(x) != old.left(x - 1)) {
            of_x = 0;
            for (uint32_t l = 0; l < old.left(x); ++l) of_x += old.parts(x, l);
        }
        slots += of_x;
    }
    WideSplit best{};
    best.us = 1.52 * whole + 2.2 * shared + 8.0 * rounds + (slots ? 6.0 + 0.05 * slots : 0.0);
    const struct { uint32_t cb; double f; } widths[] = {{11, 1.486}, {10, 1.49}, {8, 1.52}, {7, 1.59}, {6, 1.62}, {4, 1.77}};
    for (const auto &w : widths) {
        WideSplit c{};
        G3Split &sp = c.sp;
        c.cb = w.cb;
        sp.n_col = (out + 32 * w.cb - 1) / (32 * w.cb);
        sp.nb = nb; sp.mt = GM_MT; sp.single = 1; sp.gx = 32;
        sp.m_tiles = (tokens + GM_MT - 1) / GM_MT;
        sp.T = sp.m_tiles * sp.n_col;
        rounds = ((sp.T + 7) / 8 + 31) / 32;
        c.chains = 1;
        c.body = nb;
        double more = 0;
        const Rounding one = skl_chain_rounding(nb, nb, 1, 0, false);
        if (one.within(most)) {
        } else if (w.cb <= SW_HELD_CB) {
            c.body = nb - tail;
            c.chains = 0;
            for (const bool join : {true, false}) {             // the fewest (without a tail both ways are one)
                double before = 2.0 * nb;
                for (uint32_t n = join || !tail ? 2 : 1; n <= c.body && (!c.chains || n + !join < c.chains + !c.join); ++n) {
                    const Rounding now = skl_chain_rounding(nb, nb, n, tail, join);
                    if (now.within(most)) {
                        c.chains = n;
                        c.join = join;
                    }
                    if (now.like >= before) break;              // (past the least the additions outweigh what they shorten)
                    before = now.like;
                }
            }
            if (!c.chains) continue;
            c.split = w.cb;
            more = 0.16 * w.cb * (c.chains + !c.join) * rounds;
        } else {                                                // two chains, added behind the last block
            const Rounding two = skl_chain_rounding(nb, nb, 2, 0, false);
            c.chains = 2;
            for (c.split = 1; c.split <= w.cb; ++c.split) {
                const double f = (double)c.split / w.cb;
                double unlike = 0;                              // mean square of the ends' distances from the middle
                for (uint32_t i = 0; i < 8 * c.split; ++i) {
                    const double off = skl_first_chain_end(nb, c.split, i >> 3, i & 7) - 0.5 * nb;
                    unlike += off * off / (8 * c.split);
                }
                unlike *= 2.0 / nb;
                if (Rounding{one.like + f * (two.like + unlike - one.like), one.wide + f * (two.wide + unlike - one.wide)}.within(most)) break;
            }
            if (c.split > w.cb) continue;
            more = (2.0 + c.split) * rounds;
        }
        if ((uint64_t)sp.n_col * nb * w.cb * 4096 + skl_wide_part_bytes(c) > room) continue;
        for (uint32_t mu = sp.m_tiles; mu >= 1; mu /= 2) {      // the largest dealing unit that needs no further round
            if (sp.m_tiles % mu) continue;
            sp.mu = mu;
            uint32_t tiles = 0;
            for (uint32_t x = 0; x < 8; ++x) tiles = std::max(tiles, sp.tiles_of(x));
            if ((tiles + 31) / 32 <= rounds) break;
        }
        c.us = (0.6 * rounds + 0.4 * sp.T / 256.0) * nb * w.cb / 8.0 * w.f + 5.0 * rounds + more;
        if (c.us < best.us) best = c;
    }
    return best;
}

// The product of a staged call of more than 128 tokens, in the room that such calls ask for.
static inline WideSplit skl_staged_product(uint32_t out, uint32_t kb, uint32_t tokens, uint32_t tail)
{
    const uint32_t n_col = (out + GM3_NT - 1) / GM3_NT, cols = skl_staged_slab_cols(out, kb, tokens);
    if (cols == n_col) return skl_make_wide_split(out, kb, tokens, skl_staged_part_floats(out, kb, tokens) * sizeof(float) + (uint64_t)cols * kb * SG_SLOT_BYTES, tail);
    WideSplit w = skl_make_wide_split(cols * GM3_NT, kb, tokens, 0, tail);        // slab by slab, in shared tiles
    w.us *= (n_col + cols - 1) / cols;
    return w;
}

// ---- short prompts in one pass ----
// The plan of such a call: tiles of 32 * nw outputs (nw wavefronts) x 16 * rb tokens, the layer's channel blocks cut into P
// groups of consecutive blocks; one workgroup per (output tile, token tile, group).
#define SKL_PROMPT_MAX_TOKENS 512u
struct PromptPlan {
    uint32_t rb, M, rows;               // 16-token blocks per tile, token tiles, 16-token blocks of a tile that are kept
    uint32_t nw, T, P;                  // wavefronts per workgroup, output tiles, block groups
    uint64_t pack_bytes, part_bytes;
    double cost_us;                     // P == 0: no plan fits the room
};
struct PromptLayer {
    uint32_t out, d, n_blocks, kb;      // kb: 64-channel blocks of the channel list
    uint32_t steps;                     // 32-channel steps of all blocks (a block of fewer than four words is one)
    uint64_t table_bytes;               // padded tables
};

// The cheapest plan that fits `room` bytes of workspace, by a model of the three kernels fitted to 3400 plans measured on
// 13 layer shapes (2 to 8 words per state row, d = 2 to 4) x 10 token counts; 5 % rms, and the plan it picks is 2 % slower
// than the fastest one measured on average, 12 % at worst.  A block costs the larger of its copy into LDS and its
// arithmetic plus 0.38 of the smaller; fewer than six wavefronts do not hide each other's latency.
// most: groups whose sums (a chain per group) are rounded more are not taken.
static inline PromptPlan skl_make_prompt_plan(const PromptLayer &L, uint32_t tokens, uint64_t room, const Rounding &most)
{
    uint64_t groups = 0;                                        // bit P - 1: P groups may be taken
    uint32_t least = 0;
    for (uint32_t P = 1; P <= std::min(L.n_blocks, 64u); ++P)
        if (skl_prompt_rounding(L.n_blocks, L.kb, P).within(most)) {
            groups |= 1ull << (P - 1);
            if (!least) least = P;
        }
    PromptPlan best{};
    const uint32_t blocks16 = (tokens + 15) / 16;
    const uint32_t M = (blocks16 + 7) / 8, rb = std::max(2u, (blocks16 + 2 * M - 1) / (2 * M) * 2);
    const uint32_t rows = M > 1 ? rb : blocks16;
    const uint64_t pack = (uint64_t)M * 8 * L.kb * rb * 256;
    const double copy_kb = (double)(L.table_bytes + (uint64_t)8 * L.kb * rb * 256) / 1024.0 / L.n_blocks;
    const double wave_us = (double)L.steps / L.n_blocks * (0.0076 * L.d + 0.0037 * rb);
    const uint32_t units = (L.out + 31) / 32;
    for (uint32_t nw = 3; nw <= (rb >= 6 ? 8u : 12u); ++nw) {
        const uint32_t T = (units + nw - 1) / nw;
        const uint32_t one = 256 / (T * M);                      // groups that fill the chip once
        for (const uint32_t P : {one, one * 2 / 3, one / 8 * 8, 512 / (T * M), 768 / (T * M), least}) {
            if (P < 1 || P > 64 || !(groups >> (P - 1) & 1)) continue;
            const uint64_t part = (uint64_t)M * T * P * rows * 2 * nw * 1024;
            if (pack + part > room) continue;
            const uint32_t per_group = (L.n_blocks + P - 1) / P, rounds = (T * M * P + 255) / 256;
            const double copy = copy_kb * per_group * 0.0141 * (P % 8 ? 1.0 : 0.877);    // whole groups per XCD: a table enters one L2
            const double work = std::max(nw, 6u) * wave_us * per_group;
            const double group = std::max(copy, work) + 0.384 * std::min(copy, work) + 0.353 * per_group + 0.26;
            const double t = 10.67 + rounds * group + 0.219e-6 * part + 0.0455 * P;
            if (!best.P || t < best.cost_us) best = PromptPlan{rb, M, rows, nw, T, P, pack, part, t};
        }
    }
    return best;
}
