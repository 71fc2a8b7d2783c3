// Prefill of short prompts over row sketches in one pass (Sec. 3.1 Eq. 5 fused with Y = X W, Sec. 2.1): no weight
// leaves the compute unit that rebuilt it.
//   1. k_prompt_pack: activations to negated binary16, re-ordered into matrix-core operand words;
//   2. k_prompt_gemm: a workgroup owns all tokens x a tile of outputs over a group of consecutive channel blocks; it
//      streams the blocks' tables and activation words through LDS and leaves float32 partial sums;
//   3. k_prompt_reduce: adds the partial sums of a tile in group order and stores Y.
#include "skl_prefill_common.h"

//
// The staged kernels write and read the dense weights once per call; here they exist only between the LDS gathers and the
// matrix instructions of one wavefront.  The kernel is that of the batched decode with up to 128 tokens instead of 16:
// lanes are outputs, a wavefront rebuilds the operand words of 32 outputs and multiplies them with all tokens of its
// tile, whose activation words arrive in LDS beside the table (two buffers each).
// Bound by none of its units alone: of the 36 us that 4096 x 11008, d = 4, 100 tokens took before prompt_run's pipeline, on
// inputs that are not in the caches (250 workgroups of seven wavefronts), the packing launch was 5 and the reduction 5.5;
// without copies the call took 2 us less, without products 4, without the query 2.4, with gathers free of bank conflicts 2,
// without any of these 13.  What helped: chunks copied without bounds checks, an even load per stretch of code and no wait at a
// block's head (prompt_run), packing with all loads in flight.
// Whole call against the kernels it replaces: 17 tokens 45 -> 22.5 us, 48 46 -> 26, 100 59 -> 33, 256 88 -> 71; 8192 x 8192, 128
// tokens, 84 -> 42; 4096 x 4096, 64 tokens, 26 -> 18.3; 1024 x 2048, 300 tokens, 43 -> 18.5.
namespace SKL_NS {

struct PromptArgs {
    HashArgs h;
    const skl_block_meta *bmeta;
    const uint4 *tables;                // padded block tables, [r][k][rs] words
    const uint4 *Xq;                    // activation words: [word of the channel list][RB * 16 tokens]
    float *parts;                       // [tile][group][16-token block][16-output block][64 lanes] x 4 tokens
    uint32_t out, n_blocks;
    uint32_t T, M, P, per_xcd;          // output tiles, token tiles, block groups, workgroups per XCD
    uint32_t rows, n_words;             // 16-token blocks per partial tile, words of the channel list
};

// [token tile][word of the channel list][RB * 16 tokens]: the words of a block are contiguous, so that its copy into LDS is
// one piece and the matrix-core operand reads are free of bank conflicts.
template <int RB>
__global__ __launch_bounds__(SKL_WG) void k_prompt_pack(PackArgs k, uint32_t n_rows)
{
    const uint32_t t0 = blockIdx.x % n_rows * 16, lane = threadIdx.x & 63;
    pack_group<SKL_WG>(k, t0, blockIdx.x / n_rows, [&](uint32_t step) {
        return ((size_t)(t0 / (RB * 16)) * k.n_steps * 4 + step * 4 + (lane >> 4)) * (RB * 16) + t0 % (RB * 16) + (lane & 15);
    });
}

#define PG_X0 (2u * SKL_PBUF_DIST)      // LDS: two table buffers, two activation buffers
#define PG_LDS(rb) (PG_X0 + 2u * (rb) * 2048u)

template <int D, int RB>
struct PromptWalk {
    uint32_t b, b1, buf;                // next block, end of the group, its buffers
    RowBlock bm, nx;                 // block b and the one after it
    BlockAhead ahead;              // the one after those, on its way
    uint32_t lane, wave, nw, o_base, lds0, tile_m;
    float4v acc[RB][2];
};

template <int D, int RB>
__device__ __forceinline__ void prompt_copies(const PromptArgs &p, const PromptWalk<D, RB> &w, const RowBlock &bm, uint32_t buf, ChunkCopy &tab, ChunkCopy &x)
{
    tab.start(p.tables + bm.table_off16, D * bm.K * bm.rs, w.lds0 + buf * SKL_PBUF_DIST, w.wave, w.nw, w.lane);
    x.start(p.Xq + ((size_t)w.tile_m * p.n_words + (bm.chan_off >> 3)) * (RB * 16), bm.nb * (RB * 16), w.lds0 + PG_X0 + buf * (RB * 2048), w.wave, w.nw, w.lane);
}

// A run of consecutive blocks of one width class (NB words per state row): NB / 4 (at least one) steps of 32 channels
// x two 16-output sub-blocks per block, a "pair" each.  A pair is gathered, queried and multiplied in three successive
// stretches of the code, and every stretch holds the reads of one pair, the query of the pair before and the products of the
// one before that, across the blocks: LDS, vector units and matrix cores have an even load, and the barrier that hands
// the buffers over stands where the last pair of a block is gathered but not yet queried, so that its arithmetic covers
// the first gathers of the next block.  Against the gathers of three pairs in flight, the first two in one burst behind
// the barrier, and the metadata of a block waited for at its head: 4096 x 11008, whole call, 17 tokens 25.8 -> 23.4 us, 48
// 29.1 -> 26.8, 100 37.7 -> 35.7, 256 76.7 -> 71.1; 8192 x 8192, 128 tokens, 47 -> 42.5 (the same with the burst, and the
// barrier moved all the same: 38.2, 83 and 44.3 on the last three).
template <int D, int RB, int NB>
__device__ __forceinline__ void prompt_run(const PromptArgs &p, PromptWalk<D, RB> &w)
{
    constexpr uint32_t RS = NB == 1 ? 1 : NB + 1;
    constexpr int NH = NB == 8 ? 2 : 1, NP = 2 * NH;
    // Gathers a stretch ahead of their query need registers for two pairs.  Where these run out (RB = 4 and 8 have the fewest
    // per accumulator, query mode 1 has more temporaries) the gathers of a pair stand behind the query of the pair before:
    // 4096 x 11008, early -> late, mode 0: d = 8, 60 tokens 41.2 -> 39.0 us, 256 102.7 -> 97.4; d = 6, 8192 x 8192, 120 tokens
    // 48.2 -> 45.3; but d = 4, 100 tokens 33.1 -> 33.9, d = 7, 256 tokens 90.4 -> 93.7.  Mode 1: d = 4, 60 tokens 31.2 -> 27.4,
    // 256 84.8 -> 72.2; d = 6, 60 tokens 47.4 -> 30.6, 128 46.3 -> 37.6; d = 8, 256 tokens 120 -> 96.5.
    constexpr bool LATE = SKL_QM == 1 || (D >= 5 && (RB == 4 || RB == 8) && !(D == 7 && RB == 8));
    const uint32_t n = w.lane & 15, kg = w.lane >> 4;
    const uint32_t word = min(kg, (uint32_t)NB - 1);       // classes with fewer than 4 words: lanes past the last word re-read it, their activations count as zero
    const bool x_live = NB >= 4 || kg < (uint32_t)NB;
    const uint4 none = make_uint4(0, 0, 0, 0);
    uint32_t off[2][D], K_prev = 0, xa = 0;
    uint4 q[2][D], a[NH][RB], wd[2] = {none, none};
    auto gather = [&](int pr) {
#pragma unroll
        for (int r = 0; r < D; ++r) q[pr & 1][r] = lds_word_at(off[pr & 1][r] + (pr >> 1) * 64);
    };
    auto read_a = [&](int h) {
#pragma unroll
        for (int i = 0; i < RB; ++i) a[h][i] = lds_word_at(xa + h * (RB * 1024) + i * 256);
    };
    auto query = [&](int pr) {
        uint4 m = q[pr & 1][0];
#pragma unroll
        for (int r = 1; r < D; ++r) m = pk_max_u16x8(m, q[pr & 1][r]);
        wd[pr & 1].x = keys_to_neg_half2_mad(m.x); wd[pr & 1].y = keys_to_neg_half2_mad(m.y);
        wd[pr & 1].z = keys_to_neg_half2_mad(m.z); wd[pr & 1].w = keys_to_neg_half2_mad(m.w);
    };
    auto multiply = [&](int pr) {
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const uint4 ai = NB >= 4 ? a[pr >> 1][i] : keep_if(x_live, a[pr >> 1][i]);
            w.acc[i][pr & 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8v, ai), __builtin_bit_cast(half8v, wd[pr & 1]), w.acc[i][pr & 1], 0, 0, 0);
        }
    };
    auto tail = [&]() { multiply(NP - 2); query(NP - 1); };
    auto stretch = [&](auto read, auto compute) {
        if (!LATE) read();
        __builtin_amdgcn_sched_barrier(0);
        compute();
        __builtin_amdgcn_sched_barrier(0);
        if (LATE) read();
    };
    // nothing is carried into the first block: its predecessor's last pairs are products of zero activations and of keys
    // that stand for finite weights in either query mode
#pragma unroll
    for (int i = 0; i < RB; ++i) a[NH - 1][i] = none;
#pragma unroll
    for (int r = 0; r < D; ++r) q[1][r] = make_uint4(0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u);
    do {
        // block b has arrived, nobody reads the other buffers any more
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        w.nx = w.ahead.block();
        const bool more = w.b + 1 < w.b1;
        ChunkCopy ct, cx;
        prompt_copies<D, RB>(p, w, w.nx, w.buf ^ 1, ct, cx);
        if (!more) ct.off = cx.off = 0xFFFFFFFFu;
        w.ahead.request(p.bmeta + min(w.b + 2, w.b1 - 1));
        if (w.bm.K != K_prev) {
            const uint32_t K = w.bm.K, Kq = K << 8;
            uint32_t ob = w.o_base;
            asm volatile("" : "+v"(ob));
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint32_t o = min(ob + 16 * j + n, p.out - 1);
#pragma unroll
                for (int r = 0; r < D; ++r) {
                    const uint32_t t = __umul24(p.h.A[r], o) + p.h.C[r];
                    off[j][r] = w.lds0 + w.buf * SKL_PBUF_DIST + ((r * K + select_index(t, Kq)) * RS + word) * 16;
                }
            }
            K_prev = K;
        }
        xa = w.lds0 + PG_X0 + w.buf * (RB * 2048) + word * (RB * 256) + n * 16;
        stretch([&]() { gather(0); cx.some(1); ct.some(2); }, tail);    // the tail of the block before
        stretch([&]() { gather(1); if (NH == 2) read_a(0); ct.some(2); cx.some(1); }, [&]() { multiply(NP - 1); query(0); });
        if (NH == 2) {
            stretch([&]() { gather(2); ct.some(2); }, [&]() { multiply(0); query(1); });
            stretch([&]() { gather(3); read_a(1); ct.rest(); cx.rest(); }, [&]() { multiply(1); query(2); });
        } else {
            read_a(0);
            ct.rest();
            cx.rest();
        }
        const uint32_t to = w.buf ? 0u - SKL_PBUF_DIST : SKL_PBUF_DIST;     // to the other buffer
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < D; ++r) off[j][r] += to;
        w.bm = w.nx;
        w.buf ^= 1;
        ++w.b;
    } while (w.b < w.b1 && w.bm.rs == RS);
    tail();
    multiply(NP - 1);
}

// One workgroup per (block group, token tile, output tile), in that order over the XCDs: the workgroups of an XCD stage
// the same tables, which enter its L2 once.  Up to twelve wavefronts (eight where 80 tokens or more of accumulators and
// activation words want 256 registers per lane).
template <int D, int RB>
__global__ __launch_bounds__(RB >= 5 ? 512 : 768) void k_prompt_gemm(PromptArgs p)
{
    const uint32_t q = (blockIdx.x & 7) * p.per_xcd + (blockIdx.x >> 3);
    if (q >= p.T * p.M * p.P) return;
    const uint32_t g = __builtin_amdgcn_readfirstlane(q / (p.T * p.M)), tm = q - g * p.T * p.M, tile_m = __builtin_amdgcn_readfirstlane(tm / p.T), tile = tm - tile_m * p.T;
    const uint32_t b0 = __builtin_amdgcn_readfirstlane(g * p.n_blocks / p.P);
    PromptWalk<D, RB> w;
    w.b = b0;
    w.b1 = __builtin_amdgcn_readfirstlane((g + 1) * p.n_blocks / p.P);
    w.buf = 0;
    w.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    w.nw = blockDim.x >> 6;
    w.lds0 = (uint32_t)(uintptr_t)(lds_void *)smem;
    w.lane = threadIdx.x & 63;
    w.o_base = (tile * w.nw + w.wave) * 32;
    w.tile_m = tile_m;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) w.acc[i][j] = (float4v){0.f, 0.f, 0.f, 0.f};
    w.ahead.request(p.bmeta + b0);
    w.bm = w.ahead.block();
    w.ahead.request(p.bmeta + min(b0 + 1, w.b1 - 1));
    {
        ChunkCopy ct, cx;
        prompt_copies<D, RB>(p, w, w.bm, 0, ct, cx);
        ct.rest();
        cx.rest();
    }
    while (w.b < w.b1) {
        switch (w.bm.rs) {
        case 9: if constexpr (D <= 6) { prompt_run<D, RB, 8>(p, w); break; }
        case 5: prompt_run<D, RB, 4>(p, w); break;
        case 3: prompt_run<D, RB, 2>(p, w); break;
        default: prompt_run<D, RB, 1>(p, w); break;
        }
    }
    float4v *dst = reinterpret_cast<float4v *>(p.parts) + ((size_t)(tm * p.P + g) * p.rows * 2 * w.nw + w.wave * 2) * 64 + w.lane;
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        if ((uint32_t)i >= p.rows) break;
#pragma unroll
        for (int j = 0; j < 2; ++j) dst[((size_t)i * 2 * w.nw + j) * 64] = w.acc[i][j];
    }
}

// y = the sum of the P partials of every output, in group order: a wavefront adds one 16 x 16 block, four partials in
// flight, and the workgroup's 16 x 64 outputs are turned round in LDS to leave as 8- or 16-byte pieces.  Grid (ceil(out /
// 64), 16-token blocks).  The additions are in 64 bits, which the memory-bound kernel does not notice: without roundings of
// their own fewer groups do (skl_prompt_rounding).
__global__ __launch_bounds__(256) void k_prompt_reduce(const float *__restrict__ parts, uint32_t T, uint32_t P, uint32_t nw, uint32_t rows, void *Y, uint32_t y_dt,
                                                       uint32_t ldy, uint32_t tokens, uint32_t out)
{
    __shared__ __align__(16) float sm[16][68];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, rb = blockIdx.y;
    const uint32_t cb = blockIdx.x * 4 + wave, tile = cb / (2 * nw), c = cb - tile * 2 * nw, tm = rb / rows * T + tile;
    const size_t stride = (size_t)rows * 2 * nw * 64;           // float4v per group
    double s[4] = {0, 0, 0, 0};
    auto add = [&](const float4v &v) {
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] += (double)v[i];
    };
    if (cb * 16 < out) {
        const float4v *src = reinterpret_cast<const float4v *>(parts) + (size_t)tm * P * stride + ((size_t)(rb % rows) * 2 * nw + c) * 64 + lane;
        uint32_t g = 0;
        for (; g + 4 <= P; g += 4) {
            float4v v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = src[(size_t)(g + k) * stride];
#pragma unroll
            for (int k = 0; k < 4; ++k) add(v[k]);
        }
        for (; g < P; ++g) add(src[(size_t)g * stride]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) sm[(lane >> 4) * 4 + i][wave * 16 + (lane & 15)] = (float)s[i];
    __syncthreads();
    const uint32_t row = threadIdx.x >> 4, o = blockIdx.x * 64 + (threadIdx.x & 15) * 4, t = rb * 16 + row;
    if (t >= tokens || o >= out) return;
    const float4 v = *reinterpret_cast<const float4 *>(&sm[row][(threadIdx.x & 15) * 4]);
    store_four(Y, y_dt, ldy, t, o, out, v);
}

// ========================================================================
// Launcher
// ========================================================================
skl_status_t skl_launch_gemm_prompt(const skl_layer *L, const TableSrc &src, const PromptPlan &s, const uint16_t *X, skl_dtype_t x_dt,
                                    uint32_t ldx, void *Y, skl_dtype_t y_dt, uint32_t ldy, uint32_t tokens, void *ws, hipStream_t stream)
{
    const RowArgs a = make_row_args(L, src);
    PromptArgs g;
    g.h = a.h; g.bmeta = a.bmeta; g.tables = src.tables;
    g.Xq = static_cast<uint4 *>(ws);
    g.parts = reinterpret_cast<float *>(static_cast<char *>(ws) + s.pack_bytes);
    g.out = L->out; g.n_blocks = L->n_blocks;
    g.T = s.T; g.M = s.M; g.P = s.P; g.rows = s.rows; g.n_words = 8 * L->gemm_kb;
    g.per_xcd = (s.T * s.M * s.P + 7) / 8;
    const PackArgs k{X, a.chan, reinterpret_cast<const skl_pack_window *>(L->dev + L->off_windows), static_cast<uint4 *>(ws),
                     (uint32_t)x_dt, ldx, tokens, L->in, 2 * L->gemm_kb};
    const uint32_t n_rows = (tokens + 15) / 16, n_pack = n_rows * ((k.n_steps + PO_STEPS - 1) / PO_STEPS);
    skl_status_t st = SKL_OK;
    auto launch = [&](auto rb_tag, auto kernel) {
        constexpr int RB = decltype(rb_tag)::value;
        static_assert(PG_LDS(RB) <= SKL_LDS_HARD_BYTES, "two tables and two activation buffers");
        st = allow_lds(kernel, PG_LDS(RB));
        if (st != SKL_OK) return;
        hipLaunchKernelGGL((k_prompt_pack<RB>), dim3(n_pack), dim3(SKL_WG), PO_LDS_BYTES, stream, k, n_rows);
        st = check_launch("prompt packing");
        if (st == SKL_OK) hipLaunchKernelGGL(kernel, dim3(8 * g.per_xcd), dim3(64 * s.nw), PG_LDS(RB), stream, g);
    };
    DISPATCH_D(L->d, {
        // The plan's tiles are of an even number of 16-token blocks.  A lone tile that fills one less has a kernel of its own,
        // which neither copies nor multiplies the empty one: 4096 x 11008, 100 tokens 34.5 -> 33.7 us, 70 tokens 30.7 -> 29.8,
        // 40 tokens 25.7 -> 25.3; 8192 x 8192, 80 tokens 36.6 -> 35.8; 4096 x 4096, 48 tokens the same.
        switch (s.M > 1 ? s.rb : std::max(2u, s.rows)) {
        case 2: launch(std::integral_constant<int, 2>(), k_prompt_gemm<D, 2>); break;
        case 3: launch(std::integral_constant<int, 3>(), k_prompt_gemm<D, 3>); break;
        case 4: launch(std::integral_constant<int, 4>(), k_prompt_gemm<D, 4>); break;
        case 5: launch(std::integral_constant<int, 5>(), k_prompt_gemm<D, 5>); break;
        case 6: launch(std::integral_constant<int, 6>(), k_prompt_gemm<D, 6>); break;
        case 7: launch(std::integral_constant<int, 7>(), k_prompt_gemm<D, 7>); break;
        default: launch(std::integral_constant<int, 8>(), k_prompt_gemm<D, 8>);
        }
    })
    if (st == SKL_OK) st = check_launch("prompt gemm");
    if (st != SKL_OK) return st;
    hipLaunchKernelGGL(k_prompt_reduce, dim3((L->out + 63) / 64, n_rows), dim3(256), 0, stream, g.parts, s.T, s.P, s.nw, s.rows, Y, (uint32_t)y_dt,
                       ldy, tokens, L->out);
    return check_launch("prompt reduction");
}

}  // namespace SKL_NS
