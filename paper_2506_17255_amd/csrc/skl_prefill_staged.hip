// Staged prefill over row sketches (Sec. 3 inference flow: decompress the layer, compute, release -- here at
// the granularity of one call, through the workspace; W_hat of Sec. 3.1 Eq. 5, the
// product Y = X W_hat of Sec. 2.1).
//
// For long prompts, short ones, and layers whose block tables are too large for the fused kernel (wide sketches put few
// input channels behind one table: a 256-output workgroup would have to stream tables that cover all outputs, several
// times the bytes of the dense weights of its tile), every weight is rebuilt exactly once per call:
//   1. k_rebuild_operands: one workgroup per (channel block, range of output tiles) stages the block's table
//      in LDS once, runs select / gather / query / decode for all its outputs and writes the weights as
//      16-byte matrix-core operand words, already in the order the product kernel's LDS slot has;
//   2. the product of operand words that both come from memory (the workgroups of the first launch that do not rebuild
//      re-order the activations): k_staged_wide, whole tiles of 256 tokens x 128 to 352 outputs, for calls of more than
//      128 tokens where those are estimated faster (skl_make_wide_split); else k_staged_gemm, tiles of 256 tokens x 256 outputs in
//      the fused kernel's split, dealt by output-tile column, and k_staged_fixup where workgroups share tiles.  That is so for
//      layers in several slabs, for few tiles of many channels, where a whole tile would need too many chains of sums, and
//      for calls that fill the chip once with tiles of half the height.  Short prompts have a split of their own.
#include "skl_prefill_common.h"

namespace SKL_NS {


#define SG_STEP_WORDS 1024u             // 32 channels x 256 outputs (or tokens): [16-wide block 16][channel group 4][16] words of eight channels
#define SG_SLOT_WORDS (2u * SG_STEP_WORDS)
static_assert(SG_SLOT_BYTES == SG_SLOT_WORDS * 16u, "weight words of a 64-channel block of an output tile");
#define SG_EPI_BYTES 8704u              // epilogue, per wavefront: 32 rows x (64 float32 + 16 bytes)

#define SG_REBUILD_WG 512u              // threads per workgroup of the rebuild launch
struct RebuildArgs {
    HashArgs h;
    const skl_block_meta *bmeta;
    const uint4 *tables;                // padded block tables, [r][k][rs] words; low-bit states:
    const uint8_t *codes;               // codes and scales instead
    const uint4 *scales;
    uint4 *Wp;                          // [output tile of the slab][64-channel block][SG_SLOT_WORDS]
    uint32_t out, n_blocks, KB, n_words;
    uint32_t tile0, n_col, n_oseg;      // the slab: first output tile (of 256), pieces of 256 outputs, output segments
    uint32_t tb, n_tb;                  // 16-output blocks per tile of the product kernel, blocks of the slab
};

template <int D, int RS>
__device__ __forceinline__ void rebuild_body(const RebuildArgs &p, uint32_t blk, uint32_t seg, const skl_block_meta &bm, const uint4 *tab)
{
    constexpr int NB = RS == 1 ? 1 : RS - 1;
    const uint32_t lo = (uint32_t)(((uint64_t)seg * p.n_col) / p.n_oseg);
    const uint32_t hi = (uint32_t)(((uint64_t)(seg + 1) * p.n_col) / p.n_oseg);
    const uint32_t w0 = bm.chan_off >> 3;                       // first operand word of the block along the channel list
    const bool pad = blk + 1 == p.n_blocks;                     // the last block also fills the words up to the end of the last 64-channel block
    const uint32_t sub = threadIdx.x & 255;
    for (uint32_t tile = lo + (threadIdx.x >> 8); tile < hi; tile += SG_REBUILD_WG / 256) {
        // outputs past the end of the layer are rebuilt like the last one: their products are never stored
        const uint32_t o = min((p.tile0 + tile) * GM3_NT + sub, p.out - 1);
        const uint32_t ob = tile * 16 + (sub >> 4), wide = ob / p.tb, step_words = p.tb * 64;
        if (ob >= p.n_tb) continue;
        uint4 *dst = p.Wp + (size_t)wide * p.KB * 2 * step_words + (ob - wide * p.tb) * 64 + (sub & 15);
        uint32_t off[D];
        row_offsets<D>(p.h, o, bm.K, RS, off);
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            const uint32_t w = w0 + c;
            dst[(size_t)(w >> 2) * step_words + (w & 3) * 16] = keys_to_neg_half8(row_query8<D>(tab, off, c));
        }
        if (pad)
            for (uint32_t w = p.n_words; w < 8 * p.KB; ++w) dst[(size_t)(w >> 2) * step_words + (w & 3) * 16] = make_uint4(0, 0, 0, 0);
    }
}

// A block's padded table from codes and scales.  The expansion by a launch of its own, which writes all tables to the workspace
// for this kernel to read back, took 8 to 10 us of a call (4096 x 11008, 4-bit states, 100 tokens, 72.5 -> 65.4; 6784 x 11008, 8-bit,
// 237 tokens, 123 -> 112; 1024 x 2048, 8-bit, 700 tokens, 24.4 -> 22.4).
template <int D, int BITS>
__device__ __forceinline__ void expand_block(const RebuildArgs &p, const skl_block_meta &bm)
{
    const uint32_t nb = bm.nb, words = D * bm.K * nb, lg = 31 - __builtin_clz(nb);
    for (uint32_t i0 = threadIdx.x; i0 < words; i0 += 4 * SG_REBUILD_WG) {
        uint2 codes[4];
        uint4 sw[4];
        uint32_t rk[4], c[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t i = min(i0 + k * SG_REBUILD_WG, words - 1);
            codes[k] = codes_of_word<BITS>(p.codes, bm.ptable_off16 + i);
            c[k] = i & (nb - 1);
            rk[k] = i >> lg;
            uint32_t r = 0;
#pragma unroll
            for (uint32_t j = 1; j < D; ++j) r += rk[k] >= j * bm.K;
            sw[k] = p.scales[bm.scale_off16 + r * nb + c[k]];
        }
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k)
            if (i0 + k * SG_REBUILD_WG < words) smem[rk[k] * bm.rs + c[k]] = keys_of_word<BITS, SKL_QM>(codes[k], sw[k]);
    }
}

// Workgroup `idx` of n_blocks * n_oseg: channel block idx % n_blocks, output segment idx / n_blocks.
// LDS: the block's padded table.
template <int D, int BITS>
__device__ __forceinline__ void rebuild_block(const RebuildArgs &p, uint32_t idx)
{
    const uint32_t blk = idx % p.n_blocks, seg = idx / p.n_blocks;
    if (!skl_in_range(blk, p.n_blocks, SKL_DBG_BLOCK) || !skl_in_range(seg, p.n_oseg, SKL_DBG_OUTPUT)) return;
    const skl_block_meta bm = p.bmeta[blk];
    if constexpr (BITS == 16) {
        // global -> LDS without passing through registers: all of a wavefront's chunks are in flight at once
        copy_words_to_lds_async(smem, p.tables + bm.table_off16, D * bm.K * bm.rs, SG_REBUILD_WG / 64);
        wait_async_copies();
    } else {
        expand_block<D, BITS>(p, bm);
    }
    __syncthreads();
    switch (bm.rs) {
    case 9: rebuild_body<D, 9>(p, blk, seg, bm, smem); break;
    case 5: rebuild_body<D, 5>(p, blk, seg, bm, smem); break;
    case 3: rebuild_body<D, 3>(p, blk, seg, bm, smem); break;
    default: rebuild_body<D, 1>(p, blk, seg, bm, smem); break;
    }
}

// Both in one launch: a short prompt has too few activations to fill the chip and too little work for a launch of its
// own (4096 x 4096, 100 tokens, whole call: 34 -> 29 us; 1024 x 2048: 22 -> 18; 2048 tokens: 80 -> 78).  The rebuilding
// workgroups come first: they wait for tables and write the weights while the many short ones that re-order the
// activations fill the compute units around them.  512 threads, so that six wavefronts per SIMD gather from the three
// tables a compute unit has room for.  4096 x 11008, 2048 tokens, 0.5 bit, 256 threads and the activations first 39.7 us, now
// 28 (the weights alone 19; their 90 MB take a fill 13); 8192 x 28672 131 -> 106 (470 MB, a fill 69; the gathers cost
// nothing, without the stores 79); 4096 x 4096 19.7 -> 15.3.
// Channel blocks x output segments + 16-token rows x step groups workgroups, over two grid dimensions (a dimension holds
// 2^32 threads)
template <int D, int BITS>
__global__ __launch_bounds__(SG_REBUILD_WG) void k_rebuild_operands(RebuildArgs r, PackArgs k, uint32_t n_pack)
{
    const uint32_t n_rows = (k.tokens + 15) / 16, idx = blockIdx.y * gridDim.x + blockIdx.x;
    if (idx < r.n_blocks * r.n_oseg) {
        rebuild_block<D, BITS>(r, idx);
    } else if (idx < r.n_blocks * r.n_oseg + n_pack) {
        // [256-token tile][32-channel step][16-token block][channel group 4][16 tokens]
        const uint32_t i = idx - r.n_blocks * r.n_oseg, t0 = i % n_rows * 16;
        pack_group<SG_REBUILD_WG>(k, t0, i / n_rows, [&](uint32_t step) {
            return ((size_t)(t0 / GM_MT) * k.n_steps + step) * SG_STEP_WORDS + (t0 % GM_MT) / 16 * 64 + (threadIdx.x & 63);
        });
    }
}

template <class Split>
struct StagedArgs {
    const uint4 *Xp;                    // activation words: [256-token tile][32-channel step][SG_STEP_WORDS]
    const uint4 *Wp;                    // weight words: [output tile][32-channel step][SG_STEP_WORDS]
    void *Y;
    float *parts;
    uint32_t KB, tokens, out, y_dt, ldy, rows_aligned;
    uint32_t tile0;                     // first output tile of the slab (Wp and the split are slab-relative)
    Split sp;
};

// The wavefront's results (RB x 4 blocks of 16 tokens x 16 outputs) turned round in a private LDS area, 32 rows at
// a time, and stored in 16-byte pieces: every store instruction writes whole 128-byte (256 for float32) row pieces.
template <int DT, int RB, int CB = 4, int C0 = 0, int NC = 4>
__device__ __forceinline__ void staged_store_rows(const float4v (&acc)[RB][CB], uint32_t lds_wave, void *Y, uint32_t ldy, uint32_t t0,
                                                  uint32_t tokens, uint32_t o0, uint32_t out, uint32_t lane)
{
    constexpr uint32_t ES = DT == SKL_F32 ? 4 : 2, ROWB = 64 * ES + 16, CH = NC * 16 * ES / 16;      // bytes per LDS row (padded), pieces per row
    static_assert(32 * ROWB <= SG_EPI_BYTES, "32 rows have to fit the wavefront's area");
    const uint32_t n = lane & 15, q = lane >> 4;
#pragma unroll
    for (int r = 0; r < RB; r += 2) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t addr = lds_wave + (h * 16 + q * 4 + i) * ROWB + (c * 16 + n) * ES;
                    const float v = acc[r + h][C0 + c][i];
                    if (DT == SKL_F32) *(__attribute__((address_space(3))) float *)(uintptr_t)addr = v;
                    else *(__attribute__((address_space(3))) uint16_t *)(uintptr_t)addr = DT == SKL_F16 ? float_to_half_bits(v) : float_to_bf16_bits(v);
                }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (uint32_t it = 0; it < 32 * CH / 64; ++it) {
            const uint32_t idx = it * 64 + lane, row = idx / CH, c = idx % CH;
            const uint4 w = lds_word_at(lds_wave + row * ROWB + c * 16);
            const uint32_t t = t0 + r * 16 + row, o = o0 + c * (16 / ES);
            if (t < tokens && o < out) {
                char *dst = static_cast<char *>(Y) + ((size_t)t * ldy + o) * ES;
                if (o + 16 / ES <= out) {
                    *reinterpret_cast<uint4 *>(dst) = w;
                } else {                                    // ragged last piece of the layer
                    const uint32_t e[4] = {w.x, w.y, w.z, w.w};
                    for (uint32_t b = 0; b < (out - o) * ES; b += 2)
                        *reinterpret_cast<uint16_t *>(dst + b) = (uint16_t)(e[b >> 2] >> ((b & 2) * 8));
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// Y = X W on re-ordered operands, RB * 32 tokens x 256 outputs per workgroup (RB 8, or 4 in the single-round mode of
// the split).  Eight wavefronts, two per SIMD, so that one has matrix instructions to issue while the other waits;
// each owns RB * 16 tokens x 64 outputs (RB x 4 accumulator blocks).
// Bound by the chip's power: a loop of nothing but matrix instructions on random operands runs at 1.78 PFLOP/s in
// the 32x32x16 form and at 2.05 in the 16x16x32 form (half the accumulator traffic per product), hence the latter.
// Both operands go global -> LDS without passing through registers (both are stored in operand order, so that a
// copy is a contiguous KiB and an LDS read is free of bank conflicts), a stage of 32 channels at a time.  All but
// two of the stages in LDS are on their way while one is multiplied from registers and one is being read.  The
// copies are issued between the matrix instructions one by one: as a burst they queue at the address unit and hold
// the wavefronts up before the barrier.  One barrier per stage; the words of a stage are read during the stage
// before, so that no matrix instruction waits for an LDS read issued after a barrier.
// Short prompts (ShortSplit) take it with RB 2 or 4 for one token tile of 64 or 128 tokens: bound by the weight words,
// each read once, and by the partials; 4096 x 11008 at 100 tokens 22 us (56 us in the fused kernel, which multiplies a
// 256-token tile and rebuilds its weights beside it).
// On layers that take whole tiles now (2048 tokens), 8192 x 28672: 718 to 726 us at best = 1.32 to 1.34 PFLOP/s, 801 us with
// one wavefront per SIMD in the 32x32x16 form; of the difference to a loop without LDS reads and copies (525 us) the reads
// are about 80 us and the copies 120, and on all-zero data (clock not held back) the copies alone set the time: 7.6 GB
// through the L2s, 1.7 GB from behind them, in 570 us.  4096 x 11008: 186 us (200), 4096 x 4096 in half-height tiles: 63 (74).
#define SG_STAGES(rb) ((rb) == 8 ? 5u : (rb) == 4 ? 6u : 7u)
#define SG_STAGE_BYTES(rb) ((rb) * 2048u + 16384u)      // (rb * 32) tokens x 32 channels, 32 channels x 256 outputs
template <int RB, class Split>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_staged_gemm(StagedArgs<Split> p)
{
    constexpr uint32_t A_BYTES = RB * 2048, ST_BYTES = SG_STAGE_BYTES(RB), NS = SG_STAGES(RB);
    constexpr bool PARTS = RB == 8 || std::is_same<Split, ShortSplit>::value;   // (the single-round mode of the half-height tiles has no partial tiles)
    const uint32_t xcd = blockIdx.x & 7, wg = blockIdx.x >> 3;
    const Split sp = p.sp;
    if (sp.empty(xcd, wg)) return;
    uint32_t round = 0, u_next = sp.share_begin(xcd, wg);
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void *)smem;
    const uint32_t wm = wave >> 2, wn = wave & 3;               // token half and 64-output quarter of this wavefront
    const uint32_t a_lane = lds0 + wm * (RB * 1024) + lane * 16, b_lane = lds0 + A_BYTES + wn * 4096 + lane * 16;
    const uint32_t lds_wave = lds0 + wave * 1024, copy_off[2] = {wave * 1024 + lane * 16, (wave + 8) * 1024 + lane * 16};
    // 64 tokens are half a KiB per wavefront: both halves of the workgroup copy the same four KiB
    const uint32_t a_wave = RB == 2 ? lds0 + (wave & 3) * 1024 : lds_wave, a_off = RB == 2 ? (wave & 3) * 1024 + lane * 16 : copy_off[0];
    float4v acc[RB][4];
    for (;;) {
        G3Split::Seg sg;
        if (!sp.next(xcd, wg, round, u_next, sg)) break;
        uint32_t tile_m, tile_n;
        sp.tile_of(xcd, sg.k, tile_m, tile_n);
        const uint32_t n_st = __builtin_amdgcn_readfirstlane((sg.k1 - sg.k0) * 2);      // stages of the segment
        // the activation words are laid out by 256-token tiles of sixteen blocks; a half-height tile is eight of them
        // (RB 2: the short-prompt mode, whose only token tile is the first)
        const char *const xa = uniform_address(p.Xp + ((size_t)(RB == 8 ? tile_m : tile_m >> 1) * p.KB + sg.k0) * SG_SLOT_WORDS + (RB == 8 ? 0 : (tile_m & 1) * 512));
        const char *const wb = uniform_address(p.Wp + ((size_t)tile_n * p.KB + sg.k0) * SG_SLOT_WORDS);
        constexpr uint32_t NA = RB >= 4 ? RB / 4 : 1;
        constexpr int PER = NA + 2;                             // copies of a wavefront per stage: of the activations, then of the weights
        auto next_buf = [](uint32_t buf) { return buf + ST_BYTES == NS * ST_BYTES ? 0 : buf + ST_BYTES; };
        // Copy I of the wavefront's share of a stage, into the LDS buffer at offset buf.  Two source pointers step
        // through the stages, a constant lane offset per copy does the rest: with addresses formed per copy the
        // scalar instructions between the matrix instructions held up both wavefronts of a SIMD at once.
        const char *pa = xa, *pb = wb;
        auto copy_piece = [&](uint32_t buf, auto piece) {
            constexpr uint32_t I = decltype(piece)::value, J = I < NA ? I : I - NA;
            if constexpr (I == 0) lds_dma_16_offset<0>(pa, a_off, a_wave + buf);
            else lds_dma_16_offset<(I < NA ? 0 : A_BYTES) + J * 8192>(I < NA ? pa : pb, copy_off[J], lds_wave + buf);
        };
        // to the next stage of the segment (past its end: the last one again, never multiplied)
        auto next_stage = [&](uint32_t st) {
            const uint32_t step = st + 1 < n_st ? SG_STEP_WORDS * 16 : 0;
            pa += step;
            pb += step;
        };
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[r][c] = (float4v){0.f, 0.f, 0.f, 0.f};
        uint4 a[2][RB], b[2][4];
        const std::integral_constant<uint32_t, 0> c0;
        const std::integral_constant<uint32_t, 1> c1;
        const std::integral_constant<uint32_t, 2> c2;
        const std::integral_constant<uint32_t, 3> c3;
        auto read_b = [&](uint32_t buf, auto set) {             // operand words of the stage in buffer buf
            constexpr uint32_t H = decltype(set)::value;
#pragma unroll
            for (int c = 0; c < 4; ++c) b[H][c] = lds_word_at(b_lane + buf + c * 1024);
        };
        auto read_a = [&](uint32_t buf, auto set, int r) {
            constexpr uint32_t H = decltype(set)::value;
            a[H][r] = lds_word_at(a_lane + buf + r * 1024);
        };
        auto multiply_row = [&](auto set, int r) {
            constexpr uint32_t H = decltype(set)::value;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8v, a[H][r]), __builtin_bit_cast(half8v, b[H][c]), acc[r][c], 0, 0, 0);
        };
        uint32_t buf = 0;
        for (uint32_t st = 0; st < NS; ++st) {
            copy_piece(buf, c0);
            copy_piece(buf, c1);
            copy_piece(buf, c2);
            if constexpr (PER == 4) copy_piece(buf, c3);
            next_stage(st);
            buf += ST_BYTES;
        }
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * PER) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        read_b(0, c0);
#pragma unroll
        for (int r = 0; r < RB; ++r) read_a(0, c0, r);
        uint32_t from = 0;                                      // buffer of the stage in registers
        // stage st is in register set H; stage st + 1 is read into the other one, stage st + NS takes its buffer
        auto stage = [&](uint32_t st, auto set) {
            constexpr uint32_t H = decltype(set)::value;
            const std::integral_constant<uint32_t, H ^ 1> other;
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NS - 2) * PER) : "memory");    // stage st + 1 has arrived, stage st is read
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            const uint32_t nxt = next_buf(from);
            read_b(nxt, other);
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                read_a(nxt, other, r);
                __builtin_amdgcn_sched_barrier(0);
                multiply_row(set, r);
                if (r == 0) copy_piece(from, c0);
                if (r == RB / 4) copy_piece(from, c1);
                if (r == RB / 2) copy_piece(from, c2);
                if constexpr (PER == 4)
                    if (r == 3 * RB / 4) copy_piece(from, c3);
                if (r == RB - 1) next_stage(st + NS);
                __builtin_amdgcn_sched_barrier(0);
            }
            from = nxt;
        };
        for (uint32_t st = 0; st < n_st; st += 2) {             // (n_st is even: two stages per 64-channel block)
            stage(st, c0);
            stage(st + 1, c1);
        }
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __syncthreads();                                        // nothing on its way into LDS, nobody reads it: the epilogue may use it
        // the addresses of the epilogue are formed from a lane number the compiler cannot trace back, so that they are
        // not kept in registers across the loop above
        uint32_t ln = lane;
        asm volatile("" : "+v"(ln));
        const uint32_t t0 = tile_m * (RB * 32) + wm * (RB * 16), o0 = (p.tile0 + tile_n) * GM3_NT + wn * 64;
        if (sg.whole && p.rows_aligned) {
            const uint32_t lw = lds0 + wave * SG_EPI_BYTES;
            if (p.y_dt == SKL_F32) staged_store_rows<SKL_F32, RB>(acc, lw, p.Y, p.ldy, t0, p.tokens, o0, p.out, ln);
            else if (p.y_dt == SKL_F16) staged_store_rows<SKL_F16, RB>(acc, lw, p.Y, p.ldy, t0, p.tokens, o0, p.out, ln);
            else staged_store_rows<SKL_BF16, RB>(acc, lw, p.Y, p.ldy, t0, p.tokens, o0, p.out, ln);
        } else if (sg.whole) {
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t t = t0 + r * 16 + (ln >> 4) * 4 + i, o = o0 + c * 16 + (ln & 15);
                        if (t < p.tokens && o < p.out) store_out(p.Y, p.y_dt, (size_t)t * p.ldy + o, acc[r][c][i]);
                    }
        } else if constexpr (PARTS) {
            // partial tile: [token block][output block 16][lane] x 4 tokens, whole 1 KiB rows per store
            float4v *dst = reinterpret_cast<float4v *>(p.parts + sg.part_slot * (RB * 32 * GM3_NT)) + ln;
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                if (RB < 8 && t0 + r * 16 >= p.tokens) continue;        // blocks of tokens past the end: nobody reads them
#pragma unroll
                for (int c = 0; c < 4; ++c) dst[(size_t)((wm * RB + r) * 16 + wn * 4 + c) * 64] = acc[r][c];
            }
        }
        __syncthreads();                                        // the epilogue's LDS areas are free again
    }
}

// Y = X W on re-ordered operands, whole tiles of 256 tokens x 32 * CB outputs (the split is skl_make_wide_split).  A tile
// that fits the chip in whole rounds needs no partial tiles: 4096 x 11008 at 2048 tokens is 256 tiles of 352 outputs instead
// of 344 of 256, 88 of which went through 90 MB of float32 partials and a fix-up launch (product 186 us + fix-up 16 -> 151,
// with the chains below 161; 138 and 140 at best).
// As k_staged_gemm, but the eight wavefronts own 64 tokens x 16 * CB outputs each: up to 176 accumulator registers, so that
// of a stage only the activation words are held twice; weight words are read two or three columns (of 16 outputs) ahead of
// their products, into registers that the column before has left.  A stage's buffer is therefore read until its last
// column, and the copies issued during a stage go to the buffer of the stage before it.
// CHAINS: the products of an output go through several chains of float32 sums, one after the other, where shared tiles would
// have had as many.  Narrow tiles keep the sum of the earlier chains in as many registers as the accumulators; wider ones,
// which have none left, write the first chain of some columns to the workspace, a column per 64-channel block, and read it
// back at the end, where all workgroups do so at once: 4096 x 11008, 5 of 11 columns (42 MB), 177 -> 186 us for the whole call,
// 8192 x 28672, 2 of 10, 831 -> 837 (847 with all columns written at the same block).
struct WideArgs {
    const uint4 *Xp;                    // activation words: [256-token tile][32-channel step][SG_STEP_WORDS]
    const uint4 *Wp;                    // weight words: [output tile][32-channel step][2 * CB blocks of 16 outputs][64]
    void *Y;
    float *parts;                       // [workgroup][wavefront][column][64-token quarter][64 lanes] x 4: first chains
    uint32_t KB, tokens, out, y_dt, ldy, rows_aligned;
    uint32_t chains, split, body, join; // of skl_make_wide_split
    G3Split sp;
};

#define SW_STAGE_BYTES(cb) (16384u + (cb) * 2048u)
#define SW_STAGES(cb) ((cb) <= 8 ? 5u : 4u)
template <int DT, int CB, int C0>
__device__ __forceinline__ void wide_store(const float4v (&acc)[4][CB], uint32_t lds_wave, void *Y, uint32_t ldy, uint32_t t0, uint32_t tokens,
                                           uint32_t o0, uint32_t out, uint32_t lane)
{
    if constexpr (C0 < CB) {
        staged_store_rows<DT, 4, CB, C0, (CB - C0 < 4 ? CB - C0 : 4)>(acc, lds_wave, Y, ldy, t0, tokens, o0 + C0 * 16, out, lane);
        wide_store<DT, CB, C0 + 4>(acc, lds_wave, Y, ldy, t0, tokens, o0, out, lane);
    }
}

template <int CB, bool CHAINS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_staged_wide(WideArgs p)
{
    constexpr bool HELD = CHAINS && CB <= (int)SW_HELD_CB;
    constexpr uint32_t A_BYTES = 16384, ST_BYTES = SW_STAGE_BYTES(CB), NS = SW_STAGES(CB), LOOK = CB % 4 == 2 ? 2 : 3;     // (words of the next columns in registers)
    constexpr int PER = (16 + 2 * CB + 7) / 8;
    static_assert(CB % 4 == 0 || CB % 4 == (int)LOOK, "the words read ahead of the next stage land in free registers");
    const uint32_t xcd = blockIdx.x & 7, wg = blockIdx.x >> 3;
    const G3Split sp = p.sp;
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void *)smem;
    const uint32_t wm = wave >> 1, wn = wave & 1;
    const uint32_t a_lane = lds0 + wm * 4096 + lane * 16, b_lane = lds0 + A_BYTES + wn * (CB * 1024) + lane * 16;
    const uint32_t lds_wave = lds0 + wave * 1024, a_off = wave * 1024 + lane * 16;
    // the last copy of a stage repeats its last KiB where the pieces do not divide out
    const uint32_t last_b = min(wave + 8 * (PER - 3), 2u * CB - 1) * 1024;
    float4v acc[4][CB], sum[HELD ? 4 : 1][HELD ? CB : 1];
    float4v *const part = CHAINS && !HELD ? reinterpret_cast<float4v *>(p.parts) + (size_t)(blockIdx.x * 8 + wave) * p.split * 256 : nullptr;
    for (uint32_t k = wg; k < sp.tiles_of(xcd); k += 32) {
        uint32_t tile_m, tile_n;
        sp.tile_of(xcd, k, tile_m, tile_n);
        const uint32_t n_st = __builtin_amdgcn_readfirstlane(p.KB * 2);
        const char *pa = uniform_address(p.Xp + (size_t)tile_m * p.KB * SG_SLOT_WORDS);
        const char *pb = uniform_address(p.Wp + (size_t)tile_n * p.KB * 2 * (CB * 128));
        auto next_buf = [](uint32_t buf) { return buf + ST_BYTES == NS * ST_BYTES ? 0 : buf + ST_BYTES; };
        auto copy_piece = [&](uint32_t buf, auto piece) {
            constexpr int I = decltype(piece)::value;
            if constexpr (I < 2) lds_dma_16_offset<I * 8192>(pa + I * 8192, a_off, lds_wave + buf);
            else if constexpr (I + 1 < PER) lds_dma_16_offset<A_BYTES + (I - 2) * 8192>(pb + (I - 2) * 8192, a_off, lds_wave + buf);
            else lds_dma_16_offset<A_BYTES>(pb + last_b, lane * 16, lds0 + last_b + buf);
        };
        auto next_stage = [&](uint32_t st) {
            const bool more = st + 1 < n_st;
            pa += more ? SG_STEP_WORDS * 16 : 0;
            pb += more ? CB * 2048 : 0;
        };
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < CB; ++c) acc[r][c] = (float4v){0.f, 0.f, 0.f, 0.f};
        uint4 a[2][4], b[4];
        const std::integral_constant<int, 0> c0;
        const std::integral_constant<int, 1> c1;
        const std::integral_constant<int, 2> c2;
        const std::integral_constant<int, 3> c3;
        const std::integral_constant<int, 4> c4;
        uint32_t buf = 0;
        for (uint32_t st = 0; st + 1 < NS; ++st) {
            copy_piece(buf, c0);
            copy_piece(buf, c1);
            copy_piece(buf, c2);
            if constexpr (PER > 3) copy_piece(buf, c3);
            if constexpr (PER > 4) copy_piece(buf, c4);
            next_stage(st);
            buf += ST_BYTES;
        }
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * PER) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int r = 0; r < 4; ++r) a[0][r] = lds_word_at(a_lane + r * 1024);
#pragma unroll
        for (uint32_t c = 0; c < LOOK; ++c) b[c] = lds_word_at(b_lane + c * 1024);
        uint32_t from = 0, into = (NS - 1) * ST_BYTES;          // buffer of the stage being multiplied; of the stage before it
        auto stage = [&](uint32_t st, auto set) {
            constexpr int H = decltype(set)::value;
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 3) * PER) : "memory");     // stage st + 1 has arrived
            __builtin_amdgcn_s_barrier();                       // nobody reads the stage before any more
            asm volatile("" ::: "memory");
            const uint32_t nxt = next_buf(from);
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                if (c + (int)LOOK < CB && LOOK == 3) b[(c + 3) & 3] = lds_word_at(b_lane + from + (c + 3) * 1024);
                if (c + (int)LOOK < CB && LOOK == 2) b[(c + 2) & 3] = lds_word_at(b_lane + from + (c + 2) * 1024);
                if (c < 4) a[H ^ 1][c] = lds_word_at(a_lane + nxt + c * 1024);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8v, a[H][r]), __builtin_bit_cast(half8v, b[c & 3]), acc[r][c], 0, 0, 0);
                if (c == 0) copy_piece(into, c0);
                if (c == 1) copy_piece(into, c1);
                if (c == 2) copy_piece(into, c2);
                if constexpr (PER > 3) { if (c == 3) copy_piece(into, c3); }
                if constexpr (PER > 4) { if (c == 4) copy_piece(into, c4); }
                if (c == (CB > 5 ? 5 : CB - 1)) next_stage(st + NS - 1);
                __builtin_amdgcn_sched_barrier(0);
                if (c + (int)LOOK >= CB) b[c + LOOK - CB] = lds_word_at(b_lane + nxt + (c + LOOK - CB) * 1024);
            }
            into = from;
            from = nxt;
        };
        if constexpr (!CHAINS) {
            for (uint32_t st = 0; st < n_st; st += 2) {         // (n_st is even: two stages per 64-channel block)
                stage(st, c0);
                stage(st + 1, c1);
            }
        } else {
            uint32_t st = 0;
            const uint32_t n = HELD ? p.chains + (p.body < p.KB) : p.split + 1;
            for (uint32_t i = 1; i <= n; ++i) {
                uint32_t end = n_st;
                if (HELD ? i <= p.chains : i < n) end = 2 * (HELD ? i * p.body / p.chains : skl_first_chain_end(p.KB, p.split, i - 1, wg));
                for (; st < end; st += 2) {
                    stage(st, c0);
                    stage(st + 1, c1);
                }
                if constexpr (HELD) {
                    if (p.join && i > p.chains) break;          // the sum has gone through the last blocks
                    const bool go_on = i == n || (p.join && i == p.chains);
                    const float4v zero = {0.f, 0.f, 0.f, 0.f};
                    auto each = [&](auto what) {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
#pragma unroll
                            for (int c = 0; c < CB; ++c) what(sum[r][c], acc[r][c]);
                    };
                    // (branches that the empty statements keep: selects one way or the other are 128 instructions more, 0.4 us; 192
                    // outputs have no registers for both ways of the accumulators)
                    if constexpr (CB > 4) {
                        each([&](float4v &s, float4v &a) { s = i == 1 ? a : s + a; a = go_on ? s : zero; });
                    } else if (go_on) {
                        asm volatile("");
                        each([&](float4v &s, float4v &a) { a = s + a; });
                    } else if (i == 1) {
                        asm volatile("");
                        each([&](float4v &s, float4v &a) { s = a; a = zero; });
                    } else {
                        asm volatile("");
                        each([&](float4v &s, float4v &a) { s += a; a = zero; });
                    }
                } else if (i < n) {                             // (the stores only make the next waits for copies longer)
                    uint32_t ln = lane;
                    asm volatile("" : "+v"(ln));
#pragma unroll
                    for (int c = 0; c < CB; ++c)
                        if ((uint32_t)c + 1 == i) {
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                part[(c * 4 + r) * 64 + ln] = acc[r][c];
                                acc[r][c] = (float4v){0.f, 0.f, 0.f, 0.f};
                            }
                        }
                }
            }
        }
        // the first chains, two columns at a time into the registers that the operand words have left: the first two are on
        // their way while the workgroup meets (not at 352 outputs, where they would spill)
        float4v first[CHAINS && !HELD ? 2 : 1][4];
        uint32_t ln = lane;
        asm volatile("" : "+v"(ln));
        auto request = [&](int c0) {
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) first[c][r] = part[(min(c0 + c, (int)p.split - 1) * 4 + r) * 64 + ln];
        };
        if constexpr (CHAINS && !HELD && CB < 11) request(0);
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __syncthreads();                                        // nothing on its way into LDS, nobody reads it: the epilogue may use it
        if constexpr (CHAINS && !HELD) {
#pragma unroll
            for (int c0 = 0; c0 < CB; c0 += 2)
                if ((uint32_t)c0 < p.split) {
                    if (c0 || CB == 11) request(c0);
#pragma unroll
                    for (int c = 0; c < 2 && c0 + c < CB; ++c)
                        if ((uint32_t)(c0 + c) < p.split) {
#pragma unroll
                            for (int r = 0; r < 4; ++r) acc[r][c0 + c] += first[c][r];
                        }
                }
        }
        const uint32_t t0 = tile_m * GM_MT + wm * 64, o0 = tile_n * (CB * 32) + wn * (CB * 16);
        if (p.rows_aligned) {
            const uint32_t lw = lds0 + wave * SG_EPI_BYTES;
            if (p.y_dt == SKL_F32) wide_store<SKL_F32, CB, 0>(acc, lw, p.Y, p.ldy, t0, p.tokens, o0, p.out, ln);
            else if (p.y_dt == SKL_F16) wide_store<SKL_F16, CB, 0>(acc, lw, p.Y, p.ldy, t0, p.tokens, o0, p.out, ln);
            else wide_store<SKL_BF16, CB, 0>(acc, lw, p.Y, p.ldy, t0, p.tokens, o0, p.out, ln);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < CB; ++c)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t t = t0 + r * 16 + (ln >> 4) * 4 + i, o = o0 + c * 16 + (ln & 15);
                        if (t < p.tokens && o < p.out) store_out(p.Y, p.y_dt, (size_t)t * p.ldy + o, acc[r][c][i]);
                    }
        }
        __syncthreads();                                        // the epilogue's LDS areas are free again
    }
}

// Adds n_parts partials of 16 tokens x 256 outputs (the first at src, part_floats apart) in order, four of them on their way
// at a time, turns them round in LDS and stores rows in pieces of four outputs.  (One partial at a time and single elements,
// whole calls: 1024 x 11008, 8-bit states, 128 tokens, 26.4 us, now 25.7; 1408 x 10048, 4-bit, 33 tokens, 27.4, 26.8; 4096 x
// 2048, 600 tokens, 53.1, 52.4; most others the same.)
__device__ __forceinline__ void fixup_rows(const float *first, uint32_t part_floats, uint32_t n_parts, void *Y, uint32_t y_dt, uint32_t ldy,
                                           uint32_t t0, uint32_t tokens, uint32_t o0, uint32_t out)
{
    __shared__ __align__(16) float rows[16][GM3_NT + 4];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float4v *src = reinterpret_cast<const float4v *>(first) + (wave * 4) * 64 + lane;
    float4v v[4];
    for (uint32_t part = 0; part < n_parts; part += 4) {        // the slots of a tile are neighbours
        float4v w[4][4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k)
#pragma unroll
            for (int c = 0; c < 4; ++c) w[k][c] = src[(size_t)min(part + k, n_parts - 1) * (part_floats / 4) + c * 64];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (part + k == 0) v[c] = w[k][c];
                else if (part + k < n_parts) v[c] += w[k][c];
            }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) rows[(lane >> 4) * 4 + i][(wave * 4 + c) * 16 + (lane & 15)] = v[c][i];
    __syncthreads();
    const uint32_t n = (threadIdx.x & 63) * 4, o = o0 + n;
    if (o >= out) return;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
        const uint32_t row = k * 4 + (threadIdx.x >> 6);
        if (t0 + row < tokens) store_four(Y, y_dt, ldy, t0 + row, o, out, *reinterpret_cast<const float4 *>(&rows[row][n]));
    }
}

// the leftover tiles of a call; grid (8 * l_max, 16)
__global__ __launch_bounds__(256) void k_staged_fixup(G3Split sp, const float *__restrict__ parts, void *Y, uint32_t y_dt, uint32_t ldy,
                                                      uint32_t tokens, uint32_t out, uint32_t tile0)
{
    const uint32_t xcd = blockIdx.x / sp.l_max, l = blockIdx.x % sp.l_max, rb = blockIdx.y;
    if (l >= sp.left(xcd)) return;
    uint32_t tile_m, tile_n;
    sp.tile_of(xcd, sp.rounds(xcd) * sp.gx + l, tile_m, tile_n);
    const uint32_t t0 = tile_m * GM_MT + rb * 16;
    if (t0 >= tokens) return;
    fixup_rows(parts + sp.slot(xcd, l, 0) * G3_SLOT_FLOATS + rb * 16 * GM3_NT, G3_SLOT_FLOATS, sp.parts(xcd, l), Y, y_dt, ldy, t0, tokens,
               (tile0 + tile_n) * GM3_NT, out);            // tile0: first output tile of the slab the split covers
}

// the shared tiles of a short prompt; grid (tiles, ceil(tokens / 16))
__global__ __launch_bounds__(256) void k_short_fixup(ShortSplit sp, uint32_t part_floats, const float *__restrict__ parts, void *Y, uint32_t y_dt,
                                                     uint32_t ldy, uint32_t tokens, uint32_t out, uint32_t tile0)
{
    const uint32_t tile = blockIdx.x, rb = blockIdx.y;
    fixup_rows(parts + (size_t)tile * sp.P * part_floats + rb * 16 * GM3_NT, part_floats, sp.P, Y, y_dt, ldy, rb * 16, tokens,
               (tile0 + tile) * GM3_NT, out);
}

// ========================================================================
// Launcher
// ========================================================================
static uint32_t staged_slab_cols(const skl_layer *L, uint32_t tokens) { return skl_staged_slab_cols(L->out, L->gemm_kb, tokens); }

static uint64_t staged_pack_bytes(const skl_layer *L, uint32_t tokens)
{
    const uint64_t m_tiles = (tokens + GM_MT - 1) / GM_MT;
    return m_tiles * L->gemm_kb * 2 * SG_STEP_WORDS * 16ull;
}

static uint64_t staged_part_bytes(const skl_layer *L, uint32_t tokens)
{
    return skl_staged_part_floats(L->out, L->gemm_kb, tokens) * sizeof(float);
}

uint64_t skl_gemm_staged_bytes(const skl_layer *L, uint32_t tokens)
{
    return round256(staged_pack_bytes(L, tokens)) + round256(staged_part_bytes(L, tokens)) +
           (uint64_t)staged_slab_cols(L, tokens) * L->gemm_kb * SG_SLOT_BYTES;
}

template <int RB, class Split>
static skl_status_t launch_product(const StagedArgs<Split> &g, uint32_t grid, hipStream_t stream)
{
    constexpr size_t lds = SG_STAGES(RB) * SG_STAGE_BYTES(RB);
    static_assert(lds >= 8 * SG_EPI_BYTES && lds <= SKL_LDS_HARD_BYTES, "the epilogue has to fit the stages' LDS");
    const skl_status_t st = allow_lds(k_staged_gemm<RB, Split>, lds);
    if (st != SKL_OK) return st;
    hipLaunchKernelGGL((k_staged_gemm<RB, Split>), dim3(grid), dim3(512), lds, stream, g);
    return check_launch("staged gemm");
}

template <int CB>
static skl_status_t launch_wide(const WideArgs &g, hipStream_t stream)
{
    constexpr size_t lds = SW_STAGES(CB) * SW_STAGE_BYTES(CB);
    static_assert(lds >= 8 * SG_EPI_BYTES && lds <= SKL_LDS_HARD_BYTES, "the epilogue has to fit the stages' LDS");
    auto launch = [&](auto kernel) {
        const skl_status_t st = allow_lds(kernel, lds);
        if (st != SKL_OK) return st;
        hipLaunchKernelGGL(kernel, dim3(256), dim3(512), lds, stream, g);
        return check_launch("staged gemm, whole tiles");
    };
    return g.split ? launch(k_staged_wide<CB, true>) : launch(k_staged_wide<CB, false>);
}

skl_status_t skl_launch_gemm_staged(const skl_layer *L, const TableSrc &src, const uint16_t *X, skl_dtype_t x_dt, uint32_t ldx,
                                    void *Y, skl_dtype_t y_dt, uint32_t ldy, uint32_t tokens, void *ws, hipStream_t stream)
{
    const RowArgs a = make_row_args(L, src);
    char *area = static_cast<char *>(ws);
    uint4 *Xp = reinterpret_cast<uint4 *>(area);
    area += round256(staged_pack_bytes(L, tokens));
    float *parts = reinterpret_cast<float *>(area);
    area += round256(staged_part_bytes(L, tokens));
    uint4 *Wp = reinterpret_cast<uint4 *>(area);
    const uint32_t KB = L->gemm_kb, n_col = (L->out + GM3_NT - 1) / GM3_NT, slab_cols = staged_slab_cols(L, tokens);

    const skl_pack_window *windows = reinterpret_cast<const skl_pack_window *>(L->dev + L->off_windows);
    const PackArgs k{X, a.chan, windows, Xp, (uint32_t)x_dt, ldx, tokens, L->in, 2 * KB};
    skl_status_t st = SKL_OK;
    const WideSplit wide = tokens > SKL_SHORT_TOKENS ? skl_staged_product(L->out, KB, tokens, L->gemm_tail) : WideSplit{};     // (slabs: cb 0)
    const uint32_t wide_cb = wide.cb;
    // no partial tiles: their room holds the first chains and weight words
    if (wide_cb) Wp = reinterpret_cast<uint4 *>(static_cast<char *>(ws) + round256(staged_pack_bytes(L, tokens)) + skl_wide_part_bytes(wide));
    for (uint32_t tile0 = 0; tile0 < n_col; tile0 += slab_cols) {
        const uint32_t cols = wide_cb ? (wide.sp.n_col * wide_cb + 7) / 8 : std::min(slab_cols, n_col - tile0);
        RebuildArgs r;
        r.h = a.h; r.bmeta = a.bmeta; r.tables = src.tables; r.Wp = Wp;
        r.codes = L->dev + L->off_codes; r.scales = reinterpret_cast<const uint4 *>(L->dev + L->off_scales);
        r.out = L->out; r.n_blocks = L->n_blocks; r.KB = KB; r.n_words = L->n_packed / 8;
        r.tile0 = tile0; r.n_col = cols;
        r.tb = wide_cb ? 2 * wide_cb : 16; r.n_tb = wide_cb ? wide.sp.n_col * 2 * wide_cb : 16 * cols;
        r.n_oseg = skl_rebuild_segments(L->n_blocks, L->n_packed / 8, L->table_bytes, cols);
        const size_t lds = std::max<size_t>(L->max_table_bytes, PO_LDS_BYTES);
        const uint32_t n_pack = tile0 ? 0 : (tokens + 15) / 16 * ((2 * KB + PO_STEPS - 1) / PO_STEPS);     // (with the first slab)
        const uint32_t n_wg = n_pack + L->n_blocks * r.n_oseg, row = std::min(n_wg, 1u << 22);
        const dim3 grid(row, (n_wg + row - 1) / row);
        auto rebuild = [&](auto kernel) {
            st = allow_lds(kernel, lds);
            if (st == SKL_OK) hipLaunchKernelGGL(kernel, grid, dim3(SG_REBUILD_WG), lds, stream, r, k, n_pack);
        };
        DISPATCH_D(L->d, { !skl_rebuilds_from_codes(L) ? rebuild(k_rebuild_operands<D, 16>) : L->qbits == 8 ? rebuild(k_rebuild_operands<D, 8>) : rebuild(k_rebuild_operands<D, 4>); })
        if (st == SKL_OK) st = check_launch("operand rebuild");
        if (st != SKL_OK) return st;

        if (wide_cb) {
            const WideArgs g{Xp, Wp, Y, parts, KB, tokens, L->out, (uint32_t)y_dt, ldy, ((size_t)ldy * (y_dt == SKL_F32 ? 4 : 2)) % 16 == 0,
                             wide.chains, wide.split, wide.body, wide.join, wide.sp};
            return wide_cb == 6 ? launch_wide<6>(g, stream) : wide_cb == 7 ? launch_wide<7>(g, stream) : wide_cb == 8 ? launch_wide<8>(g, stream)
                 : wide_cb == 10 ? launch_wide<10>(g, stream) : wide_cb == 4 ? launch_wide<4>(g, stream) : launch_wide<11>(g, stream);
        }
        auto fill = [&](auto &g) {
            g.Xp = Xp; g.Wp = Wp; g.Y = Y; g.parts = parts;
            g.KB = KB; g.tokens = tokens; g.out = L->out; g.y_dt = (uint32_t)y_dt; g.ldy = ldy;
            g.rows_aligned = ((size_t)ldy * (y_dt == SKL_F32 ? 4 : 2)) % 16 == 0;
            g.tile0 = tile0;
        };
        if (tokens <= SKL_SHORT_TOKENS) {
            StagedArgs<ShortSplit> g;
            fill(g);
            g.sp = skl_make_short_split(cols * GM3_NT, KB);
            const uint32_t mt = skl_short_mt(tokens), n_grid = (g.sp.T * g.sp.P + 7) / 8 * 8;
            st = mt == 64 ? launch_product<2>(g, n_grid, stream) : launch_product<4>(g, n_grid, stream);
            if (st != SKL_OK) return st;
            if (g.sp.P > 1) {
                hipLaunchKernelGGL(k_short_fixup, dim3(g.sp.T, (tokens + 15) / 16), dim3(256), 0, stream, g.sp, mt * GM3_NT, parts, Y,
                                   (uint32_t)y_dt, ldy, tokens, L->out, tile0);
                st = check_launch("short-prompt fix-up");
                if (st != SKL_OK) return st;
            }
            continue;
        }
        StagedArgs<G3Split> g;
        fill(g);
        g.sp = skl_make_split(cols * GM3_NT, KB, tokens, true);
        st = g.sp.mt == GM_MT ? launch_product<8>(g, 8 * g.sp.gx, stream) : launch_product<4>(g, 8 * g.sp.gx, stream);
        if (st != SKL_OK) return st;
        if (g.sp.l_max) {
            hipLaunchKernelGGL(k_staged_fixup, dim3(8 * g.sp.l_max, 16), dim3(256), 0, stream, g.sp, parts, Y, (uint32_t)y_dt, ldy, tokens,
                               L->out, tile0);
            st = check_launch("staged gemm fix-up");
            if (st != SKL_OK) return st;
        }
    }
    return SKL_OK;
}

}  // namespace SKL_NS
