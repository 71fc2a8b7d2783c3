// Shared by the prefill kernels: tile shapes, the operand rebuild used by producers and the epilogues of
// the fused kernel.
#pragma once
#include "skl_device.h"
#include "skl_split.h"

namespace SKL_NS {
// staged prefill (skl_prefill_staged.hip): workspace bytes of a call (activation words, partial tiles, weight words)
uint64_t skl_gemm_staged_bytes(const skl_layer *L, uint32_t tokens);
skl_status_t skl_launch_gemm_staged(const skl_layer *L, const TableSrc &src, const uint16_t *X, skl_dtype_t x_dt, uint32_t ldx,
                                    void *Y, skl_dtype_t y_dt, uint32_t ldy, uint32_t tokens, void *ws, hipStream_t stream);
// short prompts in one pass (skl_prefill_short.hip)
skl_status_t skl_launch_gemm_prompt(const skl_layer *L, const TableSrc &src, const PromptPlan &s, const uint16_t *X, skl_dtype_t x_dt,
                                    uint32_t ldx, void *Y, skl_dtype_t y_dt, uint32_t ldy, uint32_t tokens, void *ws, hipStream_t stream);
}  // namespace SKL_NS

typedef float float4v __attribute__((ext_vector_type(4)));

// Whether the rebuild launch of staged calls expands low-bit states itself.  A workgroup takes longer to expand a table than to copy
// it, and with a handful of channel blocks a table beyond the LDS buffers is the tail of the launch: 47 x 6454, d = 4, four bits
// per weight as 8-bit codes (tables of 25 KB, one of 100), 24 tokens, 12.5 us with a launch of its own before, 13.6 without, 37 x
// 26524, d = 6 (103 KB), 14.9 / 15.9; but 54 x 11872 (46 KB) 10.4 / 9.95, 301 x 6206 (38 blocks, one of 100 KB), 786 tokens, 26.0 / 25.0.
inline bool skl_rebuilds_from_codes(const skl_layer *L)
{
    return L->qbits == 4 || (L->qbits == 8 && (L->n_blocks > 8 || L->max_table_bytes <= SKL_LDS_SOFT_TABLE_BYTES));
}

typedef uint32_t u32x4h __attribute__((ext_vector_type(4), aligned(2)));     // eight 16-bit elements on any 2-byte boundary

// four neighbouring results of token t, from output o (a multiple of four) on
__device__ __forceinline__ void store_four(void *Y, uint32_t y_dt, uint32_t ldy, uint32_t t, uint32_t o, uint32_t out, float4 v)
{
    const size_t at = (size_t)t * ldy + o;
    if ((ldy & 3u) == 0 && o + 4 <= out) {                      // (Y starts on a 16-byte boundary)
        if (y_dt == SKL_F32) {
            *reinterpret_cast<float4 *>(static_cast<float *>(Y) + at) = v;
        } else {
            uint16_t e[4];
            const float f[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) e[i] = y_dt == SKL_F16 ? float_to_half_bits(f[i]) : float_to_bf16_bits(f[i]);
            *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(Y) + at) = make_uint2(e[0] | (uint32_t)e[1] << 16, e[2] | (uint32_t)e[3] << 16);
        }
        return;
    }
    store_out(Y, y_dt, at, v.x);
    if (o + 1 < out) store_out(Y, y_dt, at + 1, v.y);
    if (o + 2 < out) store_out(Y, y_dt, at + 2, v.z);
    if (o + 3 < out) store_out(Y, y_dt, at + 3, v.w);
}

// two activations -> two binary16 values with inverted sign bits
__device__ __forceinline__ uint32_t neg_half_pair(uint32_t e, uint32_t x_dt)
{
    if (x_dt == SKL_BF16) {
        const uint32_t lo = float_to_half_bits(__builtin_bit_cast(float, e << 16));
        const uint32_t hi = float_to_half_bits(__builtin_bit_cast(float, e & 0xFFFF0000u));
        e = lo | (hi << 16);
    }
    return e ^ 0x80008000u;
}

// Activations to negated binary16, re-ordered into matrix-core A words, a word being eight entries of the channel list
// for one token: lane l of a wavefront builds the word of token l % 16 and channel group l / 16 of a 32-channel step,
// and place(step) says where in the caller's layout it goes.  A workgroup takes 16 tokens x PO_STEPS steps: it copies the window of X that holds
// the steps' channels into LDS in its own order (coalesced 16-byte pieces) and builds the words from
// 2-byte LDS reads, so that the channels which the width order moved away cost nothing (fetching every word that
// spans such a gap channel by channel from memory took 5 of 15 us on layers with one percent of wide channels).
// Steps whose channels are far apart (the wide channels themselves) have no window and are fetched from memory.
// 2048 tokens x 4096 channels of such a layer, 16.8 MB in and out: 10 us, 15 before (5.1 TB/s would be 6.6).
// All loads of a stretch are on their way before the first is needed, rows on any 2-byte boundary take 16-byte pieces, and a piece
// that would reach past the end of a row is fetched by element:
// with a wait after every piece, and by element where rows do not start on 16-byte boundaries, whole calls took 26.8 us
// (3001 x 7003, 77 tokens; now 22.2), 36.7 (5001 x 3000, 200 tokens; 32.0), 23.4 (4096 x 11008, 17 tokens; 22.8).
#define PO_STRIDE (PO_WINDOW + 8u)      // halfs per LDS row: 16-byte aligned rows on different banks
#define PO_LDS_BYTES (16u * PO_STRIDE * 2u)
struct PackArgs {
    const uint16_t *X;
    const uint32_t *chan;
    const skl_pack_window *windows;
    uint4 *Xp;
    uint32_t x_dt, ldx, tokens, in, n_steps;
};
// tokens t0 .. t0 + 15, group g of PO_STEPS steps; LDS: PO_LDS_BYTES at smem
template <uint32_t NT, class Place>
__device__ __forceinline__ void pack_group(const PackArgs &p, uint32_t t0, uint32_t g, Place place)
{
    uint16_t *rows = reinterpret_cast<uint16_t *>(smem);
    const uint16_t *__restrict__ X = p.X;
    const uint32_t *__restrict__ chan = p.chan;
    const skl_pack_window *__restrict__ windows = p.windows;
    uint4 *__restrict__ Xp = p.Xp;
    const uint32_t x_dt = p.x_dt, ldx = p.ldx, tokens = p.tokens, in = p.in, n_steps = p.n_steps;
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t row = lane & 15, kg = lane >> 4;
    const skl_pack_window win = windows[g];
    constexpr uint32_t WAVES = NT / 64, N = PO_STEPS / WAVES, PER_ROW = NT / 16;            // steps per wavefront
    u32x4v ch[N][2];                                            // this lane's channels (the list is padded to whole groups of steps)
#pragma unroll
    for (uint32_t i = 0; i < N; ++i) {
        const u32x4v *c = reinterpret_cast<const u32x4v *>(chan + (g * PO_STEPS + wave + WAVES * i) * 32 + kg * 8);
        ch[i][0] = c[0];
        ch[i][1] = c[1];
    }
    if (win.n) {
        // (every piece is requested before the first is stored; pieces that reach past the row's end are fetched again, by
        // element: what lies past it is never read from LDS)
        const uint32_t r = threadIdx.x / PER_ROW;               // PER_ROW threads copy one token's row
        const uint16_t *src = X + (size_t)min(t0 + r, tokens - 1) * ldx;
        constexpr uint32_t PIECES = (PO_WINDOW + 8 * PER_ROW - 1) / (8 * PER_ROW);
        u32x4v v[PIECES];
#pragma unroll
        for (uint32_t i = 0; i < PIECES; ++i) {
            const uint32_t c = (threadIdx.x % PER_ROW + PER_ROW * i) * 8;
            if (c < win.n && in >= 8) v[i] = *reinterpret_cast<const u32x4h *>(src + min(win.base + c, in - 8));
        }
#pragma unroll
        for (uint32_t i = 0; i < PIECES; ++i) {
            const uint32_t c = (threadIdx.x % PER_ROW + PER_ROW * i) * 8;
            if (c >= win.n) continue;
            if (win.base + c + 8 > in) {
                uint32_t e[8];
#pragma unroll
                for (uint32_t k = 0; k < 8; ++k) e[k] = src[min(win.base + c + k, in - 1)];
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k) v[i][k] = e[2 * k] | e[2 * k + 1] << 16;
            }
            *reinterpret_cast<u32x4v *>(rows + r * PO_STRIDE + c) = v[i];
        }
    }
    __syncthreads();
    const uint16_t *far = X + (size_t)min(t0 + row, tokens - 1) * ldx;     // rows past the end repeat the last one: their products are never stored
    const uint16_t *near = rows + row * PO_STRIDE;
    uint32_t e[N][8];
    auto fetch = [&](const uint16_t *from, uint32_t base) {     // (all on their way before the first is needed)
#pragma unroll
        for (uint32_t i = 0; i < N; ++i)
#pragma unroll
            for (uint32_t k = 0; k < 8; ++k) {
                const uint32_t c = ch[i][k >> 2][k & 3];
                if (c != SKL_NO_CHANNEL && skl_in_range(c, in, SKL_DBG_CHANNEL)) e[i][k] = from[c - base];
            }
    };
    if (win.n) fetch(near, win.base);
    else fetch(far, 0);
#pragma unroll
    for (uint32_t i = 0; i < N; ++i) {
        const uint32_t step = g * PO_STEPS + wave + WAVES * i;
        if (step >= n_steps) continue;
        uint32_t w[4];
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) {
            const uint32_t v = ch[i][k >> 2][k & 3] != SKL_NO_CHANNEL ? e[i][k] : 0;
            w[k >> 1] = k & 1 ? w[k >> 1] | v << 16 : v;
        }
        Xp[place(step)] =
            make_uint4(neg_half_pair(w[0], x_dt), neg_half_pair(w[1], x_dt), neg_half_pair(w[2], x_dt), neg_half_pair(w[3], x_dt));
    }
}

#define GM_NT 128            // outputs per workgroup
#define GM_THREADS 512       // four compute + four copy wavefronts

// Operand slot: word (cb, row = 2*step + k-group, n) at ((cb*8 + row)*34 + n);
// 34 instead of 32 words per row keeps the producers' scattered writes (eight
// rows, two neighbouring n per 16 lanes) on distinct banks.
#define G2_ROW 34u
#define G2_CB_WORDS (8u * G2_ROW)

struct Gemm2Args {
    HashArgs h;
    const uint4 *ptables;
    const skl_block_meta *bmeta;
    const uint4 *Xp;
    const uint4 *zeros;        // at least 1 KiB of zero bytes
    void *Y;
    uint32_t n_blocks, n_steps, tokens, out, y_dt, ldy, tab_words, n_col, m_tiles;
    float *parts;              // third kernel: partial tiles
    uint32_t T, gx, l_max, p_cap;
    uint32_t rows_aligned;     // every row of Y starts on a 16-byte boundary
};

// producers: table offsets (bytes from the table start) of the rows this lane gathers
template <int D, int NB>
__device__ __forceinline__ void g2_offsets(const HashArgs &h, uint32_t o_first, uint32_t out, uint32_t K, uint32_t lane,
                                           uint32_t (&off)[4][D])
{
    constexpr uint32_t OPI = 64 / NB;                       // outputs per gather instruction
    constexpr int SETS = NB >= 2 ? NB / 2 : 1;              // instructions for the 32 outputs of a column block
    const uint32_t sub = lane / NB, cw = lane % NB;
    const uint32_t Kq = K << 8;
    asm volatile("" : "+v"(o_first));                       // keep the hashes out of the loop-invariant registers
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
        const uint32_t o = min(o_first + min(OPI * s + sub, 31u), out - 1);
#pragma unroll
        for (int r = 0; r < D; ++r) {
            const uint32_t t = __umul24(h.A[r], o) + h.C[r];
            off[s][r] = ((r * K + select_index(t, Kq)) * NB + cw) * 16;
        }
    }
}

// producers: rebuild the operand words of one block for column block cb
template <int D, int NB>
__device__ __forceinline__ void g2_build(const uint32_t (&off)[4][D], uint32_t tab_addr, uint32_t slot_addr, uint32_t cb,
                                         uint32_t lane)
{
    constexpr uint32_t OPI = 64 / NB;
    constexpr int SETS = NB >= 2 ? NB / 2 : 1;
    const uint32_t sub = lane / NB, cw = lane % NB;
    uint4 q[2][D];
#pragma unroll
    for (int r = 0; r < D; ++r) q[0][r] = lds_word_at(tab_addr + off[0][r]);
#pragma unroll
    for (int s = 0; s < SETS; ++s) {
        if (s + 1 < SETS) {
#pragma unroll
            for (int r = 0; r < D; ++r) q[(s + 1) & 1][r] = lds_word_at(tab_addr + off[s + 1][r]);
            __builtin_amdgcn_sched_barrier(0);
        }
        uint4 m = q[s & 1][0];
#pragma unroll
        for (int r = 1; r < D; ++r) m = pk_max_u16x8(m, q[s & 1][r]);
        u32x4v w;
        w.x = keys_to_neg_half2_mad(m.x); w.y = keys_to_neg_half2_mad(m.y);
        w.z = keys_to_neg_half2_mad(m.z); w.w = keys_to_neg_half2_mad(m.w);
        const uint32_t n = OPI * s + sub;
        if (NB > 1 || n < 32)
            *(__attribute__((address_space(3))) u32x4v *)(uintptr_t)(slot_addr + ((cb * 8 + cw) * G2_ROW + n) * 16) = w;
        __builtin_amdgcn_sched_barrier(0);
    }
}


// ---- 256 x 256 output tiles of the fused prefill kernel ----
#define G3_CB_WORDS (8u * G2_ROW)
#define G3_SLOT_BYTES (8u * G3_CB_WORDS * 16u)

// One accumulator element, read where it is used.  Left to itself the compiler copies all 256
// elements out of the accumulation registers after the block loop and parks half of them in scratch memory.
__device__ __forceinline__ float acc_elem(float v)
{
    float r;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(r) : "a"(v));
    return r;
}

template <int DT>
__device__ __forceinline__ void gemm3_store(const float16v (&acc)[16], void *Y, uint32_t ldy, uint32_t t0, uint32_t tokens,
                                            uint32_t o0, uint32_t out, uint32_t q)
{
#pragma unroll
    for (int cb = 0; cb < 8; ++cb) {
        const uint32_t o = o0 + cb * 32;
        if (o >= out) continue;
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const uint32_t t = t0 + rb * 32 + (i >> 2) * 8 + q * 4 + (i & 3);
                if (t < tokens) {
                    const size_t idx = (size_t)t * ldy + o;
                    const float v = acc_elem(acc[rb * 8 + cb][i]);
                    if (DT == SKL_F32) static_cast<float *>(Y)[idx] = v;
                    else if (DT == SKL_F16) static_cast<uint16_t *>(Y)[idx] = float_to_half_bits(v);
                    else static_cast<uint16_t *>(Y)[idx] = float_to_bf16_bits(v);
                }
            }
        }
    }
}

// Row-major epilogue of the third kernel: a wavefront turns its 64 x 256 results round in a private LDS
// area, one group of rows at a time, and stores 16-byte pieces, so that every store instruction writes
// whole 512-byte (1 KiB for float32) rows of Y instead of 2-byte elements.  Needs 16-byte aligned rows.
#define G3_EPI_BYTES 16896u             // per wavefront: 32 rows x (512 + 16) bytes, or 16 rows x (1024 + 16)
static_assert(4 * G3_EPI_BYTES <= 2 * G3_SLOT_BYTES + 1024, "the epilogue areas must end below the block metadata");
template <int DT>
__device__ __forceinline__ void gemm3_store_rows(const float16v (&acc)[16], uint32_t lds_wave, void *Y, uint32_t ldy,
                                                 uint32_t t0, uint32_t tokens, uint32_t o_tile, uint32_t out, uint32_t lane)
{
    constexpr uint32_t ES = DT == SKL_F32 ? 4 : 2;
    constexpr uint32_t ROWB = 256 * ES + 16;                    // padded: the two token groups of a store land on other banks
    constexpr int GROUPS = DT == SKL_F32 ? 2 : 1;               // row groups per 32-row block
    constexpr uint32_t ROWS = 32 / GROUPS, CH = 256 * ES / 16;  // rows per group, 16-byte pieces per row
    const uint32_t n = lane & 31, q = lane >> 5;
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int gr = 0; gr < GROUPS; ++gr) {
#pragma unroll
            for (int cb = 0; cb < 8; ++cb)
#pragma unroll
                for (int ii = 0; ii < 16 / GROUPS; ++ii) {
                    const int i = gr * (16 / GROUPS) + ii;
                    const uint32_t row = (ii >> 2) * 8 + q * 4 + (ii & 3);
                    const uint32_t addr = lds_wave + row * ROWB + (cb * 32 + n) * ES;
                    const float v = acc_elem(acc[rb * 8 + cb][i]);
                    if (DT == SKL_F32) *(__attribute__((address_space(3))) float *)(uintptr_t)addr = v;
                    else *(__attribute__((address_space(3))) uint16_t *)(uintptr_t)addr =
                        DT == SKL_F16 ? float_to_half_bits(v) : float_to_bf16_bits(v);
                }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (uint32_t it = 0; it < ROWS * CH / 64; ++it) {
                const uint32_t idx = it * 64 + lane, row = idx / CH, c = idx % CH;
                const uint4 w = lds_word_at(lds_wave + row * ROWB + c * 16);
                const uint32_t t = t0 + rb * 32 + gr * ROWS + row, o = o_tile + c * (16 / ES);
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


