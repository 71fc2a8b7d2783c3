// Per-weight path: 2-D groups, one hash evaluation (Sec. 3.1 Eq. 3) per
// weight and sketch row.
#include <cmath>

#include "skl_prefill_common.h"

namespace SKL_NS {


// ========================================================================
// Path 0: 2-D groups, one hash evaluation per weight and sketch row.
// A workgroup owns (group, chunk of the group's input rows, 256 outputs).
// ========================================================================
struct TileArgs {
    HashArgs h;
    const skl_group_meta *gmeta;
    const uint16_t *keys;
    uint32_t in, out, tj, to, n_ob, jc_rows, n_jc;
};

// every `stride`-th word from word t on, BATCH loads in flight
template <uint32_t BATCH, typename Word>
__device__ __forceinline__ void copy_words(Word *dst, const Word *src, uint32_t n, uint32_t t, uint32_t stride)
{
    uint32_t i = t;
    for (; i + (BATCH - 1) * stride < n; i += BATCH * stride) {
        Word w[BATCH];
#pragma unroll
        for (uint32_t k = 0; k < BATCH; ++k) w[k] = src[i + k * stride];
#pragma unroll
        for (uint32_t k = 0; k < BATCH; ++k) dst[i + k * stride] = w[k];
    }
    for (; i < n; i += stride) dst[i] = src[i];
}

// a group's table to LDS by `stride` threads, this one number t: in pieces of 16 or 4 bytes where it starts on such
// a boundary (the widths before it decide), key by key elsewhere and at its end
__device__ __forceinline__ void stage_keys(uint16_t *dst, const uint16_t *src, uint32_t n, uint32_t t, uint32_t stride)
{
    const uintptr_t at = reinterpret_cast<uintptr_t>(src);
    uint32_t done = 0;
    if ((at & 15u) == 0) {
        done = n & ~7u;
        for (uint32_t i = t; i < n / 8; i += stride) reinterpret_cast<uint4 *>(dst)[i] = reinterpret_cast<const uint4 *>(src)[i];
    } else if ((at & 3u) == 0) {
        done = n & ~1u;
        for (uint32_t i = t; i < n / 2; i += stride) reinterpret_cast<uint32_t *>(dst)[i] = reinterpret_cast<const uint32_t *>(src)[i];
    }
    for (uint32_t i = done + t; i < n; i += stride) dst[i] = src[i];
}

// The same by a workgroup, tables of more than two 16-byte pieces per thread with several loads in flight (bound by
// their latency) and key by key where they lie off 4-byte boundaries (a plain loop, which the compiler unrolls).  1024 x
// 8192 in groups of 64 x 8192 (tables of 32 KiB), d = 4: batch 16 46.9 us with all keys one by one, 48.5 with pieces one at a
// time, 41.5 so; 100 tokens 89.3, 103.2, 78.4.  Smaller tables gain nothing and would pay for the longer code (1 %),
// the smallest even for the choice of a piece (2048 x 512 in groups of 32 x 32, 100 tokens: 134 us, 141).
__device__ __forceinline__ void stage_table(uint16_t *dst, const uint16_t *src, uint32_t n)
{
    const uint32_t t = threadIdx.x;
    if (n <= SKL_WG) {
        if (t < n) dst[t] = src[t];
        return;
    }
    if (n <= 16 * SKL_WG) return stage_keys(dst, src, n, t, SKL_WG);
    const uintptr_t at = reinterpret_cast<uintptr_t>(src);
    if ((at & 15u) == 0) {
        copy_words<4>(reinterpret_cast<uint4 *>(dst), reinterpret_cast<const uint4 *>(src), n / 8, t, SKL_WG);
        if (t < (n & 7u)) dst[(n & ~7u) + t] = src[(n & ~7u) + t];
    } else if ((at & 3u) == 0) {
        copy_words<8>(reinterpret_cast<uint32_t *>(dst), reinterpret_cast<const uint32_t *>(src), n / 2, t, SKL_WG);
        if (t < (n & 1u)) dst[n - 1] = src[n - 1];
    } else {
        for (uint32_t i = t; i < n; i += SKL_WG) dst[i] = src[i];
    }
}

struct TileUnit {
    uint32_t g, jb, ob, jc, j_lo, j_hi, K, key_off;
};

__device__ __forceinline__ TileUnit tile_unit(const TileArgs &p, uint32_t unit)
{
    TileUnit u;
    u.g = unit / p.n_jc;
    u.jc = unit - u.g * p.n_jc;
    u.jb = u.g / p.n_ob;
    u.ob = u.g - u.jb * p.n_ob;
    u.j_lo = u.jc * p.jc_rows;
    u.j_hi = min(u.j_lo + p.jc_rows, p.tj);
    const skl_group_meta gm = p.gmeta[u.g];
    u.K = gm.K;
    u.key_off = gm.key_off;
    return u;
}

// running hash state of one lane: t_r for the current address, advanced by one
// input row (tile_out addresses) per step
template <int D>
struct TileHash {
    uint32_t t[D], step[D];
    __device__ __forceinline__ void init(const HashArgs &h, uint32_t a0, uint32_t to)
    {
#pragma unroll
        for (int r = 0; r < D; ++r) {
            t[r] = __umul24(h.A[r], a0) + h.C[r];
            step[r] = __umul24(h.A[r], to);
        }
    }
    __device__ __forceinline__ uint16_t query(const uint16_t *tab, uint32_t K, uint32_t Kq)
    {
        uint16_t m = 0;
#pragma unroll
        for (int r = 0; r < D; ++r) {
            const uint16_t k = tab[r * K + select_index(t[r], Kq)];
            m = k > m ? k : m;
            t[r] += step[r];
        }
        return m;
    }
};


template <int D>
__global__ __launch_bounds__(SKL_WG) void k_tile_reconstruct(TileArgs p, uint16_t *__restrict__ W_hat)
{
    uint16_t *tab = reinterpret_cast<uint16_t *>(smem);
    const TileUnit u = tile_unit(p, blockIdx.x);
    stage_table(tab, p.keys + u.key_off, D * u.K);
    __syncthreads();
    const uint32_t ol = blockIdx.y * SKL_WG + threadIdx.x;
    if (ol >= p.to) return;
    TileHash<D> th;
    th.init(p.h, u.j_lo * p.to + ol, p.to);
    const uint32_t Kq = u.K << 8;
    for (uint32_t jl = u.j_lo; jl < u.j_hi; ++jl) {
        const uint16_t k = th.query(tab, u.K, Kq);
        W_hat[(size_t)(u.jb * p.tj + jl) * p.out + u.ob * p.to + ol] = key_to_half_bits(k);
    }
}

// decode GEMV for BT batch rows per pass (grid z walks the batch)
template <int D, int BT>
__global__ __launch_bounds__(SKL_WG) void k_tile_gemv(TileArgs p, const uint16_t *__restrict__ x, uint32_t ldx,
                                                      uint32_t batch, float *__restrict__ partial, uint32_t key_words)
{
    uint16_t *tab = reinterpret_cast<uint16_t *>(smem);
    float *xs = reinterpret_cast<float *>(smem + key_words);   // [BT][jc_rows]
    const TileUnit u = tile_unit(p, blockIdx.x);
    stage_table(tab, p.keys + u.key_off, D * u.K);
    const uint32_t b0 = blockIdx.z * BT;
    const uint32_t rows = u.j_hi - u.j_lo;
    for (uint32_t i = threadIdx.x; i < BT * rows; i += SKL_WG) {
        const uint32_t b = i / rows, jr = i - b * rows;
        xs[b * p.jc_rows + jr] =
            b0 + b < batch ? half_bits_to_float(x[(size_t)(b0 + b) * ldx + u.jb * p.tj + u.j_lo + jr]) : 0.f;
    }
    __syncthreads();
    const uint32_t ol = blockIdx.y * SKL_WG + threadIdx.x;
    if (ol >= p.to) return;
    TileHash<D> th;
    th.init(p.h, u.j_lo * p.to + ol, p.to);
    const uint32_t Kq = u.K << 8;
    float acc[BT];
#pragma unroll
    for (int b = 0; b < BT; ++b) acc[b] = 0.f;
    // four rows' gathers in flight: a chunk is a chain of rows, each a dependent LDS read otherwise
#pragma unroll 4
    for (uint32_t jr = 0; jr < rows; ++jr) {
        const float w = half_bits_to_float(key_to_half_bits(th.query(tab, u.K, Kq)));
#pragma unroll
        for (int b = 0; b < BT; ++b) acc[b] = fmaf(w, xs[b * p.jc_rows + jr], acc[b]);
    }
    const uint32_t unit = u.jb * p.n_jc + u.jc;   // partial-sum slot of this chunk
#pragma unroll
    for (int b = 0; b < BT; ++b)
        if (b0 + b < batch)
            partial[((size_t)unit * batch + b0 + b) * p.out + u.ob * p.to + ol] = acc[b];
}

// Decode GEMV of a small layer in one launch.  Bound by latency: the work is under a microsecond, and the partial
// sums and the second launch of a split reduction took longer.  A workgroup owns 16 outputs and every input row:
// the tables above these outputs all sit in LDS, each staged by wavefronts of its own at the same time; the 64
// threads of an output take every 64th row of a table, and their sums are added in LDS in a fixed order.  grid z
// walks the batch, BT rows per pass.
// Whole call, split -> one launch: 256 x 256, batch 1 6.4-8.1 -> 4.1-4.6 us, batch 16 8.2 -> 4.5; 1024 x 1024 in groups
// of 256, batch 1 8.9 -> 5.5, in groups of 128, batch 16 14.9 -> 8.1; 1024 x 2048 in groups of 128, batch 1 8.2 -> 6.6.
#define TS_O 16
#define TS_SLICES 64
#define TS_MAX_IN 1024
#define TS_WIDTHS (TS_MAX_IN / TS_SLICES)       // most tables above an output

template <int D, int BT>
__global__ __launch_bounds__(TS_O * TS_SLICES) void k_tile_gemv_small(TileArgs p, const uint16_t *__restrict__ x, uint32_t ldx,
                                                                       uint32_t batch, void *__restrict__ y, uint32_t y_dt,
                                                                       uint32_t ldy, uint32_t key_words)
{
    const uint32_t n_jb = p.in / p.tj;
    const uint32_t n_oc = (p.to + TS_O - 1) / TS_O;                 // 16-wide output chunks per group column
    const uint32_t ob = blockIdx.x / n_oc, oc = blockIdx.x - ob * n_oc;
    float *xs = reinterpret_cast<float *>(smem + n_jb * key_words);          // [BT][in]
    float *red = xs + (size_t)BT * p.in;                                      // [BT][TS_SLICES][TS_O]
    __shared__ uint32_t width[TS_WIDTHS];                            // (a fixed address: 0.1 us less than behind the sums)
    const uint32_t b0 = blockIdx.z * BT;
    // a wavefront or more to a table, all tables at once (one after the other, eight tables took 8.6 us a call, now 6.6)
    uint32_t tables = 1;                                             // side by side: n_jb rounded up to a power of two
    while (tables < n_jb) tables *= 2;
    const uint32_t per_table = TS_O * TS_SLICES / tables;
    const uint32_t my_jb = threadIdx.x / per_table;
    if (my_jb < n_jb) {
        const skl_group_meta gm = p.gmeta[my_jb * p.n_ob + ob];
        const uint32_t t = threadIdx.x & (per_table - 1);
        if (t == 0) width[my_jb] = gm.K;
        stage_keys(reinterpret_cast<uint16_t *>(smem + my_jb * key_words), p.keys + gm.key_off, D * gm.K, t, per_table);
    }
#pragma unroll
    for (int b = 0; b < BT; ++b)
        for (uint32_t j = threadIdx.x; j < p.in; j += TS_O * TS_SLICES)
            xs[b * p.in + j] = b0 + b < batch ? half_bits_to_float(x[(size_t)(b0 + b) * ldx + j]) : 0.f;
    __syncthreads();
    const uint32_t n = threadIdx.x & (TS_O - 1), slice = threadIdx.x / TS_O;
    const uint32_t ol = min(oc * TS_O + n, p.to - 1);               // a lane past the group repeats its last output
    float acc[BT];
#pragma unroll
    for (int b = 0; b < BT; ++b) acc[b] = 0.f;
    for (uint32_t jb = 0; jb < n_jb; ++jb) {
        const uint16_t *tab = reinterpret_cast<const uint16_t *>(smem + jb * key_words);
        const uint32_t K = __builtin_amdgcn_readfirstlane(width[jb]), Kq = K << 8;
        TileHash<D> th;
        th.init(p.h, slice * p.to + ol, TS_SLICES * p.to);
#pragma unroll 4
        for (uint32_t jl = slice; jl < p.tj; jl += TS_SLICES) {
            const float w = half_bits_to_float(key_to_half_bits(th.query(tab, K, Kq)));
#pragma unroll
            for (int b = 0; b < BT; ++b) acc[b] = fmaf(w, xs[b * p.in + jb * p.tj + jl], acc[b]);
        }
    }
#pragma unroll
    for (int b = 0; b < BT; ++b) red[(b * TS_SLICES + slice) * TS_O + n] = acc[b];
    __syncthreads();
    // 16 x 4 threads per batch row: four quarters of the slices, then across the quarters
    const uint32_t b = threadIdx.x >> 6, q = (threadIdx.x >> 4) & 3u;
    if (b >= BT) return;
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < TS_SLICES / 4; ++i) t += red[(b * TS_SLICES + q * (TS_SLICES / 4) + i) * TS_O + n];
    t += __shfl_xor(t, 16);
    t += __shfl_xor(t, 32);
    if (q == 0 && oc * TS_O + n < p.to && b0 + b < batch)
        store_out(y, y_dt, (size_t)(b0 + b) * ldy + ob * p.to + ol, t);
}

// prefill GEMM on path 0, any geometry: 64 tokens x 64 outputs per workgroup; per 16 input
// rows the weights are reconstructed once into LDS (transposed, binary16 with
// inverted sign) and fed to 32x32x16 MFMAs.
#define TG_T 64
#define TG_AS 24   // halfs per LDS row of the 16-wide operand tiles (16 + 8)

template <int D>
__global__ __launch_bounds__(SKL_WG) void k_tile_gemm(TileArgs p, const uint16_t *__restrict__ X, uint32_t x_dt,
                                                      uint32_t ldx, uint32_t tokens, void *__restrict__ Y, uint32_t y_dt,
                                                      uint32_t ldy, uint32_t key_words)
{
    uint16_t *tab = reinterpret_cast<uint16_t *>(smem);
    uint16_t *As = reinterpret_cast<uint16_t *>(smem + key_words);   // [64 tokens][TG_AS]
    uint16_t *Bs = As + TG_T * TG_AS;                                // [64 outputs][TG_AS]
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t wm = wave >> 1, wn = wave & 1;
    const uint32_t n = lane & 31, q = lane >> 5;
    const uint32_t n_oc = (p.to + TG_T - 1) / TG_T;       // 64-wide output chunks per group column
    const uint32_t ob = blockIdx.x / n_oc, oc = blockIdx.x - ob * n_oc;
    const uint32_t t0 = blockIdx.y * TG_T;
    const uint32_t ol_b = oc * TG_T + (threadIdx.x & 63);   // output (inside the group) this thread reconstructs
    const uint32_t jsub = threadIdx.x >> 6;                 // ... for input rows jsub*4 .. jsub*4+3 of each 16
    float16v acc = {0.f};
    const uint32_t n_jb = p.in / p.tj;
    for (uint32_t jb = 0; jb < n_jb; ++jb) {
        const skl_group_meta gm = p.gmeta[jb * p.n_ob + ob];
        __syncthreads();
        stage_table(tab, p.keys + gm.key_off, D * gm.K);
        __syncthreads();
        const uint32_t Kq = gm.K << 8;
        for (uint32_t j0 = 0; j0 < p.tj; j0 += 16) {
            // reconstruct 16 x 64 weights: thread -> (output ol_b, rows j0 + jsub*4 .. +3)
            {
                TileHash<D> th;
                const uint32_t olc = min(ol_b, p.to - 1);
                th.init(p.h, (j0 + jsub * 4) * p.to + olc, p.to);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t jl = j0 + jsub * 4 + i;
                    uint16_t v = 0;
                    const uint16_t k = th.query(tab, gm.K, Kq);   // addresses past the group are never used below
                    if (jl < p.tj && ol_b < p.to) v = key_to_half_bits(k) ^ 0x8000u;
                    Bs[(threadIdx.x & 63) * TG_AS + jsub * 4 + i] = v;
                }
            }
            // activations: 64 tokens x 16 input rows, thread -> (token, 4 rows)
            {
                const uint32_t tr = threadIdx.x >> 2, js = (threadIdx.x & 3) * 4;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t jl = j0 + js + i;
                    uint16_t v = 0;
                    if (t0 + tr < tokens && jl < p.tj) v = load_neg_half(X, x_dt, (size_t)(t0 + tr) * ldx + jb * p.tj + jl);
                    As[tr * TG_AS + js + i] = v;
                }
            }
            __syncthreads();
            const uint4 a = *reinterpret_cast<const uint4 *>(As + (wm * 32 + n) * TG_AS + q * 8);
            const uint4 b = *reinterpret_cast<const uint4 *>(Bs + (wn * 32 + n) * TG_AS + q * 8);
            // both operands carry an inverted sign: the product is x * w
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8v, a), __builtin_bit_cast(half8v, b), acc, 0, 0, 0);
            __syncthreads();
        }
    }
    const uint32_t ol = oc * TG_T + wn * 32 + n;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const uint32_t t = t0 + wm * 32 + (i >> 2) * 8 + q * 4 + (i & 3);
        if (t < tokens && ol < p.to) store_out(Y, y_dt, (size_t)t * ldy + ob * p.to + ol, acc[i]);
    }
}


// Prefill GEMM on path 0 where a lane's eight consecutive input rows lie in one group (group heights that are multiples of 8)
// and a 16-wide output tile does (widths that are multiples of 16).  A workgroup owns RB * 16 tokens x OB * 16 outputs; its
// wavefronts divide the input rows among themselves, 32 at a time: a lane rebuilds the eight weights of one output that
// the matrix instruction takes from it (one key per row and sketch row from the tables above the outputs, which all sit in
// LDS), and the activations come from memory in operand order as they lie.  No barrier between the first table and the last
// product; the wavefronts' sums are added in their order at the end.
// Bound by the vector units (four instructions per weight and sketch row); every weight is rebuilt once per RB * 16 tokens.
// Whole call against 64 x 64 tiles that walk all rows, 16 at a time between two barriers (k_tile_gemm, for the other
// geometries): 256 x 256, 17 tokens, 15.5 -> 4.6 us, 512 x 512, 256 tokens, 32.7 -> 6.3, 1024 x 1024, 64 tokens, 62 -> 7.9, 2048 x 512,
// 100 tokens, 120 -> 11.8, 2048 x 2048, 512 tokens, 130 -> 31.
// The wavefronts' chains of float32 sums are shorter: errors against 64 bits 0.39 to 0.69 of those before (24 drawn layers).
#define TP_RED_BYTES 65536u             // sums of all wavefronts for some of the 16 x 16 blocks of the tile

// a group's table to LDS by one wavefront, wherever it starts, four loads in flight
__device__ __forceinline__ void stage_by_wave(uint16_t *dst, const uint16_t *src, uint32_t n, uint32_t lane)
{
    const uint32_t pieces = n / 8;
    for (uint32_t i0 = lane; i0 < pieces; i0 += 256) {
        u32x4v v[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) v[k] = *reinterpret_cast<const u32x4h *>(src + 8 * min(i0 + 64 * k, pieces - 1));
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k)
            if (i0 + 64 * k < pieces) reinterpret_cast<u32x4v *>(dst)[i0 + 64 * k] = v[k];
    }
    if (lane < (n & 7u)) dst[pieces * 8 + lane] = src[pieces * 8 + lane];
}

template <int D, int RB, int OB>
__global__ __launch_bounds__(OB == 2 ? 512 : 1024) void k_tile_prompt(TileArgs p, const uint16_t *__restrict__ X, uint32_t x_dt, uint32_t ldx, uint32_t tokens,
                                                      void *__restrict__ Y, uint32_t y_dt, uint32_t ldy, uint32_t key_words, uint32_t at_once)
{
    uint32_t *const width = reinterpret_cast<uint32_t *>(smem + at_once * key_words);           // of the tables in LDS
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const uint32_t n = lane & 15, kg = lane >> 4;
    const uint32_t n_jb = p.in / p.tj, n_ot = p.to / (16 * OB);
    const uint32_t ob = __builtin_amdgcn_readfirstlane(blockIdx.x / n_ot), o0 = (blockIdx.x - ob * n_ot) * (16 * OB);
    const uint32_t t0 = blockIdx.y * (RB * 16);
    const uint16_t *row[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) row[i] = X + (size_t)min(t0 + i * 16 + n, tokens - 1) * ldx;   // (rows past the end: never stored)
    float4v acc[RB][OB];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int b = 0; b < OB; ++b) acc[i][b] = (float4v){0.f, 0.f, 0.f, 0.f};
    u32x4v next[RB];
    auto request = [&](uint32_t j) {                            // (steps past the last row fetch the last eight again)
#pragma unroll
        for (int i = 0; i < RB; ++i) next[i] = *reinterpret_cast<const u32x4h *>(row[i] + min(j, p.in - 8));
    };
    for (uint32_t jb0 = 0; jb0 < n_jb; jb0 += at_once) {        // as many tables as fit, all of them in most layers
        const uint32_t jb1 = min(jb0 + at_once, n_jb), j_hi = jb1 * p.tj;
        uint32_t j = jb0 * p.tj + wave * 32 + kg * 8, left = wave * 32 < j_hi - jb0 * p.tj ? (j_hi - jb0 * p.tj - wave * 32 + 32 * nw - 1) / (32 * nw) : 0;
        request(j);
        if (jb0) __syncthreads();                               // nobody reads the tables before these any more
        for (uint32_t jb = jb0 + wave; jb < jb1; jb += nw) {
            const skl_group_meta gm = p.gmeta[jb * p.n_ob + ob];
            if (!skl_in_range(D * gm.K, key_words * 8 + 1, SKL_DBG_LDS_COPY)) continue;
            if (lane == 0) width[jb - jb0] = gm.K;
            stage_by_wave(reinterpret_cast<uint16_t *>(smem + (jb - jb0) * key_words), p.keys + gm.key_off, D * gm.K, lane);
        }
        __syncthreads();
        for (; left; --left, j += 32 * nw) {
            const bool live = j < j_hi;
            const uint32_t jc = live ? j : jb0 * p.tj, jb = jc / p.tj, jl = jc - jb * p.tj;
            const uint32_t K = width[jb - jb0], Kq = K << 8, tab = (uint32_t)(uintptr_t)(lds_void *)smem + (jb - jb0) * key_words * 16;
            u32x4v x[RB];
#pragma unroll
            for (int i = 0; i < RB; ++i) {
#pragma unroll
                for (int k = 0; k < 4; ++k) x[i][k] = live ? neg_half_pair(next[i][k], x_dt) : 0;
            }
            request(j + 32 * nw);
#pragma unroll
            for (int b = 0; b < OB; ++b) {
                TileHash<D> th;
                th.init(p.h, jl * p.to + o0 + b * 16 + n, p.to);
                uint32_t w[4];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    uint32_t m = 0;
#pragma unroll
                    for (int r = 0; r < D; ++r) {
                        uint32_t at = r * K + select_index(th.t[r], Kq);
                        if (!skl_in_range(at, key_words * 8, SKL_DBG_LDS_READ)) at = 0;
                        m = max(m, (uint32_t)*(const __attribute__((address_space(3))) uint16_t *)(uintptr_t)(tab + at * 2));
                        th.t[r] += th.step[r];
                    }
                    w[k >> 1] = k & 1 ? w[k >> 1] | m << 16 : m;
                }
                uint4 v;
                v.x = keys_to_neg_half2_mad(w[0]); v.y = keys_to_neg_half2_mad(w[1]);
                v.z = keys_to_neg_half2_mad(w[2]); v.w = keys_to_neg_half2_mad(w[3]);
                v = keep_if(live, v);
                // both operands carry an inverted sign: the product is x * w
#pragma unroll
                for (int i = 0; i < RB; ++i)
                    acc[i][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8v, x[i]), __builtin_bit_cast(half8v, v), acc[i][b], 0, 0, 0);
            }
        }
    }
    // the blocks of the tile, as many at a time as their sums fit: every wavefront leaves its own, and one adds them in order
    const uint32_t some = min((uint32_t)(RB * OB), TP_RED_BYTES / 1024 / nw);
    float4v *const red = reinterpret_cast<float4v *>(smem);
    for (uint32_t r0 = 0; r0 < RB * OB; r0 += some) {
        __syncthreads();
#pragma unroll
        for (uint32_t i = 0; i < RB; ++i)
#pragma unroll
            for (uint32_t b = 0; b < OB; ++b)
                if (i * OB + b >= r0 && i * OB + b < r0 + some) red[(wave * some + i * OB + b - r0) * 64 + lane] = acc[i][b];
        __syncthreads();
        for (uint32_t k = wave; k < some && r0 + k < RB * OB; k += nw) {
            float4v s = red[k * 64 + lane];
            for (uint32_t v = 1; v < nw; ++v) s += red[(v * some + k) * 64 + lane];
            const uint32_t i = (r0 + k) / OB, b = (r0 + k) % OB;
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e) {
                const uint32_t t = t0 + i * 16 + kg * 4 + e;
                if (t < tokens) store_out(Y, y_dt, (size_t)t * ldy + ob * p.to + o0 + b * 16 + n, s[e]);
            }
        }
    }
}

static TileArgs make_tile_args(const skl_layer *L, const TableSrc &src)
{
    TileArgs a;
    for (int r = 0; r < SKL_MAX_D; ++r) { a.h.A[r] = L->A[r]; a.h.C[r] = L->C[r]; }
    a.gmeta = reinterpret_cast<const skl_group_meta *>(L->dev + L->off_gmeta);
    a.keys = src.keys;
    a.in = L->in; a.out = L->out; a.tj = L->tj; a.to = L->to; a.n_ob = L->n_ob;
    a.jc_rows = L->jc_rows; a.n_jc = L->n_jc;
    return a;
}

static inline size_t tile_key_words(const skl_layer *L) { return ((size_t)L->d * L->max_K * 2 + 15) / 16; }


skl_status_t skl_tile_launch_reconstruct(const skl_layer *L, const TableSrc &src, uint16_t *W_hat, hipStream_t stream)
{
    skl_status_t st = SKL_OK;
    const TileArgs a = make_tile_args(L, src);
    const size_t lds = tile_key_words(L) * 16;
    const dim3 grid(L->n_jb * L->n_ob * L->n_jc, (L->to + SKL_WG - 1) / SKL_WG);
    DISPATCH_D(L->d, {
        st = allow_lds(k_tile_reconstruct<D>, lds);
        if (st == SKL_OK) hipLaunchKernelGGL(k_tile_reconstruct<D>, grid, dim3(SKL_WG), lds, stream, a, W_hat);
    });
    return st == SKL_OK ? check_launch("reconstruct") : st;
}

// first kernel of the decode call: one partial sum per (group chunk, output); the caller adds the reduction
skl_status_t skl_tile_launch_gemv(const skl_layer *L, const TableSrc &src, const uint16_t *x, uint32_t ldx, uint32_t batch,
                                  float *partial, hipStream_t stream)
{
    skl_status_t st = SKL_OK;
    const TileArgs a = make_tile_args(L, src);
    const uint32_t kw = (uint32_t)tile_key_words(L);
    const uint32_t units = L->n_jb * L->n_ob * L->n_jc, noc = (L->to + SKL_WG - 1) / SKL_WG;
    if (batch == 1) {
        const size_t lds = (size_t)kw * 16 + (size_t)L->jc_rows * sizeof(float);
        DISPATCH_D(L->d, {
            st = allow_lds(k_tile_gemv<D, 1>, lds);
            if (st == SKL_OK)
                hipLaunchKernelGGL((k_tile_gemv<D, 1>), dim3(units, noc, 1), dim3(SKL_WG), lds, stream, a, x, ldx,
                                   batch, partial, kw);
        });
    } else {
        const size_t lds = (size_t)kw * 16 + (size_t)4 * L->jc_rows * sizeof(float);
        DISPATCH_D(L->d, {
            st = allow_lds(k_tile_gemv<D, 4>, lds);
            if (st == SKL_OK)
                hipLaunchKernelGGL((k_tile_gemv<D, 4>), dim3(units, noc, (batch + 3) / 4), dim3(SKL_WG), lds, stream,
                                   a, x, ldx, batch, partial, kw);
        });
    }
    return st;
}

// Where one launch is taken: groups of at least 64 rows (fewer leave threads idle), at most 1024 input rows (the gain,
// 3.5 us at 256 rows, is down to 1.6 there: every workgroup walks all rows), tables that leave room for two workgroups on
// a compute unit, and no more workgroups than that one round (512 of them: 512 x 2048, batch 16, 13.3 -> 7.3 us); beyond, each table
// would be staged by workgroups that wait for their turn.
static inline size_t tile_small_lds(const skl_layer *L, uint32_t bt)
{
    return (size_t)L->n_jb * tile_key_words(L) * 16 + (size_t)bt * (L->in + TS_SLICES * TS_O) * sizeof(float);
}

bool skl_tile_gemv_is_small(const skl_layer *L, uint32_t batch)
{
    const uint64_t wgs = (uint64_t)L->n_ob * ((L->to + TS_O - 1) / TS_O) * (batch == 1 ? 1 : (batch + 3) / 4);
    return L->tj >= TS_SLICES && L->in <= TS_MAX_IN && wgs <= 512 && tile_small_lds(L, batch == 1 ? 1 : 4) <= 65536;
}

skl_status_t skl_tile_launch_gemv_small(const skl_layer *L, const TableSrc &src, const uint16_t *x, uint32_t ldx, uint32_t batch,
                                        void *y, skl_dtype_t y_dt, uint32_t ldy, hipStream_t stream)
{
    skl_status_t st = SKL_OK;
    const TileArgs a = make_tile_args(L, src);
    const uint32_t kw = (uint32_t)tile_key_words(L);
    const uint32_t n_oc = (L->to + TS_O - 1) / TS_O;
    if (batch == 1) {
        const size_t lds = tile_small_lds(L, 1);
        DISPATCH_D(L->d, {
            st = allow_lds(k_tile_gemv_small<D, 1>, lds + TS_WIDTHS * sizeof(uint32_t));
            if (st == SKL_OK)
                hipLaunchKernelGGL((k_tile_gemv_small<D, 1>), dim3(L->n_ob * n_oc), dim3(TS_O * TS_SLICES), lds, stream, a, x, ldx,
                                   batch, y, (uint32_t)y_dt, ldy, kw);
        });
    } else {
        const size_t lds = tile_small_lds(L, 4);
        DISPATCH_D(L->d, {
            st = allow_lds(k_tile_gemv_small<D, 4>, lds + TS_WIDTHS * sizeof(uint32_t));
            if (st == SKL_OK)
                hipLaunchKernelGGL((k_tile_gemv_small<D, 4>), dim3(L->n_ob * n_oc, 1, (batch + 3) / 4), dim3(TS_O * TS_SLICES), lds,
                                   stream, a, x, ldx, batch, y, (uint32_t)y_dt, ldy, kw);
        });
    }
    return st == SKL_OK ? check_launch("gemv") : st;
}

// tables above an output tile that are in LDS together
static uint32_t tile_prompt_tables(const skl_layer *L) { return std::min(L->n_jb, std::max(1u, 49152u / (uint32_t)(tile_key_words(L) * 16))); }
static size_t tile_prompt_table_bytes(const skl_layer *L) { return (size_t)tile_prompt_tables(L) * (tile_key_words(L) * 16 + 4); }

bool skl_tile_prompt_fits(const skl_layer *L) { return L->tj % 8 == 0 && L->to % 16 == 0 && tile_prompt_table_bytes(L) <= SKL_LDS_HARD_BYTES; }

struct TilePromptShape {
    uint32_t RB, ob, nw;            // tiles of RB * 16 tokens x ob * 16 outputs, wavefronts to each
};

static TilePromptShape tile_prompt_shape(const skl_layer *L, uint32_t tokens)
{
    // The smallest tile that is no more than three workgroups for two CUs: a larger one re-uses weights and activations
    // more, a smaller one fills the chip and is over sooner.  Whole calls by tokens x outputs per tile, in us: 512 x 512,
    // 256 tokens 32 x 16 (256 workgroups) 6.7, 64 x 16 7.7, 128 x 16 10.9; 2048 x 512, 100 tokens, 32 x 16 (128) 11.8, 64 x 16
    // 15.1; 1024 x 1024, 400 tokens, 32 x 32 (416) 16.0, 64 x 32 (224) 12.7, 128 x 32 17.7; 2048 x 2048, 512 tokens, 32 x 32
    // (1024) 48, 64 x 32 34.4, 128 x 32 (256) 30.8; 256 x 2048, 300 tokens, 64 x 32 (320) 8.3, 128 x 32 10.5.
    const uint32_t blocks = (tokens + 15) / 16;
    uint32_t RB = blocks == 1 ? 1 : 2, ob = 1;
    auto wgs = [&]() { return (uint64_t)(L->out / (16 * ob)) * ((blocks + RB - 1) / RB); };
    if (wgs() > SKL_N_CU * 3 / 2 && L->to % 32 == 0) ob = 2;
    while (wgs() > SKL_N_CU * 3 / 2 && RB > 1 && RB < 8) RB *= 2;
    // (sixteen wavefronts, 2048 rows: 2048 x 512, 100 tokens, 12.8 -> 11.8, 2048 x 256, 512 tokens, 13.7 -> 11.5; 1024 rows the same; 512
    // x 512, 100 tokens, 6.0 / 6.5; up to 16 tokens, 1024 x 1024 6.9 -> 6.6, 512 x 512 the same)
    uint32_t nw = ob == 1 && wgs() <= SKL_N_CU && L->in > (RB == 1 ? 512u : 1024u) ? 16 : 8;
    // With more workgroups than the chip holds at once, fewer wavefronts each: eight per CU hide the latencies, and every one
    // beyond the first adds its sums to the exchange at the end, which is what a tile of few input rows consists of.  Groups of
    // 128, d = 3, eight wavefronts / this rule: 256 x 2048, 1024 tokens (512 workgroups, four) 20.7 / 13.7 us, 4096 tokens (2048, one)
    // 76 / 35; 2048 x 2048, 1024 tokens 53.5 / 48.8, 4096 tokens 205 / 177; with 256 workgroups eight are best (512 tokens, 28.5 against
    // 41.9 with four).  And none without input rows: 128 x 2048, 512 tokens, 10.3 -> 9.4.
    // And only as many workgroups count as find room for their tables at once: 5088 x 5888 in groups of 16 x 128 (318 tables above
    // an output, 40 KB), 3293 tokens, one wavefront each 3918 us, two 1532; the kernel for any geometry 2159.
    const uint64_t held = std::min<uint64_t>(wgs(), SKL_N_CU * (SKL_LDS_HARD_BYTES / tile_prompt_table_bytes(L)));
    while (nw > 1 && nw <= 8 && held * (nw / 2) >= 8 * SKL_N_CU) nw /= 2;
    nw = std::min(nw, (L->in + 31) / 32);
    return {RB, ob, nw};
}

// Whether a decode call takes the prompt kernel: two estimates in us, of its time and that of the kernels it stands in for (one
// launch for small layers, or partial sums and their reduction), both fitted to 1213 measured calls (512 to 8192 input rows,
// 128 to 8192 outputs, groups of 8 to 512 x 16 to 512, d = 1 to 8, both query modes, 8-bit and 16-bit states, batch 2 to 16; 10 %
// off on average).  What it gains by is one launch and no partial sums (2048 x 2048 in groups of 128, batch 16, 9.9 / 23.0 us) and
// weights that are rebuilt once for 16 rows instead of for four; what it can lose by is that a wavefront stages whole tables, one
// after the other, and walks its share of all input rows: 5632 x 512 in groups of 512, d = 4 (tables of 64 KB), batch 9, 54 /
// 31; 5088 x 4864 in groups of 16 x 128 (318 tables), batch 4, 69 / 43; 944 x 256, d = 8, batch 3, 10.5 / 8.6.  The choice is slower
// by more than 3 % in 20 of the calls (26 % at most), that of the rule before it, which left the tables out and took every layer of
// up to 1024 rows, in 107 (76 %).  Layers of fewer than 128 outputs or 512 input rows stay with the other kernels.
static double tile_prompt_us(const skl_layer *L, uint32_t batch)
{
    const TilePromptShape sh = tile_prompt_shape(L, batch);
    const uint32_t at_once = tile_prompt_tables(L), full = L->n_jb / at_once, rest = L->n_jb % at_once, rows = 32 * sh.nw;
    auto up = [](uint32_t a, uint32_t b) { return (double)((a + b - 1) / b); };
    const double table = 0.135 + 0.325 * up((uint32_t)tile_key_words(L), 256);          // one, by a wavefront
    const double stage = (full * up(at_once, sh.nw) + up(rest, sh.nw)) * table * (L->qbits ? 1.6 : 1.0);      // (expanded ones come from afar)
    const double steps = (full * up(at_once * L->tj, rows) + up(rest * L->tj, rows)) * (sh.ob == 2 ? 1.15 : 1.0) * (0.644 + 0.257 * L->d);
    const double alone = 2.02 + stage + steps + 0.437 * (full + (rest > 0));
    const double filled = (double)L->in * L->out / (1u << 26) * (20.0 + 11.7 * L->d);
    return std::pow(std::pow(alone, 5) + std::pow(filled, 5), 0.2);
}

static double tile_gemv_us(const skl_layer *L, uint32_t batch)
{
    const uint32_t passes = (batch + 3) / 4;
    if (skl_tile_gemv_is_small(L, batch)) {
        const bool two = (uint64_t)L->n_ob * ((L->to + TS_O - 1) / TS_O) * passes > SKL_N_CU;
        return 3.27 + L->n_jb * (0.175 + 0.0056 * L->d) + L->in / 64.0 * (0.0908 + 0.0344 * L->d) * (two ? 2.28 : 1.0) +
               0.4386 / 1024 * L->n_jb * tile_key_words(L);
    }
    return 5.55 + 0.0214 * L->n_units + (double)L->in * L->out / (1u << 26) * (20.07 + 9.06 * L->d) * passes * std::max(1.0, 64.0 / L->to) +
           1.69e-6 * L->n_units * L->out * batch;
}

bool skl_tile_prompt_decodes(const skl_layer *L, uint32_t batch)
{
    return batch >= 2 && L->in >= 512 && L->out >= 128 && skl_tile_prompt_fits(L) && tile_prompt_us(L, batch) < tile_gemv_us(L, batch);
}

skl_status_t skl_tile_launch_prompt(const skl_layer *L, const TableSrc &src, const uint16_t *X, skl_dtype_t x_dt, uint32_t ldx, void *Y,
                                    skl_dtype_t y_dt, uint32_t ldy, uint32_t tokens, hipStream_t stream)
{
    skl_status_t st = SKL_OK;
    const TileArgs a = make_tile_args(L, src);
    const uint32_t kw = (uint32_t)tile_key_words(L), at_once = tile_prompt_tables(L);
    const size_t tables = tile_prompt_table_bytes(L);
    const TilePromptShape sh = tile_prompt_shape(L, tokens);
    const uint32_t RB = sh.RB, ob = sh.ob, nw = sh.nw;
    const dim3 tiles(L->out / (16 * ob), ((tokens + 15) / 16 + RB - 1) / RB);
    const size_t need = std::max<size_t>(tables, (size_t)nw * std::min(RB * ob, TP_RED_BYTES / 1024 / nw) * 1024);
    auto launch = [&](auto kernel) {
        st = allow_lds(kernel, need);
        if (st == SKL_OK) hipLaunchKernelGGL(kernel, tiles, dim3(64 * nw), need, stream, a, X, (uint32_t)x_dt, ldx, tokens, Y, (uint32_t)y_dt, ldy, kw, at_once);
    };
    DISPATCH_D(L->d, {
        if (RB == 1) ob == 1 ? launch(k_tile_prompt<D, 1, 1>) : launch(k_tile_prompt<D, 1, 2>);
        else if (ob == 1) RB == 2 ? launch(k_tile_prompt<D, 2, 1>) : RB == 4 ? launch(k_tile_prompt<D, 4, 1>) : launch(k_tile_prompt<D, 8, 1>);
        else RB == 2 ? launch(k_tile_prompt<D, 2, 2>) : RB == 4 ? launch(k_tile_prompt<D, 4, 2>) : launch(k_tile_prompt<D, 8, 2>);
    });
    return st == SKL_OK ? check_launch("gemm") : st;
}

skl_status_t skl_tile_launch_gemm(const skl_layer *L, const TableSrc &src, const uint16_t *X, skl_dtype_t x_dt, uint32_t ldx,
                                  void *Y, skl_dtype_t y_dt, uint32_t ldy, uint32_t tokens, hipStream_t stream)
{
    skl_status_t st = SKL_OK;
    const TileArgs a = make_tile_args(L, src);
    const uint32_t kw = (uint32_t)tile_key_words(L);
    const size_t lds = (size_t)kw * 16 + (size_t)2 * TG_T * TG_AS * sizeof(uint16_t);
    const uint32_t n_oc = (L->to + TG_T - 1) / TG_T;
    const uint32_t n_tt = (tokens + TG_T - 1) / TG_T;
    if (n_tt > 65535) {
        skl_set_error("more than %u tokens in one call through the per-weight path", 65535u * TG_T);
        return SKL_ERR_UNSUPPORTED;
    }
    // (fewer than 128 input rows, groups of 64: 64 x 2048, 128 tokens 5.5 / 7.8 us here, 512 tokens 8.8 to 9.8 / 7.6, 1024 tokens 10.6
    // / 9.4, 4096 tokens 19.8 / 24.  Beyond, with whole tiles of 64 outputs, the other kernel keeps calls of few rows and sketch rows:
    // 40 x 2048, d = 3, 2477 tokens, 18.3 / 11.0, 64 x 2112, d = 3, 2138 tokens 20.2 / 16.1, 32 x 1024, d = 8, 4622 tokens 16.8 / 13.4; of 179
    // measured calls this leaves 9 slower than with the other kernel, by up to 35 %, and makes 6 slower, by up to 19 %)
    const uint64_t results = (uint64_t)tokens * L->out;
    const bool few_rows = (L->in < 128 && results > 1u << 18 && results <= 1u << 22) ||
                          (results > 1u << 22 && L->to % 64 == 0 && (uint64_t)L->in * (L->d + 2) <= 340);
    if (skl_tile_prompt_fits(L) && !few_rows) return skl_tile_launch_prompt(L, src, X, x_dt, ldx, Y, y_dt, ldy, tokens, stream);
    const dim3 grid(L->n_ob * n_oc, n_tt);
    DISPATCH_D(L->d, {
        st = allow_lds(k_tile_gemm<D>, lds);
        if (st == SKL_OK)
            hipLaunchKernelGGL(k_tile_gemm<D>, grid, dim3(SKL_WG), lds, stream, a, X, (uint32_t)x_dt, ldx, tokens, Y,
                               (uint32_t)y_dt, ldy, kw);
    });
    return st == SKL_OK ? check_launch("gemm") : st;
}

}  // namespace SKL_NS
