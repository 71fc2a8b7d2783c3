#include "skl_device.h"

// ========================================================================
// Sketch construction (Eq. 4).  One thread per weight: for every sketch row
// an atomic minimum on a 64-bit key (magnitude, address inside the group,
// sign) in the state's slot.  The smallest key is the weight of smallest
// magnitude and, among equals, of smallest address -- the one the sequential
// update stream keeps -- whatever the order in which threads arrive.
// ========================================================================
struct BuildArgs {
    HashArgs h;
    const uint16_t *W;
    const uint64_t *base;       // state offset of every group (row sketches: null where the kernel sums the widths)
    const uint32_t *width;
    unsigned long long *keys;
    uint32_t in, out, tj, to, n_ob, d;
    uint32_t lg_ch, max_states;     // row sketches: log2 of the channels per workgroup; d x the largest width
};

__global__ __launch_bounds__(SKL_WG) void k_build_clear(unsigned long long *keys, uint64_t n)
{
    for (uint64_t i = (uint64_t)blockIdx.x * SKL_WG + threadIdx.x; i < n; i += (uint64_t)gridDim.x * SKL_WG) keys[i] = ~0ull;
}

// grid (ceil(out / 256), min(in, 65535)): a thread owns one output column and walks the input rows of its grid row
__global__ __launch_bounds__(SKL_WG) void k_build_scatter(BuildArgs p)
{
    const uint32_t o = blockIdx.x * SKL_WG + threadIdx.x;
    if (o >= p.out) return;
    for (uint32_t j = blockIdx.y; j < p.in; j += gridDim.y) {
        const uint32_t g = (j / p.tj) * p.n_ob + o / p.to;
        const uint32_t a = (j % p.tj) * p.to + o % p.to;
        const uint32_t K = p.width[g];
        const uint16_t w = p.W[(size_t)j * p.out + o];
        const unsigned long long key = ((unsigned long long)(w & 0x7FFFu) << 25) | ((unsigned long long)a << 1) | (w >> 15);
        unsigned long long *S = p.keys + p.base[g];
        for (uint32_t r = 0; r < p.d; ++r) {
            const uint32_t t = __umul24(p.h.A[r], a) + p.h.C[r];
            atomicMin(S + (size_t)r * K + select_index(t, K << 8), key);
        }
    }
}

// Row sketches (one group per input channel).  A workgroup owns 1 << p.lg_ch neighbouring channels, keeps their
// d x K keys in LDS as [state][channel] and takes the minima with LDS atomics.  The state index depends on the
// output only, so the lanes that hold one output of the channels (of one width) update neighbouring words.
//
// Bound by the rate of the LDS atomics, d per weight.  Measured per wavefront and CU: 16.6 clocks for 64-bit minima
// at 64 random states of one channel (the layout this kernel had before), 11.7 for 32-bit ones, 4.6 for 32-bit
// ones in rows of eight channels, 4.1 if nothing collides.  Hence eight channels, and 32-bit keys wherever a
// group has at most 2^16 weights: magnitude (15 bits) | output (16) | sign.
// 4096 x 11008, d = 4: the kernel takes 31 us (78 us with one channel and 64-bit keys per workgroup); the whole call 47 us, 95 to 98 before.
#define BR_THREADS 1024u
template <typename Key>
__device__ __forceinline__ Key build_key(uint32_t w, uint32_t o)
{
    return sizeof(Key) == 4 ? (Key)((w & 0x7FFFu) << 17 | o << 1 | w >> 15) : (Key)((uint64_t)(w & 0x7FFFu) << 25 | (uint64_t)o << 1 | w >> 15);
}

// grid ceil(in / channels per workgroup); LDS: channels x d x (largest width) keys, then a sum per wavefront
#define BR_SUMS_BYTES (BR_THREADS / 64 * 4)
template <int D, typename Key, uint32_t T>
__global__ __launch_bounds__(T) void k_build_rows(BuildArgs p, uint16_t *__restrict__ states)
{
    constexpr uint32_t KEY_SHIFT = sizeof(Key) == 4 ? 17 : 25;
    Key *S = reinterpret_cast<Key *>(smem);
    const uint32_t lg = p.lg_ch, ch = 1u << lg, j0 = blockIdx.x << lg;
    const uint32_t c = threadIdx.x & (ch - 1);                  // this thread's channel
    const uint32_t j = min(j0 + c, p.in - 1), K = p.width[j];
    for (uint32_t i = threadIdx.x; i < (p.max_states << lg); i += T) S[i] = (Key)~(Key)0;
    __syncthreads();
    const uint16_t *row = p.W + (size_t)j * p.out;
    // LDS byte address of (row r, state 0, channel c), and log2 of the bytes per state
    const uint32_t sh = lg + (sizeof(Key) == 4 ? 2 : 3), Kq = K << 8;
    const uint32_t out = p.out, step = (T >> lg) * 8;
    uint32_t Sr[D], A[D], A_next[D];                            // A_next: from a thread's eighth output to the first of its next eight
#pragma unroll
    for (int r = 0; r < D; ++r) A[r] = p.h.A[r], A_next[r] = (step - 8) * p.h.A[r];
#pragma unroll
    for (int r = 0; r < D; ++r) Sr[r] = (uint32_t)(uintptr_t)(lds_void *)smem + (r * K << sh) + c * (uint32_t)sizeof(Key);
    // every thread takes eight outputs of its channel at a time, the next eight on their way meanwhile
    uint32_t o0 = (threadIdx.x >> lg) * 8;
    uint32_t t[D];
#pragma unroll
    for (int r = 0; r < D; ++r) t[r] = __umul24(A[r], o0) + p.h.C[r];
    auto update = [&](uint32_t w, uint32_t o) {
        const Key key = build_key<Key>(w, o);
#pragma unroll
        for (int r = 0; r < D; ++r) {
            uint32_t at;            // as one instruction (left to itself the compiler splits Sr[r] into a shifted part and a rest)
            asm("v_lshl_add_u32 %0, %1, %2, %3" : "=v"(at) : "v"(select_index(t[r], Kq)), "s"(sh), "v"(Sr[r]));
            __hip_atomic_fetch_min((__attribute__((address_space(3))) Key *)(uintptr_t)at, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            t[r] += A[r];           // (only the low 24 bits of t count)
        }
    };
    if (j0 + c >= p.in) {
        // a slot of the last workgroup without a channel
    } else if ((out & 7u) == 0) {   // rows are whole, aligned 16-byte pieces
        u32x4v next = {0, 0, 0, 0};
        if (o0 < out) next = *reinterpret_cast<const u32x4v *>(row + o0);
        for (; o0 < out; o0 += step) {
            const u32x4v e = next;
            if (o0 + step < out) next = *reinterpret_cast<const u32x4v *>(row + o0 + step);
#pragma unroll
            for (uint32_t i = 0; i < 8; ++i) update((e[i >> 1] >> ((i & 1) * 16)) & 0xFFFFu, o0 + i);
#pragma unroll
            for (int r = 0; r < D; ++r) t[r] += A_next[r];
        }
    } else {
        for (; o0 < out; o0 += step) {
            const uint32_t n = min(8u, out - o0);
            uint32_t next = row[o0];
            for (uint32_t i = 0; i < n; ++i) {
                const uint32_t w = next;
                next = row[min(o0 + i + 1, out - 1)];
                update(w, o0 + i);
            }
#pragma unroll
            for (int r = 0; r < D; ++r) t[r] += A_next[r];      // (only the last piece may be short)
        }
    }
    // the states of the channels before this workgroup's: summed here where that is a few loads per thread, so that the
    // widths are all the host has to send
    uint16_t *dst = states;
    if (p.base) {
        __syncthreads();
        dst += p.base[j0];
    } else {
        uint32_t before = 0;
        for (uint32_t i = threadIdx.x; i < j0; i += T) before += p.width[i];
        for (int m = 32; m; m >>= 1) before += __shfl_xor(before, m);
        uint32_t *part = reinterpret_cast<uint32_t *>(S + (p.max_states << lg));
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = before;
        __syncthreads();
        before = 0;
        for (uint32_t i = 0; i < T / 64; ++i) before += part[i];
        dst += (size_t)before * D;
    }
    for (uint32_t cc = 0; cc < ch && j0 + cc < p.in; ++cc) {
        const uint32_t n = D * p.width[j0 + cc];
        for (uint32_t i = threadIdx.x; i < n; i += T) {
            const Key k = S[(i << lg) + cc];
            dst[i] = k == (Key)~(Key)0 ? (uint16_t)0 : (uint16_t)(((k & 1) << 15) | (k >> KEY_SHIFT));
        }
        dst += n;
    }
}

__global__ __launch_bounds__(SKL_WG) void k_build_finish(const unsigned long long *keys, uint64_t n, uint16_t *states)
{
    for (uint64_t i = (uint64_t)blockIdx.x * SKL_WG + threadIdx.x; i < n; i += (uint64_t)gridDim.x * SKL_WG) {
        const unsigned long long k = keys[i];
        states[i] = k == ~0ull ? (uint16_t)0 : (uint16_t)(((k & 1) << 15) | (k >> 25));
    }
}


skl_status_t skl_launch_build(const skl_desc_t *d, uint64_t n_groups, const uint64_t *group_base, const uint16_t *W,
                              uint16_t *states, void *ws, void *stream_)
{
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    char *area = static_cast<char *>(ws);
    BuildArgs a;
    for (int r = 0; r < SKL_MAX_D; ++r) { a.h.A[r] = r < (int)d->d ? d->hash_a[r] : 0; a.h.C[r] = r < (int)d->d ? d->hash_c[r] : 0; }
    a.W = W;
    a.keys = reinterpret_cast<unsigned long long *>(area);
    area += round256(d->n_states * 8);
    uint64_t *base_dev = reinterpret_cast<uint64_t *>(area);
    area += round256((n_groups + 1) * 8);
    uint32_t *width_dev = reinterpret_cast<uint32_t *>(area);
    a.width = width_dev;
    a.in = d->in_features; a.out = d->out_features; a.tj = d->tile_in; a.to = d->tile_out;
    a.n_ob = d->out_features / d->tile_out; a.d = d->d;
    const bool key32 = d->tile_out <= 65536;
    uint32_t max_K = 0;
    for (uint64_t g = 0; g < n_groups; ++g) max_K = std::max(max_K, d->group_width[g]);
    const uint64_t ch_lds = (uint64_t)d->d * max_K * (key32 ? 4 : 8);       // row sketches: LDS bytes per channel
    bool rows = d->tile_in == 1 && d->tile_out == d->out_features && ch_lds <= 64 * 1024;
    if (rows) {
        // eight channels per workgroup, fewer where their keys exceed 64 KiB or the chip would not be filled
        a.lg_ch = 3;
        while (a.lg_ch && ((ch_lds << a.lg_ch) > 64 * 1024 || ((a.in + (1u << a.lg_ch) - 1) >> a.lg_ch) < SKL_N_CU)) --a.lg_ch;
        a.max_states = d->d * max_K;
        rows = ((a.in + (1u << a.lg_ch) - 1) >> a.lg_ch) < (1ull << 32) / BR_THREADS;      // a grid dimension holds 2^32 threads
    }
    // Many channels: every workgroup would sum the widths of half of them on the average, which grows with the square of
    // their number, so the host sends the offsets (8 bytes per channel); and short rows then want small workgroups.
    // Whole call, summed / sent: 16384 x 4096 85 / 90 us, 24576 x 4096 124 / 130, 32768 x 4096 151 / 138, 65536 x 4096
    // 320 / 242.  Rows of 256 outputs, summed by 1024 threads / sent to 256: 24576 73 / 66, 65536 197 / 120.
    const bool short_rows = d->out_features <= 256 && d->in_features > 16384;
    const bool send_base = !rows || short_rows || d->in_features > 24576;
    a.base = send_base ? base_dev : nullptr;
    hipError_t e = hipMemcpyAsync(width_dev, d->group_width, n_groups * 4, hipMemcpyHostToDevice, stream);
    if (e == hipSuccess && send_base) e = hipMemcpyAsync(base_dev, group_base, (n_groups + 1) * 8, hipMemcpyHostToDevice, stream);
    if (e != hipSuccess) {
        skl_set_error("copy of the group widths failed: %s", hipGetErrorString(e));
        return SKL_ERR_HIP;
    }
    skl_status_t st = SKL_OK;
    if (rows) {
        const dim3 grid((a.in + (1u << a.lg_ch) - 1) >> a.lg_ch);
        const size_t lds = (size_t)(ch_lds << a.lg_ch) + BR_SUMS_BYTES;
        auto launch = [&](auto kernel, uint32_t threads) {
            st = allow_lds(kernel, lds);
            if (st == SKL_OK) hipLaunchKernelGGL(kernel, grid, dim3(threads), lds, stream, a, states);
        };
        DISPATCH_D(d->d, {
            if (!key32) launch(k_build_rows<D, unsigned long long, BR_THREADS>, BR_THREADS);
            else if (!short_rows) launch(k_build_rows<D, uint32_t, BR_THREADS>, BR_THREADS);
            else launch(k_build_rows<D, uint32_t, BR_THREADS / 4>, BR_THREADS / 4);
        })
        if (st != SKL_OK) return st;
    } else {
        const uint32_t sweep = (uint32_t)std::min<uint64_t>((d->n_states + SKL_WG - 1) / SKL_WG, 4096);
        hipLaunchKernelGGL(k_build_clear, dim3(sweep), dim3(SKL_WG), 0, stream, a.keys, d->n_states);
        hipLaunchKernelGGL(k_build_scatter, dim3((a.out + SKL_WG - 1) / SKL_WG, std::min(a.in, 65535u)), dim3(SKL_WG), 0, stream, a);
        hipLaunchKernelGGL(k_build_finish, dim3(sweep), dim3(SKL_WG), 0, stream, a.keys, d->n_states, states);
    }
    st = check_launch("sketch construction");
    if (st != SKL_OK) return st;
    e = hipStreamSynchronize(stream);          // the host arrays behind the copies may go away now
    if (e != hipSuccess) {
        skl_set_error("sketch construction failed: %s", hipGetErrorString(e));
        return SKL_ERR_HIP;
    }
    return SKL_OK;
}

