// Block-aligned symmetric quantizer (paper Sec. 4.3 (1)): one scale per group of `block` tokens
// x d channels of one head, aligned with the attention block.  Bound by HBM bandwidth: every
// element is read once (2 or 4 bytes) and written once (0.5, 1 or 2 bytes).
//
// One workgroup of 256 threads owns one group.  The tile stays in registers between the absmax
// pass and the code pass, so HBM is touched exactly once in each direction.  The absmax is
// reduced inside each wavefront with cross-lane shuffles and across the four wavefronts through
// LDS.  For the PARO_VT layout the codes are transposed through LDS so that the global stores
// stay 16 bytes per lane and contiguous.
#include <hip/hip_bf16.h>
#include <string.h>

#include <algorithm>

#include "common.h"

namespace paro {

template <typename T>
__device__ inline void load8(const T* p, float (&x)[8]);

template <>
__device__ inline void load8<float>(const float* p, float (&x)[8]) {
    const float4 a = ((const float4*)p)[0];
    const float4 b = ((const float4*)p)[1];
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
    x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
}

template <>
__device__ inline void load8<uint16_t>(const uint16_t* p, float (&x)[8]) {  // bf16 bit patterns
    // the input is read exactly once: a non-temporal load keeps it from displacing the codes in the caches
    // (-3 % on the one-grid quantizer; the same hint on the stores of the codes, which the attention kernel reads
    // next, gains nothing)
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    const v4u a = __builtin_nontemporal_load((const v4u*)p);
    const unsigned w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[2 * i] = __uint_as_float(w[i] << 16);
        x[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
}

// eight values that load8 read, as they were
__device__ inline void store8(float* p, const float (&x)[8]) {
    ((float4*)p)[0] = make_float4(x[0], x[1], x[2], x[3]);
    ((float4*)p)[1] = make_float4(x[4], x[5], x[6], x[7]);
}
__device__ inline void store8(uint16_t* p, const float (&x)[8]) {
    unsigned w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = (__float_as_uint(x[2 * i]) >> 16) | (__float_as_uint(x[2 * i + 1]) & 0xffff0000u);
    *(uint4*)p = make_uint4(w[0], w[1], w[2], w[3]);
}

__device__ inline unsigned f32_to_bf16_bits(float f) {  // round to nearest even
    const unsigned u = __float_as_uint(f);
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

__device__ inline float wave_max(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
    return v;
}

// GATHER = false: the input is the reordered, padded tensor xp [bh][Npad][D].
// GATHER = true : the input is x [bh][N][D] in the default token order and the reorder of
//                 Sec. 4.1 happens on the way in (row n' of the group reads row idx(n') of x), so
//                 the reordered tensor never exists in memory.
// SMOOTH: the per-(head, channel) constant sub[bh][c] is subtracted from every real token before anything else
//         (padded rows stay zero): the smoothed tensor never exists in memory either.
// KEEP: the reordered, padded tensor is wanted as well and goes to `kept` from the registers that the codes are made from.
template <typename InT, int BLK, int D, int BITS, int LAYOUT, bool GATHER, bool SMOOTH = false, bool KEEP = false>
__device__ __forceinline__ void quantize_group(const InT* __restrict__ xp, uint8_t* __restrict__ codes, float* __restrict__ scales,
                                               int n_tokens, int kblocks, const ReorderTable& table, int nh, int blk, int bh,
                                               const float* __restrict__ sub = nullptr, InT* __restrict__ kept = nullptr) {
    constexpr int ELEMS = BLK * D;
    constexpr int CHUNKS = ELEMS / 8;  // 8 consecutive channels of one token per chunk
    constexpr int IT = (CHUNKS + 255) / 256;
    constexpr int OUT_BYTES = ELEMS * BITS / 8;
    constexpr float QMAX = BITS == 4 ? 7.0f : 127.0f;
    // LDS staging of the transposed tile: bytes for 8- and 4-bit codes, 16-bit words for bf16.
    // Rows of the staged transposed tile (one channel each) are 4 bytes longer than the block for the
    // integer codes, so that the byte stores of the 8 lanes that hold one token's 64 channels fall into
    // different LDS banks.
    constexpr int SSTR = BITS == 16 ? BLK : BLK + 4;
    constexpr int STAGE_BYTES = LAYOUT == PARO_VT ? D * SSTR * (BITS == 16 ? 2 : 1) : 16;
    __shared__ __attribute__((aligned(16))) uint8_t stage[STAGE_BYTES];
    __shared__ float wave_amax[4];

    const int tid = threadIdx.x;
    const size_t group = (size_t)bh * kblocks + blk;
    const InT* tile = GATHER ? xp + (size_t)bh * n_tokens * D : xp + group * ELEMS;
    uint8_t* out = codes + group * OUT_BYTES;

    // source row of every token of the group, computed once per row rather than once per chunk
    __shared__ int src_row[GATHER ? BLK : 1];
    if constexpr (GATHER) {
        if (tid < BLK) src_row[tid] = blk * BLK + tid < n_tokens ? reorder_source(table, bh % nh, blk * BLK + tid) : 0;
        __syncthreads();
    }

    float x[IT][8];
    float amax = 0.0f;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int chunk = tid + 256 * it;
        const int row = (chunk * 8) / D;
        const bool live = chunk < CHUNKS && blk * BLK + row < n_tokens;
        if (live) {
            if constexpr (GATHER) {
                load8<InT>(tile + (size_t)src_row[row] * D + (chunk * 8) % D, x[it]);
            } else {
                load8<InT>(tile + (size_t)chunk * 8, x[it]);
            }
            if constexpr (SMOOTH) {
                float mu[8];
                load8<float>(sub + (size_t)bh * D + (chunk * 8) % D, mu);
#pragma unroll
                for (int e = 0; e < 8; ++e) x[it][e] -= mu[e];  // one binary32 subtraction per element
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) x[it][e] = 0.0f;
        }
        if constexpr (KEEP) {
            if (chunk < CHUNKS) store8(kept + group * ELEMS + (size_t)chunk * 8, x[it]);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf(x[it][e]));
    }

    float scale = 1.0f;
    if constexpr (BITS != 16) {
        amax = wave_max(amax);
        if ((tid & 63) == 0) wave_amax[tid >> 6] = amax;
        __syncthreads();
        amax = fmaxf(fmaxf(wave_amax[0], wave_amax[1]), fmaxf(wave_amax[2], wave_amax[3]));
        if (amax > 0.0f) scale = amax / QMAX;  // correctly rounded binary32 divide
    }
    if (tid == 0) scales[group] = scale;
    const GroupDivider quotient(scale);  // fl32(x / scale) for every element of the group

#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int chunk = tid + 256 * it;
        if (chunk >= CHUNKS) continue;
        const int row = (chunk * 8) / D;
        const int c0 = (chunk * 8) % D;
        if constexpr (BITS == 16) {
            unsigned h[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) h[e] = f32_to_bf16_bits(x[it][e]);
            if constexpr (LAYOUT == PARO_ROWS) {
                uint4 w = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
                *(uint4*)(out + (size_t)chunk * 16) = w;
            } else {
                uint16_t* st = (uint16_t*)stage;
                const int slot = vt_slot(row);
#pragma unroll
                for (int e = 0; e < 8; ++e) st[(c0 + e) * BLK + slot] = (uint16_t)h[e];
            }
        } else {
            int q[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float r = rintf(quotient(x[it][e]));  // v_rndne_f32: round half to even
                q[e] = (int)fminf(fmaxf(r, -QMAX), QMAX);
            }
            if constexpr (LAYOUT == PARO_ROWS) {
                if constexpr (BITS == 8) {
                    uint2 w;
                    w.x = (q[0] & 0xff) | ((q[1] & 0xff) << 8) | ((q[2] & 0xff) << 16) | ((unsigned)q[3] << 24);
                    w.y = (q[4] & 0xff) | ((q[5] & 0xff) << 8) | ((q[6] & 0xff) << 16) | ((unsigned)q[7] << 24);
                    *(uint2*)(out + (size_t)chunk * 8) = w;
                } else {
                    unsigned w = 0;
#pragma unroll
                    for (int e = 0; e < 8; ++e) w |= (unsigned)(q[e] & 0xf) << (4 * e);
                    *(unsigned*)(out + (size_t)chunk * 4) = w;
                }
            } else {
                const int slot = vt_slot(row);
#pragma unroll
                for (int e = 0; e < 8; ++e) stage[(c0 + e) * SSTR + slot] = (uint8_t)q[e];
            }
        }
    }

    if constexpr (LAYOUT == PARO_VT) {
        __syncthreads();
        if constexpr (BITS == 4) {
            // 8 consecutive slots of one channel -> 4 bytes: byte t = slot t | slot 4+t << 4
            constexpr int GROUPS = ELEMS / 8;
            for (int g = tid; g < GROUPS; g += 256) {
                const unsigned* src = (const unsigned*)(stage + (g / (BLK / 8)) * SSTR + (g % (BLK / 8)) * 8);
                *(unsigned*)(out + (size_t)g * 4) = (src[0] & 0x0f0f0f0fu) | ((src[1] & 0x0f0f0f0fu) << 4);
            }
        } else if constexpr (BITS == 8) {
            constexpr int VEC = ELEMS / 16;
            for (int v = tid; v < VEC; v += 256) {
                const unsigned* src = (const unsigned*)(stage + (v / (BLK / 16)) * SSTR + (v % (BLK / 16)) * 16);
                ((uint4*)out)[v] = make_uint4(src[0], src[1], src[2], src[3]);
            }
        } else {
            constexpr int VEC = STAGE_BYTES / 16;
            for (int v = tid; v < VEC; v += 256) ((uint4*)out)[v] = ((const uint4*)stage)[v];
        }
    }
}

template <typename InT, int BLK, int D, int BITS, int LAYOUT, bool GATHER>
__global__ __launch_bounds__(256) void quantize_kernel(const InT* __restrict__ xp, uint8_t* __restrict__ codes,
                                                       float* __restrict__ scales, int n_tokens, int kblocks,
                                                       ReorderTable table, int nh) {
    quantize_group<InT, BLK, D, BITS, LAYOUT, GATHER>(xp, codes, scales, n_tokens, kblocks, table, nh, blockIdx.x, blockIdx.y);
}

// K with a per-channel constant removed (see paro_k_channel_mean): rows, reorder fused into the loads.
template <typename InT, int BLK, int D, int BITS>
__global__ __launch_bounds__(256) void quantize_smoothed_kernel(const InT* __restrict__ x, const float* __restrict__ sub,
                                                                uint8_t* __restrict__ codes, float* __restrict__ scales, int n_tokens,
                                                                int kblocks, ReorderTable table, int nh) {
    quantize_group<InT, BLK, D, BITS, PARO_ROWS, true, true>(x, codes, scales, n_tokens, kblocks, table, nh, blockIdx.x, blockIdx.y, sub);
}

// Sums of 8 channels per thread over the tokens first, first + ROWS, .. below last of one (batch, head), met across the wavefront's
// row lanes; part: [wavefront][channel] (base and first are the thread's own).
template <typename InT, int CHUNKS, int THREADS>
__device__ __forceinline__ void sum_channels(const InT* __restrict__ base, int D, int first, int last, double (*part)[CHUNKS * 8]) {
    constexpr int ROWS = THREADS / CHUNKS;  // tokens per pass of the workgroup
    const int tid = threadIdx.x, cc = tid % CHUNKS;
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    // 8 (bf16) or 4 (fp32) loads in flight per thread, held as loaded (16 or 32 bytes each) and widened only when they are added
    constexpr int INFLIGHT = sizeof(InT) == 2 ? 8 : 4;
    constexpr int WORDS = sizeof(InT) * 8 / 4;  // 32-bit words per 8 channels
    for (int r0 = first; r0 < last; r0 += INFLIGHT * ROWS) {
        unsigned raw[INFLIGHT][WORDS];
#pragma unroll
        for (int u = 0; u < INFLIGHT; ++u) {
            const int r = r0 + u * ROWS;
            if (r < last) {
                const uint4* src = (const uint4*)(base + (size_t)r * D);
#pragma unroll
                for (int q = 0; q < WORDS / 4; ++q) {
                    const uint4 t = src[q];
                    raw[u][4 * q] = t.x; raw[u][4 * q + 1] = t.y; raw[u][4 * q + 2] = t.z; raw[u][4 * q + 3] = t.w;
                }
            } else {
#pragma unroll
                for (int q = 0; q < WORDS; ++q) raw[u][q] = 0u;
            }
        }
#pragma unroll
        for (int u = 0; u < INFLIGHT; ++u)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float f;
                if constexpr (sizeof(InT) == 2) f = __uint_as_float((e & 1) ? (raw[u][e >> 1] & 0xffff0000u) : (raw[u][e >> 1] << 16));
                else f = __uint_as_float(raw[u][e]);
                acc[e] += (double)f;
            }
    }
    // lanes of a wavefront that own the same chunk are CHUNKS apart
#pragma unroll
    for (int off = CHUNKS; off < 64; off <<= 1)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += __shfl_xor(acc[e], off);
    if ((tid & 63) < CHUNKS) {
#pragma unroll
        for (int e = 0; e < 8; ++e) part[tid >> 6][cc * 8 + e] = acc[e];
    }
}

// Mean over the N tokens of every channel of every (batch, head), accumulated in binary64 and rounded to
// bfloat16 (returned as float).  A workgroup of 1024 threads owns CHUNKS groups of 8 channels of one (batch, head), a thread
// one of the groups of every (1024 / CHUNKS)-th token; partial sums meet across the row lanes of a wavefront by shuffles
// and across the 16 wavefronts through LDS.  Any constant would do for the smoothing (the softmax does not see it); the
// coarse rounding makes this one independent of the order of the additions.
//
// Bound by the few compute units that a launch of one workgroup per head uses.  The channels of a head are split over several
// workgroups (mean_chunks), which need no scratch memory and no second launch to meet, as a split over the tokens would.
// They read parts of the same 128-byte lines, so they are numbered to run on one XCD, whose L2 then fetches a line
// once: workgroup b runs on XCD b % 8, and the parts of a head are 8 apart.  Whole head -> split, 17550 tokens: 30 bf16
// heads 47 -> 35 us, 48 bf16 heads 49 -> 37, 30 fp32 heads 87 -> 45; 24 bf16 heads of 4096 tokens, d = 128: 18 -> 9.
template <typename InT, int CHUNKS>
__global__ __launch_bounds__(1024) void channel_mean_kernel(const InT* __restrict__ x, float* __restrict__ mean, int n_tokens, int heads, int D) {
    __shared__ double part[16][CHUNKS * 8];
    const int parts = D / (CHUNKS * 8);
    const int octet = blockIdx.x / (8 * parts), in_octet = blockIdx.x - octet * 8 * parts;
    const int head = octet * 8 + (in_octet & 7), c0 = (in_octet >> 3) * CHUNKS * 8;
    if (head >= heads) return;
    const int tid = threadIdx.x;
    const int cc = tid % CHUNKS;
    const int rl = tid / CHUNKS;
    const InT* base = x + (size_t)head * n_tokens * D + c0 + cc * 8;
    sum_channels<InT, CHUNKS, 1024>(base, D, rl, n_tokens, part);
    __syncthreads();
    if (tid < CHUNKS * 8) {
        double sum = 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) sum += part[w][tid];
        const float m = (float)(sum / (double)n_tokens);
        mean[(size_t)head * D + c0 + tid] = __uint_as_float(f32_to_bf16_bits(m) << 16);
    }
}

// 8-channel groups per workgroup: halved from the whole head until the launch covers the 256 compute units, as long as a
// workgroup has more tokens than it keeps in flight (4 heads of 128 tokens: 5.4 us whole, 6.2 split to the end) and its share
// of a token stays 32 bytes or more (48 bf16 heads of 17550 tokens: 37 us at 32 bytes, 67 at 16).
template <typename InT>
static int mean_chunks(int n, int heads, int d) {
    constexpr int least = sizeof(InT) == 2 ? 2 : 1, in_flight = sizeof(InT) == 2 ? 8 : 4;
    int chunks = d / 8;
    while (chunks > least && 2 * heads * (d / (8 * chunks)) <= 256 && n > in_flight * (1024 / chunks)) chunks /= 2;
    return chunks;
}

template <typename InT>
static void launch_channel_mean(const InT* k, float* k_mean, int n, int heads, int d, hipStream_t st) {
    const int chunks = mean_chunks<InT>(n, heads, d);
    const dim3 grid((unsigned)((heads + 7) / 8 * 8 * (d / (8 * chunks))));
#define PARO_MEAN(C) \
    case C: hipLaunchKernelGGL((channel_mean_kernel<InT, C>), grid, dim3(1024), 0, st, k, k_mean, n, heads, d); break
    if constexpr (sizeof(InT) == 4)
        switch (chunks) { PARO_MEAN(1); }
    switch (chunks) {
        PARO_MEAN(2);
        PARO_MEAN(4);
        PARO_MEAN(8);
        PARO_MEAN(16);
    }
#undef PARO_MEAN
}

// The same mean where a call has memory to meet in: workgroup (p, head) adds up the tokens p span .. of all channels of a head into
// partial[head][p], the next launch adds those.  Whole rows are read in order by workgroups on every compute unit, so it is bound by
// HBM and not by one workgroup's loads: mean, second launch and the quantizers behind them, 17550 tokens, 30 bf16 heads 93.5 -> 74.1 us,
// 8 heads 42.1 -> 28.6, 30 fp32 heads 118 -> 103; 30 bf16 heads of 5120 32.4 -> 29.9.
template <typename InT, int D>
__global__ __launch_bounds__(256) void channel_sums_kernel(const InT* __restrict__ x, double* __restrict__ partial, int n_tokens, int span) {
    constexpr int CHUNKS = D / 8;
    __shared__ double part[4][D];
    const int head = blockIdx.y, tid = threadIdx.x, first = blockIdx.x * span;
    sum_channels<InT, CHUNKS, 256>(x + (size_t)head * n_tokens * D + tid % CHUNKS * 8, D, first + tid / CHUNKS, min(first + span, n_tokens), part);
    __syncthreads();
    if (tid < D) partial[((size_t)head * gridDim.x + blockIdx.x) * D + tid] = (part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]);
}

template <int D>
__global__ __launch_bounds__(256) void channel_mean_of_sums_kernel(const double* __restrict__ partial, float* __restrict__ mean, int n_tokens, int parts) {
    __shared__ double part[256 / D][D];
    const int head = blockIdx.x, c = threadIdx.x % D, g = threadIdx.x / D;
    const double* mine = partial + (size_t)head * parts * D + c;
    double sum = 0.0;
#pragma unroll 4
    for (int p = g; p < parts; p += 256 / D) sum += mine[(size_t)p * D];
    part[g][c] = sum;
    __syncthreads();
    if (g == 0) {
#pragma unroll
        for (int u = 1; u < 256 / D; ++u) sum += part[u][c];
        mean[(size_t)head * D + c] = __uint_as_float(f32_to_bf16_bits((float)(sum / (double)n_tokens)) << 16);
    }
}

// 512 workgroups in all: two for each compute unit (256: 30 bf16 heads of 17550 tokens 1 us more; 2048: their sums take as much).
constexpr int kMeanGroups = 512;
// scratch: at least n D / 2 bytes per head.
template <typename InT, int D>
static void launch_channel_mean_by_sums(const InT* k, float* k_mean, double* scratch, int n, int heads, hipStream_t st) {
    constexpr int pass = 256 / (D / 8) * (sizeof(InT) == 2 ? 8 : 4);  // tokens that a workgroup keeps in flight
    int parts = std::min((n + 2 * pass - 1) / (2 * pass), std::max(kMeanGroups / heads, 1));
    const int span = ((n + parts - 1) / parts + pass - 1) / pass * pass;
    parts = (n + span - 1) / span;
    hipLaunchKernelGGL((channel_sums_kernel<InT, D>), dim3(parts, heads), dim3(256), 0, st, k, scratch, n, span);
    hipLaunchKernelGGL((channel_mean_of_sums_kernel<D>), dim3(heads), dim3(256), 0, st, scratch, k_mean, n, parts);
}

// Q, K and V of one attention call in a single launch (blockIdx.z selects the tensor): Q and K as
// row-major codes of QKBITS, V as transposed blocks of PVBITS, all three reordered on the way in.
// Same arithmetic as three quantize_kernel launches, two launch gaps fewer.
//
// KEEP: the reordered tensors are stored too (the separate-step form, where a program looks at them): one launch in place of
// three reorders and three quantizers, and the reordered tensors are not read back.  2 x 6 heads of 1955 fp32 tokens, block
// 32: the whole call 55.2 -> 41.7 us in three launches instead of eight (runs of one side differ by 0.2 %).
struct QkvPointers {
    const void* in[3];
    uint8_t* codes[3];
    float* scales[3];
    void* kept[3];
    int first;  // 0, or 1 where the grid holds K and V alone
};

template <typename InT, int BLK, int D, int QKBITS, int PVBITS, bool KEEP>
__global__ __launch_bounds__(256) void quantize_qkv_kernel(QkvPointers p, int n_tokens, int kblocks, ReorderTable table, int nh) {
    const int z = p.first + blockIdx.z;
    if (z < 2)
        quantize_group<InT, BLK, D, QKBITS, PARO_ROWS, true, false, KEEP>((const InT*)p.in[z], p.codes[z], p.scales[z], n_tokens, kblocks, table,
                                                                          nh, blockIdx.x, blockIdx.y, nullptr, (InT*)p.kept[z]);
    else
        quantize_group<InT, BLK, D, PVBITS, PARO_VT, true, false, KEEP>((const InT*)p.in[2], p.codes[2], p.scales[2], n_tokens, kblocks, table, nh,
                                                                        blockIdx.x, blockIdx.y, nullptr, (InT*)p.kept[2]);
}

// The same grid with the channel mean of K removed from it on the way in.
template <typename InT, int BLK, int D, int QKBITS, int PVBITS>
__global__ __launch_bounds__(256) void quantize_qkv_smoothed_kernel(QkvPointers p, const float* __restrict__ mean, int n_tokens, int kblocks,
                                                                    ReorderTable table, int nh) {
    const int z = blockIdx.z;
    if (z == 0)
        quantize_group<InT, BLK, D, QKBITS, PARO_ROWS, true>((const InT*)p.in[0], p.codes[0], p.scales[0], n_tokens, kblocks, table, nh, blockIdx.x,
                                                             blockIdx.y);
    else if (z == 1)
        quantize_group<InT, BLK, D, QKBITS, PARO_ROWS, true, true>((const InT*)p.in[1], p.codes[1], p.scales[1], n_tokens, kblocks, table, nh,
                                                                   blockIdx.x, blockIdx.y, mean);
    else
        quantize_group<InT, BLK, D, PVBITS, PARO_VT, true>((const InT*)p.in[2], p.codes[2], p.scales[2], n_tokens, kblocks, table, nh, blockIdx.x,
                                                           blockIdx.y);
}

struct QuantLaunch {
    dim3 grid;
    hipStream_t stream;
    const void* in;
    void* codes;
    float* scales;
    int n, k, nh;
    bool gather;
    ReorderTable table;
};

template <typename InT, int BLK, int D, int BITS, int LAYOUT>
static void launch_gather(const QuantLaunch& q) {
    if (q.gather)
        hipLaunchKernelGGL((quantize_kernel<InT, BLK, D, BITS, LAYOUT, true>), q.grid, dim3(256), 0, q.stream, (const InT*)q.in,
                           (uint8_t*)q.codes, q.scales, q.n, q.k, q.table, q.nh);
    else
        hipLaunchKernelGGL((quantize_kernel<InT, BLK, D, BITS, LAYOUT, false>), q.grid, dim3(256), 0, q.stream, (const InT*)q.in,
                           (uint8_t*)q.codes, q.scales, q.n, q.k, q.table, q.nh);
}

template <typename InT, int BLK, int D, int BITS>
static void launch_layout(paro_layout layout, const QuantLaunch& q) {
    if (layout == PARO_ROWS) launch_gather<InT, BLK, D, BITS, PARO_ROWS>(q);
    else launch_gather<InT, BLK, D, BITS, PARO_VT>(q);
}

template <typename InT, int BLK, int D>
static void launch_bits(int bits, paro_layout layout, const QuantLaunch& q) {
    if (bits == 8) launch_layout<InT, BLK, D, 8>(layout, q);
    else if (bits == 4) launch_layout<InT, BLK, D, 4>(layout, q);
    else launch_layout<InT, BLK, D, 16>(layout, q);
}

template <typename InT>
static void launch_shape(int blk, int d, int bits, paro_layout layout, const QuantLaunch& q) {
    if (blk == 64 && d == 64) launch_bits<InT, 64, 64>(bits, layout, q);
    else if (blk == 64 && d == 128) launch_bits<InT, 64, 128>(bits, layout, q);
    else if (blk == 32 && d == 64) launch_bits<InT, 32, 64>(bits, layout, q);
    else launch_bits<InT, 32, 128>(bits, layout, q);
}

static int quantize_entry(const char* what, const paro_shape* s, paro_dtype dtype, int bits, paro_layout layout,
                          const uint8_t* h_perm_ids, const void* in, void* codes, float* scales, void* stream) {
    int64_t n, k;
    if (int st = check_shape(s, &n, &k)) return st;
    if (dtype != PARO_F32 && dtype != PARO_BF16) return fail(PARO_EINVAL, "dtype=%d is not a paro_dtype", (int)dtype);
    if (bits != 8 && bits != 4 && bits != 16) return fail(PARO_EINVAL, "bits=%d: expected 8, 4 or 16", bits);
    if (layout != PARO_ROWS && layout != PARO_VT) return fail(PARO_EINVAL, "layout=%d is not a paro_layout", (int)layout);
    if (!in || !codes || !scales) return fail(PARO_EINVAL, "input, codes and scales must not be NULL");
    if (((uintptr_t)in | (uintptr_t)codes) & 15) return fail(PARO_EINVAL, "input and codes must be 16-byte aligned");
    if (in == codes) return fail(PARO_EINVAL, "input and codes must not alias");
    QuantLaunch q;
    q.gather = h_perm_ids != nullptr;
    if (q.gather) {
        if (int st = make_reorder_table(s, h_perm_ids, &q.table)) return st;
    } else {
        memset(&q.table, 0, sizeof(q.table));
    }
    q.grid = dim3((unsigned)k, (unsigned)(s->B * s->nh));
    q.stream = (hipStream_t)stream;
    q.in = in;
    q.codes = codes;
    q.scales = scales;
    q.n = (int)n;
    q.k = (int)k;
    q.nh = s->nh;
    if (dtype == PARO_F32) launch_shape<float>(s->block, s->d, bits, layout, q);
    else launch_shape<uint16_t>(s->block, s->d, bits, layout, q);
    return check_launch(what);
}

template <typename InT, int BLK, int D, bool KEEP>
static bool launch_qkv_bits(int bits_qk, int bits_pv, dim3 grid, hipStream_t st, const QkvPointers& p, int n, int k, const ReorderTable& t, int nh) {
#define PARO_QKV_CASE(QK, PV)                                                                                              \
    if (bits_qk == QK && bits_pv == PV) {                                                                                  \
        hipLaunchKernelGGL((quantize_qkv_kernel<InT, BLK, D, QK, PV, KEEP>), grid, dim3(256), 0, st, p, n, k, t, nh);            \
        return true;                                                                                                       \
    }
    PARO_QKV_CASE(8, 8)
    PARO_QKV_CASE(8, 4)
    PARO_QKV_CASE(4, 4)
    PARO_QKV_CASE(4, 8)
    PARO_QKV_CASE(16, 16)
#undef PARO_QKV_CASE
    return false;
}

template <typename InT, bool KEEP>
static bool launch_qkv_shape(int blk, int d, int bits_qk, int bits_pv, dim3 grid, hipStream_t st, const QkvPointers& p, int n, int k,
                             const ReorderTable& t, int nh) {
    if (blk == 64 && d == 64) return launch_qkv_bits<InT, 64, 64, KEEP>(bits_qk, bits_pv, grid, st, p, n, k, t, nh);
    if (blk == 64 && d == 128) return launch_qkv_bits<InT, 64, 128, KEEP>(bits_qk, bits_pv, grid, st, p, n, k, t, nh);
    if (blk == 32 && d == 64) return launch_qkv_bits<InT, 32, 64, KEEP>(bits_qk, bits_pv, grid, st, p, n, k, t, nh);
    return launch_qkv_bits<InT, 32, 128, KEEP>(bits_qk, bits_pv, grid, st, p, n, k, t, nh);
}

// The channel mean of K and, with it removed, the three tensors in one grid.  (Q and V beside the mean and K behind them, also two launches:
// 16 bf16 heads of 17550 tokens 67 -> 56 us, but 48 heads 127 -> 145, 30 of 5120 33 -> 35, and smaller ones the same.)
template <typename InT, int BLK, int D, int QKBITS, int PVBITS>
static void launch_smoothed_qkv(dim3 grid, hipStream_t st, const QkvPointers& p, float* mean, int n, int k, int heads, const ReorderTable& t, int nh) {
    // Rows of 8 KB of one channel and more by sums, which meet in Q's codes: these are written behind the mean and have n D / 2 bytes per head
    // or more, the sums (at most one of 8 bytes per channel and 128 tokens) n D / 16.  The third launch costs 0.5 .. 1 us: 24 bf16 heads of
    // 1024 tokens 10.7 by channels, 11.5 by sums, of 4096 21.1 and 20.8, of 8100 42.3 and 35.0; 8 fp32 heads of 1024 9.7 and 10.0, of 2048
    // 11.7 and 10.5.  (48 fp32 heads of 4096 .. 5120, whose channels fill the chip: 37.9 and 38.7, 45.2 and 46.4.)
    if ((long long)n * (int)sizeof(InT) >= 8192) launch_channel_mean_by_sums<InT, D>((const InT*)p.in[1], mean, (double*)p.codes[0], n, heads, st);
    else launch_channel_mean((const InT*)p.in[1], mean, n, heads, D, st);
    hipLaunchKernelGGL((quantize_qkv_smoothed_kernel<InT, BLK, D, QKBITS, PVBITS>), grid, dim3(256), 0, st, p, mean, n, k, t, nh);
}
template <typename InT, int BLK, int D>
static bool launch_smoothed_qkv_bits(int bits_qk, int bits_pv, dim3 grid, hipStream_t st, const QkvPointers& p, float* mean, int n, int k, int heads,
                                     const ReorderTable& t, int nh) {
    if (bits_qk == 8 && bits_pv == 8) launch_smoothed_qkv<InT, BLK, D, 8, 8>(grid, st, p, mean, n, k, heads, t, nh);
    else if (bits_qk == 8 && bits_pv == 4) launch_smoothed_qkv<InT, BLK, D, 8, 4>(grid, st, p, mean, n, k, heads, t, nh);
    else if (bits_qk == 4 && bits_pv == 4) launch_smoothed_qkv<InT, BLK, D, 4, 4>(grid, st, p, mean, n, k, heads, t, nh);
    else if (bits_qk == 4 && bits_pv == 8) launch_smoothed_qkv<InT, BLK, D, 4, 8>(grid, st, p, mean, n, k, heads, t, nh);
    else return false;
    return true;
}
template <typename InT>
static bool launch_smoothed_qkv_shape(int blk, int d, int bits_qk, int bits_pv, dim3 grid, hipStream_t st, const QkvPointers& p, float* mean, int n, int k,
                                      int heads, const ReorderTable& t, int nh) {
    if (blk == 64 && d == 64) return launch_smoothed_qkv_bits<InT, 64, 64>(bits_qk, bits_pv, grid, st, p, mean, n, k, heads, t, nh);
    if (blk == 64 && d == 128) return launch_smoothed_qkv_bits<InT, 64, 128>(bits_qk, bits_pv, grid, st, p, mean, n, k, heads, t, nh);
    if (blk == 32 && d == 64) return launch_smoothed_qkv_bits<InT, 32, 64>(bits_qk, bits_pv, grid, st, p, mean, n, k, heads, t, nh);
    return launch_smoothed_qkv_bits<InT, 32, 128>(bits_qk, bits_pv, grid, st, p, mean, n, k, heads, t, nh);
}

// outputs: codes of Q, K, V (from tensor `first` on) and, with `keep`, their reordered rows; with `mean`, the channel mean of K, removed from K
static int qkv_entry(const char* what, const paro_shape* s, paro_dtype dtype, int bits_qk, int bits_pv, const uint8_t* h_perm_ids,
                     const void* const (&ins)[3], void* const (&codes)[3], float* const (&scales)[3], void* const (&kept)[3], bool keep, void* stream,
                     int first = 0, float* mean = nullptr) {
    int64_t n, kb;
    if (int st = check_shape(s, &n, &kb)) return st;
    if (dtype != PARO_F32 && dtype != PARO_BF16) return fail(PARO_EINVAL, "dtype=%d is not a paro_dtype", (int)dtype);
    if (!h_perm_ids) return fail(PARO_EINVAL, "perm_ids is NULL");
    uintptr_t bits = 0;
    for (int a = first; a < 3; ++a) {
        if (!ins[a] || !codes[a] || !scales[a] || (keep && !kept[a])) return fail(PARO_EINVAL, "inputs, codes, scales and reordered rows must not be NULL");
        bits |= (uintptr_t)ins[a] | (uintptr_t)codes[a] | (keep ? (uintptr_t)kept[a] : 0);
    }
    if (bits & 15) return fail(PARO_EINVAL, "inputs, codes and reordered rows must be 16-byte aligned");
    const void* outs[6] = {codes[0], codes[1], codes[2], kept[0], kept[1], kept[2]};
    const int n_out = keep ? 6 : 3;
    for (int b = first; b < n_out; ++b) {
        for (int a = first; a < 3; ++a)
            if (ins[a] == outs[b]) return fail(PARO_EINVAL, "inputs and outputs must not alias");
        for (int a = first; a < b; ++a)
            if (outs[a] == outs[b]) return fail(PARO_EINVAL, "inputs and outputs must not alias");
    }
    QkvPointers p;
    p.first = first;
    for (int a = 0; a < 3; ++a) {
        p.in[a] = ins[a];
        p.codes[a] = (uint8_t*)codes[a];
        p.scales[a] = scales[a];
        p.kept[a] = kept[a];
    }
    ReorderTable table;
    if (int st = make_reorder_table(s, h_perm_ids, &table)) return st;
    const dim3 grid((unsigned)kb, (unsigned)(s->B * s->nh), (unsigned)(3 - first));
    const auto st = (hipStream_t)stream;
    if (mean) {
        const int heads = s->B * s->nh;
        const auto smoothed = dtype == PARO_F32 ? launch_smoothed_qkv_shape<float> : launch_smoothed_qkv_shape<uint16_t>;
        if (!smoothed(s->block, s->d, bits_qk, bits_pv, grid, st, p, mean, (int)n, (int)kb, heads, table, s->nh))
            return fail(PARO_EINVAL, "bits (qk=%d, pv=%d): expected (8,8), (8,4), (4,4) or (4,8)", bits_qk, bits_pv);
        return check_launch(what);
    }
    const auto run = dtype == PARO_F32 ? (keep ? launch_qkv_shape<float, true> : launch_qkv_shape<float, false>)
                                       : (keep ? launch_qkv_shape<uint16_t, true> : launch_qkv_shape<uint16_t, false>);
    if (!run(s->block, s->d, bits_qk, bits_pv, grid, st, p, (int)n, (int)kb, table, s->nh))
        return fail(PARO_EINVAL, "bits (qk=%d, pv=%d): expected (8,8), (8,4), (4,4), (4,8) or (16,16)", bits_qk, bits_pv);
    return check_launch(what);
}

}  // namespace paro

extern "C" int paro_permute_quantize_qkv(const paro_shape* s, paro_dtype dtype, int bits_qk, int bits_pv, const uint8_t* h_perm_ids,
                                         const void* q, const void* k, const void* v, void* q_codes, float* sq, void* k_codes,
                                         float* sk, void* v_codes, float* sv, void* stream) {
    return paro::qkv_entry("paro_permute_quantize_qkv", s, dtype, bits_qk, bits_pv, h_perm_ids, {q, k, v}, {q_codes, k_codes, v_codes}, {sq, sk, sv},
                           {nullptr, nullptr, nullptr}, false, stream);
}

extern "C" int paro_permute_quantize_kv(const paro_shape* s, paro_dtype dtype, int bits_qk, int bits_pv, const uint8_t* h_perm_ids, const void* k,
                                        const void* v, void* k_codes, float* sk, void* v_codes, float* sv, void* stream) {
    return paro::qkv_entry("paro_permute_quantize_kv", s, dtype, bits_qk, bits_pv, h_perm_ids, {nullptr, k, v}, {nullptr, k_codes, v_codes},
                           {nullptr, sk, sv}, {nullptr, nullptr, nullptr}, false, stream, 1);
}

extern "C" int paro_permute_quantize_qkv_smoothed(const paro_shape* s, paro_dtype dtype, int bits_qk, int bits_pv, const uint8_t* h_perm_ids,
                                                  const void* q, const void* k, const void* v, float* k_mean, void* q_codes, float* sq,
                                                  void* k_codes, float* sk, void* v_codes, float* sv, void* stream) {
    if (!k_mean || ((uintptr_t)k_mean & 15)) return paro::fail(PARO_EINVAL, "k_mean must be a 16-byte aligned buffer");
    for (const void* x : {q, k, v, (const void*)q_codes, (const void*)k_codes, (const void*)v_codes})
        if (x == k_mean) return paro::fail(PARO_EINVAL, "k_mean must not alias the other arguments");
    return paro::qkv_entry("paro_permute_quantize_qkv_smoothed", s, dtype, bits_qk, bits_pv, h_perm_ids, {q, k, v}, {q_codes, k_codes, v_codes},
                           {sq, sk, sv}, {nullptr, nullptr, nullptr}, false, stream, 0, k_mean);
}

extern "C" int paro_permute_quantize_qkv_keep(const paro_shape* s, paro_dtype dtype, int bits_qk, int bits_pv, const uint8_t* h_perm_ids,
                                              const void* q, const void* k, const void* v, void* qp, void* kp, void* vp, void* q_codes, float* sq,
                                              void* k_codes, float* sk, void* v_codes, float* sv, void* stream) {
    return paro::qkv_entry("paro_permute_quantize_qkv_keep", s, dtype, bits_qk, bits_pv, h_perm_ids, {q, k, v}, {q_codes, k_codes, v_codes},
                           {sq, sk, sv}, {qp, kp, vp}, true, stream);
}

extern "C" int paro_quantize(const paro_shape* s, paro_dtype dtype, int bits, paro_layout layout, const void* xp,
                             void* codes, float* scales, void* stream) {
    return paro::quantize_entry("paro_quantize", s, dtype, bits, layout, nullptr, xp, codes, scales, stream);
}

extern "C" int paro_permute_quantize(const paro_shape* s, paro_dtype dtype, int bits, paro_layout layout,
                                     const uint8_t* h_perm_ids, const void* x, void* codes, float* scales, void* stream) {
    if (!h_perm_ids) return paro::fail(PARO_EINVAL, "perm_ids is NULL");
    return paro::quantize_entry("paro_permute_quantize", s, dtype, bits, layout, h_perm_ids, x, codes, scales, stream);
}


namespace paro {
template <typename InT, int BLK, int D>
static void launch_smoothed(int bits, dim3 grid, hipStream_t st, const void* x, const float* sub, void* codes, float* scales, int n, int k,
                            const ReorderTable& t, int nh) {
    if (bits == 8)
        hipLaunchKernelGGL((quantize_smoothed_kernel<InT, BLK, D, 8>), grid, dim3(256), 0, st, (const InT*)x, sub, (uint8_t*)codes, scales, n, k, t, nh);
    else
        hipLaunchKernelGGL((quantize_smoothed_kernel<InT, BLK, D, 4>), grid, dim3(256), 0, st, (const InT*)x, sub, (uint8_t*)codes, scales, n, k, t, nh);
}
template <typename InT>
static void launch_smoothed_shape(int blk, int d, int bits, dim3 grid, hipStream_t st, const void* x, const float* sub, void* codes,
                                  float* scales, int n, int k, const ReorderTable& t, int nh) {
    if (blk == 64 && d == 64) launch_smoothed<InT, 64, 64>(bits, grid, st, x, sub, codes, scales, n, k, t, nh);
    else if (blk == 64 && d == 128) launch_smoothed<InT, 64, 128>(bits, grid, st, x, sub, codes, scales, n, k, t, nh);
    else if (blk == 32 && d == 64) launch_smoothed<InT, 32, 64>(bits, grid, st, x, sub, codes, scales, n, k, t, nh);
    else launch_smoothed<InT, 32, 128>(bits, grid, st, x, sub, codes, scales, n, k, t, nh);
}
}  // namespace paro

extern "C" int paro_k_channel_mean(const paro_shape* s, paro_dtype dtype, const void* k, float* k_mean, void* stream) {
    using namespace paro;
    int64_t n, kb;
    if (int st = check_shape(s, &n, &kb)) return st;
    if (dtype != PARO_F32 && dtype != PARO_BF16) return fail(PARO_EINVAL, "dtype=%d is not a paro_dtype", (int)dtype);
    if (!k || !k_mean) return fail(PARO_EINVAL, "k and k_mean must not be NULL");
    if (((uintptr_t)k | (uintptr_t)k_mean) & 15) return fail(PARO_EINVAL, "k and k_mean must be 16-byte aligned");
    if (dtype == PARO_F32) launch_channel_mean((const float*)k, k_mean, (int)n, s->B * s->nh, s->d, (hipStream_t)stream);
    else launch_channel_mean((const uint16_t*)k, k_mean, (int)n, s->B * s->nh, s->d, (hipStream_t)stream);
    return check_launch("paro_k_channel_mean");
}

extern "C" int paro_permute_quantize_smoothed(const paro_shape* s, paro_dtype dtype, int bits, const uint8_t* h_perm_ids, const void* k,
                                              const float* k_mean, void* codes, float* scales, void* stream) {
    using namespace paro;
    int64_t n, kb;
    if (int st = check_shape(s, &n, &kb)) return st;
    if (dtype != PARO_F32 && dtype != PARO_BF16) return fail(PARO_EINVAL, "dtype=%d is not a paro_dtype", (int)dtype);
    if (bits != 8 && bits != 4) return fail(PARO_EINVAL, "bits=%d: expected 8 or 4", bits);
    if (!h_perm_ids) return fail(PARO_EINVAL, "perm_ids is NULL");
    if (!k || !k_mean || !codes || !scales) return fail(PARO_EINVAL, "k, k_mean, codes and scales must not be NULL");
    if (((uintptr_t)k | (uintptr_t)k_mean | (uintptr_t)codes) & 15) return fail(PARO_EINVAL, "k, k_mean and codes must be 16-byte aligned");
    if (k == codes) return fail(PARO_EINVAL, "input and codes must not alias");
    ReorderTable table;
    if (int st = make_reorder_table(s, h_perm_ids, &table)) return st;
    const dim3 grid((unsigned)kb, (unsigned)(s->B * s->nh));
    if (dtype == PARO_F32)
        launch_smoothed_shape<float>(s->block, s->d, bits, grid, (hipStream_t)stream, k, k_mean, codes, scales, (int)n, (int)kb, table, s->nh);
    else
        launch_smoothed_shape<uint16_t>(s->block, s->d, bits, grid, (hipStream_t)stream, k, k_mean, codes, scales, (int)n, (int)kb, table, s->nh);
    return check_launch("paro_permute_quantize_smoothed");
}
