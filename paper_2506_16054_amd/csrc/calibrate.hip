// Offline calibration of PAROAttention on the GPU (paper Sec. 4.1 "Metric for Permutation Order",
// Sec. 4.2 (3) "Efficient Offline Mask Generation"), for gfx950.
//
//   paro_calib_block_stats   per b x b block of the post-softmax map P = softmax(Q K^T / sqrt(d)) of
//                            already reordered 16-bit operands: sum, maximum, and the number of
//                            entries below eps (the n_ij of Eq. (M_sparse)).  The map is never
//                            stored: a workgroup owns four row blocks (one, where that would leave
//                            the chip idle) and sweeps all column blocks three times, for the row
//                            maxima, for the denominators and for the block statistics, on
//                            v_mfma_f32_32x32x16_bf16 in the transposed orientation (a lane holds
//                            16 keys of ONE query, so the row statistics are in-lane plus one
//                            cross-lane step).
//   paro_calib_row_stats, paro_calib_block_stats_from_rows
//                            the first two sweeps and the third apart, each split into column chunks:
//                            the first two serve every axis order of the same Q and K.
//   paro_calib_metrics       M_sparse and M_quant of Eq. (M_sparse) / (M_quant) per head.
//   paro_calib_choose        the combined metric over the six orders and the order that minimises it.
//   paro_calib_mask          block-sum thresholding with explicit density control: the n_live
//                            largest block sums of a head stay live (exact selection on the bit
//                            patterns, equal sums resolved by position), written as the bitmask
//                            the attention path consumes.
//
// This is an offline step (the paper runs it once per model on one or two prompts); it is written
// for exactness of the integer decisions first and is not on the measured hot path.
#include <math.h>
#include <string.h>

#include "common.h"

namespace paro {

typedef __bf16 c_v8bf __attribute__((ext_vector_type(8)));
typedef float c_v16f __attribute__((ext_vector_type(16)));

// Row statistics of the map are kept in column chunks, so that a launch has several times more workgroups than
// the chip has room for: [kRowChunks][B * nh][npad] row maxima (float, log2 units) and, behind them, as many
// denominators (double).
constexpr int kRowChunks = 4;

struct CalibArgs {
    const uint8_t* q;  // bf16 [B, nh, Npad, d], reordered, padded rows zero
    const uint8_t* k;
    float* bsum;       // [B, nh, k, k]
    float* bmax;
    int* bcnt;
    float* row_max;    // row statistics in the DEFAULT token order (unused by the kernel that makes its own)
    double* row_den;
    int nh;
    int kblocks;
    int n_tokens;
    int npad;
    int bh_total;      // B * nh
    int groups;        // groups of four row blocks per (batch, head)
    int chunks;        // column chunks per group
    int total_wg;
    int per_xcd;
    float qk_scale;  // log2(e) / sqrt(d)
    float eps;
    float log2_eps;
    ReorderTable table;  // order of the operands (kernels that read row statistics of the default order)
};

// max / sum over the wavefront in lane 63; x >= 0 (0 is the identity of both)
template <typename F>
__device__ inline float lane63_fold(float x, F op) {
#define PARO_FOLD(ctrl, rows) \
    x = op(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), ctrl, rows, 0xf, false)));
    PARO_FOLD(0xB1, 0xf)   // quad_perm [1,0,3,2]
    PARO_FOLD(0x4E, 0xf)   // quad_perm [2,3,0,1]
    PARO_FOLD(0x141, 0xf)  // row_half_mirror
    PARO_FOLD(0x140, 0xf)  // row_mirror
    PARO_FOLD(0x142, 0xa)  // row_bcast 15 into rows 1 and 3
    PARO_FOLD(0x143, 0xc)  // row_bcast 31 into rows 2 and 3
#undef PARO_FOLD
    return x;
}
__device__ inline int lane63_sum(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x141, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x140, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}

enum CalibPhase { kRowMax = 0, kRowDen = 1, kBlockStats = 2, kBlockStatsAnyEps = 3 };

// One workgroup = four row blocks of one (batch, head), one wavefront each, that sweep a range of column blocks
// together: every K tile is fetched once for the four (global_load_lds into a ring of two slots, one barrier per
// tile) and the 16-byte pieces of a 128-byte line sit at position piece ^ (row % 8), which spreads the fragment
// reads over all banks.  A wavefront holds its queries as halves of 32 (one half at block 32) in the transposed
// orientation: the lanes n and n + 32 share query n of the half.
//
// Phases.  kRowMax: the row's largest logit (exact in any order).  kRowDen: its denominator against that maximum,
// accumulated in binary64, so that - rounded to binary32 - it depends on the order of the keys only where the sum lies
// within its own rounding of a binary32 boundary: the row statistics of one axis order serve all six.  Taking both
// in one sweep would save the first, but not with a denominator that is the same in every order.  kBlockStats: the exponent is formed against eps,
//     y = c S - (m + log2 l + log2 eps),   p = eps 2^y,
// so that its sign bit IS the comparison p < eps: the 32 signs of a half are shifted into one register
// (v_alignbit) and counted by one v_bcnt; the maximum is taken on y.  The offset is rounded to binary32; what that
// changes is put back by the row's factor, computed from the rounded offset.  kBlockStatsAnyEps: the same with eps = 1 in
// the exponent and p itself compared, for the eps that 2^y could not be scaled by (calib_exponent_eps).
//
// ONE_ROW_BLOCK: the four wavefronts have the same row block and every fourth column block each, through a ring of their
// own and without a barrier in the loop; their row statistics meet in meet().
template <int BLK, int D, bool ONE_ROW_BLOCK = false>
struct CalibSweep {
    static constexpr int QH = BLK / 32;
    static constexpr int KT = BLK / 32;
    static constexpr int KS = D / 16;
    static constexpr int TILE = BLK * D * 2;
    static constexpr int PIECES = TILE / (ONE_ROW_BLOCK ? 1024 : 4096);  // 1 KB pieces of a tile that a wavefront moves
    static constexpr int LDS_BYTES = (ONE_ROW_BLOCK ? 8 : 2) * TILE;
    static constexpr int STEP = ONE_ROW_BLOCK ? 4 : 1;  // column blocks from one of a wavefront's tiles to its next

    const CalibArgs& a;
    uint8_t* ring;  // LDS [2][TILE]
    int first;      // piece of a tile that this wavefront's transfers start at
    int bh, i, lane, n, g, w;
    const uint8_t* kbase;
    unsigned fill[PIECES];
    unsigned kread[KS];
    c_v8bf qf[QH][KS];
    float m[QH];      // kRowMax: running maximum; afterwards the final one
    double den[QH];
    float off[QH], factor[QH];

    __device__ CalibSweep(const CalibArgs& args, uint8_t* lds, int bh_, int group) : a(args), bh(bh_) {
        lane = threadIdx.x & 63;
        w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        n = lane & 31;
        g = lane >> 5;
        i = ONE_ROW_BLOCK ? group : min(4 * group + w, a.kblocks - 1);  // past the last row block: repeats it and stores nothing
        ring = lds + (ONE_ROW_BLOCK ? 2 * TILE * w : 0);
        first = ONE_ROW_BLOCK ? 0 : PIECES * w;
        kbase = a.k + (size_t)bh * a.npad * D * 2;
#pragma unroll
        for (int u = 0; u < PIECES; ++u) {
            const unsigned p = (first + u) * 1024u + 16u * lane;
            const unsigned row = p / (2 * D), pos = (p % (2 * D)) / 16;
            fill[u] = row * 2 * D + 16 * ((pos & ~7u) | ((pos ^ row) & 7u));
        }
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const unsigned piece = 2 * s + g;
            kread[s] = 2u * D * n + 16u * ((piece & ~7u) | ((piece ^ n) & 7u));
        }
#pragma unroll
        for (int H = 0; H < QH; ++H) {
            // a lane past the last token repeats it, query and statistics, and enters the block with factor 0 (a query of
            // zeros against that token's statistics could overflow, and 0 times infinity is not 0)
            const uint8_t* qrow = a.q + ((size_t)bh * a.npad + real_row(H)) * D * 2 + 16 * g;
#pragma unroll
            for (int s = 0; s < KS; ++s) qf[H][s] = *(const c_v8bf*)(qrow + 32 * s);
        }
    }
    __device__ int row_of(int H) const { return i * BLK + 32 * H + n; }
    __device__ int real_row(int H) const { return min(row_of(H), a.n_tokens - 1); }
    __device__ bool row_valid(int H) const { return row_of(H) < a.n_tokens; }

    __device__ void request(int t, int slot) {
        const uint8_t* kp = kbase + (size_t)t * TILE;
#pragma unroll
        for (int u = 0; u < PIECES; ++u)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(kp + fill[u]),
                                             (__attribute__((address_space(3))) void*)(ring + slot * TILE + (first + u) * 1024), 16, 0, 0);
    }

    template <int PHASE>
    __device__ void tile(int t, int slot, bool store) {
        constexpr bool STATS = PHASE == kBlockStats || PHASE == kBlockStatsAnyEps;
        const uint8_t* ks = ring + slot * TILE;
        const int nkeys = a.n_tokens - t * BLK;  // real keys of the tile
        float ps = 0.0f, pm = 0.0f;
        int pc = 0;
#pragma unroll
        for (int H = 0; H < QH; ++H) {
            c_v16f S[KT];
#pragma unroll
            for (int T = 0; T < KT; ++T) {
#pragma unroll
                for (int r = 0; r < 16; ++r) S[T][r] = 0.0f;
#pragma unroll
                for (int s = 0; s < KS; ++s)
                    S[T] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const c_v8bf*)(ks + 64 * D * T + kread[s]), qf[H][s], S[T], 0, 0, 0);
            }
            int pad = 0;  // this lane's keys past N: they do not exist
            if (nkeys < BLK) {
#pragma unroll
                for (int T = 0; T < KT; ++T)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (32 * T + 8 * (r >> 2) + 4 * g + (r & 3) >= nkeys) {
                            S[T][r] = -INFINITY;
                            ++pad;
                        }
            }
            const float o = PHASE == kRowMax ? 0.0f : PHASE == kRowDen ? -m[H] : off[H];
#pragma unroll
            for (int T = 0; T < KT; ++T)
#pragma unroll
                for (int r = 0; r < 16; ++r) S[T][r] = fmaf(S[T][r], a.qk_scale, o);
            if constexpr (PHASE != kRowDen) {
                float part[4];
#pragma unroll
                for (int T = 0; T < KT; ++T)
#pragma unroll
                    for (int r = 0; r < 16; ++r) part[r & 3] = (T == 0 && r < 4) ? S[T][r] : fmaxf(part[r & 3], S[T][r]);
                const float top = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
                if constexpr (PHASE == kRowMax) m[H] = fmaxf(m[H], top);
                else pm = fmaxf(pm, factor[H] * __builtin_amdgcn_exp2f(top));
            }
            if constexpr (PHASE == kBlockStats) {
                unsigned signs = 0;
#pragma unroll
                for (int T = 0; T < KT; ++T)
#pragma unroll
                    for (int r = 0; r < 16; ++r) signs = __builtin_amdgcn_alignbit(signs, __float_as_uint(S[T][r]), 31);
                pc += factor[H] > 0.0f ? __popc(signs) - pad : 0;  // not past N and not NaN, whose signs say nothing
            }
            if constexpr (PHASE != kRowMax) {
#pragma unroll
                for (int T = 0; T < KT; ++T)
#pragma unroll
                    for (int r = 0; r < 16; ++r) S[T][r] = __builtin_amdgcn_exp2f(S[T][r]);
            }
            if constexpr (PHASE == kRowDen) {
#pragma unroll
                for (int T = 0; T < KT; ++T)
#pragma unroll
                    for (int r = 0; r < 16; ++r) den[H] += (double)S[T][r];
            }
            if constexpr (PHASE == kBlockStatsAnyEps) {
                int below = 0;
#pragma unroll
                for (int T = 0; T < KT; ++T)
#pragma unroll
                    for (int r = 0; r < 16; ++r) below += factor[H] * S[T][r] < a.eps ? 1 : 0;
                pc += factor[H] > 0.0f ? below - pad : 0;
            }
            if constexpr (STATS) {
                float part[4];
#pragma unroll
                for (int T = 0; T < KT; ++T)
#pragma unroll
                    for (int r = 0; r < 16; ++r) part[r & 3] = (T == 0 && r < 4) ? S[T][r] : part[r & 3] + S[T][r];
                ps = fmaf(factor[H], (part[0] + part[1]) + (part[2] + part[3]), ps);
            }
        }
        if constexpr (STATS) {
            ps = lane63_fold(ps, [](float x, float y) { return x + y; });
            pm = lane63_fold(pm, [](float x, float y) { return fmaxf(x, y); });
            pc = lane63_sum(pc);
            if (store && lane == 63) {
                const size_t at = ((size_t)bh * a.kblocks + i) * a.kblocks + t;
                a.bsum[at] = ps;
                a.bmax[at] = pm;
                a.bcnt[at] = pc;
            }
        }
    }

    template <int PHASE>
    __device__ void sweep(int t0, int t1, bool store) {
        if constexpr (PHASE == kRowMax)
#pragma unroll
            for (int H = 0; H < QH; ++H) m[H] = -INFINITY;
        if constexpr (PHASE == kRowDen)
#pragma unroll
            for (int H = 0; H < QH; ++H) den[H] = 0.0;
        __syncthreads();  // the previous sweep is done with the ring
        if constexpr (ONE_ROW_BLOCK) t0 += w;
        if (t0 < t1) request(t0, 0);
        for (int t = t0, slot = 0; t < t1; t += STEP, slot ^= 1) {
            __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0), lgkmcnt(0): this wavefront's share of tile t has landed
            if constexpr (!ONE_ROW_BLOCK) __syncthreads();  // and everybody's; the tile before it has been read by all
            if (t + STEP < t1) request(t + STEP, slot ^ 1);
            tile<PHASE>(t, slot, store);
        }
#pragma unroll
        for (int H = 0; H < QH; ++H) {  // the two lanes of a query hold half of its keys each
            if constexpr (PHASE == kRowMax) m[H] = fmaxf(m[H], __shfl_xor(m[H], 32));
            if constexpr (PHASE == kRowDen) den[H] += __shfl_xor(den[H], 32);
        }
    }

    // ONE_ROW_BLOCK: the maxima or denominators of the four wavefronts' column blocks, joined in all of them
    template <int PHASE, typename T>
    __device__ void meet(T (*rows)[BLK], T (&mine)[QH]) {
#pragma unroll
        for (int H = 0; H < QH; ++H)
            if (g == 0) rows[w][32 * H + n] = mine[H];
        __syncthreads();
#pragma unroll
        for (int H = 0; H < QH; ++H) {
            T x = rows[0][32 * H + n];
            for (int v = 1; v < 4; ++v) {
                if constexpr (PHASE == kRowMax) x = fmaxf(x, rows[v][32 * H + n]);
                else x += rows[v][32 * H + n];
            }
            mine[H] = x;
        }
    }

    // offset and factor of a row from its maximum and its denominator in binary32:  p = factor 2^(c S + off)
    __device__ void finish_row(int H, float l) {
        off[H] = -m[H] - (__builtin_amdgcn_logf(l) + a.log2_eps);
        factor[H] = row_valid(H) ? __builtin_amdgcn_exp2f(-m[H] - off[H]) / l : 0.0f;
    }
};

template <int BLK, int D>
constexpr int calib_waves() { return BLK == 64 && D == 128 ? 2 : 3; }

// the three sweeps of four row blocks, or of one, by their own workgroup (operands in any order, nothing kept)
template <int BLK, int D, int STATS, bool ONE_ROW_BLOCK>
__global__ __launch_bounds__(256, (ONE_ROW_BLOCK ? (BLK * D > 4096 ? 1 : 2) : calib_waves<BLK, D>())) void calib_stats_kernel(CalibArgs a) {
    using Sweep = CalibSweep<BLK, D, ONE_ROW_BLOCK>;
    __shared__ __attribute__((aligned(16))) uint8_t lds[Sweep::LDS_BYTES];
    const int item = (blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3);  // a head's K stays in one XCD's L2
    if (item >= a.total_wg) return;
    const int per_head = ONE_ROW_BLOCK ? a.kblocks : a.groups;
    const int bh = item / per_head, group = item - bh * per_head;
    Sweep c(a, lds, bh, group);
    c.template sweep<kRowMax>(0, a.kblocks, false);
    if constexpr (ONE_ROW_BLOCK) {
        __shared__ float rows[4][BLK];
        c.template meet<kRowMax>(rows, c.m);
    }
    c.template sweep<kRowDen>(0, a.kblocks, false);
    if constexpr (ONE_ROW_BLOCK) {
        __shared__ double rows[4][BLK];
        c.template meet<kRowDen>(rows, c.den);
    }
#pragma unroll
    for (int H = 0; H < c.QH; ++H) c.finish_row(H, (float)c.den[H]);
    c.template sweep<STATS>(0, a.kblocks, ONE_ROW_BLOCK || 4 * group + c.w < a.kblocks);
}

// the same sweeps as one launch each, a workgroup per (four row blocks, column chunk)
template <int BLK, int D, int PHASE>
__global__ __launch_bounds__(256, (calib_waves<BLK, D>())) void calib_phase_kernel(CalibArgs a) {
    constexpr bool STATS = PHASE == kBlockStats || PHASE == kBlockStatsAnyEps;
    __shared__ __attribute__((aligned(16))) uint8_t lds[CalibSweep<BLK, D>::LDS_BYTES];
    const int item = (blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3);
    if (item >= a.total_wg) return;
    const int bh = item / (a.groups * a.chunks);
    const int rest = item - bh * (a.groups * a.chunks);
    const int group = rest / a.chunks, chunk = rest - group * a.chunks;
    const int t0 = (int)((long long)a.kblocks * chunk / a.chunks), t1 = (int)((long long)a.kblocks * (chunk + 1) / a.chunks);
    CalibSweep<BLK, D> c(a, lds, bh, group);
    const bool store = 4 * group + c.w < a.kblocks;
    const size_t plane = (size_t)a.bh_total * a.npad;
    if constexpr (PHASE != kRowMax) {
#pragma unroll
        for (int H = 0; H < c.QH; ++H) {
            const int row = c.real_row(H);
            const size_t at = (size_t)bh * a.npad + (STATS ? reorder_source(a.table, bh % a.nh, row) : row);
            float m = a.row_max[at];
            for (int z = 1; z < kRowChunks; ++z) m = fmaxf(m, a.row_max[z * plane + at]);
            c.m[H] = m;
            if constexpr (STATS) {
                double l = a.row_den[at];
                for (int z = 1; z < kRowChunks; ++z) l += a.row_den[z * plane + at];
                c.finish_row(H, (float)l);
            }
        }
    }
    c.template sweep<PHASE>(t0, t1, store);
    if constexpr (!STATS) {
#pragma unroll
        for (int H = 0; H < c.QH; ++H)
            if (store && c.g == 0) {
                const size_t at = chunk * plane + (size_t)bh * a.npad + c.row_of(H);
                if constexpr (PHASE == kRowMax) a.row_max[at] = c.m[H];
                else a.row_den[at] = c.den[H];
            }
    }
}

// -------------------------------------------------------------------------------------------
// M_sparse and M_quant: one workgroup per (head, axis order) reduces the head's B * k * k blocks.  Bound by latency
// and the binary64 division per block, hence 1024 threads per workgroup and all orders in one launch.
// -------------------------------------------------------------------------------------------
constexpr int kMetricThreads = 1024;

__global__ __launch_bounds__(kMetricThreads) void calib_metrics_kernel(int B, int nh, int kb, int n_tokens, int blk, const float* __restrict__ bsum,
                                                                       const float* __restrict__ bmax, const int* __restrict__ bcnt, float sigma,
                                                                       float* __restrict__ m_sparse, float* __restrict__ m_quant) {
    __shared__ double s_psi[kMetricThreads];
    __shared__ int s_sparse[kMetricThreads];
    const int h = blockIdx.x;
    const int order = blockIdx.y;
    const int t = threadIdx.x;
    const int per_head = kb * kb;
    double psi = 0.0;
    int sparse = 0;
    for (int b = 0; b < B; ++b) {
        const size_t base = (((size_t)order * B + b) * nh + h) * per_head;
        for (int e = t; e < per_head; e += kMetricThreads) {
            const int i = e / kb, j = e - i * kb;
            const int rows = min(blk, n_tokens - i * blk), cols = min(blk, n_tokens - j * blk);
            const float entries = (float)(rows * cols);
            sparse += ((float)bcnt[base + e] >= sigma * entries) ? 1 : 0;
            const float s = bsum[base + e];
            if (s > 0.0f) psi += (double)bmax[base + e] * (double)entries / (double)s;
        }
    }
    s_psi[t] = psi;
    s_sparse[t] = sparse;
    __syncthreads();
    for (int off = kMetricThreads / 2; off >= 1; off >>= 1) {
        if (t < off) {
            s_psi[t] += s_psi[t + off];
            s_sparse[t] += s_sparse[t + off];
        }
        __syncthreads();
    }
    if (t == 0) {
        const double total = (double)B * per_head;
        m_sparse[order * nh + h] = (float)((double)s_sparse[0] / total);
        m_quant[order * nh + h] = (float)(s_psi[0] / total);
    }
}

// block sums of every head's chosen order out of the six: out[b][h] = in[perm_ids[h]][b][h]
__global__ __launch_bounds__(256) void calib_pick_kernel(int B, int nh, int per_head, const float* __restrict__ in,
                                                         const uint8_t* __restrict__ perm_ids, float* __restrict__ out) {
    const int bh = blockIdx.y;
    const size_t from = ((size_t)min((int)perm_ids[bh % nh], 5) * B * nh + bh) * per_head;
    for (int e = blockIdx.x * 256 + threadIdx.x; e < per_head; e += gridDim.x * 256) out[(size_t)bh * per_head + e] = in[from + e];
}

__global__ __launch_bounds__(256) void calib_choose_kernel(int nh, const float* __restrict__ ms, const float* __restrict__ mq, float alpha,
                                                           float* __restrict__ m_out, uint8_t* __restrict__ perm_ids) {
    const int h = blockIdx.x * 256 + threadIdx.x;
    if (h >= nh) return;
    double dense[6], quant[6], sd = 0.0, sq = 0.0;
    for (int t = 0; t < 6; ++t) {
        dense[t] = 1.0 - (double)ms[t * nh + h];  // share of blocks that are not sparse: lower is better
        quant[t] = (double)mq[t * nh + h];
        sd += dense[t];
        sq += quant[t];
    }
    int best = 0;
    double best_m = 0.0;
    for (int t = 0; t < 6; ++t) {
        const double mt = (double)alpha * (sd > 0.0 ? dense[t] / sd : 0.0) + (1.0 - (double)alpha) * (sq > 0.0 ? quant[t] / sq : 0.0);
        m_out[t * nh + h] = (float)mt;
        if (t == 0 || mt < best_m) {
            best = t;
            best_m = mt;
        }
    }
    perm_ids[h] = (uint8_t)best;
}

// -------------------------------------------------------------------------------------------
// Block-sum thresholding with density control, one workgroup per head.
// -------------------------------------------------------------------------------------------
constexpr int kMaskThreads = 1024;
constexpr int kMaskMaxWords = 12288;  // k*k <= 393216 mask bits held in LDS

// Heads of up to kMaskRegBlocks blocks: the keys stay in registers (thread t holds the blocks u * 1024 + t), the
// threshold is found by bisection on the key values - one compare per key and step, counted by ballots - and the
// bits of 64 consecutive blocks are one ballot, stored as they are.
constexpr int kMaskRegKeys = 80;
constexpr int kMaskRegBlocks = kMaskRegKeys * kMaskThreads;

template <int PER>
__global__ __launch_bounds__(kMaskThreads) void calib_mask_reg_kernel(int B, int nh, int kb, int k_img, int n_live, const float* __restrict__ bsum,
                                                                      uint8_t* __restrict__ bitmask) {
    __shared__ unsigned words[PER * kMaskThreads / 32];
    __shared__ int part[2][kMaskThreads / 64];
    constexpr int WAVES = kMaskThreads / 64;
    const int h = blockIdx.x;
    const int t = threadIdx.x;
    const int lane = t & 63, w = t >> 6;
    const int per_head = kb * kb;
    const int nbytes = (per_head + 7) / 8;
    // the sum over the calibration samples, in sample order; non-negative, so its bit pattern orders it
    float sums[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) sums[u] = 0.0f;
    for (int b = 0; b < B; ++b) {
        // a buffer of exactly the head's sums: what lies past them reads as 0, with no compare per key
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(bsum + ((size_t)b * nh + h) * per_head), 0, per_head * 4, 0x00020000);
#pragma unroll
        for (int u = 0; u < PER; ++u)
            sums[u] += __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, t * 4, u * kMaskThreads * 4, 0));
    }
    // key: bit pattern + 1; 0 for text blocks and what lies past the end, which no step below counts
    unsigned keys[PER];
    unsigned top = 0u;
    const int step_i = kMaskThreads / kb, step_j = kMaskThreads % kb;
    int i = t / kb, j = t % kb;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        keys[u] = i < k_img && j < k_img ? __float_as_uint(sums[u]) + 1u : 0u;
        asm volatile("" : "+v"(keys[u]));  // `key != 0` stays a compare: kept as flags, 80 of them would fill the scalar registers
        top = max(top, keys[u]);
        i += step_i;
        j += step_j;
        if (j >= kb) {
            j -= kb;
            ++i;
        }
    }
    auto block_total = [&](int n, int slot) {  // sum over the wavefronts of a value that is uniform in each
        if (lane == 0) part[slot][w] = n;
        __syncthreads();
        n = 0;
#pragma unroll
        for (int v = 0; v < WAVES; ++v) n += part[slot][v];
        return n;
    };
    // count(key >= below) >= n_live > count(key >= above)
    unsigned below = 1u, above = 2u;
    int at_above = 0;
    const bool select = n_live > 0 && n_live < k_img * k_img;
    if (select) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) top = max(top, (unsigned)__shfl_xor((int)top, off));
        if (lane == 0) part[1][w] = (int)top;
        __syncthreads();
        for (int v = 0; v < WAVES; ++v) top = max(top, (unsigned)part[1][v]);
        above = top + 1u;
        for (int step = 0; above - below > 1u; ++step) {  // at most 32 steps
            const unsigned mid = below + (above - below) / 2u;
            int n = 0;
#pragma unroll
            for (int u = 0; u < PER; ++u) n += __popcll(__builtin_amdgcn_ballot_w64(keys[u] >= mid));
            n = block_total(n, step & 1);
            if (n >= n_live) {
                below = mid;
                if (n == n_live) break;  // exactly the wanted blocks are >= below: all of them are live
            } else {
                above = mid;
                at_above = n;
            }
        }
        __syncthreads();
    }
    // blocks above the threshold `below` are live, and of those equal to it `remaining` in ascending position
    const unsigned thr = below;
    int equal = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u)
        equal += __popcll(__builtin_amdgcn_ballot_w64(keys[u] == thr));
    equal = block_total(equal, 0);
    const int remaining = n_live - at_above;
    const bool all_equal = equal <= remaining;
    int seen = 0;  // equal blocks in front of this pass's (only needed when some of them are not live)
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const bool in = keys[u] != 0u;
        const bool eq = keys[u] == thr;
        bool live = !in || (select ? keys[u] > thr || (eq && all_equal) : n_live > 0);
        if (select && !all_equal) {
            const unsigned long long eqs = __builtin_amdgcn_ballot_w64(eq);
            __syncthreads();
            if (lane == 0) part[1][w] = __popcll(eqs);
            __syncthreads();
            int rank = seen + __popcll(eqs & ((1ull << lane) - 1ull));
            for (int v = 0; v < WAVES; ++v) {
                rank += v < w ? part[1][v] : 0;
                seen += part[1][v];
            }
            live = live || (eq && rank < remaining);
        }
        const unsigned long long bits = __builtin_amdgcn_ballot_w64(live);
        if (lane < 2) words[u * (kMaskThreads / 32) + 2 * w + lane] = (unsigned)(bits >> (32 * lane));
    }
    __syncthreads();
    // bits past the last block stay zero
    const int last_bits = per_head & 31;
    uint8_t* out = bitmask + (size_t)h * nbytes;
    for (int b = t; b < nbytes; b += kMaskThreads) {
        unsigned word = words[b >> 2];
        if (last_bits && (b >> 2) == per_head >> 5) word &= (1u << last_bits) - 1u;
        out[b] = (uint8_t)((word >> (8 * (b & 3))) & 255u);
    }
}

// Heads with more blocks: radix selection, 8 bits a pass, that reads the sums again in every pass.  (Its LDS histogram
// is slow where many keys share their leading byte: at 275 x 275 blocks 235 us against the kernel above.)
__global__ __launch_bounds__(kMaskThreads) void calib_mask_kernel(int B, int nh, int kb, int k_img, int n_live, const float* __restrict__ bsum,
                                                                  uint8_t* __restrict__ bitmask) {
    __shared__ unsigned words[kMaskMaxWords];
    __shared__ int hist[256];
    __shared__ int part[kMaskThreads];
    __shared__ int sel_bin, sel_remaining;
    const int h = blockIdx.x;
    const int t = threadIdx.x;
    const int per_head = kb * kb;
    const int nwords = (per_head + 31) / 32;
    const int nbytes = (per_head + 7) / 8;
    // the sum over the calibration samples, in sample order; non-negative, so the bit pattern orders it
    auto key_of = [&](int e) {
        float s = 0.0f;
        for (int b = 0; b < B; ++b) s += bsum[((size_t)b * nh + h) * per_head + e];
        return __float_as_uint(s);
    };
    auto is_img = [&](int e) { return e / kb < k_img && e % kb < k_img; };

    for (int wd = t; wd < nwords; wd += kMaskThreads) words[wd] = 0u;

    // ---- exact n_live-th largest key among the image x image blocks: radix selection, 8 bits a pass
    unsigned prefix = 0u, decided = 0u;
    int remaining = n_live;  // afterwards: how many blocks equal to the threshold stay live
    const bool select = n_live > 0 && n_live < k_img * k_img;
    if (select) {
        for (int shift = 24; shift >= 0; shift -= 8) {
            if (t < 256) hist[t] = 0;
            __syncthreads();
            for (int e = t; e < per_head; e += kMaskThreads) {
                if (!is_img(e)) continue;
                const unsigned key = key_of(e);
                if ((key & decided) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1);
            }
            __syncthreads();
            if (t == 0) {
                int above = 0, bin = 255;
                for (; bin > 0; --bin) {
                    if (above + hist[bin] >= remaining) break;
                    above += hist[bin];
                }
                sel_bin = bin;
                sel_remaining = remaining - above;
            }
            __syncthreads();
            prefix |= (unsigned)sel_bin << shift;
            decided |= 255u << shift;
            remaining = sel_remaining;
            __syncthreads();
        }
    }
    const unsigned thr = prefix;

    // ---- live bits; blocks equal to the threshold are taken in ascending position until `remaining`
    const int per = (per_head + kMaskThreads - 1) / kMaskThreads;
    const int lo = min(t * per, per_head), hi = min(lo + per, per_head);
    int equal = 0;
    if (select)
        for (int e = lo; e < hi; ++e) equal += (is_img(e) && key_of(e) == thr) ? 1 : 0;
    part[t] = equal;
    __syncthreads();
    for (int off = 1; off < kMaskThreads; off <<= 1) {
        const int add = t >= off ? part[t - off] : 0;
        __syncthreads();
        part[t] += add;
        __syncthreads();
    }
    int rank = part[t] - equal;
    for (int e = lo; e < hi; ++e) {
        bool live;
        if (!is_img(e)) {
            live = true;  // rows and columns of text blocks are never sparsified
        } else if (!select) {
            live = n_live > 0;
        } else {
            const unsigned key = key_of(e);
            live = key > thr || (key == thr && rank < remaining);
            rank += key == thr ? 1 : 0;
        }
        if (live) atomicOr(&words[e >> 5], 1u << (e & 31));
    }
    __syncthreads();
    uint8_t* out = bitmask + (size_t)h * nbytes;
    for (int b = t; b < nbytes; b += kMaskThreads) out[b] = (uint8_t)((words[b >> 2] >> (8 * (b & 3))) & 255u);
}

static int calib_shape(const paro_shape* s, int64_t* n, int64_t* kb) {
    if (int st = check_shape(s, n, kb)) return st;
    if (s->T_text > 0 && ((int64_t)s->F * s->Hg * s->Wg) % s->block != 0)
        return fail(PARO_EUNSUPPORTED, "with text tokens the image tokens must fill whole blocks (F*Hg*Wg=%lld, block=%d)",
                    (long long)s->F * s->Hg * s->Wg, s->block);
    return PARO_OK;
}

}  // namespace paro

namespace paro {
static int calib_args(const paro_shape* s, const void* q16, const void* k16, CalibArgs* a) {
    int64_t n, kb;
    if (int st = calib_shape(s, &n, &kb)) return st;
    if (!q16 || !k16) return fail(PARO_EINVAL, "q16 and k16 must not be NULL");
    if (((uintptr_t)q16 | (uintptr_t)k16) & 15) return fail(PARO_EINVAL, "q16 and k16 must be 16-byte aligned");
    memset(a, 0, sizeof(*a));
    a->q = (const uint8_t*)q16;
    a->k = (const uint8_t*)k16;
    a->nh = s->nh;
    a->kblocks = (int)kb;
    a->n_tokens = (int)n;
    a->npad = (int)(kb * s->block);
    a->bh_total = s->B * s->nh;
    a->groups = (int)((kb + 3) / 4);
    a->qk_scale = (float)(1.4426950408889634 / sqrt((double)s->d));
    return PARO_OK;
}
static dim3 calib_grid(CalibArgs* a, int per_head, int chunks) {
    a->chunks = chunks;
    a->total_wg = a->bh_total * per_head * chunks;
    a->per_xcd = (a->total_wg + 7) / 8;
    return dim3((unsigned)(a->per_xcd * 8));
}
// Whether 2^y with y = log2(p / eps) can stand for p: 1 / eps and the sums of 2^y over a block stay far from overflow above
// 2^-100 (below 2^-126 the factor eps would flush to zero), and up to 1 nothing is flushed that p itself would keep.
static bool calib_exponent_eps(float eps) { return eps >= 0x1p-100f && eps <= 1.0f; }

static int calib_outputs(CalibArgs* a, float eps, float* block_sum, float* block_max, int32_t* block_cnt) {
    if (!block_sum || !block_max || !block_cnt) return fail(PARO_EINVAL, "block_sum, block_max and block_cnt must not be NULL");
    if (!(eps > 0.0f)) return fail(PARO_EINVAL, "eps=%g must be positive", (double)eps);
    a->bsum = block_sum;
    a->bmax = block_max;
    a->bcnt = block_cnt;
    a->eps = eps;
    a->log2_eps = calib_exponent_eps(eps) ? (float)log2((double)eps) : 0.0f;
    return PARO_OK;
}
// the row statistics in a buffer of paro_calib_row_stats_bytes(): denominators first (8-byte aligned), then maxima
static void calib_row_buffers(CalibArgs* a, void* row_stats) {
    const size_t rows = (size_t)kRowChunks * a->bh_total * a->npad;
    a->row_den = (double*)row_stats;
    a->row_max = (float*)((double*)row_stats + rows);
}
template <int PHASE>
static void launch_phase(const paro_shape* s, dim3 grid, hipStream_t st, const CalibArgs& a) {
    if (s->block == 64 && s->d == 64) hipLaunchKernelGGL((calib_phase_kernel<64, 64, PHASE>), grid, dim3(256), 0, st, a);
    else if (s->block == 64 && s->d == 128) hipLaunchKernelGGL((calib_phase_kernel<64, 128, PHASE>), grid, dim3(256), 0, st, a);
    else if (s->block == 32 && s->d == 64) hipLaunchKernelGGL((calib_phase_kernel<32, 64, PHASE>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((calib_phase_kernel<32, 128, PHASE>), grid, dim3(256), 0, st, a);
}
// Whether every row block gets a workgroup of its own in the one-call form: while the workgroups of four row blocks leave compute
// units idle or nearly so, a quarter of the chain per wavefront is worth more than K tiles that four of them share (and than
// a quarter of the LDS, which lets fewer workgroups in).  The line, in workgroups of four, both sides in us (four / one):
// block 64, d = 64, 17550 tokens: 1 head (69) 807 / 361, 8 heads (552) 1711 / 1512, 16 heads (1104) 2872 / 2997;
// block 64, d = 128, 4096 tokens: 4 heads (64) 256 / 81, 24 heads (384) 389 / 472;
// block 32, d = 64, 17550 tokens: 1 head (138) 615 / 324, 8 heads (1104) 1641 / 1718, 48 heads of 1955 (768) 130 / 142;
// block 32, d = 128, 4096 tokens: 4 heads (128) 185 / 89, 8 heads (256) 190 / 173, 16 heads (512) 260 / 329.
static bool calib_one_row_block(const paro_shape* s, const CalibArgs& a) {
    return a.bh_total * a.groups <= (s->block == 64 && s->d == 64 ? 768 : 256);
}
template <int STATS, bool ONE_ROW_BLOCK>
static void launch_stats(const paro_shape* s, hipStream_t st, CalibArgs& a) {
    const dim3 grid = calib_grid(&a, ONE_ROW_BLOCK ? a.kblocks : a.groups, 1);
    if (s->block == 64 && s->d == 64) hipLaunchKernelGGL((calib_stats_kernel<64, 64, STATS, ONE_ROW_BLOCK>), grid, dim3(256), 0, st, a);
    else if (s->block == 64 && s->d == 128) hipLaunchKernelGGL((calib_stats_kernel<64, 128, STATS, ONE_ROW_BLOCK>), grid, dim3(256), 0, st, a);
    else if (s->block == 32 && s->d == 64) hipLaunchKernelGGL((calib_stats_kernel<32, 64, STATS, ONE_ROW_BLOCK>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((calib_stats_kernel<32, 128, STATS, ONE_ROW_BLOCK>), grid, dim3(256), 0, st, a);
}
}  // namespace paro

extern "C" int paro_calib_block_stats(const paro_shape* s, const void* q16, const void* k16, float eps, float* block_sum,
                                      float* block_max, int32_t* block_cnt, void* stream) {
    using namespace paro;
    CalibArgs a;
    if (int st = calib_args(s, q16, k16, &a)) return st;
    if (int st = calib_outputs(&a, eps, block_sum, block_max, block_cnt)) return st;
    hipStream_t st = (hipStream_t)stream;
    if (!calib_exponent_eps(eps)) launch_stats<kBlockStatsAnyEps, false>(s, st, a);
    else if (calib_one_row_block(s, a)) launch_stats<kBlockStats, true>(s, st, a);
    else launch_stats<kBlockStats, false>(s, st, a);
    return check_launch("paro_calib_block_stats");
}

extern "C" int64_t paro_calib_row_stats_bytes(const paro_shape* s) {
    using namespace paro;
    int64_t n, kb;
    if (int st = calib_shape(s, &n, &kb)) return st;
    return (int64_t)kRowChunks * s->B * s->nh * kb * s->block * (int64_t)(sizeof(double) + sizeof(float));
}

extern "C" int paro_calib_row_stats(const paro_shape* s, const void* q16, const void* k16, void* row_stats, void* stream) {
    using namespace paro;
    CalibArgs a;
    if (int st = calib_args(s, q16, k16, &a)) return st;
    if (!row_stats || ((uintptr_t)row_stats & 15)) return fail(PARO_EINVAL, "row_stats must be a 16-byte aligned buffer");
    calib_row_buffers(&a, row_stats);
    const dim3 grid = calib_grid(&a, a.groups, kRowChunks);
    launch_phase<kRowMax>(s, grid, (hipStream_t)stream, a);
    launch_phase<kRowDen>(s, grid, (hipStream_t)stream, a);
    return check_launch("paro_calib_row_stats");
}

extern "C" int paro_calib_block_stats_from_rows(const paro_shape* s, const uint8_t* h_perm_ids, const void* q16, const void* k16,
                                                const void* row_stats, float eps, float* block_sum, float* block_max,
                                                int32_t* block_cnt, void* stream) {
    using namespace paro;
    CalibArgs a;
    if (int st = calib_args(s, q16, k16, &a)) return st;
    if (int st = calib_outputs(&a, eps, block_sum, block_max, block_cnt)) return st;
    if (!h_perm_ids) return fail(PARO_EINVAL, "perm_ids is NULL");
    if (!row_stats || ((uintptr_t)row_stats & 15)) return fail(PARO_EINVAL, "row_stats must be a 16-byte aligned buffer");
    if (int st = make_reorder_table(s, h_perm_ids, &a.table)) return st;
    calib_row_buffers(&a, (void*)row_stats);
    // column chunks of about 16 blocks: a launch of many short workgroups ends evenly
    const dim3 grid = calib_grid(&a, a.groups, (a.kblocks + 15) / 16);
    if (calib_exponent_eps(eps)) launch_phase<kBlockStats>(s, grid, (hipStream_t)stream, a);
    else launch_phase<kBlockStatsAnyEps>(s, grid, (hipStream_t)stream, a);
    return check_launch("paro_calib_block_stats_from_rows");
}

extern "C" int paro_calib_metrics_orders(const paro_shape* s, int orders, const float* block_sum, const float* block_max,
                                         const int32_t* block_cnt, float sigma, float* m_sparse, float* m_quant, void* stream) {
    using namespace paro;
    int64_t n, kb;
    if (int st = calib_shape(s, &n, &kb)) return st;
    if (orders < 1 || orders > 6) return fail(PARO_EINVAL, "orders=%d out of range [1, 6]", orders);
    if (!block_sum || !block_max || !block_cnt || !m_sparse || !m_quant)
        return fail(PARO_EINVAL, "block_sum, block_max, block_cnt, m_sparse and m_quant must not be NULL");
    if (!(sigma >= 0.0f && sigma <= 1.0f)) return fail(PARO_EINVAL, "sigma=%g must lie in [0, 1]", (double)sigma);
    hipLaunchKernelGGL(calib_metrics_kernel, dim3((unsigned)s->nh, (unsigned)orders), dim3(kMetricThreads), 0, (hipStream_t)stream, s->B, s->nh,
                       (int)kb, (int)n, s->block, block_sum, block_max, block_cnt, sigma, m_sparse, m_quant);
    return check_launch("paro_calib_metrics");
}

extern "C" int paro_calib_metrics(const paro_shape* s, const float* block_sum, const float* block_max, const int32_t* block_cnt,
                                  float sigma, float* m_sparse, float* m_quant, void* stream) {
    return paro_calib_metrics_orders(s, 1, block_sum, block_max, block_cnt, sigma, m_sparse, m_quant, stream);
}

extern "C" int paro_calib_pick(const paro_shape* s, const float* block_sum6, const uint8_t* perm_ids, float* block_sum, void* stream) {
    using namespace paro;
    int64_t n, kb;
    if (int st = calib_shape(s, &n, &kb)) return st;
    if (!block_sum6 || !perm_ids || !block_sum) return fail(PARO_EINVAL, "block_sum6, perm_ids and block_sum must not be NULL");
    const int per_head = (int)(kb * kb);
    hipLaunchKernelGGL(calib_pick_kernel, dim3((unsigned)((per_head + 2047) / 2048), (unsigned)(s->B * s->nh)), dim3(256), 0, (hipStream_t)stream,
                       s->B, s->nh, per_head, block_sum6, perm_ids, block_sum);
    return check_launch("paro_calib_pick");
}

extern "C" int paro_calib_choose(int nh, const float* m_sparse6, const float* m_quant6, float alpha, float* m_combined6,
                                 uint8_t* perm_ids, void* stream) {
    using namespace paro;
    if (nh < 1 || nh > kMaxHeads) return fail(PARO_EINVAL, "nh=%d out of range [1, %d]", nh, kMaxHeads);
    if (!m_sparse6 || !m_quant6 || !m_combined6 || !perm_ids) return fail(PARO_EINVAL, "m_sparse6, m_quant6, m_combined6 and perm_ids must not be NULL");
    if (!(alpha >= 0.0f && alpha <= 1.0f)) return fail(PARO_EINVAL, "alpha=%g must lie in [0, 1]", (double)alpha);
    hipLaunchKernelGGL(calib_choose_kernel, dim3((unsigned)((nh + 255) / 256)), dim3(256), 0, (hipStream_t)stream, nh, m_sparse6, m_quant6,
                       alpha, m_combined6, perm_ids);
    return check_launch("paro_calib_choose");
}

extern "C" int paro_calib_mask(const paro_shape* s, const float* block_sum, float density, uint8_t* bitmask, void* stream) {
    using namespace paro;
    int64_t n, kb;
    if (int st = calib_shape(s, &n, &kb)) return st;
    if (!block_sum || !bitmask) return fail(PARO_EINVAL, "block_sum and bitmask must not be NULL");
    if (!(density >= 0.0f && density <= 1.0f)) return fail(PARO_EINVAL, "density=%g must lie in [0, 1]", (double)density);
    if (kb * kb > (int64_t)kMaskMaxWords * 32)
        return fail(PARO_EUNSUPPORTED, "k=%lld: masks of more than %d blocks per head are not supported", (long long)kb, kMaskMaxWords * 32);
    const int64_t k_img = ((int64_t)s->F * s->Hg * s->Wg + s->block - 1) / s->block;
    const int64_t n_live = (int64_t)nearbyint((double)density * (double)(k_img * k_img));  // ties to even
#define PARO_MASK(KERNEL)                                                                                                       \
    hipLaunchKernelGGL((KERNEL), dim3((unsigned)s->nh), dim3(kMaskThreads), 0, (hipStream_t)stream, s->B, s->nh, (int)kb, (int)k_img, \
                       (int)n_live, block_sum, bitmask)
    if (kb * kb <= 8 * kMaskThreads) PARO_MASK(calib_mask_reg_kernel<8>);
    else if (kb * kb <= kMaskRegBlocks) PARO_MASK(calib_mask_reg_kernel<kMaskRegKeys>);
    else PARO_MASK(calib_mask_kernel);
#undef PARO_MASK
    return check_launch("paro_calib_mask");
}
