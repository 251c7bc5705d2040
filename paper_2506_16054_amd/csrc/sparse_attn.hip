// Block-sparse attention over the live blocks of a static per-head mask with INT8 QK^T and
// INT8 / INT4 PV under block-wise scales (paper Sec. 4.2 (2) and Sec. 4.3), for gfx950.
//
// Work split.  One workgroup owns one row block (BLK queries) of one head and walks that row's
// compacted live-block list in ascending order.  Integer codes have three kernels: attn_i8_w64_kernel (d = 64, block 64, many row
// blocks: one wavefront of 64 queries), attn_i8_q16_kernel (d = 128, block 64, and d = 64 with few row blocks: four wavefronts of
// 16) and attn_i8_b32_kernel (block 32: one wavefront of 32).  Both products run on v_mfma_i32_32x32x32_i8 (16x16x64 with 16
// queries) in the transposed orientation
//        S^T (keys x queries)   = K_j (A operand)   x Q_i^T (B operand, registers)
//        O^T (channels x queries) = V_j^T (A operand) x P^T   (B operand, registers)
// because the accumulator layout of a 32x32 result tile gives every lane 16 values of ONE
// query (keys 8q + 4g + p of the tile, q,p = 0..3, g = lane / 32): row reductions of the
// softmax are in-lane plus one cross-lane step, and the 16 quantized probabilities pack into
// exactly the four registers the next matrix instruction wants as its B operand.  The key
// order this imposes on the contraction is matched by the PARO_VT storage order of V, so V
// fragments are plain 16-byte reads.  The P quantization group is the whole BLK x BLK tile; cross-lane reductions use DPP,
// v_permlane32_swap and scalar reads, never LDS.
//
// Arithmetic per live block (X in log2 units, c = sq_i * sk_j * log2(e) / sqrt(d)):
//   m' = max(m, c * rowmax S)  (the row maximum is taken on the integers, c > 0);  e = max over valid rows of (c * rowmax S - m')   (<= 0)
//   E  = qmaxP * 2^(c*S - m' - e)  in (0, qmaxP]  ->  Pc = round-half-even(E), two codes per
//        v_cvt_pknorm_u16_f32 (E is formed pre-divided by 65535), four codes packed by one v_perm_b32.
//        Folded form (8-bit P codes at block 64): the exponent is ONE fma on the raw accumulator register, which read as a float
//        is B + S in units of 2^-26 (B = kStartI), so c*S + off = c*(B + S) + (off - c*B); the offset off - c*B is
//        rounded to binary32 once per row and block, and that rounding (at most half an ulp of c*B, about
//        1e-4 relative in E) is computed and returned to the block's weight, so the sums see the
//        scale the codes were really formed with,
//   l  = l * 2^(m - m') + sP * rowsum(E),  sP = 2^e / qmaxP   (the P tile maximum over qmaxP)
//   acc = acc * 2^(m - m') + (sP * sv_j) * float(Pc V_j)
// The two running sums are held divided by 2^(m' - m_ref), m_ref being the row's maximum after its
// first block: then the factor 2^(m - m') never has to be applied to them (the new term is
// multiplied by 2^(m' - m_ref) instead, one scalar per row), and since the output is acc / l the
// common factor cancels.  If a row's maximum climbs more than 64 octaves above its reference the
// sums are brought back to the current maximum (a rare, wavefront-uniform branch).
#include <string.h>

#include <type_traits>

#include "common.h"

namespace paro {

typedef unsigned v2u __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// Measurement build only (lib/libparo_timeline.so, read by `python -m paper_2506_16054_amd.probe --timeline`; the
// product library is compiled without it): every wavefront of the two main integer kernels records the constant-rate
// clock when it starts and when it has stored its rows, and the number of column blocks it visited, at slot
// (launch item) x (wavefronts per workgroup) + wavefront.  paro_timeline_read copies the records to the host.
#ifndef PARO_TIMELINE
#define PARO_TIMELINE 0
#endif
#if PARO_TIMELINE
constexpr int kTimelineSlots = 1 << 16;
constexpr int kTimelineFields = 8;  // start, end (constant-rate clock), column blocks, shader cycles of phases 0..4
__device__ long long timeline_records[kTimelineSlots][kTimelineFields];
// (on: whether this instantiation records; some have no registers to hold it)
#define PARO_TIMELINE_BEGIN(on)                                      \
    constexpr bool timeline_on = on;                                 \
    const long long timeline_start = timeline_on ? wall_clock64() : 0; \
    long long timeline_last = timeline_on ? clock64() : 0, timeline_phase[5] = {0, 0, 0, 0, 0};
// closes phase i of the block loop (shader clock at issue, not at completion, of the instructions in front of it)
#define PARO_TIMELINE_PHASE(i)                             \
    if constexpr (timeline_on) {                           \
        const long long now_ = clock64();                  \
        timeline_phase[i] += now_ - timeline_last;         \
        timeline_last = now_;                              \
    }
// without phases
#define PARO_TIMELINE_STOP(slot, lane, blocks)                                        \
    if ((lane) == 0 && (slot) < kTimelineSlots) {                                     \
        timeline_records[slot][0] = timeline_start;                                   \
        timeline_records[slot][1] = wall_clock64();                                   \
        timeline_records[slot][2] = (blocks);                                         \
    }
#define PARO_TIMELINE_END(slot, lane, blocks)                                         \
    if constexpr (timeline_on) { PARO_TIMELINE_STOP(slot, lane, blocks) }             \
    if (timeline_on && (lane) == 0 && (slot) < kTimelineSlots) {                      \
        for (int f_ = 0; f_ < 5; ++f_) timeline_records[slot][3 + f_] = timeline_phase[f_]; \
    }
#else
#define PARO_TIMELINE_BEGIN(on)
#define PARO_TIMELINE_PHASE(i)
#define PARO_TIMELINE_STOP(slot, lane, blocks)
#define PARO_TIMELINE_END(slot, lane, blocks)
#endif

struct AttnArgs {
    const uint8_t* q;
    const uint8_t* k;
    const uint8_t* v;
    const float* sq;
    const float* sk;
    const float* sv;
    const int* row_ptr;
    const int* col_idx;
    void* op;
    int nnz;
    int nh;
    int kblocks;
    int n_tokens;
    int total_wg;  // B * nh * kblocks
    int per_xcd;   // ceil(total_wg / 8)
    const int* row_order;  // optional [total_wg]: (b*nh + h)*k + i of the row block that runs at each launch position
    float qk_scale;  // log2(e) / sqrt(d)
    int scatter;     // 1: store row n' of the result at row idx(n') of o [B,nh,N,d] (Sec. 4.1 inverse reorder
                     //    done by adjusting the write-back address); 0: store op [B,nh,Npad,d]
    ReorderTable table;
};

// Where this lane's query row goes: element offset of the row in the output tensor, or -1 if the
// row is not stored (a padded row when the output is the unpadded, default-order tensor).
template <int D>
__device__ inline long long out_row_offset(const AttnArgs& a, int bh, int h, size_t head_rows, int row, bool row_valid) {
    if (!a.scatter) return (long long)((head_rows + row) * D);
    if (!row_valid) return -1;
    return (long long)(((size_t)bh * a.n_tokens + reorder_source(a.table, h, row)) * D);
}

__device__ inline unsigned bf16_rne(float f) {
    const unsigned u = __float_as_uint(f);
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

__device__ inline void store4(float* p, float a, float b, float c, float d) { *(float4*)p = make_float4(a, b, c, d); }
__device__ inline void store4(uint16_t* p, float a, float b, float c, float d) {
    *(uint2*)p = make_uint2(bf16_rne(a) | (bf16_rne(b) << 16), bf16_rne(c) | (bf16_rne(d) << 16));
}

// ---- cross-lane helpers (no LDS traffic) ---------------------------------------------------
template <int CTRL>
__device__ inline int dpp_mov(int x) {
    return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, true);
}

// max over lanes n and n + 32 (the two lanes that share a query), returned in both
__device__ inline int xor32_max(int x) {
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return max((int)r[0], (int)r[1]);
}

// Minimum over the wavefront of unsigned values that are equal in lanes l and l + 32 (the two
// lanes of a query), as a wave-uniform value.  Rows of 16 lanes are reduced with DPP (xor 1, xor 2,
// half mirror, mirror); rows 0 and 1 then cover the wave and are combined through scalar registers.
// Used on the bit patterns of floats that are all <= 0 (or -inf): for those a larger value has the
// smaller bit pattern, so this is their maximum.
__device__ inline unsigned wave_umin(unsigned x) {
    x = min(x, (unsigned)dpp_mov<0xB1>((int)x));   // quad_perm [1,0,3,2]
    x = min(x, (unsigned)dpp_mov<0x4E>((int)x));   // quad_perm [2,3,0,1]
    x = min(x, (unsigned)dpp_mov<0x141>((int)x));  // row_half_mirror
    x = min(x, (unsigned)dpp_mov<0x140>((int)x));  // row_mirror
    const unsigned r0 = __builtin_amdgcn_readlane(x, 0), r1 = __builtin_amdgcn_readlane(x, 16);
    return min(r0, r1);
}

// The folded exponent is taken where the logit scales of the row block's tiles keep the rounding of its offset small:
// c * 1.5 * 2^23 < 2^13 for the largest K scale among the live column blocks, i.e. at most 2^-12 in the exponent.  Row blocks whose inputs
// have an unusual magnitude take the exact form.  The decision is the same in every lane of the workgroup (one row block, one list).
constexpr float kFoldBound = 12582912.0f;

// Smallest scale of a block of logits that may meet the -inf of a masked key: scales of Q and K that are both of some 2^-75 have a product
// of 0, and 0 times -inf is NaN.  Rows whose scale in the ragged block is below it take the exact form of the exponent, which
// raises the scale to it: |c S| <= 2^-126 * 2^21 changes no bit of an exponent of -9 or below.
constexpr float kLogitScaleMin = 0x1p-126f;

// The scale of a column block is the same for every lane and is written by the quantizer before this kernel
// starts: read through the constant address space it becomes a scalar load, needs no vector register while it is
// carried from one block to the next, and enters its one multiplication as a scalar operand.
__device__ inline float uniform_load(const float* p) { return *(const __attribute__((address_space(4))) float*)(unsigned long long)p; }

// 1: with 8-bit P codes the accumulator bias of the logits is folded into the offset of the exponent's
// fma (one vector instruction per logit less); 0: the bias is always subtracted first and the exponent is
// exact to fp32 rounding.  With 4-bit P codes a code that flips at a rounding tie moves an output element
// by up to a seventh of its largest term, so that mode always keeps the exact exponent.
#ifndef PARO_FOLD_LOGIT_BIAS
#define PARO_FOLD_LOGIT_BIAS 1
#endif

// 16 bytes of packed 4-bit codes -> 32 signed bytes holding the codes times 16: a nibble moved to
// the top of its byte is the two's-complement code scaled by 16; the factor is undone in the
// scale.  Of every 8 codes the four even ones come first, then the four odd ones - a fixed
// permutation of the contraction index that Q and K (or P and V) share.
__device__ inline void unpack_nibbles(const v4i x, v4i& first, v4i& second) {
    const v4i lo = (x << 4) & (int)0xF0F0F0F0;
    const v4i hi = x & (int)0xF0F0F0F0;
    first = v4i{lo.x, hi.x, lo.y, hi.y};
    second = v4i{lo.z, hi.z, lo.w, hi.w};
}

// -------------------------------------------------------------------------------------------
// d = 64, block 64, 8-bit Q and K codes (P and V 8-bit or 4-bit): ONE wavefront per row block, no barrier.
//
// The wavefront owns all 64 queries of the row block as two halves of 32 (H = 0, 1; a lane holds query
// n of each half).  The P quantization group - the whole 64 x 64 tile - then lives in one wavefront: its
// maximum is an in-wave reduction, nothing is exchanged between wavefronts and nothing has to be
// synchronised.
//
// What bounds it: issue slots and, under sustained load, the energy of a block (the card holds 1 380 W of its 1 400 W limit
// throughout and lowers the clock, 2.4 -> about 2.1 GHz), so both instructions and bytes moved on the chip count.  Two
// wavefronts of a SIMD issue together only where neither issues an exponential (a v_exp_f32 takes all of 8.5 cycles), a
// matrix instruction costs 8 issue cycles beside exponentials and blocks the second slot for its 32 cycles beside
// anything else.  Therefore:
//   * the 64 exponentials of a lane come in four bursts of 16 (half x key tile) with raised priority: a wavefront in its burst is
//     not interleaved with the other one's fp32 work, which could not issue beside it, and outside of bursts both issue at once;
//   * the 16 matrix instructions sit in the bursts, one in front of every four exponentials (34 cycles).  For that, products
//     run ahead or behind: the bursts of block t hold, in turn, P V of half 1 of block t - 1, K Q of half 1 of block t + 1,
//     P V of half 0 of block t and K Q of half 0 of block t + 1;
//   * the chain from the row maxima to the tile's scale runs beside the sum and the codes of the previous block's last tile;
//   * K and V^T fragments (16 bytes per lane; a lane pair reads 32 contiguous bytes of a 64-byte row) go from global memory (L2)
//     to registers, each as soon as the last product of its predecessor is issued: K has two bursts, V one and two halves of
//     vector work to arrive.  No LDS (a copy through LDS cost 21.9 pJ/B against 16.7);
//   * the accumulators of the products start at an instruction's own constant (acc_start): 16 registers less, and 16 register
//     reads less in every second matrix instruction.
// Before: K and V by way of an LDS ring, products, maxima and exponentials of a block one after the other, 1.00 of the
// summed issue cost.  Sustained, us per call with the quantizer: 48 heads of 17550 tokens at 30 % 1 175 -> 1 089, 30 heads
// at 50 % 1 196 -> 1 090; 48 heads at 20 % with 4-bit P and V 840 -> 791, all 4-bit 839 -> 807.
// -------------------------------------------------------------------------------------------

// Lane L's 16 bytes at base + lane_off + OFFSET land at slot + OFFSET + 16 L (slot wave-uniform).  The instruction's immediate
// offset moves the global AND the LDS address, so the requests of a tile share one address register pair and one LDS base
// instead of costing a per-lane 64-bit addition each.
template <int OFFSET>
__device__ inline void lds_dma16(const uint8_t* base, unsigned lane_off, uint8_t* slot) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(base + lane_off),
                                     (__attribute__((address_space(3))) void*)slot, 16, OFFSET, 0);
}

// The lane number, computed where it stands: in rarely taken branches, so that nothing derived from it is kept in
// registers through the loop around them.
__device__ __forceinline__ int lane_here() {
    int zero = 0;
    asm volatile("" : "+v"(zero));
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
}

// 64 column indices per fetch, one per lane, one chunk ahead; at(u) is called with u = 0, 1, 2, ...
struct ColumnList {
    const int* cols;
    int cnt, kblocks, cur, nxt, chunk;
    __device__ ColumnList(const int* cols_, int cnt_, int kblocks_) : cols(cols_), cnt(cnt_), kblocks(kblocks_), chunk(0) {
        cur = load(0);
        nxt = load(1);
    }
    __device__ int load(int ch) const {
        const int idx = min(ch * 64 + lane_here(), cnt - 1);
        return cnt > 0 && ch * 64 < cnt ? min(max(cols[idx], 0), kblocks - 1) : 0;
    }
    __device__ int at(int u) {
        if ((u & 63) == 0 && u > 0) {
            cur = nxt;
            ++chunk;
            nxt = load(chunk + 1);
        }
        return __builtin_amdgcn_readlane(cur, u & 63);
    }
};

// Start of an integer accumulator chain that costs no registers: 1 / (2 pi), one of the constants that an instruction can
// name in place of a register.  As a float its bits 0x3E22F983 are kStartI * 2^-26, so the register of a chain that started
// there, read as a float, is (kStartI + result) * 2^-26 exactly while -2292099 <= result <= 6096508 (|result| <= 127 * 127 * 128
// here), and one subtraction leaves result * 2^-26.
constexpr float kStartI = 10680707.0f;
constexpr float kStartF = kStartI * 0x1p-26f;
__device__ inline v16i acc_start() {
    v16i x;
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = 0x3E22F983;
    return x;
}
__device__ inline float start_result(int raw) { return fmaf(__int_as_float(raw), 0x1p26f, -kStartI); }  // exact
// The offset of the folded exponent, off_n - c_up * kStartF rounded once, and by how much it lies above the exact value (to the last
// place of off_n: the second fma cancels to off_n plus that).  Left to the compiler, the product was rounded by itself in one of the
// two halves, and kStartI has 24 significant bits: that is no less than the difference's own rounding.  Error against binary64, fp32
// outputs of 8-bit codes, all heads of 17550 tokens: 48 heads at 30 % 3.41e-4 -> 3.15e-4, 30 heads at 50 % 3.40e-4 -> 3.14e-4, 30 heads with
// 4-bit Q and K at 30 % 3.58e-4 -> 3.34e-4 (with a start of 1.5 * 2^23 3.19e-4, 3.18e-4 and 3.91e-4).
__device__ __forceinline__ float folded_offset(float off_n, float c_up, float& above) {
    const float off = fmaf(-c_up, kStartF, off_n);
    above = fmaf(c_up, kStartF, off) - off_n;
    return off;
}
// Ends a basic block without an instruction.  The compiler names the constant above in the instruction only where a
// basic block uses it once; two chains that start in one block would get it in 16 registers.
__device__ __forceinline__ void end_basic_block() {
    __label__ next;
    asm goto("" : : : : next);
next:;
}
// How the exponent is formed from the raw logit: in one fma on the biased value; after one subtraction, with 2^26 in the scale; or
// from the integer itself, for scales that 2^26 could take out of range.
enum LogitMode { kFold = 0, kScaled = 1, kExact = 2 };

typedef const __attribute__((address_space(1))) uint8_t* global_bytes;
typedef __attribute__((address_space(1))) v4i global_v4i;
typedef __attribute__((address_space(1))) v2u global_v2u;

// QSRC: 0 = Q codes and scale from the quantizer; 1 (bf16) / 2 (fp32) = the unquantized Q in the default token order, reordered and
// quantized here - the quantization group of Q is the row block this wavefront owns (Sec. 4.3 (1)), so no other workgroup needs the
// result and its absmax is one in-wave reduction.
// QKBITS 4: Q and K rows are 32 bytes of packed 4-bit codes; a lane fetches the 16 bytes that hold its 32 channels
// (32 g .. 32 g + 31) of a K row - one fragment per key tile instead of two - and widens them to two 16-byte operands
// (codes times 16, undone in the scale) right before their products; Q is widened the same way once.
template <int QKBITS, int PVBITS, typename OutT, int QSRC>
__device__ __forceinline__ void attn_i8_w64_body(const AttnArgs& a) {
    static_assert(QSRC == 0 || QKBITS == 8, "in-kernel quantization of Q produces 8-bit codes");
    constexpr int BLK = 64, D = 64;
    constexpr int KPACK = QKBITS == 4 ? 2 : 1;
    constexpr int VPACK = PVBITS == 4 ? 2 : 1;
    constexpr float LOG2_QMAXP = PVBITS == 4 ? 2.807354922057604f : 6.988684686772166f;
    constexpr float kLog2_65535 = 15.999977986052736f;

    const int wg = blockIdx.x;
    const int logical = (wg & 7) * a.per_xcd + (wg >> 3);
    if (logical >= a.total_wg) return;
    const int item = a.row_order ? min(max(a.row_order[logical], 0), a.total_wg - 1) : logical;
    const int bh = item / a.kblocks;
    const int i = item - bh * a.kblocks;
    const int h = bh % a.nh;
    const int lane = threadIdx.x;
    const int n = lane & 31;
    const int g = lane >> 5;
#if PARO_TIMELINE
    const long long timeline_start = QKBITS == 8 ? wall_clock64() : 0;  // 4-bit Q and K leave no registers to hold it
#endif

    const int* rp = a.row_ptr + (size_t)h * (a.kblocks + 1) + i;
    const int beg = __builtin_amdgcn_readfirstlane(min(max(rp[0], 0), a.nnz));
    const int end = __builtin_amdgcn_readfirstlane(min(max(rp[1], beg), a.nnz));
    const int cnt = end - beg;
    const int* cols = a.col_idx + beg;

    const size_t head_rows = (size_t)bh * a.kblocks * BLK;
    const uint8_t* kbase = a.k + head_rows * D / KPACK;  // the head's K codes (wave-uniform)
    const uint8_t* vbase = a.v + head_rows * D / VPACK;  // the head's V^T codes (wave-uniform)
    const unsigned klane = n * (D / KPACK) + 16 * g;     // this lane's K fragment of key tile 0, step 0, inside a block
    const unsigned vlane = n * (BLK / VPACK) + 16 / VPACK * g;  // its V^T fragment of channel tile 0, key tile 0
    const float* skp = a.sk + (size_t)bh * a.kblocks;
    const float sk_last = uniform_load(skp + a.kblocks - 1);  // asked for here, used below
    const float* svp = a.sv + (size_t)bh * a.kblocks;
    float sq_i;
    int row[2];
    bool row_valid[2];
    v4i qf[2][2];  // [half][contraction step]
#pragma unroll
    for (int H = 0; H < 2; ++H) {
        row[H] = i * BLK + 32 * H + n;
        row_valid[H] = row[H] < a.n_tokens;
    }
    if constexpr (QSRC == 0 && QKBITS == 4) {
        sq_i = a.sq[(size_t)bh * a.kblocks + i] * a.qk_scale * (1.0f / 256.0f);  // Q and K codes both enter times 16
#pragma unroll
        for (int H = 0; H < 2; ++H) unpack_nibbles(*(const v4i*)(a.q + (head_rows + row[H]) * (D / 2) + 16 * g), qf[H][0], qf[H][1]);
    } else if constexpr (QSRC == 0) {
        sq_i = a.sq[(size_t)bh * a.kblocks + i] * a.qk_scale;
#pragma unroll
        for (int H = 0; H < 2; ++H) {
            const uint8_t* qrow = a.q + (head_rows + row[H]) * D + 16 * g;
#pragma unroll
            for (int s = 0; s < 2; ++s) qf[H][s] = *(const v4i*)(qrow + 32 * s);
        }
    } else {
        // same arithmetic as the quantizer: absmax over the real rows of the block, scale = absmax / 127 in
        // binary32, code = rint(fl32(x / scale))
        using RawT = std::conditional_t<QSRC == 1, uint16_t, float>;
        float x[2][2][16];  // this lane's slices of its two unquantized rows
        float amax = 0.0f;
#pragma unroll
        for (int H = 0; H < 2; ++H) {
            const RawT* qsrc = (const RawT*)a.q + ((size_t)bh * a.n_tokens + (row_valid[H] ? reorder_source(a.table, h, row[H]) : 0)) * D + 16 * g;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                if (row_valid[H]) {
                    if constexpr (QSRC == 1) {
                        const uint4 lo = *(const uint4*)(qsrc + 32 * s), hi = *(const uint4*)(qsrc + 32 * s + 8);
                        const unsigned wv[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            x[H][s][2 * e] = __uint_as_float(wv[e] << 16);
                            x[H][s][2 * e + 1] = __uint_as_float(wv[e] & 0xffff0000u);
                        }
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float4 f = *(const float4*)(qsrc + 32 * s + 4 * e);
                            x[H][s][4 * e] = f.x;
                            x[H][s][4 * e + 1] = f.y;
                            x[H][s][4 * e + 2] = f.z;
                            x[H][s][4 * e + 3] = f.w;
                        }
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 16; ++e) x[H][s][e] = 0.0f;
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) amax = fmaxf(amax, fabsf(x[H][s][e]));
            }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
        const float scale = amax > 0.0f ? amax / 127.0f : 1.0f;
        const GroupDivider quotient(scale);
#pragma unroll
        for (int H = 0; H < 2; ++H)
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int e4 = 0; e4 < 4; ++e4) {
                    unsigned word = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float r = fminf(fmaxf(rintf(quotient(x[H][s][4 * e4 + e])), -127.0f), 127.0f);
                        word |= ((unsigned)(int)r & 0xffu) << (8 * e);
                    }
                    qf[H][s][e4] = (int)word;
                }
        sq_i = scale * a.qk_scale;
    }

    v4i kf[2][2];  // K fragments of the next block [key tile][contraction step]
    v4i vf[2][2];  // V^T fragments [channel tile][key tile]
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int T = 0; T < 2; ++T) vf[dt][T] = v4i{0, 0, 0, 0};
    v4i kraw[2];   // 4-bit K: a lane's 32 channels of a key of either tile
    auto load_k = [&](int j) {
        global_bytes kp = (global_bytes)kbase + (size_t)j * (BLK * D / KPACK);  // j comes from a scalar register
        unsigned off = klane;
        asm volatile("" : "+s"(kp), "+v"(off));  // scalar base + lane offset, not a 64-bit address per lane
#pragma unroll
        for (int T = 0; T < 2; ++T) {
            if constexpr (QKBITS == 4) {
                kraw[T] = *(const global_v4i*)(kp + off + 32 * T * (D / 2));
            } else {
#pragma unroll
                for (int s = 0; s < 2; ++s) kf[T][s] = *(const global_v4i*)(kp + off + 32 * T * D + 32 * s);
            }
        }
    };
    auto widen_k = [&]() {
        if constexpr (QKBITS == 4) {
#pragma unroll
            for (int T = 0; T < 2; ++T) unpack_nibbles(kraw[T], kf[T][0], kf[T][1]);
        }
    };
    v2u vraw[2][2];  // 4-bit V: a lane's 16 slots of a channel
    auto load_v = [&](int j) {
        global_bytes vp = (global_bytes)vbase + (size_t)j * (BLK * D / VPACK);
        unsigned off = vlane;
        asm volatile("" : "+s"(vp), "+v"(off));
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int T = 0; T < 2; ++T) {
                if constexpr (PVBITS == 4) vraw[dt][T] = *(const global_v2u*)(vp + off + 32 * dt * (BLK / 2) + 16 * T);
                else vf[dt][T] = *(const global_v4i*)(vp + off + 32 * dt * BLK + 32 * T);
            }
    };
    auto widen_v = [&]() {
        if constexpr (PVBITS == 4) {
            // a nibble moved to the top of its byte is the code times 16 (undone in the scale), and the PARO_VT nibble order
            // makes the bytes come out in slot order
#pragma unroll
            for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                for (int T = 0; T < 2; ++T)
                    vf[dt][T] = v4i{(int)((vraw[dt][T].x << 4) & 0xF0F0F0F0u), (int)(vraw[dt][T].x & 0xF0F0F0F0u),
                                    (int)((vraw[dt][T].y << 4) & 0xF0F0F0F0u), (int)(vraw[dt][T].y & 0xF0F0F0F0u)};
        }
    };
    // product number p (0 .. 3) of S^T = K Q^T / of O^T = V^T P^T: the two chains of two alternate
    auto qk = [&](int p, int H, v16i (&S)[2]) {
        const int T = p & 1, s = p >> 1;
        S[T] = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf[T][s], qf[H][s], s == 0 ? acc_start() : S[T], 0, 0, 0);
    };
    auto pv = [&](int p, const v4i (&pf)[2], v16i (&o)[2]) {
        const int dt = p & 1, T = p >> 1;
        o[dt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf[dt][T], pf[T], T == 0 ? acc_start() : o[dt], 0, 0, 0);
    };

    // Padded rows hold +inf: their share of the tile's scale is then -inf, they never ask for a new reference, and what their own
    // sums become (NaN) is not stored.
    float m[2], m_ref[2];
#pragma unroll
    for (int H = 0; H < 2; ++H) m[H] = m_ref[H] = row_valid[H] ? -INFINITY : INFINITY;
    float l[2] = {0.0f, 0.0f};
    float acc[2][2][16];  // [half][channel tile][register]
#pragma unroll
    for (int H = 0; H < 2; ++H)
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[H][dt][r] = 0.0f;
    auto update = [&](int H, const v16i (&o)[2], float sv_eff) {
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc[H][dt][r] = fmaf(__int_as_float(o[dt][r]) - kStartF, sv_eff, acc[H][dt][r]);
                asm volatile("" : "+v"(acc[H][dt][r]));  // here, not where the sum is next used: the product's registers are needed
            }
    };

    // 64 column indices per fetch, one per lane; past the end of the row any column, read and not used
    auto load_cols = [&](int chunk) {
        const int idx = min(chunk * 64 + lane_here(), cnt - 1);
        return chunk * 64 < cnt ? min(max(cols[idx], 0), a.kblocks - 1) : 0;
    };
    int cols64 = load_cols(0);
    auto column = [&](int u) {  // u advances by one per call
        if ((u & 63) == 0) cols64 = load_cols(u >> 6);
        return __builtin_amdgcn_readlane(cols64, u & 63);
    };
    // The scaled and the folded form multiply the logit scale by 2^26.  Folded: the rule of kFoldBound.  Scaled: where that
    // cannot overflow; beyond 2^90 (inputs of some 2^50 each) the exact form takes over.
    constexpr bool FOLDABLE = PARO_FOLD_LOGIT_BIAS && PVBITS == 8;
    bool fast = false;
    float acc_down = 0x1p13f;  // the sums are held divided by this (half of the 2^26 of start_result), or by 2^26 where V is huge
    {   // the largest scales of the row block (a lane past the end of the list holds the row's last column)
        float sk_max = cnt > 0 ? skp[cols64] : 0.0f, sv_max = cnt > 0 ? svp[cols64] : 0.0f;
        for (int base = 64; base < cnt; base += 64)
            if (base + lane < cnt) {
                const int j = min(max(cols[base + lane], 0), a.kblocks - 1);
                sk_max = fmaxf(sk_max, skp[j]);
                sv_max = fmaxf(sv_max, svp[j]);
            }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) sk_max = fmaxf(sk_max, __shfl_xor(sk_max, off));
        if (__builtin_amdgcn_ballot_w64(sv_max > 0x1p90f) != 0) acc_down = 1.0f;
        sq_i = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(sq_i)));
        fast = FOLDABLE ? sq_i * sk_max * kFoldBound < 8192.0f : sq_i * sk_max < 0x1p90f;
    }
    const int tail_block = (a.n_tokens % BLK) != 0 ? a.kblocks - 1 : -1;  // the column block with padded keys, if any
    if (tail_block >= 0 && sq_i * sk_last < kLogitScaleMin) fast = false;

    v16i S0[2], Sa[2], Sb[2];  // raw logits [key tile]: of half 0; of half 1, this block's and the next one's in turn
    v4i pf1[2] = {v4i{0, 0, 0, 0}, v4i{0, 0, 0, 0}};
    float sv_eff1 = 0.0f;
    float sk_cur = 0.0f, sv_cur = 0.0f;
    int j0 = 0, j1 = 0;  // columns of the first block and of block t + 1 (past the end: any column, read and not used)
    if (cnt > 0) {
        j0 = __builtin_amdgcn_readlane(cols64, 0);
        j1 = column(1);
        load_k(j0);
        widen_k();
        sk_cur = uniform_load(skp + j0);
        sv_cur = uniform_load(svp + j0);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            qk(p, 0, S0);
            if (p < 2) end_basic_block();
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            qk(p, 1, Sa);
            if (p < 1) end_basic_block();
        }
        load_k(j1);
    }

    auto codes = [&](const float (&E)[16], v4i& f) {
#pragma unroll
        for (int r = 0; r < 16; r += 4) {
            const unsigned lo = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pknorm_u16(E[r], E[r + 1]));
            const unsigned hi = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pknorm_u16(E[r + 2], E[r + 3]));
            f[r >> 2] = (int)__builtin_amdgcn_perm(hi, lo, 0x06040200u);
        }
    };
    auto add16 = [&](const float (&E)[16], float (&sum)[4], bool first) {
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[r & 3] = first && r < 4 ? E[r] : sum[r & 3] + E[r];
        asm volatile("" : "+v"(sum[0]), "+v"(sum[1]), "+v"(sum[2]), "+v"(sum[3]));  // here: the exponentials' registers are needed
    };
    // what is left of half 1 of the block before when a block begins: its second tile's exponentials (E), the sum over its
    // first one, its weight, and (pf1, sv_eff1) its product P V
    float sum1[4] = {0.0f, 0.0f, 0.0f, 0.0f}, w_blk1 = 0.0f;

    auto close = [&](const float (&E)[16]) {
        add16(E, sum1, false);
        codes(E, pf1[1]);
        l[1] = fmaf((sum1[0] + sum1[1]) + (sum1[2] + sum1[3]), w_blk1, l[1]);
    };

    // What has to be known of a block before its exponentials: row maxima and the tile's scale.  `last`: the tile of the block before
    // whose sum and codes are still to be made; they keep the wavefront busy through this chain of dependent steps.
    float e = 0.0f;
    auto open = [&](int j, float sk_next, v16i (&S1)[2], const float (&last)[16]) {
        // Keys past N (ragged last column block) never receive probability mass: their raw logits become the
        // bit pattern of -inf, which as an integer loses every maximum and as a float sends the exponent's fma
        // (c > 0) to -inf, i.e. E = 0.  A wave-uniform branch, taken for that one column block only.
        if (j == tail_block) {
            const int nkeys = a.n_tokens - (a.kblocks - 1) * BLK, gg = lane_here() >> 5;
#pragma unroll
            for (int T = 0; T < 2; ++T)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (32 * T + 8 * (r >> 2) + 4 * gg + (r & 3) >= nkeys) {
                        S0[T][r] = (int)0xFF800000;
                        S1[T][r] = (int)0xFF800000;
                    }
        }
        int part[2][4] = {{0, 0, 0, 0}, {0, 0, 0, 0}};  // below every real value (those carry the accumulators' start)
#pragma unroll
        for (int T = 0; T < 2; ++T)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                part[0][r & 3] = max(part[0][r & 3], S0[T][r]);
                part[1][r & 3] = max(part[1][r & 3], S1[T][r]);
            }
        // ---- running maxima of both halves and the tile's quantization scale (one in-wave reduction), beside the sum and the
        // codes of the last quarter of the block before, which keep the wavefront busy through this chain of dependent steps
        const float c = sq_i * sk_next;
        float m_new[2];
        unsigned eb = 0xFF800000u;
#pragma unroll
        for (int H = 0; H < 2; ++H) {
            const float ymax = c * start_result(xor32_max(max(max(part[H][0], part[H][1]), max(part[H][2], part[H][3]))));
            m_new[H] = fmaxf(m[H], ymax);
            eb = min(eb, __float_as_uint(ymax - m_new[H]));  // a padded row has -inf here and loses the minimum
        }
        e = __uint_as_float(wave_umin(eb));
        close(last);
        if (__builtin_amdgcn_ballot_w64(m_new[0] - m_ref[0] > 64.0f || m_new[1] - m_ref[1] > 64.0f) != 0) {
#pragma unroll
            for (int H = 0; H < 2; ++H) {
                const float down = __builtin_amdgcn_exp2f(m_ref[H] - m_new[H]);  // first block: 2^-inf = 0 on zero sums
                l[H] *= down;
#pragma unroll
                for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[H][dt][r] *= down;
                m_ref[H] = m_new[H];
                if (H == 1) sv_eff1 *= down;  // of the product that is still to be added
            }
        }
        m[0] = m_new[0];
        m[1] = m_new[1];
    };
    float E[16] = {};  // exponentials of the tile at hand
    // one live block; S1 and N1: the raw logits of half 1, this block's and the next one's
    auto step = [&](auto mode_tag, int t, v16i (&S1)[2], v16i (&N1)[2]) {
        constexpr int MODE = decltype(mode_tag)::value;
        float c = sq_i * sk_cur;
        if (MODE == kExact && c < kLogitScaleMin) c = kLogitScaleMin;
        v16i o[2];
        const float sv_now = sv_cur * (PVBITS == 4 ? acc_down * 0.0625f : acc_down);
        float off_f[2], w_blk[2];
        const float c_up = c * 0x1p26f;
#pragma unroll
        for (int H = 0; H < 2; ++H) {
            const float off_n = (LOG2_QMAXP - kLog2_65535) - m[H] - e;
            off_f[H] = off_n;
            if constexpr (MODE == kFold) {
                float above;
                off_f[H] = folded_offset(off_n, c_up, above);
                w_blk[H] = __builtin_amdgcn_exp2f(((-kLog2_65535 - m_ref[H]) - off_n) - above);
            } else {
                w_blk[H] = __builtin_amdgcn_exp2f((-kLog2_65535 - m_ref[H]) - off_n);
            }
        }
        auto exponents = [&](const v16i& S, int H, float (&E)[16]) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if constexpr (MODE == kFold) E[r] = fmaf(__int_as_float(S[r]), c_up, off_f[H]);
                else if constexpr (MODE == kScaled) E[r] = fmaf(__int_as_float(S[r]) - kStartF, c_up, off_f[H]);
                else E[r] = fmaf(start_result(S[r]), c, off_f[H]);
            }
        };
        // a tile's exponentials, four behind each of four matrix instructions
        auto burst = [&](float (&E)[16], auto product) {
            end_basic_block();
            __builtin_amdgcn_s_setprio(3);
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                product(p);
                if (p == 0) end_basic_block();
#pragma unroll
                for (int r = 4 * p; r < 4 * p + 4; ++r) E[r] = __builtin_amdgcn_exp2f(E[r]);
                __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_s_setprio(0);
        };
        float sum[4];
        v4i pf0[2];
        exponents(S0[0], 0, E);
        burst(E, [&](int p) { pv(p, pf1, o); });  // P V of half 1 of the block before
        load_v(j0);
        j0 = j1;
        sk_cur = uniform_load(skp + j0);
        sv_cur = uniform_load(svp + j0);
        add16(E, sum, true);
        codes(E, pf0[0]);
        exponents(S0[1], 0, E);
        update(1, o, sv_eff1);
        widen_k();
        burst(E, [&](int p) { qk(p, 1, N1); });  // the next block's logits of half 1
        add16(E, sum, false);
        codes(E, pf0[1]);
        l[0] = fmaf((sum[0] + sum[1]) + (sum[2] + sum[3]), w_blk[0], l[0]);
        asm volatile("" : "+v"(l[0]));
        exponents(S1[0], 1, E);
        widen_v();
        burst(E, [&](int p) { pv(p, pf0, o); });  // P V of half 0
        add16(E, sum1, true);
        codes(E, pf1[0]);
        exponents(S1[1], 1, E);
        update(0, o, w_blk[0] * sv_now);
        burst(E, [&](int p) { qk(p, 0, S0); });  // the next block's logits of half 0
        j1 = column(t + 2);
        load_k(j1);
        w_blk1 = w_blk[1];
        sv_eff1 = w_blk[1] * sv_now;
        if (t + 1 < cnt) open(j0, sk_cur, N1, E);
    };
    auto visit_all = [&](auto mode_tag) {
        int t = 0;
        for (; t + 1 < cnt; t += 2) {  // one exit: a second one would cost waits for loads that only its path has in flight
            step(mode_tag, t, Sa, Sb);
            step(mode_tag, t + 1, Sb, Sa);
        }
        if (t < cnt) step(mode_tag, t, Sa, Sb);
    };
    if (cnt > 0) open(j0, sk_cur, Sa, E);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // nothing pending at the loop's entry: the compiler would wait for it in every pass
    if (fast) visit_all(std::integral_constant<int, FOLDABLE ? kFold : kScaled>{});
    else visit_all(std::integral_constant<int, kExact>{});
    if (cnt > 0) {
        v16i o[2];
        close(E);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            if (p < 2) end_basic_block();
            pv(p, pf1, o);
        }
        update(1, o, sv_eff1);
    }

#pragma unroll
    for (int H = 0; H < 2; ++H) {
        const int ln = lane_here();  // nothing that only these stores need is kept through the loop
        const int orow_no = i * BLK + 32 * H + (ln & 31);
        const bool valid = orow_no < a.n_tokens;
        const float l_tot = (l[H] + __shfl_xor(l[H], 32)) * 65535.0f;
        const float inv = (valid && l_tot > 0.0f) ? (0x1p26f / acc_down) / l_tot : 0.0f;
        const long long ooff = out_row_offset<D>(a, bh, h, head_rows, orow_no, valid);
        if (ooff >= 0) {
            OutT* orow = (OutT*)a.op + ooff + 4 * (ln >> 5);
#pragma unroll
            for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                for (int qd = 0; qd < 4; ++qd) {
                    float x[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) x[r] = valid ? acc[H][dt][4 * qd + r] * inv : 0.0f;
                    store4(orow + 32 * dt + 8 * qd, x[0], x[1], x[2], x[3]);
                }
        }
    }
    if constexpr (QKBITS == 8) { PARO_TIMELINE_STOP(item, lane, cnt) }
}

template <int PVBITS, typename OutT, int QSRC = 0>
__global__ __launch_bounds__(64, 2) void attn_i8_w64_kernel(AttnArgs a) {
    attn_i8_w64_body<8, PVBITS, OutT, QSRC>(a);
}

// the same wavefront program on 4-bit Q and K codes (Tab. 1, "QK (INT4)")
template <int PVBITS, typename OutT>
__global__ __launch_bounds__(64, 2) void attn_i8_w64_qk4_kernel(AttnArgs a) {
    attn_i8_w64_body<4, PVBITS, OutT, 0>(a);
}

// -------------------------------------------------------------------------------------------
// block 32: ONE wavefront per row block of 32 queries, no barrier.
//
// The same wavefront program as above with one half: the 16 exponentials of a lane stand in one burst at raised priority,
// and inside it run K Q of block t + 1 and P V of block t - 1 (at d = 64 one matrix instruction in front of every four
// exponentials; at d = 128 six of the eight fit, the others run beside the vector work).  K and V^T fragments go from global memory
// straight to registers, each requested as soon as the last product of its predecessor is issued; the chain from the row maxima
// to the tile's scale runs beside the codes of the block before.  Rows of 128 bytes of K are the exception: a lane pair reads 32 of a row, so
// every request would touch 32 lines and the next three the same ones, more than the L1 of a compute unit holds for its wavefronts; they
// go through LDS in whole lines.
// Bound by the issue of the vector work where the chip is full (184 vector instructions per block at d = 64, 256 at d = 128), by the
// chain of one block where it is not.  Attention call alone, us, before (tiles exchanged through LDS with a barrier per block) -> now,
// 8-bit codes / all 4-bit, 30 % density: d = 64, 30 heads of 17550 tokens 975 -> 827 / 956 -> 797, 24 heads of 4096 54.3 -> 45.3 /
// 56.3 -> 46.7, 4 heads of 4096 35.1 -> 26.1 / 36.7 -> 27.1; d = 128, 30 heads of 17550 1780 -> 1400 (K of 8-bit codes by registers took
// 1.2 times as long) / 1834 -> 1301, 4 heads of 4096 45.0 -> 32.4 / 48.3 -> 35.5.
//
// The exponent is formed after one exact subtraction per logit (the folded form of the kernel above is 2.5 % faster here and
// decides P codes within 6e-5 of a tie differently: error against binary64 3e-4 with it, 4e-5 without).
// -------------------------------------------------------------------------------------------

// A P V product enters the sums as the integer that it is: its chain starts at kStartI (see acc_start), one subtraction per element leaves
// the result times 2^-26, of which 2^13 come back in the weights and 2^13 at the end, whatever the scales: nothing is asked about them in
// front of a row.  (Left in the sums and taken out every few blocks the start would save the subtraction, 773 us instead of 833 for 30
// heads of 17550 tokens, d = 64; but it is as large as the largest result, times a weight that says nothing about a query's own codes, and a
// block of V some 2^12 larger than the rest, or one of zeros, whose scale is 1, pushes the digits of the others out of the sum: 5e-3 of the
// output at 2^12, all of it at 2^20.)
template <int D, int QKBITS, int PVBITS, typename OutT>
__global__ __launch_bounds__(64, (D == 64 ? 3 : 2)) void attn_i8_b32_kernel(AttnArgs a) {
    constexpr int BLK = 32;
    constexpr int KPACK = QKBITS == 4 ? 2 : 1;
    constexpr int VPACK = PVBITS == 4 ? 2 : 1;
    constexpr int KS = D / 32;  // contraction steps of QK^T
    constexpr int DT = D / 32;  // 32-channel tiles of the output
    constexpr float LOG2_QMAXP = PVBITS == 4 ? 2.807354922057604f : 6.988684686772166f;
    constexpr float kLog2_65535 = 15.999977986052736f;
    constexpr bool K_BY_LDS = D / KPACK == 128;
    constexpr float kClimb = 32.0f;  // octaves above its reference at which a row takes a new one (64 in the other kernels, whose weights carry less)
    __shared__ __attribute__((aligned(16))) uint8_t kslot[K_BY_LDS ? BLK * D : 16];

    const int wg = blockIdx.x;
    const int logical = (wg & 7) * a.per_xcd + (wg >> 3);
    if (logical >= a.total_wg) return;
    const int item = a.row_order ? min(max(a.row_order[logical], 0), a.total_wg - 1) : logical;
    const int bh = item / a.kblocks;
    const int i = item - bh * a.kblocks;
    const int h = bh % a.nh;
    const int lane = threadIdx.x;
    const int n = lane & 31;
    const int g = lane >> 5;

    const int* rp = a.row_ptr + (size_t)h * (a.kblocks + 1) + i;
    const int beg = __builtin_amdgcn_readfirstlane(min(max(rp[0], 0), a.nnz));
    const int end = __builtin_amdgcn_readfirstlane(min(max(rp[1], beg), a.nnz));
    const int cnt = end - beg;
    const int* cols = a.col_idx + beg;

    const size_t head_rows = (size_t)bh * a.kblocks * BLK;
    const uint8_t* kbase = a.k + head_rows * D / KPACK;
    const uint8_t* vbase = a.v + head_rows * D / VPACK;
    const unsigned klane = n * (D / KPACK) + 16 * g;            // this lane's K fragment of step 0, inside a block
    const unsigned vlane = n * (BLK / VPACK) + 16 / VPACK * g;  // its V^T fragment of channel tile 0
    const float* skp = a.sk + (size_t)bh * a.kblocks;
    const float* svp = a.sv + (size_t)bh * a.kblocks;
    float sq_i = a.sq[(size_t)bh * a.kblocks + i] * (QKBITS == 4 ? a.qk_scale * (1.0f / 256.0f) : a.qk_scale);  // 4-bit codes enter times 16
    sq_i = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(sq_i)));
    const int row = i * BLK + n;
    const bool row_valid = row < a.n_tokens;
    v4i qf[KS];
    if constexpr (QKBITS == 4) {
        const uint8_t* qrow = a.q + (head_rows + row) * (D / 2) + 16 * g;
#pragma unroll
        for (int s = 0; s < KS; s += 2) unpack_nibbles(*(const v4i*)(qrow + 16 * s), qf[s], qf[s + 1]);
    } else {
        const uint8_t* qrow = a.q + (head_rows + row) * D + 16 * g;
#pragma unroll
        for (int s = 0; s < KS; ++s) qf[s] = *(const v4i*)(qrow + 32 * s);
    }

    v4i kf[KS], kraw[KS / 2];  // K fragments of the next block; 4-bit: 32 channels each, widened in front of the products
    v4i vf[DT];                // V^T fragments [channel tile]
    v2u vraw[DT];              // 4-bit V: a lane's 16 slots of a channel
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
        vf[dt] = v4i{0, 0, 0, 0};
        vraw[dt] = v2u{0, 0};
    }
    // lane L of a request fills bytes 16 L of a 1 KB piece: position L % 8 of line L / 8, which holds the line's piece (L % 8) ^ (L / 8)
    const unsigned kfill = 128u * (lane >> 3) + 16u * ((lane & 7) ^ (lane >> 3));
    auto load_k = [&](int j) {
        if constexpr (K_BY_LDS) {
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): what the slot held has been read
            const uint8_t* kp = kbase + (size_t)j * (BLK * D);
            lds_dma16<0>(kp, kfill, kslot);
            lds_dma16<1024>(kp, kfill, kslot);
            lds_dma16<2048>(kp, kfill, kslot);
            lds_dma16<3072>(kp, kfill, kslot);
            return;
        }
        global_bytes kp = (global_bytes)kbase + (size_t)j * (BLK * D / KPACK);
        unsigned off = klane;
        asm volatile("" : "+s"(kp), "+v"(off));  // scalar base + lane offset, not a 64-bit address per lane
#pragma unroll
        for (int s = 0; s < KS / KPACK; ++s) {
            if constexpr (QKBITS == 4) kraw[s] = *(const global_v4i*)(kp + off + 32 * s);
            else kf[s] = *(const global_v4i*)(kp + off + 32 * s);
        }
    };
    auto widen_k = [&]() {  // what was requested, as operands
        if constexpr (K_BY_LDS) {
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
#pragma unroll
            for (int s = 0; s < KS; ++s) kf[s] = *(const v4i*)(kslot + 128 * n + 16 * ((2 * s + g) ^ (n & 7)));
        }
        if constexpr (QKBITS == 4) {
#pragma unroll
            for (int s = 0; s < KS; s += 2) unpack_nibbles(kraw[s / 2], kf[s], kf[s + 1]);
        }
    };
    auto load_v = [&](int j) {
        global_bytes vp = (global_bytes)vbase + (size_t)j * (BLK * D / VPACK);
        unsigned off = vlane;
        asm volatile("" : "+s"(vp), "+v"(off));
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            if constexpr (PVBITS == 4) vraw[dt] = *(const global_v2u*)(vp + off + 32 * dt * (BLK / 2));
            else vf[dt] = *(const global_v4i*)(vp + off + 32 * dt * BLK);
        }
    };
    auto widen_v = [&]() {  // codes times 16, undone in the scale; the PARO_VT nibble order makes the bytes come out in slot order
        if constexpr (PVBITS == 4) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
                vf[dt] = v4i{(int)((vraw[dt].x << 4) & 0xF0F0F0F0u), (int)(vraw[dt].x & 0xF0F0F0F0u),
                             (int)((vraw[dt].y << 4) & 0xF0F0F0F0u), (int)(vraw[dt].y & 0xF0F0F0F0u)};
        }
    };

    // 64 column indices per fetch, one per lane; past the end of the row its last column again
    auto load_cols = [&](int chunk) { return min(max(cols[min(chunk * 64 + lane_here(), cnt - 1)], 0), a.kblocks - 1); };
    int cols64 = cnt > 0 ? load_cols(0) : 0;
    auto column = [&](int u) {  // u advances by one per call
        if ((u & 63) == 0) cols64 = load_cols(u >> 6);
        return __builtin_amdgcn_readlane(cols64, u & 63);
    };

    float sk_cur = 0.0f, sv_cur = 0.0f;
    int j0 = 0, j1 = 0;
    if (cnt > 0) {
        j0 = __builtin_amdgcn_readlane(cols64, 0);
        j1 = column(1);
        load_k(j0);
        sk_cur = uniform_load(skp + j0);
        sv_cur = uniform_load(svp + j0);
    }

    // a padded row holds +inf, as above
    float m = row_valid ? -INFINITY : INFINITY, m_ref = m, l = 0.0f;
    float acc[DT][16];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[dt][r] = 0.0f;

    const int tail_block = (a.n_tokens % BLK) != 0 ? a.kblocks - 1 : -1;
    v16i start = acc_start();  // of the P V products: several in a basic block
    asm volatile("" : "+v"(start));

    v16i Sa, Sb;  // raw logits, this block's and the next one's in turn
    v4i pf = {0, 0, 0, 0};
    float weight = 0.0f;  // of the product that is still to be added
    auto qk = [&](int s, v16i& S) { S = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf[s], qf[s], s == 0 ? acc_start() : S, 0, 0, 0); };

    float e = 0.0f;
    // row maxima and the tile's scale of a block, from its raw logits; `beside` is what keeps the wavefront busy meanwhile
    auto open = [&](int j, float sk_next, v16i& S, auto beside) __attribute__((always_inline)) {
        if (j == tail_block) {  // keys past N, as in the kernel above
            const int real = a.n_tokens - (a.kblocks - 1) * BLK - 4 * (lane_here() >> 5);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                S[r] = 8 * (r >> 2) + (r & 3) >= real ? (int)0xFF800000 : S[r];
                asm volatile("" : "+v"(S[r]));
            }
        }
        int part[4] = {0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 16; ++r) part[r & 3] = max(part[r & 3], S[r]);
        const float c = sq_i * sk_next;
        const float ymax = c * start_result(xor32_max(max(max(part[0], part[1]), max(part[2], part[3]))));
        const float m_new = fmaxf(m, ymax);
        const unsigned eb = wave_umin(min(0xFF800000u, __float_as_uint(ymax - m_new)));  // a padded row has -inf here
        beside();
        e = __uint_as_float(eb);
        if (__builtin_amdgcn_ballot_w64(m_new - m_ref > kClimb) != 0) {
            const float down = __builtin_amdgcn_exp2f(m_ref - m_new);  // first block: 2^-inf = 0 on zero sums
            l *= down;
            weight *= down;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[dt][r] *= down;
            m_ref = m_new;
        }
        m = m_new;
    };
    // block t, whose logits are in S; N: the next one's, unless it is the last
    auto step = [&](auto last_tag, int t, v16i& S, v16i& N) __attribute__((always_inline)) {
        constexpr bool LAST = decltype(last_tag)::value;
        // at least kLogitScaleMin where the ragged block's masked keys need it (it changes no other exponent), and 0 stays 0 under any scale
        const float c_up = __builtin_amdgcn_fmed3f(sq_i * sk_cur * 0x1p26f, kLogitScaleMin * 0x1p26f, 3.402823466e+38f);
        const float off_n = (LOG2_QMAXP - kLog2_65535) - m - e;
        const float w_blk = __builtin_amdgcn_exp2f((-kLog2_65535 - m_ref) - off_n) * 0x1p13f;
        float E[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) E[r] = fmaf(__int_as_float(S[r]) - kStartF, c_up, off_n);
        int j2 = j1;
        if constexpr (!LAST) {
            widen_k();
            j2 = column(t + 2);
        }
        widen_v();
        auto add = [&](int dt, const v16i& o) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc[dt][r] = fmaf(__int_as_float(o[r]) - kStartF, weight, acc[dt][r]);
                asm volatile("" : "+v"(acc[dt][r]));
            }
        };
        v16i o[DT];
        end_basic_block();
        __builtin_amdgcn_s_setprio(3);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            if constexpr (LAST) {
                if (p < 2) o[p] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf[p], pf, start, 0, 0, 0);
            } else if constexpr (D == 64) {
                if (p < 2) qk(p, N);
                else o[p - 2] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf[p - 2], pf, start, 0, 0, 0);
            } else {
                qk(p, N);
                if (p & 1) o[p >> 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf[p >> 1], pf, start, 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 4 * p; r < 4 * p + 4; ++r) E[r] = __builtin_amdgcn_exp2f(E[r]);
            __builtin_amdgcn_sched_barrier(0);
            if (!LAST && p == D / 32 - 1) load_k(j2);
        }
        __builtin_amdgcn_s_setprio(0);
        float sum[4];
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[r & 3] = r < 4 ? E[r] : sum[r & 3] + E[r];
        asm volatile("" : "+v"(sum[0]), "+v"(sum[1]), "+v"(sum[2]), "+v"(sum[3]));
        add(0, o[0]);
        add(1, o[1]);
        if constexpr (D == 128) {
#pragma unroll
            for (int dt = 2; dt < DT; ++dt) o[dt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf[dt], pf, start, 0, 0, 0);
        }
        load_v(j0);
        const float sv_now = sv_cur * (PVBITS == 4 ? 0.0625f : 1.0f);
        auto rest = [&]() __attribute__((always_inline)) {
            if constexpr (D == 128) {
                add(2, o[2]);
                add(3, o[3]);
            }
#pragma unroll
            for (int r = 0; r < 16; r += 4) {
                const unsigned lo = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pknorm_u16(E[r], E[r + 1]));
                const unsigned hi = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pknorm_u16(E[r + 2], E[r + 3]));
                pf[r >> 2] = (int)__builtin_amdgcn_perm(hi, lo, 0x06040200u);
            }
            asm volatile("" : "+v"(pf));
            l = fmaf((sum[0] + sum[1]) + (sum[2] + sum[3]), w_blk, l);
            weight = w_blk * sv_now;
        };
        if constexpr (LAST) {
            rest();
        } else {
            j0 = j1;
            sk_cur = uniform_load(skp + j0);
            sv_cur = uniform_load(svp + j0);
            j1 = j2;
            open(j0, sk_cur, N, rest);
        }
    };
    if (cnt > 0) {
        widen_k();
#pragma unroll
        for (int s = 0; s < KS; ++s) qk(s, Sa);
        load_k(j1);
        open(j0, sk_cur, Sa, [] {});
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // nothing pending at the loop's entry: the compiler would wait for it in every pass
    // The last block stands apart, without a product behind it.  One loop, and no look at the row's scales in front of it, where a loop for each of
    // two ranges of them and a scan stood: a launch of short rows is mostly instructions that are fetched once.  Attention alone, 8-bit Q and K
    // with 4-bit P and V, us, (tiles exchanged through LDS with a barrier per block) / scan and two loops -> now: 85 heads of 96 tokens, d = 64
    // 4.3 / 4.7 -> 4.3, d = 128 5.1 / 5.7 -> 5.2; 128 heads of 256 at 50 % 7.2 / 7.3 -> 6.7; 128 heads of 96 in 32 batches 26.0 / 28.4 -> 27.0; long rows
    // 0 to 3 % slower, 4 heads of 4096 8-bit 25.5 -> 26.0, 30 heads of 17550 817 -> 819.  (V in two sets of registers, and it, the scales and two blocks
    // of K requested together in front of a row: no difference, d = 128 5 % slower.)
    {
        const std::false_type inner;
        int t = 0;
        for (; t + 2 < cnt; t += 2) {
            step(inner, t, Sa, Sb);
            step(inner, t + 1, Sb, Sa);
        }
        if (t + 1 < cnt) {
            step(inner, t, Sa, Sb);
            Sa = Sb;
        }
        if (cnt > 0) step(std::true_type(), cnt - 1, Sa, Sb);
    }
    if (cnt > 0) {  // the last block's P V, one tile at a time
        widen_v();
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            const v16i o = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf[dt], pf, start, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[dt][r] = fmaf(__int_as_float(o[r]) - kStartF, weight, acc[dt][r]);
        }
    }

    const int ln = lane_here();
    const int orow_no = i * BLK + (ln & 31);
    const bool valid = orow_no < a.n_tokens;
    const float l_tot = (l + __shfl_xor(l, 32)) * 65535.0f;
    const float inv = (valid && l_tot > 0.0f) ? 0x1p26f / l_tot : 0.0f;
    const long long ooff = out_row_offset<D>(a, bh, h, head_rows, orow_no, valid);
    if (ooff >= 0) {
        OutT* orow = (OutT*)a.op + ooff + 4 * (ln >> 5);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                float x[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) x[r] = valid ? acc[dt][4 * qd + r] * inv : 0.0f;
                store4(orow + 32 * dt + 8 * qd, x[0], x[1], x[2], x[3]);
            }
    }
}

// -------------------------------------------------------------------------------------------
// block 64, d = 128, and d = 64 where the row blocks are few: FOUR wavefronts per row block, 16 queries each, on
// v_mfma_i32_16x16x64_i8.
//
// Why 16 queries.  At d = 128 a wavefront of 32 carries 64 accumulator registers and needs some 200: two wavefronts per SIMD.  With 16
// it needs 128 or fewer - four per SIMD, four workgroups per compute unit - and a block is a quarter of the instructions per wavefront, which
// is what counts where a row's chain of blocks bounds the launch: rows of text (Sec. 4.2 (1)) that attend every column block, and
// launches with fewer row blocks than the chip has room for.
//
// Order of things.  Between two barriers a wavefront exponentiates block t and multiplies K Q of block t + 1: its four matrix
// instructions per two key tiles run beside the exponentials of two tiles of block t (at raised priority), and the chain from the
// maxima of block t + 1 to this wavefront's share of its tile exponent, four numbers that meet in LDS across the barrier, runs beside
// the sum, the codes, P V and the accumulator update of block t.  192 vector instructions per wavefront and block at d = 128 (207 with
// products, maxima and exponentials of one block in turn), 152 at d = 64.  What bounds it: issue where the chip is full (the matrix
// time is added where it is not beside an exponential), the chain of one block, some 1 100 (d = 64) to 1 500 cycles, where it is not.
// Exponentials in whole bursts with one matrix instruction per two of them: 1 % slower, registers.
//
// Layouts.  S^T tile T (16 keys x 16 queries): lane (n = lane % 16, G = lane / 16) holds query n, keys
// 4 G + r (r = 0..3) of the tile.  Which key sits in which row of a tile is free - K rows are fetched from
// LDS by address - and is chosen so that the four codes of a lane's tile T land, packed into register T
// of the B operand, on the contraction slots 16 G + 4 T + r that lane group G of the PV instruction
// covers: row 4 G + r of tile T is the key whose PARO_VT slot is 16 G + 4 T + r, i.e. token
// 32 (G >> 1) + 8 T + 4 (G & 1) + r of the block.  V^T fragments are then plain 16-byte reads of PARO_VT rows.
//
// Tiles.  K_j and V_j^T of 8-bit codes go to LDS as they are with global_load_lds_dwordx4, each wavefront moving a quarter, 4-bit codes by
// way of registers in which they are widened once for all four wavefronts.  Inside every 128-byte line the eight 16-byte pieces are
// stored at position (piece ^ line % 8): the reads of 16 lanes that walk down a column of pieces then spread over all banks.  Two K
// slots and two V slots, arrays of their own in a loop unrolled by two: with one array the compiler makes every read wait for all
// requests before it.  ONE barrier per block, after the wavefront has waited for its own requests: behind it K_{t+2} may overwrite
// K_t and V_{t+1} V_{t-1}, and they have the whole block to land.
//
// Attention call alone, us, before -> now, 30 % density, 8-bit codes / 8-bit Q K with 4-bit P V / all 4-bit.  d = 128 (before: the same split without
// the overlap for 8-bit codes, two wavefronts of 32 queries otherwise): 30 heads of 17550 tokens 1146 -> 1103 / 1264 -> 1118 / 1279 -> 1083,
// 24 heads of 4096 59.4 -> 57.9 / 76.7 -> 59.2 / 77.4 -> 58.9, 4 heads of 4096 23.0 -> 19.3 / 33.8 -> 22.0 / 35.0 -> 22.7, 24 heads of
// 4096 image and 512 text tokens 105 -> 101 / 119 -> 103 / 119 -> 104.  d = 64 (before: one wavefront of 64 queries): 24 heads of 4096
// 42.0 -> 39.7 / 45.6 -> 41.9 / 47.4 -> 42.9, 4 heads of 4096 29.5 -> 15.3 / 32.3 -> 16.1 / 32.9 -> 17.1.
// -------------------------------------------------------------------------------------------
typedef int v4acc __attribute__((ext_vector_type(4)));

// max over the four lanes n, n + 16, n + 32, n + 48 (the lanes that share a query), returned in all four
__device__ inline int quad_rows_max(int x) {
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    return xor32_max(max((int)r[0], (int)r[1]));
}
__device__ inline float quad_rows_sum(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(x), false, false);
    const float y = __int_as_float((int)r[0]) + __int_as_float((int)r[1]);
    const auto z = __builtin_amdgcn_permlane32_swap(__float_as_int(y), __float_as_int(y), false, false);
    return __int_as_float((int)z[0]) + __int_as_float((int)z[1]);
}

template <int D, int QKBITS, int PVBITS, typename OutT, int QSRC = 0>
__global__ __launch_bounds__(256, (QSRC != 0 ? 3 : 4)) void attn_i8_q16_kernel(AttnArgs a) {
    static_assert(QSRC == 0 || QKBITS == 8, "in-kernel quantization of Q produces 8-bit codes");
    constexpr int BLK = 64;
    constexpr int KPACK = QKBITS == 4 ? 2 : 1;
    constexpr int VPACK = PVBITS == 4 ? 2 : 1;
    constexpr int KS = D / 64;        // contraction steps of QK^T (64 channels each)
    constexpr int CT = D / 16;        // 16-channel tiles of the output
    constexpr int TILE = BLK * D;     // bytes of a K and of a V^T tile in LDS
    constexpr float LOG2_QMAXP = PVBITS == 4 ? 2.807354922057604f : 6.988684686772166f;
    constexpr float kLog2_65535 = 15.999977986052736f;
    __shared__ __attribute__((aligned(16))) uint8_t kring0[TILE];
    __shared__ __attribute__((aligned(16))) uint8_t kring1[TILE];
    __shared__ __attribute__((aligned(16))) uint8_t vring0[TILE];
    __shared__ __attribute__((aligned(16))) uint8_t vring1[TILE];
    __shared__ __attribute__((aligned(16))) unsigned tile_e[2][4];

    const int wg = blockIdx.x;
    const int logical = (wg & 7) * a.per_xcd + (wg >> 3);
    if (logical >= a.total_wg) return;
    const int item = a.row_order ? min(max(a.row_order[logical], 0), a.total_wg - 1) : logical;
    const int bh = item / a.kblocks;
    const int i = item - bh * a.kblocks;
    const int h = bh % a.nh;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15;
    const int G = lane >> 4;
    PARO_TIMELINE_BEGIN(QKBITS == 8 && PVBITS == 8)

    const int* rp = a.row_ptr + (size_t)h * (a.kblocks + 1) + i;
    const int beg = __builtin_amdgcn_readfirstlane(min(max(rp[0], 0), a.nnz));
    const int end = __builtin_amdgcn_readfirstlane(min(max(rp[1], beg), a.nnz));
    const int cnt = end - beg;
    const int* cols = a.col_idx + beg;

    const size_t head_rows = (size_t)bh * a.kblocks * BLK;
    const uint8_t* kbase = a.k + head_rows * D / KPACK;
    const uint8_t* vbase = a.v + head_rows * D / VPACK;
    const float* skp = a.sk + (size_t)bh * a.kblocks;
    const float sk_last = uniform_load(skp + a.kblocks - 1);  // asked for here, used below
    const float* svp = a.sv + (size_t)bh * a.kblocks;
    const int row = i * BLK + 16 * w + n;  // this lane's query, in the reordered sequence
    const bool row_valid = row < a.n_tokens;

    // ---- tiles to LDS, as 128-byte lines of eight 16-byte pieces (one K row at d = 128, two rows otherwise); piece p of line x sits at
    // position p ^ (x % 8).  8-bit codes are requested straight into LDS, 1 KB a request, lane L filling bytes 16 L: position L % 8 of
    // a line L / 8.  4-bit codes come in registers, a whole block earlier, and are widened on the way (codes times 16, undone in the scale).
    const unsigned fill = 128u * (lane >> 3) + 16u * ((lane & 7) ^ (lane >> 3));
    auto request = [&](const uint8_t* tile, uint8_t* slot) __attribute__((always_inline)) {
        constexpr int EACH = TILE / 4;
        const uint8_t* from = tile + EACH * w;
        unsigned off = fill;
        asm volatile("" : "+s"(from), "+v"(off));  // scalar base + lane offset, not a 64-bit address per lane
        lds_dma16<0>(from, off, slot + EACH * w);
        if constexpr (EACH == 2048) lds_dma16<1024>(from, off, slot + EACH * w);
    };
    using Packed = std::conditional_t<D == 128, v4i, v2u>;  // a thread's share of a tile of 4-bit codes
    const int tid = threadIdx.x;
    Packed kreg{}, vreg{};
    auto place = [](int line, int piece) { return 128u * line + 16u * (piece ^ (line & 7)); };
    auto widen = [&](const Packed& x, uint8_t* slot, unsigned at, unsigned apart) __attribute__((always_inline)) {
        v4i first, second;
        if constexpr (D == 128) {
            unpack_nibbles(x, first, second);
            *(v4i*)(slot + at) = first;
            *(v4i*)(slot + (at ^ apart)) = second;
        } else {
            unpack_nibbles(v4i{(int)x.x, (int)x.y, 0, 0}, first, second);
            *(v4i*)(slot + at) = first;
        }
    };
    // K: a quarter of row tid / 4, 32 channels as pieces p and 4 + p of 16 (Q is split the same way) or 16 channels as one piece;
    // V^T: half of row tid / 2, 32 slots as two pieces, or a quarter of row tid / 4, one piece
    const unsigned kat = D == 128 ? place(tid >> 2, tid & 3) : place(tid >> 3, tid & 7);
    const unsigned vat = D == 128 ? place(tid >> 2, 2 * (tid & 3)) : place(tid >> 3, tid & 7);
    auto fetch = [&](const uint8_t* tile, Packed& x) __attribute__((always_inline)) {
        global_bytes from = (global_bytes)tile;
        unsigned off = sizeof(Packed) * (64u * w + lane_here());
        asm volatile("" : "+s"(from), "+v"(off));
        x = *(const __attribute__((address_space(1))) Packed*)(from + off);
    };
    auto fetch_k = [&](int j) __attribute__((always_inline)) { fetch(kbase + (size_t)j * (TILE / 2), kreg); };
    auto fetch_v = [&](int j) __attribute__((always_inline)) { fetch(vbase + (size_t)j * (TILE / 2), vreg); };
    // the next tile into a free slot: requested (8-bit, block j) or written from the registers, which then fetch block j_after
    auto bring_k = [&](int j, int j_after, uint8_t* slot) __attribute__((always_inline)) {
        if constexpr (QKBITS == 8) request(kbase + (size_t)j * TILE, slot);
        else {
            widen(kreg, slot, kat, 64);
            fetch_k(j_after);
        }
    };
    auto bring_v = [&](int j, int j_after, uint8_t* slot) __attribute__((always_inline)) {
        if constexpr (PVBITS == 8) request(vbase + (size_t)j * TILE, slot);
        else {
            widen(vreg, slot, vat, 16);
            fetch_v(j_after);
        }
    };

    // 64 column indices per fetch, one per lane; past the end of the row its last column again
    auto load_cols = [&](int chunk) { return min(max(cols[min(chunk * 64 + lane_here(), cnt - 1)], 0), a.kblocks - 1); };
    int cols64 = cnt > 0 ? load_cols(0) : 0;
    auto column = [&](int u) {  // u advances by one per call
        if ((u & 63) == 0) cols64 = load_cols(u >> 6);
        return __builtin_amdgcn_readlane(cols64, u & 63);
    };
    int j0 = 0, j1 = 0, j2 = 0;  // columns of the first block and of blocks t + 1 and t + 2
    float sk0 = 0.0f, sv0 = 0.0f, sk1 = 0.0f, sv1 = 0.0f;  // their scales
    const int first_cols = cols64;
    if (cnt > 0) {
        j0 = __builtin_amdgcn_readlane(cols64, 0);
        j1 = column(1);
        j2 = column(2);
        if constexpr (QKBITS == 4) fetch_k(j0);
        if constexpr (PVBITS == 4) fetch_v(j0);
        bring_k(j0, j1, kring0);
        bring_v(j0, j1, vring0);
        if (cnt > 1) bring_k(j1, j2, kring1);
        sk0 = uniform_load(skp + j0);
        sv0 = uniform_load(svp + j0);
        sk1 = uniform_load(skp + j1);
        sv1 = uniform_load(svp + j1);
    }

    // ---- Q
    v4i qf[KS];
    float sq_i = 0.0f;
    if constexpr (QSRC == 0) {
        sq_i = a.sq[(size_t)bh * a.kblocks + i] * (QKBITS == 4 ? a.qk_scale * (1.0f / 256.0f) : a.qk_scale);  // 4-bit codes enter times 16
        const uint8_t* qrow = a.q + (head_rows + row) * (D / KPACK);
        if constexpr (QKBITS == 8) {
#pragma unroll
            for (int s = 0; s < KS; ++s) qf[s] = *(const v4i*)(qrow + 64 * s + 16 * G);
        } else if constexpr (KS == 2) {
            unpack_nibbles(*(const v4i*)(qrow + 16 * G), qf[0], qf[1]);
        } else {
            v4i unused;
            const v2u x = *(const v2u*)(qrow + 8 * G);
            unpack_nibbles(v4i{(int)x.x, (int)x.y, 0, 0}, qf[0], unused);
        }
    } else {
        // same arithmetic as the quantizer: absmax over the real rows of the block, scale = absmax / 127 in binary32,
        // code = rint(fl32(x / scale))
        using RawT = std::conditional_t<QSRC == 1, uint16_t, float>;
        __shared__ float q_amax[4];
        const RawT* qsrc = (const RawT*)a.q + ((size_t)bh * a.n_tokens + (row_valid ? reorder_source(a.table, h, row) : 0)) * D + 16 * G;
        float x[KS][16];
        float amax = 0.0f;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if (row_valid) {
                if constexpr (QSRC == 1) {
                    const uint4 lo = *(const uint4*)(qsrc + 64 * s), hi = *(const uint4*)(qsrc + 64 * s + 8);
                    const unsigned wv[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        x[s][2 * e] = __uint_as_float(wv[e] << 16);
                        x[s][2 * e + 1] = __uint_as_float(wv[e] & 0xffff0000u);
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float4 f = *(const float4*)(qsrc + 64 * s + 4 * e);
                        x[s][4 * e] = f.x;
                        x[s][4 * e + 1] = f.y;
                        x[s][4 * e + 2] = f.z;
                        x[s][4 * e + 3] = f.w;
                    }
                }
            } else {
#pragma unroll
                for (int e = 0; e < 16; ++e) x[s][e] = 0.0f;
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) amax = fmaxf(amax, fabsf(x[s][e]));
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
        if (lane == 0) q_amax[w] = amax;
        __syncthreads();
        amax = fmaxf(fmaxf(q_amax[0], q_amax[1]), fmaxf(q_amax[2], q_amax[3]));
        const float scale = amax > 0.0f ? amax / 127.0f : 1.0f;
        const GroupDivider quotient(scale);
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
                unsigned word = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float r = fminf(fmaxf(rintf(quotient(x[s][4 * e4 + e])), -127.0f), 127.0f);
                    word |= ((unsigned)(int)r & 0xffu) << (8 * e);
                }
                qf[s][e4] = (int)word;
            }
        sq_i = scale * a.qk_scale;
    }
    sq_i = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(sq_i)));

    // ---- which of the loops the row block's scales allow (as in the kernels above)
    constexpr bool FOLDABLE = PARO_FOLD_LOGIT_BIAS && PVBITS == 8;
    bool fast = false;
    float sv_up = 0x1p26f;  // what a V scale is multiplied by to give a weight, as in the kernel above
    {
        float sk_max = 0.0f, sv_max = 0.0f;
        for (int base = 0; base < cnt; base += 64)
            if (base + lane < cnt) {
                const int j = base == 0 ? first_cols : min(max(cols[base + lane], 0), a.kblocks - 1);
                sk_max = fmaxf(sk_max, skp[j]);
                sv_max = fmaxf(sv_max, svp[j]);
            }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) sk_max = fmaxf(sk_max, __shfl_xor(sk_max, off));
        fast = FOLDABLE ? sq_i * sk_max * kFoldBound < 8192.0f : sq_i * sk_max < 0x1p90f;
        if (__builtin_amdgcn_ballot_w64(sv_max > 0x1p40f) != 0) sv_up = 1.0f;
    }
    const int tail_block = (a.n_tokens % BLK) != 0 ? a.kblocks - 1 : -1;  // the column block with padded keys, if any
    if (tail_block >= 0 && sq_i * sk_last < kLogitScaleMin) fast = false;
    v4acc start;  // of every chain of products: four registers
#pragma unroll
    for (int r = 0; r < 4; ++r) start[r] = 0x3E22F983;
    asm volatile("" : "+v"(start));

    // ---- fragments.  K, tile T: row 32 (n >> 3) + 8 T + (n & 7) of the block; V^T, channel tile ct: row 16 ct + n
    unsigned kread[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        // d = 128: contraction step x.  d = 64: even and odd tiles, which sit four lines further on
        if constexpr (D == 128) kread[x] = 128u * (32 * (n >> 3) + (n & 7)) + 16u * ((4 * x + G) ^ (n & 7));
        else kread[x] = 128u * (16 * (n >> 3) + ((n & 7) >> 1)) + 16u * ((4 * (n & 1) + G) ^ ((n & 7) >> 1) ^ (4 * x));
    }
    const unsigned vread = 128u * (n >> 1) + 16u * ((4 * (n & 1) + G) ^ (n >> 1));
    auto k_fragment = [&](const uint8_t* slot, int T, int s) __attribute__((always_inline)) {
        return D == 128 ? *(const v4i*)(slot + 1024 * T + kread[s]) : *(const v4i*)(slot + 512 * T + kread[T & 1]);
    };
    auto logits = [&](const uint8_t* slot, v4acc (&S)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int T = 0; T < 4; ++T) {
#pragma unroll
            for (int s = 0; s < KS; ++s) S[T] = __builtin_amdgcn_mfma_i32_16x16x64_i8(k_fragment(slot, T, s), qf[s], s == 0 ? start : S[T], 0, 0, 0);
        }
    };

    float m = row_valid ? -INFINITY : INFINITY, m_ref = m, l = 0.0f;  // a padded row holds +inf, as above
    float acc[CT][4];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[ct][r] = 0.0f;

    auto mask_tail = [&](int j, v4acc (&S)[4]) __attribute__((always_inline)) {
        if (j == tail_block) {  // keys past N: the bit pattern of -inf loses every maximum and gives E = 0 (c > 0)
            const int GG = lane_here() >> 4;
            const int real = a.n_tokens - (a.kblocks - 1) * BLK - 32 * (GG >> 1) - 4 * (GG & 1);
#pragma unroll
            for (int T = 0; T < 4; ++T)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    S[T][r] = 8 * T + r >= real ? (int)0xFF800000 : S[T][r];
                    asm volatile("" : "+v"(S[T][r]));
                }
        }
    };
    // new running maximum from a block's raw logits, and this wavefront's share of the tile's quantization scale
    auto maxima = [&](const v4acc (&S)[4], float c, unsigned& eb) __attribute__((always_inline)) {
        int part[4] = {0, 0, 0, 0};  // below every real value (those carry the accumulators' start)
#pragma unroll
        for (int T = 0; T < 4; ++T)
#pragma unroll
            for (int r = 0; r < 4; ++r) part[r] = max(part[r], S[T][r]);
        const float ymax = c * start_result(quad_rows_max(max(max(part[0], part[1]), max(part[2], part[3]))));
        const float m_new = fmaxf(m, ymax);
        eb = __float_as_uint(ymax - m_new);              // a padded row has -inf here and loses the minimum
        eb = min(eb, (unsigned)dpp_mov<0xB1>((int)eb));  // the four rows of 16 lanes hold the same 16 queries:
        eb = min(eb, (unsigned)dpp_mov<0x4E>((int)eb));  // one row is reduced
        eb = min(eb, (unsigned)dpp_mov<0x141>((int)eb));
        eb = min(eb, (unsigned)dpp_mov<0x140>((int)eb));
        return m_new;
    };
    auto refer = [&](float m_new) __attribute__((always_inline)) {  // keeps the stored sums far from overflow; takes the maximum over
        if (__builtin_amdgcn_ballot_w64(m_new - m_ref > 64.0f) != 0) {
            const float down = __builtin_amdgcn_exp2f(m_ref - m_new);  // first block: 2^-inf = 0 on zero sums
            l *= down;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[ct][r] *= down;
            m_ref = m_new;
        }
        m = m_new;
    };
    v4acc Sa[4], Sb[4];  // raw logits, this block's and the next one's in turn
    // block t, whose logits are in S and whose tile exponents are in tile_e; K_{t+1} is in k_next and V_t in v_now.  parity: that of t, or kLast
    // in the last block, which brings no tile and multiplies for no block behind it: a third of the work of a row of one block, d = 128, 85 heads of
    // 192 tokens 6.7 -> 6.4 us (6.5 in the kernel before), 128 heads of 192 in 16 batches at 50 % 57.5 -> 54.4 (54.4), 24 heads of 4096 and 512 102.3 -> 100.5
    constexpr int kLast = 2;
    auto step = [&](auto mode_tag, auto parity_tag, int t, v4acc (&S)[4], v4acc (&N)[4]) __attribute__((always_inline)) {
        constexpr int MODE = decltype(mode_tag)::value;
        constexpr bool LAST = decltype(parity_tag)::value == kLast;
        const int PARITY = LAST ? t & 1 : decltype(parity_tag)::value;
        uint8_t* const k_next = PARITY ? kring0 : kring1;  // K_{t+1}
        uint8_t* const k_free = PARITY ? kring1 : kring0;  // held K_t
        uint8_t* const v_now = PARITY ? vring1 : vring0;   // V_t
        uint8_t* const v_free = PARITY ? vring0 : vring1;  // held V_{t-1}
        const uint4 eq = *(const uint4*)tile_e[PARITY];
        v4i kf[2][KS];
        auto read_k = [&](int T0) __attribute__((always_inline)) {
#pragma unroll
            for (int T = 0; T < 2; ++T)
#pragma unroll
                for (int s = 0; s < KS; ++s) kf[T][s] = k_fragment(k_next, T0 + T, s);
        };
        auto products_k = [&](int T0) __attribute__((always_inline)) {
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int T = 0; T < 2; ++T) N[T0 + T] = __builtin_amdgcn_mfma_i32_16x16x64_i8(kf[T][s], qf[s], s == 0 ? start : N[T0 + T], 0, 0, 0);
        };
        v4i vf[4];
        auto read_v = [&](int ct0) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < 4; ++x) vf[x] = *(const v4i*)(v_now + 1024 * (ct0 + x) + vread);
        };
        int j3 = j2;
        if constexpr (!LAST) {
            read_k(0);
            j3 = column(t + 3);
            bring_k(j2, j3, k_free);
            bring_v(j1, j2, v_free);
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(3);
        if constexpr (!LAST) {
            products_k(0);
            read_k(2);
        }
        const float e = __uint_as_float(min(min(eq.x, eq.y), min(eq.z, eq.w)));
        float c = sq_i * sk0;
        if (MODE == kExact && c < kLogitScaleMin) c = kLogitScaleMin;
        const float c_up = c * 0x1p26f;
        const float off_n = (LOG2_QMAXP - kLog2_65535) - m - e;
        float off_f = off_n, w_blk;
        if constexpr (MODE == kFold) {
            float above;
            off_f = folded_offset(off_n, c_up, above);
            w_blk = __builtin_amdgcn_exp2f(((-kLog2_65535 - m_ref) - off_n) - above);
        } else {
            w_blk = __builtin_amdgcn_exp2f((-kLog2_65535 - m_ref) - off_n);
        }
        float E[4][4];
        auto exponentials = [&](int T0) __attribute__((always_inline)) {
#pragma unroll
            for (int T = T0; T < T0 + 2; ++T)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float y;
                    if constexpr (MODE == kFold) y = fmaf(__int_as_float(S[T][r]), c_up, off_f);
                    else if constexpr (MODE == kScaled) y = fmaf(__int_as_float(S[T][r]) - kStartF, c_up, off_f);
                    else y = fmaf(start_result(S[T][r]), c, off_f);
                    E[T][r] = __builtin_amdgcn_exp2f(y);
                }
            asm volatile("" : "+v"(E[T0][0]), "+v"(E[T0][1]), "+v"(E[T0][2]), "+v"(E[T0][3]), "+v"(E[T0 + 1][0]), "+v"(E[T0 + 1][1]), "+v"(E[T0 + 1][2]), "+v"(E[T0 + 1][3]));
        };
        exponentials(0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!LAST) products_k(2);
        __builtin_amdgcn_sched_barrier(0);
        read_v(0);
        exponentials(2);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(0);
        PARO_TIMELINE_PHASE(0)  // products K Q of the next block, exponentials
        unsigned eb = 0;
        float m_new = 0.0f;
        if constexpr (!LAST) {
            mask_tail(j1, N);
            m_new = maxima(N, sq_i * sk1, eb);
        }
        const float rs = ((E[0][0] + E[0][1]) + (E[0][2] + E[0][3])) + ((E[1][0] + E[1][1]) + (E[1][2] + E[1][3])) +
                         (((E[2][0] + E[2][1]) + (E[2][2] + E[2][3])) + ((E[3][0] + E[3][1]) + (E[3][2] + E[3][3])));
        v4i pf;
#pragma unroll
        for (int T = 0; T < 4; ++T) {
            const unsigned lo = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pknorm_u16(E[T][0], E[T][1]));
            const unsigned hi = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pknorm_u16(E[T][2], E[T][3]));
            pf[T] = (int)__builtin_amdgcn_perm(hi, lo, 0x06040200u);
        }
        l = fmaf(rs, w_blk, l);
        const float weight = w_blk * (sv0 * sv_up * (PVBITS == 4 ? 0.0625f : 1.0f));
        v4acc o[4];
        auto products_v = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < 4; ++x) o[x] = __builtin_amdgcn_mfma_i32_16x16x64_i8(vf[x], pf, start, 0, 0, 0);
        };
        auto add = [&](int ct0) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[ct0 + x][r] = fmaf(__int_as_float(o[x][r]) - kStartF, weight, acc[ct0 + x][r]);
        };
        products_v();
        if constexpr (CT == 8) {
            read_v(4);
            add(0);
            products_v();
            add(4);
        } else {
            add(0);
        }
        if constexpr (LAST) return;
        tile_e[PARITY ^ 1][w] = eb;  // (the same in every lane)
        refer(m_new);
        sk0 = sk1;
        sv0 = sv1;
        j1 = j2;
        j2 = j3;
        sk1 = uniform_load(skp + j1);
        sv1 = uniform_load(svp + j1);
        PARO_TIMELINE_PHASE(2)  // maxima of the next block, sum, codes, products P V, accumulators
        // what this wavefront has asked for has landed; behind the barrier both tiles and all four exponents are whole, and what
        // this block read is free
        if constexpr (QKBITS == 8 || PVBITS == 8) __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
        PARO_TIMELINE_PHASE(1)  // wait for the tiles and for the other wavefronts
    };
    auto visit_all = [&](auto mode_tag) __attribute__((always_inline)) {
        int t = 0;
        for (; t + 2 < cnt; t += 2) {
            step(mode_tag, std::integral_constant<int, 0>{}, t, Sa, Sb);
            step(mode_tag, std::integral_constant<int, 1>{}, t + 1, Sb, Sa);
        }
        if (t + 1 < cnt) {
            step(mode_tag, std::integral_constant<int, 0>{}, t, Sa, Sb);
#pragma unroll
            for (int T = 0; T < 4; ++T) Sa[T] = Sb[T];
        }
        if (cnt > 0) step(mode_tag, std::integral_constant<int, kLast>{}, cnt - 1, Sa, Sb);
    };
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __syncthreads();
    if (cnt > 0) {
        logits(kring0, Sa);
        mask_tail(j0, Sa);
        unsigned eb;
        const float m_new = maxima(Sa, sq_i * sk0, eb);
        tile_e[0][w] = eb;
        refer(m_new);
    }
    __syncthreads();
    PARO_TIMELINE_PHASE(4)  // everything in front of the block loop
    if (fast) visit_all(std::integral_constant<int, FOLDABLE ? kFold : kScaled>{});
    else visit_all(std::integral_constant<int, kExact>{});
    PARO_TIMELINE_PHASE(3)

    const float l_tot = quad_rows_sum(l) * 65535.0f;
    const int ln = lane_here();  // nothing that only these stores need is kept through the loop
    const int orow_no = i * BLK + 16 * w + (ln & 15);
    const bool valid = orow_no < a.n_tokens;
    const float inv = (valid && l_tot > 0.0f) ? (0x1p26f / sv_up) / l_tot : 0.0f;
    const long long ooff = out_row_offset<D>(a, bh, h, head_rows, orow_no, valid);
    if (ooff >= 0) {
        OutT* orow = (OutT*)a.op + ooff + 4 * (ln >> 4);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            float x[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = valid ? acc[ct][r] * inv : 0.0f;
            store4(orow + 16 * ct, x[0], x[1], x[2], x[3]);
        }
    }
    PARO_TIMELINE_END(4 * item + w, threadIdx.x & 63, cnt)
}

// -------------------------------------------------------------------------------------------
// bf16 unquantized block-sparse mode (the sparse-only rows of the paper's tables), on v_mfma_f32_16x16x32_bf16 in the same transposed
// orientation.  P is not quantized, so there is no tile-wide scale; P enters the PV product rounded to bf16 while the denominator
// accumulates it in fp32.
// -------------------------------------------------------------------------------------------
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

// -------------------------------------------------------------------------------------------
// bf16 mode, block 64: the wavefronts of a row block split its KEYS.  P is not quantized, so nothing ties the keys of a
// block together: each wavefront takes 32 of the 64 keys of every live block against its own fixed reference and keeps
// its own sums, which meet once, at the end of the row.
// -------------------------------------------------------------------------------------------

// Running state of NG groups of 16 queries over one wavefront's 32 keys of every block, in 16 x 16 x 32 products.  Lane n + 16 G
// holds query n of each group: in S[T], tile T of 16 keys, the four keys 4 G .. of the tile, in acc the channels 4 G .. of each 16.
// The rows of K's tiles are chosen (bf16_krow) so that a lane's eight keys are one piece of V^T's rows, and its exponentials one
// operand of the second product.
// Exponentials are taken against the first maximum that is seen; a lane whose sum of one block passes 2^64 sends the wavefront
// through a rare branch that moves the references to the rows' maxima.  (Looking at the sum takes one compare where the row maximum
// took 16 operands; a logit 64 octaves above the reference shows in the sum, and one that overflows the exponential shows as
// infinity.)
__device__ __forceinline__ int bf16_krow(int n) { return 16 * ((n >> 2) & 1) + 4 * (n >> 3) + (n & 3); }  // of tile 0; tile 1: + 8
constexpr float kBf16SumLimit = 18446744073709551616.0f;  // 2^64
template <int NG, int CT>
struct Bf16Groups {
    float off[NG];  // minus the reference, what is added to c S; 0 while there is none
    float l[NG];    // this lane's share of the row sum
    unsigned seen;  // bit H: group H's query has a reference (a real key has been seen)
    v4f acc[CT][NG];

    __device__ __forceinline__ void init() {
        seen = 0;
#pragma unroll
        for (int H = 0; H < NG; ++H) {
            off[H] = 0.0f;
            l[H] = 0.0f;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) acc[ct][H] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        }
    }
    __device__ __forceinline__ bool open() const { return __builtin_amdgcn_ballot_w64(seen != (1u << NG) - 1) != 0; }
    // keys at or past nkeys never receive probability mass; the wavefront's keys start at `first`
    static __device__ __forceinline__ void mask(v4f (&S)[2][NG], int first, int nkeys) {
        const int ln = lane_here();
        first += 16 * ((ln >> 4) & 1) + 4 * (ln >> 5);
#pragma unroll
        for (int T = 0; T < 2; ++T)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int H = 0; H < NG; ++H)
                    if (first + 8 * T + r >= nkeys) S[T][H][r] = -INFINITY;
    }
    // queries without a reference take their maximum in S; with `all`, those that climbed past theirs as well
    __device__ __forceinline__ void reference(const v4f (&S)[2][NG], float c, bool all) {
#pragma unroll
        for (int H = 0; H < NG; ++H) {
            float mx = -INFINITY;
#pragma unroll
            for (int T = 0; T < 2; ++T)
#pragma unroll
                for (int r = 0; r < 4; ++r) mx = fmaxf(mx, S[T][H][r]);
            float ymax = c * mx;
            const int ln = lane_here();
            ymax = fmaxf(ymax, __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (ln ^ 16), __float_as_int(ymax))));
            ymax = fmaxf(ymax, __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (ln ^ 32), __float_as_int(ymax))));
            if (!(seen >> H & 1)) {
                if (ymax > -INFINITY) {
                    off[H] = -ymax;
                    seen |= 1u << H;
                }
            } else if (all) {
                const float up = fmaxf(ymax + off[H], 0.0f);
                const float down = __builtin_amdgcn_exp2f(-up);
                l[H] *= down;
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[ct][H][r] *= down;
                off[H] -= up;
            }
        }
    }
    // P = 2^(c S + off) in place of S, and this lane's sums.  True if some sum calls for the rare branch: one compare for the lane's
    // queries.  A sum that is NaN stays out of it: it neither hides another's climb nor sends the wavefront there in every block.
    __device__ __forceinline__ bool exponentials(v4f (&S)[2][NG], float c, float (&rs)[NG]) const {
#pragma unroll
        for (int H = 0; H < NG; ++H)
#pragma unroll
            for (int T = 0; T < 2; ++T)
#pragma unroll
                for (int r = 0; r < 4; ++r) S[T][H][r] = __builtin_amdgcn_exp2f(fmaf(S[T][H][r], c, off[H]));
        float all = 0.0f;
#pragma unroll
        for (int H = 0; H < NG; ++H) {
            rs[H] = ((S[0][H][0] + S[1][H][0]) + (S[0][H][1] + S[1][H][1])) + ((S[0][H][2] + S[1][H][2]) + (S[0][H][3] + S[1][H][3]));
            all = H ? fmaxf(all, rs[H]) : rs[H];
        }
        return __builtin_amdgcn_ballot_w64(all > kBf16SumLimit) != 0;
    }
    __device__ __forceinline__ void add(const float (&rs)[NG]) {
#pragma unroll
        for (int H = 0; H < NG; ++H) l[H] += rs[H];
    }
    static __device__ __forceinline__ v8bf pack(const v4f (&S)[2][NG], int H) {
        v8bf f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const v2bf pb = __builtin_convertvector(v2f{S[e >> 1][H][2 * (e & 1)], S[e >> 1][H][2 * (e & 1) + 1]}, v2bf);
            f[2 * e] = pb[0];
            f[2 * e + 1] = pb[1];
        }
        return f;
    }
    // The end of a row: the sums of 64 channels of two groups (from group H0 and channel tile C0), with their references and row
    // sums, handed to another wavefront ...
    template <int H0, int C0>
    __device__ __forceinline__ void hand_over(float* tiles, float (*row)[64], int ln) const {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            row[u][ln] = seen >> (H0 + u) & 1 ? off[H0 + u] : INFINITY;
            row[2 + u][ln] = l[H0 + u];
#pragma unroll
            for (int ct = 0; ct < 4; ++ct)
#pragma unroll
                for (int r = 0; r < 4; ++r) tiles[(16 * u + 4 * ct + r) * 64 + ln] = acc[C0 + ct][H0 + u][r];
        }
    }
    // ... and joined there with its own, normalised and stored.  row0: the row (of the block's matrix) of query 0 of group H0;
    // offset(row): of its first channel in op, negative if it is not stored.
    template <int H0, int C0, typename OutT, typename Offset>
    __device__ __forceinline__ void finish(OutT* op, Offset offset, int row0, int n_tokens, const float* tiles, const float (*meet)[64], int ln) const {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int row = row0 + 16 * u + (ln & 15);
            const float mine = seen >> (H0 + u) & 1 ? off[H0 + u] : INFINITY, other = meet[u][ln];
            const float top = fminf(mine, other);  // minus the larger reference; +inf if neither saw a key
            const float fa = mine < INFINITY ? __builtin_amdgcn_exp2f(top - mine) : 0.0f;
            const float fb = other < INFINITY ? __builtin_amdgcn_exp2f(top - other) : 0.0f;
            float l_tot = l[H0 + u] * fa + meet[2 + u][ln] * fb;
            l_tot += __shfl_xor(l_tot, 16);
            l_tot += __shfl_xor(l_tot, 32);
            const float inv = (row < n_tokens && l_tot > 0.0f) ? 1.0f / l_tot : 0.0f;
            const float ia = fa * inv, ib = fb * inv;
            const long long ooff = offset(row);
            if (ooff >= 0) {
                OutT* orow = op + ooff + 16 * C0 + 4 * (ln >> 4);
#pragma unroll
                for (int ct = 0; ct < 4; ++ct) {
                    float o[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) o[r] = acc[C0 + ct][H0 + u][r] * ia + tiles[(16 * u + 4 * ct + r) * 64 + ln] * ib;
                    store4(orow + 16 * ct, o[0], o[1], o[2], o[3]);
                }
            }
        }
    }
};

// d = 64: TWO wavefronts per row block, each with all 64 queries and one half of the keys, so that every byte of K and V
// is read from LDS once per row block (four wavefronts of 16 queries read it four times: 64 KB of reads and 16 KB of
// writes per block, 640 of the 777 cycles a block took).  A wavefront's half tiles are its own: it moves them to
// LDS itself (global_load_lds, 4 KB of K and 4 KB of V, one slot each) and there is no barrier in the loop.  K_{t+1} is
// requested behind the reads of K_t, V_{t+1} behind those of V_t.
// What bounds it is power: under this load the card stands at its limit (1.4 kW) and lowers its clock to 1.7 GHz, so time
// follows the energy of a block, of which the products are nearly half.  Hence the 16 x 16 x 32 form of the products: 7.2 nJ
// for half the work of a 32 x 32 x 16 one, which takes 16.7.  48 heads of 17550 tokens at 30 % density, quantizer included:
// 1423 -> 1355 us (with 32 x 32 x 16 products before).  K and V straight to registers, without LDS and with two wavefronts
// per SIMD instead of three: 2080 us.
template <typename OutT>
__global__ __launch_bounds__(128, 3) void attn_bf16_d64_kernel(AttnArgs a) {
    constexpr int BLK = 64, D = 64;
    constexpr int TILE = BLK * D * 2;
    __shared__ __attribute__((aligned(16))) uint8_t kbuf[2][TILE / 2];  // [wavefront]; later half of the exchange buffer
    __shared__ __attribute__((aligned(16))) uint8_t vbuf[1024 + TILE];  // [1 KB in front, see request_v][wavefront]; later the other half
    __shared__ float meet[2][4][64];  // [half of the queries][2 references, 2 sums][lane]

    const int wg = blockIdx.x;
    const int logical = (wg & 7) * a.per_xcd + (wg >> 3);
    if (logical >= a.total_wg) return;
    const int item = a.row_order ? min(max(a.row_order[logical], 0), a.total_wg - 1) : logical;
    const int bh = item / a.kblocks;
    const int i = item - bh * a.kblocks;
    const int h = bh % a.nh;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15;
    const int G = lane >> 4;

    const int* rp = a.row_ptr + (size_t)h * (a.kblocks + 1) + i;
    const int beg = __builtin_amdgcn_readfirstlane(min(max(rp[0], 0), a.nnz));
    const int end = __builtin_amdgcn_readfirstlane(min(max(rp[1], beg), a.nnz));
    const int cnt = end - beg;
    if (2 * cnt > a.kblocks) __builtin_amdgcn_s_setprio(2);
    ColumnList list(a.col_idx + beg, cnt, a.kblocks);

    const size_t head_rows = (size_t)bh * a.kblocks * BLK;
    const uint8_t* kbase = a.k + head_rows * D * 2 + (TILE / 2) * w;  // rows 32 w .. of a K tile
    const uint8_t* vbase = a.v + head_rows * D * 2 + 64 * w;          // slots 32 w .. of every row of a V^T tile
    const float c = a.qk_scale;
    v8bf qf[4][2];  // [group of 16 queries][32 channels]
#pragma unroll
    for (int H = 0; H < 4; ++H) {
        const uint8_t* qrow = a.q + (head_rows + i * BLK + 16 * H + n) * D * 2 + 16 * G;
#pragma unroll
        for (int s = 0; s < 2; ++s) qf[H][s] = *(const v8bf*)(qrow + 64 * s);
    }
    const int krow = bf16_krow(n);
    // K half: 32 rows of 128 bytes, piece p of row r at position p ^ (r % 4 + 4 (r / 16)), different for the eight rows that
    // neighbouring lanes read.  V^T half: 64 rows of 64 bytes, piece p of row r at position p ^ (r / 2) % 4.
    unsigned kfill = 128u * (lane >> 3) + 16u * ((lane & 7) ^ ((lane >> 3) & 3));
    const unsigned vfill = 128u * (lane >> 2) + 16u * ((lane & 3) ^ ((lane >> 3) & 3));
    unsigned kread = 128u * krow + 16u * (G ^ ((krow & 3) | ((krow >> 2) & 4)));
    unsigned vread = 64u * n + 16u * (G ^ ((n >> 1) & 3));
    uint8_t* const vslot = vbuf + 1024 + (TILE / 2) * w;
    auto request_k = [&](int j) {
        const uint8_t* kp = kbase + (size_t)j * TILE;
        asm volatile("" : "+s"(kp), "+v"(kfill));  // scalar base + lane offset; the flipped offset is made here, not kept
        lds_dma16<0>(kp, kfill, &kbuf[w][0]);
        lds_dma16<1024>(kp, kfill, &kbuf[w][0]);
        lds_dma16<2048>(kp, kfill ^ 64u, &kbuf[w][0]);
        lds_dma16<3072>(kp, kfill ^ 64u, &kbuf[w][0]);
    };
    auto request_v = [&](int j) {
        const uint8_t* vp = vbase + (size_t)j * TILE;
        asm volatile("" : "+s"(vp));
        // a request further is 2048 bytes in memory and 1024 in LDS, while the offset counts in both: the LDS base is 1 KB lower, inside vbuf.  (The
        // step in four addresses instead: 0.7 % of the layer.)
        lds_dma16<0>(vp, vfill, vslot);
        lds_dma16<2048>(vp, vfill, vslot - 1024);
        lds_dma16<0>(vp + 4096, vfill, vslot + 2048);
        lds_dma16<2048>(vp + 4096, vfill, vslot + 1024);
    };
    Bf16Groups<4, 4> rows;
    rows.init();
    v4f S[2][4];
    const int tail_block = (a.n_tokens % BLK) != 0 ? a.kblocks - 1 : -1;
    const int nkeys = a.n_tokens - (a.kblocks - 1) * BLK;
    // Columns of the steps t, t + 1; behind the last step its own column is requested once more and not used: requests
    // under a condition would make the compiler wait for V_t in front of K_t's reads.
    int j0 = 0, j1 = 0;
    if (cnt > 0) {
        j0 = list.at(0);
        request_k(j0);
        request_v(j0);
        j1 = cnt > 1 ? list.at(1) : j0;
    }
    bool open = true;  // some row has no reference yet
    __builtin_amdgcn_s_waitcnt(0x0F70);  // Q is in registers: otherwise the compiler waits for everything in every pass
    const v4f zero = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int t = 0; t < cnt; ++t) {
        __builtin_amdgcn_s_waitcnt(0x0F74);  // vmcnt(4): all but the last request, V_t's, have landed
        asm volatile("" : "+v"(kread), "+v"(vread));  // the flipped address is made here, not kept
        // ---- S^T = K_j Q_i^T, 32 keys of this wavefront against 64 queries
        v8bf kf[2][2];
#pragma unroll
        for (int T = 0; T < 2; ++T)
#pragma unroll
            for (int s = 0; s < 2; ++s) kf[T][s] = *(const v8bf*)(&kbuf[w][0] + (kread ^ (64u * s)) + 1024 * T);
#pragma unroll
        for (int T = 0; T < 2; ++T) {
#pragma unroll
            for (int H = 0; H < 4; ++H) S[T][H] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[T][0], qf[H][0], zero, 0, 0, 0);
#pragma unroll
            for (int H = 0; H < 4; ++H) S[T][H] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[T][1], qf[H][1], S[T][H], 0, 0, 0);
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): K_t has been read
        request_k(j1);
        if (j0 == tail_block) rows.mask(S, 32 * w, nkeys);
        if (open) {
            rows.reference(S, c, false);
            open = rows.open();
        }
        float rs[4];
        if (rows.exponentials(S, c, rs)) {
            // rare: the logits once more, from K in global memory (its LDS slot is being refilled)
            const int ln = lane_here();
            const uint8_t* kp = kbase + (size_t)j0 * TILE + 128 * bf16_krow(ln & 15) + 16 * (ln >> 4);
#pragma unroll
            for (int T = 0; T < 2; ++T)
#pragma unroll
                for (int H = 0; H < 4; ++H) {
                    S[T][H] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(const v8bf*)(kp + 1024 * T), qf[H][0], zero, 0, 0, 0);
                    S[T][H] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(const v8bf*)(kp + 1024 * T + 64), qf[H][1], S[T][H], 0, 0, 0);
                }
            if (j0 == tail_block) rows.mask(S, 32 * w, nkeys);
            rows.reference(S, c, true);
            rows.exponentials(S, c, rs);
        }
        // ---- O^T += V_j^T P^T over this wavefront's keys
        rows.add(rs);
        v8bf pf[4];
#pragma unroll
        for (int H = 0; H < 4; ++H) pf[H] = rows.pack(S, H);
        __builtin_amdgcn_s_waitcnt(0x0F74);  // V_t has landed; K_{t+1} may be on its way
        v8bf vf[4];
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) vf[ct] = *(const v8bf*)(vslot + vread + 1024 * ct);
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
            for (int H = 0; H < 4; ++H) rows.acc[ct][H] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[ct], pf[H], rows.acc[ct][H], 0, 0, 0);
        __builtin_amdgcn_s_waitcnt(0xC07F);  // V_t has been read
        request_v(j1);
        j0 = j1;
        if (t + 2 < cnt) j1 = list.at(t + 2);
    }
    // ---- wavefront w finishes the queries of half w: it hands its sums of the other half over through LDS
    __builtin_amdgcn_s_waitcnt(0x0F70);  // nothing is in flight to the buffers any more
    __syncthreads();
    float* give = (float*)(w == 0 ? &kbuf[0][0] : vbuf);  // 8 KB each: [32 registers][64 lanes]
    const float* take = (const float*)(w == 0 ? vbuf : &kbuf[0][0]);
    const int ln = lane_here();  // nothing of the lane's number is kept through the loop for this
    auto offset = [&](int row) { return out_row_offset<D>(a, bh, h, head_rows, row, row < a.n_tokens); };
    if (w == 0) rows.template hand_over<2, 0>(give, meet[1], ln);
    else rows.template hand_over<0, 0>(give, meet[0], ln);
    __syncthreads();
    if (w == 0) rows.template finish<0, 0>((OutT*)a.op, offset, i * BLK, a.n_tokens, take, meet[0], ln);
    else rows.template finish<2, 0>((OutT*)a.op, offset, i * BLK + 32, a.n_tokens, take, meet[1], ln);
}

// d = 128: FOUR wavefronts per row block, wavefront w with the queries 32 (w & 1) .. and the keys 32 (w >> 1) .. of every
// block.  (Two wavefronts of 32 queries with all keys, the form this replaces, moved the tiles through registers - 64 of
// them - and a row's chain of blocks was twice as long: 72-block rows of text queries are the end of such a launch.)
// The tiles are shared: each wavefront moves a quarter of K and of V^T to LDS (global_load_lds), one slot each.
// Two barriers per block: V_t is requested behind the first (V_{t-1} has been read by all, K_t is whole) and K_{t+1}
// behind the second (K_t has been read by all, V_t is whole), so each has half a block of work to hide behind.
// 24 heads of 4096 + 512 tokens at 30 % density, two layers with quantizer and mask prefetch: 419 -> 387 us (runs of one
// side differ by 0.3 %; 406 -> 377 and 470 -> 411 elsewhere).  In 16 x 16 x 32 products, 389 -> 354 us: a lane's logits are four
// chains of four products, not one chain of eight that each wait for the one before, and they take less energy.
template <typename OutT>
__global__ __launch_bounds__(256, 3) void attn_bf16_d128_kernel(AttnArgs a) {
    constexpr int BLK = 64, D = 128;
    constexpr int TILE = BLK * D * 2;
    constexpr int KS = D / 32, CT = D / 16;
    __shared__ __attribute__((aligned(16))) uint8_t kbuf[TILE];  // later half of the exchange buffer
    __shared__ __attribute__((aligned(16))) uint8_t vbuf[TILE];
    __shared__ float meet[4][4][64];  // [wavefront][2 references, 2 sums][lane]

    const int wg = blockIdx.x;
    const int logical = (wg & 7) * a.per_xcd + (wg >> 3);
    if (logical >= a.total_wg) return;
    const int item = a.row_order ? min(max(a.row_order[logical], 0), a.total_wg - 1) : logical;
    const int bh = item / a.kblocks;
    const int i = item - bh * a.kblocks;
    const int h = bh % a.nh;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kh = w >> 1;
    const int n = lane & 15;
    const int G = lane >> 4;

    const int* rp = a.row_ptr + (size_t)h * (a.kblocks + 1) + i;
    const int beg = __builtin_amdgcn_readfirstlane(min(max(rp[0], 0), a.nnz));
    const int end = __builtin_amdgcn_readfirstlane(min(max(rp[1], beg), a.nnz));
    const int cnt = end - beg;
    if (2 * cnt > a.kblocks) __builtin_amdgcn_s_setprio(2);
    ColumnList list(a.col_idx + beg, cnt, a.kblocks);

    const size_t head_rows = (size_t)bh * a.kblocks * BLK;
    const uint8_t* kbase = a.k + head_rows * D * 2 + 4096 * w;  // rows 16 w .. of a K tile
    const uint8_t* vbase = a.v + head_rows * D * 2 + 4096 * w;  // rows 32 w .. of a V^T tile
    const float c = a.qk_scale;
    const int row0 = i * BLK + 32 * (w & 1);
    v8bf qf[2][KS];  // [group of 16 queries][32 channels]
#pragma unroll
    for (int H = 0; H < 2; ++H) {
        const uint8_t* qrow = a.q + (head_rows + row0 + 16 * H + n) * D * 2 + 16 * G;
#pragma unroll
        for (int s = 0; s < KS; ++s) qf[H][s] = *(const v8bf*)(qrow + 64 * s);
    }
    // K rows have two 128-byte lines, V^T rows one; piece p of a line sits at position p ^ (r % 4 + 4 (r / 16 % 2)) for row r of K and
    // p ^ r % 8 for row r of V^T, different for the eight rows that neighbouring lanes read
    const int krow = bf16_krow(n);
    const unsigned kfill = 256u * (lane >> 4) + 16u * ((lane & 8) | ((lane & 7) ^ ((lane >> 4) | 4 * (w & 1))));
    const unsigned vfill = 128u * (lane >> 3) + 16u * ((lane & 7) ^ (lane >> 3));
    unsigned kread = 256u * (32 * kh + krow) + 16u * (G ^ ((krow & 3) | ((krow >> 2) & 4)));  // 32 channels s: piece 4 s + G
    const unsigned vread = 128u * n + 16u * ((4 * kh + G) ^ (n & 7));                         // piece 4 kh + G
    auto request_k = [&](int j) {
        const uint8_t* kp = kbase + (size_t)j * TILE;
        asm volatile("" : "+s"(kp));
        lds_dma16<0>(kp, kfill, &kbuf[4096 * w]);
        lds_dma16<1024>(kp, kfill, &kbuf[4096 * w]);
        lds_dma16<2048>(kp, kfill, &kbuf[4096 * w]);
        lds_dma16<3072>(kp, kfill, &kbuf[4096 * w]);
    };
    auto request_v = [&](int j) {
        const uint8_t* vp = vbase + (size_t)j * TILE;
        asm volatile("" : "+s"(vp));
        lds_dma16<0>(vp, vfill, &vbuf[4096 * w]);
        lds_dma16<1024>(vp, vfill, &vbuf[4096 * w]);
        lds_dma16<2048>(vp, vfill, &vbuf[4096 * w]);
        lds_dma16<3072>(vp, vfill, &vbuf[4096 * w]);
    };
    const int tail_block = (a.n_tokens % BLK) != 0 ? a.kblocks - 1 : -1;
    const int nkeys = a.n_tokens - (a.kblocks - 1) * BLK;

    Bf16Groups<2, CT> rows;
    rows.init();
    bool open = true;  // some row has no reference yet
    const v4f zero = {0.0f, 0.0f, 0.0f, 0.0f};
    int j0 = 0, j1 = 0;  // columns of the steps t, t + 1
    if (cnt > 0) {
        j0 = list.at(0);
        request_k(j0);
        if (cnt > 1) j1 = list.at(1);
    }

    for (int t = 0; t < cnt; ++t) {
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wavefront's part of K_t has landed
        __syncthreads();                     // and everybody's; V_{t-1} has been read by all
        request_v(j0);
        asm volatile("" : "+v"(kread));  // the flipped address is made here, not kept
        // ---- S^T = K_j Q_i^T, this wavefront's 32 keys against its 32 queries
        v4f S[2][2];
        auto logits = [&]() {
            v8bf kf[2][KS];  // all requested before the first product: each would otherwise wait out its own latency
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int T = 0; T < 2; ++T) kf[T][s] = *(const v8bf*)(kbuf + (kread ^ (64u * (s & 1))) + 128 * (s >> 1) + 2048 * T);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int T = 0; T < 2; ++T)
#pragma unroll
                    for (int H = 0; H < 2; ++H) S[T][H] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[T][s], qf[H][s], s ? S[T][H] : zero, 0, 0, 0);
            if (j0 == tail_block) rows.mask(S, 32 * kh, nkeys);
        };
        logits();
        if (open) {
            rows.reference(S, c, false);
            open = rows.open();
        }
        float rs[2];
        if (rows.exponentials(S, c, rs)) {  // rare
            logits();
            rows.reference(S, c, true);
            rows.exponentials(S, c, rs);
        }
        rows.add(rs);
        v8bf pf[2];
#pragma unroll
        for (int H = 0; H < 2; ++H) pf[H] = rows.pack(S, H);
        __builtin_amdgcn_s_waitcnt(0x0F70);  // this wavefront's part of V_t has landed
        __syncthreads();                     // and everybody's; K_t has been read by all
        if (t + 1 < cnt) request_k(j1);
        // ---- O^T += V_j^T P^T over this wavefront's keys
        v8bf vf[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) vf[ct] = *(const v8bf*)(vbuf + 2048 * ct + vread);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int H = 0; H < 2; ++H) rows.acc[ct][H] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[ct], pf[H], rows.acc[ct][H], 0, 0, 0);
        j0 = j1;
        if (t + 2 < cnt) j1 = list.at(t + 2);
    }

    // ---- the wavefronts w and w ^ 2 share their queries: the one with the lower keys finishes channels 0 .. 63
    __syncthreads();
    float* give = (float*)((w & 1 ? vbuf : kbuf) + 8192 * kh);  // 8 KB each: [32 registers][64 lanes]
    const float* take = (const float*)((w & 1 ? vbuf : kbuf) + 8192 * (kh ^ 1));
    const int ln = lane_here();  // nothing of the lane's number is kept through the loop for this
    auto offset = [&](int row) { return out_row_offset<D>(a, bh, h, head_rows, row, row < a.n_tokens); };
    if (kh == 0) rows.template hand_over<0, 4>(give, meet[w], ln);
    else rows.template hand_over<0, 0>(give, meet[w], ln);
    __syncthreads();
    if (kh == 0) rows.template finish<0, 0>((OutT*)a.op, offset, row0, a.n_tokens, take, meet[w ^ 2], ln);
    else rows.template finish<0, 4>((OutT*)a.op, offset, row0, a.n_tokens, take, meet[w ^ 2], ln);
}

// Block 32, and d = 64, block 64 with few row blocks: a wavefront has 32 queries and 32 keys of every live block, at block 32 the whole of
// it, at block 64 the queries 32 (w & 1) .. and the keys 32 (w >> 1) .. of a row block that four wavefronts share until their sums meet at
// its end.  A wavefront moves its part of the tiles to LDS itself (one slot each; K_{t+2} is requested behind the reads of K_{t+1}, V_{t+1}
// behind those of V_t), so there is no barrier in the loop, and K Q of block t + 1 runs beside the exponentials of block t.
// Bound by the chain of a block where the chip is not full; where it is, a wavefront waits for its own tiles in 44 (d = 64) to 48 % of its cycles,
// with vector issue at 0.62 and the matrix pipe at 0.40 of the time.  Attention call alone, us, before (block 32: tiles
// through registers with two barriers per block; block 64: attn_bf16_d64_kernel) -> now, 30 % density: block 32, d = 64, 30 heads of 17550 tokens
// 1129 -> 915, 4 heads of 4096 32.2 -> 23.8; d = 128 2343 -> 1988 (three wavefronts per SIMD instead of two: 2186) and 40.9 -> 32.8; block 64,
// d = 64, 4 heads of 4096 20.5 -> 15.2, 6 heads of 1955 14.2 -> 10.7.  At block 64, d = 128 each byte that two wavefronts share would be
// moved to LDS twice: 73.6 -> 107.8 for 24 heads of 4096.
template <int BLK, int D, typename OutT>
__global__ __launch_bounds__(BLK == 32 ? 64 : 256, (D == 64 ? 4 : 2)) void attn_bf16_q32_kernel(AttnArgs a) {
    constexpr int NW = BLK == 32 ? 1 : 4;
    static_assert(BLK == 32 || D == 64, "shapes that are launched");
    constexpr int TILE = 32 * D * 2;  // bytes of a wavefront's part of a K or V^T tile
    constexpr int KS = D / 32, CT = D / 16;
    constexpr int REQUESTS = TILE / 1024;  // per tile
    __shared__ __attribute__((aligned(16))) uint8_t kslots[NW][TILE];
    constexpr int LEAD = 32 * BLK - 1024;  // of V's array in front of its slots, see request_v
    __shared__ __attribute__((aligned(16))) uint8_t vslots[LEAD + NW * TILE];
    __shared__ float meet[NW > 1 ? 2 : 1][4][64];  // [half of the queries][2 references, 2 sums][lane]

    const int wg = blockIdx.x;
    const int logical = (wg & 7) * a.per_xcd + (wg >> 3);
    if (logical >= a.total_wg) return;
    const int item = a.row_order ? min(max(a.row_order[logical], 0), a.total_wg - 1) : logical;
    const int bh = item / a.kblocks;
    const int i = item - bh * a.kblocks;
    const int h = bh % a.nh;
    const int lane = threadIdx.x & 63;
    const int w = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kh = w >> 1;                           // which 32 keys of a block
    const int row0 = i * BLK + 32 * (w & 1);         // first query
    uint8_t* const kbuf = &kslots[w][0];
    uint8_t* const vbuf = vslots + LEAD + TILE * w;
    const int n = lane & 15;
    const int G = lane >> 4;

    const int* rp = a.row_ptr + (size_t)h * (a.kblocks + 1) + i;
    const int beg = __builtin_amdgcn_readfirstlane(min(max(rp[0], 0), a.nnz));
    const int end = __builtin_amdgcn_readfirstlane(min(max(rp[1], beg), a.nnz));
    const int cnt = end - beg;
    const int* cols = a.col_idx + beg;

    const size_t head_rows = (size_t)bh * a.kblocks * BLK;
    const uint8_t* kbase = a.k + head_rows * D * 2 + TILE * kh;  // rows 32 kh .. of a K tile
    const uint8_t* vbase = a.v + head_rows * D * 2 + 64 * kh;    // slots 32 kh .. of every row of a V^T tile
    const float c = a.qk_scale;
    v8bf qf[2][KS];  // [group of 16 queries][32 channels]
#pragma unroll
    for (int H = 0; H < 2; ++H) {
        const uint8_t* qrow = a.q + (head_rows + row0 + 16 * H + n) * D * 2 + 16 * G;
#pragma unroll
        for (int s = 0; s < KS; ++s) qf[H][s] = *(const v8bf*)(qrow + 64 * s);
    }
    // K rows are one 128-byte line or two; piece p of a line of row r sits at position p ^ (r % 4 + 4 (r / 16)), different for the
    // eight rows that neighbouring lanes read.  V^T: rows of 64 bytes, piece p of row r at position p ^ (r / 2) % 4.
    const int krow = bf16_krow(n);
    unsigned kfill = D == 64 ? 128u * (lane >> 3) + 16u * ((lane & 7) ^ ((lane >> 3) & 3))
                             : 256u * (lane >> 4) + 16u * ((lane & 8) | ((lane & 7) ^ (lane >> 4)));
    const unsigned vfill = 2u * BLK * (lane >> 2) + 16u * ((lane & 3) ^ ((lane >> 3) & 3));
    unsigned kread = 2u * D * krow + 16u * (G ^ ((krow & 3) | ((krow >> 2) & 4)));  // 32 channels s: piece 4 s + G
    const unsigned vread = 64u * n + 16u * (G ^ ((n >> 1) & 3));
    auto request_k = [&](int j) __attribute__((always_inline)) {
        const uint8_t* kp = kbase + (size_t)j * (BLK * D * 2);
        asm volatile("" : "+s"(kp), "+v"(kfill));  // scalar base + lane offset; the flipped offset of rows 16 .. is made here, not kept
        if constexpr (D == 64) {
            lds_dma16<0>(kp, kfill, &kbuf[0]);
            lds_dma16<1024>(kp, kfill, &kbuf[0]);
            lds_dma16<2048>(kp, kfill ^ 64u, &kbuf[0]);
            lds_dma16<3072>(kp, kfill ^ 64u, &kbuf[0]);
        } else {
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const uint8_t* from = kp + 4096 * half;
                const unsigned off = kfill ^ (64u * half);
                lds_dma16<0>(from, off, &kbuf[4096 * half]);
                lds_dma16<1024>(from, off, &kbuf[4096 * half]);
                lds_dma16<2048>(from, off, &kbuf[4096 * half]);
                lds_dma16<3072>(from, off, &kbuf[4096 * half]);
            }
        }
    };
    auto request_v = [&](int j) __attribute__((always_inline)) {
        const uint8_t* vp = vbase + (size_t)j * (BLK * D * 2);
        asm volatile("" : "+s"(vp));
        // 16 rows each.  The second request of a pair is 32 BLK bytes further in memory and 1 KB in LDS, while the offset counts in both: its LDS
        // base is LEAD lower, inside vslots.  (The step in addresses of their own: 8 heads of 2048 tokens at 50 %, block 64, 18.1 -> 21.2 us.)
#pragma unroll
        for (int u = 0; u < REQUESTS; u += 2) {
            const uint8_t* from = vp + 32 * BLK * u;
            lds_dma16<0>(from, vfill, vbuf + 1024 * u);
            lds_dma16<32 * BLK>(from, vfill, vbuf + 1024 * u - LEAD);
        }
    };
    // 64 column indices per fetch, one per lane; past the end of the row its last column again
    auto load_cols = [&](int chunk) { return min(max(cols[min(chunk * 64 + lane_here(), cnt - 1)], 0), a.kblocks - 1); };
    int cols64 = cnt > 0 ? load_cols(0) : 0;
    auto column = [&](int u) {  // u advances by one per call
        if ((u & 63) == 0) cols64 = load_cols(u >> 6);
        return __builtin_amdgcn_readlane(cols64, u & 63);
    };
    const int tail_block = (a.n_tokens % BLK) != 0 ? a.kblocks - 1 : -1;
    const int nkeys = a.n_tokens - (a.kblocks - 1) * BLK;
    const v4f zero = {0.0f, 0.0f, 0.0f, 0.0f};
    Bf16Groups<2, CT> rows;
    rows.init();
    auto logits = [&](v4f (&S)[2][2]) __attribute__((always_inline)) {
        asm volatile("" : "+v"(kread));  // the flipped address is made here, not kept
        v8bf kf[2][KS];
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int T = 0; T < 2; ++T) kf[T][s] = *(const v8bf*)(kbuf + (kread ^ (64u * (s & 1))) + 128 * (s >> 1) + 16 * D * T);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int T = 0; T < 2; ++T)
#pragma unroll
                for (int H = 0; H < 2; ++H) S[T][H] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[T][s], qf[H][s], s ? S[T][H] : zero, 0, 0, 0);
    };

    int j0 = 0, j1 = 0;  // columns of the blocks t, t + 1
    bool open = true;    // some row has no reference yet
    v4f Sa[2][2], Sb[2][2];  // logits, this block's and the next one's in turn
    if (cnt > 0) {
        j0 = __builtin_amdgcn_readlane(cols64, 0);
        j1 = column(1);
        request_k(j0);
        request_v(j0);
        __builtin_amdgcn_s_waitcnt(REQUESTS == 4 ? 0x0F74 : 0x0F78);  // all but V_0's requests have landed
        logits(Sa);
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): K_0 has been read
        // (the order of the loop: K_{t+1}, then V_t; V_0 is older here and has landed when K_1 is waited for)
        request_k(j1);
    }
    // The last block stands apart: no product for a block behind it, no request that the end would wait for.  Layer of 8 heads of 221
    // tokens, block 32, d = 128: 10.65 -> 10.22 us (d = 64: 8.7 and 8.9, runs differ by 2 %; 8 heads of 4096, d = 128, 61).
    auto step = [&](auto last_tag, int t, v4f (&S)[2][2], v4f (&N)[2][2]) __attribute__((always_inline)) {
        constexpr bool LAST = decltype(last_tag)::value;
        if (j0 == tail_block) rows.mask(S, 32 * kh, nkeys);
        if (open) {
            rows.reference(S, c, false);
            open = rows.open();
        }
        int j2 = j1;
        if constexpr (!LAST) {
            j2 = column(t + 2);
            // K_{t+1} has landed (in the first block nothing is younger: everything has)
            if (t == 0) __builtin_amdgcn_s_waitcnt(0x0F70);
            else __builtin_amdgcn_s_waitcnt(REQUESTS == 4 ? 0x0F74 : 0x0F78);
            logits(N);
        }
        float rs[2];
        if (rows.exponentials(S, c, rs)) {
            // rare: the logits once more, from K in global memory (its LDS slot holds the next block)
            const int ln = lane_here();
            const uint8_t* kp = kbase + (size_t)j0 * (BLK * D * 2) + 2 * D * bf16_krow(ln & 15) + 16 * (ln >> 4);
#pragma unroll
            for (int T = 0; T < 2; ++T)
#pragma unroll
                for (int H = 0; H < 2; ++H)
#pragma unroll
                    for (int s = 0; s < KS; ++s)
                        S[T][H] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(const v8bf*)(kp + 16 * D * T + 64 * s), qf[H][s], s ? S[T][H] : zero, 0, 0, 0);
            if (j0 == tail_block) rows.mask(S, 32 * kh, nkeys);
            rows.reference(S, c, true);
            rows.exponentials(S, c, rs);
        }
        if constexpr (!LAST) {
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): K_{t+1} has been read
            request_k(j2);
        }
        rows.add(rs);
        v8bf pf[2];
#pragma unroll
        for (int H = 0; H < 2; ++H) pf[H] = rows.pack(S, H);
        // V_t has landed; K_{t+2} may be on its way
        if constexpr (LAST) __builtin_amdgcn_s_waitcnt(0x0F70);
        else __builtin_amdgcn_s_waitcnt(REQUESTS == 4 ? 0x0F74 : 0x0F78);
        // ---- O^T += V_j^T P^T
#pragma unroll
        for (int c0 = 0; c0 < CT; c0 += 4) {
            v8bf vf[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) vf[x] = *(const v8bf*)(vbuf + vread + 1024 * (c0 + x));
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int H = 0; H < 2; ++H) rows.acc[c0 + x][H] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[x], pf[H], rows.acc[c0 + x][H], 0, 0, 0);
        }
        if constexpr (!LAST) {
            __builtin_amdgcn_s_waitcnt(0xC07F);  // V_t has been read
            request_v(j1);
            j0 = j1;
            j1 = j2;
        }
    };
    const std::false_type inner;
    int t = 0;
    if constexpr (NW == 1)
        for (; t + 2 < cnt; t += 2) {  // by two, so that the logits change hands without copies: 4 heads of 4096 tokens, d = 64, 26.6 -> 24.3 us
            step(inner, t, Sa, Sb);
            step(inner, t + 1, Sb, Sa);
        }
    for (; t + 1 < cnt; ++t) {  // (the rest; no difference with four wavefronts)
        step(inner, t, Sa, Sb);
#pragma unroll
        for (int T = 0; T < 2; ++T)
#pragma unroll
            for (int H = 0; H < 2; ++H) Sa[T][H] = Sb[T][H];
    }
    if (t < cnt) step(std::true_type(), t, Sa, Sb);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // nothing is in flight to the buffers when they are given up

    const int ln = lane_here();  // nothing of the lane's number is kept through the loop for this
    auto offset = [&](int row) { return out_row_offset<D>(a, bh, h, head_rows, row, row < a.n_tokens); };
    if constexpr (NW == 1) {
#pragma unroll
        for (int H = 0; H < 2; ++H) {
            const int row = row0 + 16 * H + (ln & 15);
            float l_tot = rows.l[H] + __shfl_xor(rows.l[H], 16);
            l_tot += __shfl_xor(l_tot, 32);
            const float inv = (row < a.n_tokens && l_tot > 0.0f) ? 1.0f / l_tot : 0.0f;
            const long long ooff = offset(row);
            if (ooff >= 0) {
                OutT* orow = (OutT*)a.op + ooff + 4 * (ln >> 4);
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
                    store4(orow + 16 * ct, rows.acc[ct][H][0] * inv, rows.acc[ct][H][1] * inv, rows.acc[ct][H][2] * inv, rows.acc[ct][H][3] * inv);
            }
        }
    } else {
        // ---- the wavefronts w and w + 2 share their queries: the one with the lower keys finishes them, the other hands its sums over
        // through two of the K slots, 8 KB ([32 registers][64 lanes])
        __syncthreads();
        float* exchange = (float*)&kslots[2 * (w & 1)][0];
        if (kh == 1) rows.template hand_over<0, 0>(exchange, meet[w & 1], ln);
        __syncthreads();
        if (kh == 0) rows.template finish<0, 0>((OutT*)a.op, offset, row0, a.n_tokens, exchange, meet[w], ln);
    }
}

// Block 64, d = 64: with few row blocks four wavefronts per row block instead of two.  The line, in row blocks R of the launch, both sides
// in us (four / two wavefronts) at 20 and 50 % of K column blocks: K = 4 R = 512 6.8 / 7.4 and 7.6 / 8.8, R = 768 8.2 / 8.5 and 9.0 / 9.7, R = 896 9.3 / 9.6 and 10.5 / 10.8; K = 16 R = 768 10.2 / 11.0 and
// 14.6 / 16.7, R = 896 12.0 / 12.5 and 17.4 / 17.5; K = 32 R = 768 13.0 / 15.0 and 23.5 / 30.8, R = 896 15.5 / 15.8 and 31.0 / 40.5; K = 128 R = 768
// 67.9 / 94.6 and 95.8 / 140; masks of 3-D neighbours, K = 64, R = 768 21.0 / 23.0 and 41.7 / 47.1, R = 875 42.3 / 39.1 and 94.5 / 90.1, R = 1024 27.9 / 24.9
// and 57.5 / 51.5.
constexpr int kBf16Q32Rows = 768;

template <typename OutT>
static int launch_bf16(int blk, int d, const AttnArgs& a, hipStream_t st) {
    const dim3 grid((unsigned)(a.per_xcd * 8));
    if (blk == 64 && d == 64 && a.total_wg > kBf16Q32Rows) hipLaunchKernelGGL((attn_bf16_d64_kernel<OutT>), grid, dim3(128), 0, st, a);
    else if (blk == 64 && d == 64) hipLaunchKernelGGL((attn_bf16_q32_kernel<64, 64, OutT>), grid, dim3(256), 0, st, a);
    else if (blk == 64) hipLaunchKernelGGL((attn_bf16_d128_kernel<OutT>), grid, dim3(256), 0, st, a);
    else if (d == 64) hipLaunchKernelGGL((attn_bf16_q32_kernel<32, 64, OutT>), grid, dim3(64), 0, st, a);
    else hipLaunchKernelGGL((attn_bf16_q32_kernel<32, 128, OutT>), grid, dim3(64), 0, st, a);
    return PARO_OK;
}

template <int D, int QKBITS, int PVBITS>
static void launch_b32(paro_dtype out_dtype, const AttnArgs& a, hipStream_t st) {
    dim3 grid((unsigned)(a.per_xcd * 8));
    if (out_dtype == PARO_F32) hipLaunchKernelGGL((attn_i8_b32_kernel<D, QKBITS, PVBITS, float>), grid, dim3(64), 0, st, a);
    else hipLaunchKernelGGL((attn_i8_b32_kernel<D, QKBITS, PVBITS, uint16_t>), grid, dim3(64), 0, st, a);
}

template <int D, int QKBITS, int PVBITS, int QSRC = 0>
static void launch_q16(paro_dtype out_dtype, const AttnArgs& a, hipStream_t st) {
    dim3 grid((unsigned)(a.per_xcd * 8));
    if (out_dtype == PARO_F32) hipLaunchKernelGGL((attn_i8_q16_kernel<D, QKBITS, PVBITS, float, QSRC>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((attn_i8_q16_kernel<D, QKBITS, PVBITS, uint16_t, QSRC>), grid, dim3(256), 0, st, a);
}

template <int QKBITS, int PVBITS, int QSRC = 0>
static void launch_w64(paro_dtype out_dtype, const AttnArgs& a, hipStream_t st) {
    dim3 grid((unsigned)(a.per_xcd * 8));
    if constexpr (QKBITS == 8) {
        if (out_dtype == PARO_F32) hipLaunchKernelGGL((attn_i8_w64_kernel<PVBITS, float, QSRC>), grid, dim3(64), 0, st, a);
        else hipLaunchKernelGGL((attn_i8_w64_kernel<PVBITS, uint16_t, QSRC>), grid, dim3(64), 0, st, a);
    } else {
        if (out_dtype == PARO_F32) hipLaunchKernelGGL((attn_i8_w64_qk4_kernel<PVBITS, float>), grid, dim3(64), 0, st, a);
        else hipLaunchKernelGGL((attn_i8_w64_qk4_kernel<PVBITS, uint16_t>), grid, dim3(64), 0, st, a);
    }
}

// Block 64; QSRC as in the kernels.  d = 64: with few row blocks the chain of a row's blocks is the launch, and four wavefronts of 16
// queries are through a block in half the time that one wavefront of 64 needs; with many the chip is full and the 152 x 4 instructions
// per block of the former lose to the 495 of the latter.  Rows of fewer than 8 blocks on average are over before a chain counts: there four
// wavefronts win while all workgroups are resident at once - five per compute unit, four with 4-bit codes throughout (96 and 97
// registers) - and lose in a second round.  The lines, both sides in us (four wavefronts / one), 8-bit codes, then all 4-bit; R row blocks,
// K column blocks:
//   20 % of K = 4 .. 16 (1 .. 3 blocks a row):  R = 1024  7.8 .. 10.7 / 9.0 .. 11.8   7.8 .. 11.2 / 9.1 .. 12.6
//                                               R = 1152  8.7 .. 11.3 / 10.0 .. 12.8  10.6 .. 13.5 / 10.1 .. 13.5
//                                               R = 1280  8.8 .. 11.9 / 10.2 .. 13.2  10.8 .. 14.5 / 10.3 .. 14.3
//                                               R = 1408  11.2 .. 13.8 / 10.8 .. 13.5 11.7 .. 14.9 / 10.9 .. 14.5
//   20 % of K = 32 (6):                         R = 1280  16.1 / 18.2   19.0 / 19.7;  R = 1536  18.9 / 19.0   20.6 / 20.5
//   25 % of K = 32, 50 % of K = 16 (8):         R = 1408  21.2 / 21.8, 21.1 / 20.5;   R = 1536  21.5 / 22.2, 21.5 / 21.5
//   50 % of K = 24, 32 (12, 16):                R = 1536  28.6 / 36.8, 34.7 / 47.0    32.1 / 41.2, 39.3 / 53.1
//   20, 50 % of K = 64 (13, 32):                R = 1536  40.7 / 82.7, 67.0 / 87.7;   R = 2048  42.8 / 84.5, 79.9 / 89.0
//   20, 50 % of K = 256 (51, 128):              R = 1536  181 / 317, 306 / 321;       R = 2048  178 / 314, 313 / 325
//   30 % of K = 65, 275 (20, 83):               R = 1690  44.5 / 45.1, 49.0 / 49.9;   R = 8250  727 / 615, 792 / 688
constexpr int kQ16Rows = 1536;
template <int QKBITS, int PVBITS, int QSRC = 0>
static void launch_b64(int d, paro_dtype out_dtype, const AttnArgs& a, hipStream_t st) {
    constexpr int resident = QKBITS == 4 && PVBITS == 4 ? 1024 : 1280;
    const bool short_rows = a.nnz < 8LL * a.nh * a.kblocks;
    if (d == 128) launch_q16<128, QKBITS, PVBITS, QSRC>(out_dtype, a, st);
    else if (a.total_wg <= (short_rows ? resident : kQ16Rows)) launch_q16<64, QKBITS, PVBITS, QSRC>(out_dtype, a, st);
    else launch_w64<QKBITS, PVBITS, QSRC>(out_dtype, a, st);
}

template <int QKBITS, int PVBITS>
static void launch_i8(int blk, int d, paro_dtype out_dtype, const AttnArgs& a, hipStream_t st) {
    if (blk == 64) launch_b64<QKBITS, PVBITS>(d, out_dtype, a, st);
    else if (d == 64) launch_b32<64, QKBITS, PVBITS>(out_dtype, a, st);
    else launch_b32<128, QKBITS, PVBITS>(out_dtype, a, st);
}

// Q taken from the unquantized tensor (block 64 only): QSRC 1 = bf16, 2 = fp32
template <int QSRC>
static void launch_rawq(int d, int bits_pv, paro_dtype out_dtype, const AttnArgs& a, hipStream_t st) {
    if (bits_pv == 8) launch_b64<8, 8, QSRC>(d, out_dtype, a, st);
    else launch_b64<8, 4, QSRC>(d, out_dtype, a, st);
}

}  // namespace paro

namespace paro {
static int attn_entry(const char* what, const paro_shape* s, int bits_qk, int bits_pv, const void* q, const float* sq, const void* k,
                      const float* sk, const void* v, const float* sv, const int32_t* row_ptr, const int32_t* col_idx,
                      int64_t nnz, const int32_t* row_order, const uint8_t* h_perm_ids, paro_dtype out_dtype, void* op,
                      void* stream, int q_raw = 0) {
    int64_t n, kb;
    if (int st = check_shape(s, &n, &kb)) return st;
    if (q_raw) {
        if (bits_qk != 8 || (bits_pv != 8 && bits_pv != 4))
            return fail(PARO_EUNSUPPORTED, "in-kernel quantization of Q: bits (qk=%d, pv=%d), supported qk 8 with pv 8 or 4", bits_qk, bits_pv);
        if (s->block != 64) return fail(PARO_EUNSUPPORTED, "in-kernel quantization of Q needs block 64, got %d", s->block);
    }
    const bool i8 = (bits_qk == 8 || bits_qk == 4) && (bits_pv == 8 || bits_pv == 4);
    const bool b16 = bits_qk == 16 && bits_pv == 16;
    if (!i8 && !b16) {
        const bool known = (bits_qk == 8 || bits_qk == 4 || bits_qk == 16) && (bits_pv == 8 || bits_pv == 4 || bits_pv == 16);
        return fail(known ? PARO_EUNSUPPORTED : PARO_EINVAL,
                    "bits (qk=%d, pv=%d): supported pairs are qk in {8,4} with pv in {8,4}, and (16,16)", bits_qk, bits_pv);
    }
    if (out_dtype != PARO_F32 && out_dtype != PARO_BF16) return fail(PARO_EINVAL, "out_dtype=%d is not a paro_dtype", (int)out_dtype);
    if (!q || !k || !v || !op || !row_ptr) return fail(PARO_EINVAL, "q, k, v, op and row_ptr must not be NULL");
    if (i8 && ((!sq && !q_raw) || !sk || !sv)) return fail(PARO_EINVAL, "sq, sk and sv are required for integer operands");
    if (nnz < 0 || nnz > 0x7fffffffLL) return fail(PARO_EINVAL, "nnz=%lld out of range", (long long)nnz);
    if (nnz > 0 && !col_idx) return fail(PARO_EINVAL, "col_idx is NULL but nnz=%lld", (long long)nnz);
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)op) & 15) return fail(PARO_EINVAL, "q, k, v and op must be 16-byte aligned");

    AttnArgs a;
    a.q = (const uint8_t*)q;
    a.k = (const uint8_t*)k;
    a.v = (const uint8_t*)v;
    a.sq = sq;
    a.sk = sk;
    a.sv = sv;
    a.row_ptr = row_ptr;
    a.col_idx = col_idx;
    a.op = op;
    a.nnz = (int)nnz;
    a.nh = s->nh;
    a.kblocks = (int)kb;
    a.n_tokens = (int)n;
    a.total_wg = (int)((int64_t)s->B * s->nh * kb);
    a.per_xcd = (a.total_wg + 7) / 8;
    a.row_order = row_order;
    a.qk_scale = (float)(1.4426950408889634 / sqrt((double)s->d));
    a.scatter = h_perm_ids != nullptr;
    if (a.scatter) {
        if (int st = make_reorder_table(s, h_perm_ids, &a.table)) return st;
    } else {
        memset(&a.table, 0, sizeof(a.table));
    }
    if (b16) {
        const int st = out_dtype == PARO_F32 ? launch_bf16<float>(s->block, s->d, a, (hipStream_t)stream)
                                             : launch_bf16<uint16_t>(s->block, s->d, a, (hipStream_t)stream);
        if (st) return st;
    } else if (q_raw) {
        if (q_raw == 1) launch_rawq<1>(s->d, bits_pv, out_dtype, a, (hipStream_t)stream);
        else launch_rawq<2>(s->d, bits_pv, out_dtype, a, (hipStream_t)stream);
    } else if (bits_qk == 8) {
        if (bits_pv == 8) launch_i8<8, 8>(s->block, s->d, out_dtype, a, (hipStream_t)stream);
        else launch_i8<8, 4>(s->block, s->d, out_dtype, a, (hipStream_t)stream);
    } else {
        if (bits_pv == 8) launch_i8<4, 8>(s->block, s->d, out_dtype, a, (hipStream_t)stream);
        else launch_i8<4, 4>(s->block, s->d, out_dtype, a, (hipStream_t)stream);
    }
    return check_launch(what);
}
}  // namespace paro

extern "C" int paro_sparse_attn(const paro_shape* s, int bits_qk, int bits_pv, const void* q, const float* sq, const void* k,
                                const float* sk, const void* v, const float* sv, const int32_t* row_ptr,
                                const int32_t* col_idx, int64_t nnz, const int32_t* row_order, paro_dtype out_dtype, void* op,
                                void* stream) {
    return paro::attn_entry("paro_sparse_attn", s, bits_qk, bits_pv, q, sq, k, sk, v, sv, row_ptr, col_idx, nnz, row_order, nullptr,
                            out_dtype, op, stream);
}

extern "C" int paro_sparse_attn_unpermuted(const paro_shape* s, int bits_qk, int bits_pv, const void* q, const float* sq,
                                           const void* k, const float* sk, const void* v, const float* sv,
                                           const int32_t* row_ptr, const int32_t* col_idx, int64_t nnz,
                                           const int32_t* row_order, const uint8_t* h_perm_ids, paro_dtype out_dtype,
                                           void* o, void* stream) {
    if (!h_perm_ids) return paro::fail(PARO_EINVAL, "perm_ids is NULL");
    return paro::attn_entry("paro_sparse_attn_unpermuted", s, bits_qk, bits_pv, q, sq, k, sk, v, sv, row_ptr, col_idx, nnz,
                            row_order, h_perm_ids, out_dtype, o, stream);
}

extern "C" int paro_sparse_attn_unpermuted_rawq(const paro_shape* s, paro_dtype q_dtype, int bits_pv, const void* q, const void* k,
                                                const float* sk, const void* v, const float* sv, const int32_t* row_ptr,
                                                const int32_t* col_idx, int64_t nnz, const int32_t* row_order,
                                                const uint8_t* h_perm_ids, paro_dtype out_dtype, void* o, void* stream) {
    if (!h_perm_ids) return paro::fail(PARO_EINVAL, "perm_ids is NULL");
    if (q_dtype != PARO_F32 && q_dtype != PARO_BF16) return paro::fail(PARO_EINVAL, "q_dtype=%d is not a paro_dtype", (int)q_dtype);
    return paro::attn_entry("paro_sparse_attn_unpermuted_rawq", s, 8, bits_pv, q, nullptr, k, sk, v, sv, row_ptr, col_idx, nnz, row_order,
                            h_perm_ids, out_dtype, o, stream, q_dtype == PARO_BF16 ? 1 : 2);
}

#if PARO_TIMELINE
// h_records: int64 [slots][8] (HOST; start clock, end clock, column blocks visited, shader cycles of the block loop's
// phases 0..3 and of the part in front of the loop); returns the rate of the start/end clock in kHz (> 0)
// or a negative status.  Synchronises the device.
extern "C" int64_t paro_timeline_read(int64_t* h_records, int64_t slots) {
    if (!h_records || slots < 0 || slots > paro::kTimelineSlots) return PARO_EINVAL;
    if (hipMemcpyFromSymbol(h_records, HIP_SYMBOL(paro::timeline_records), sizeof(long long) * paro::kTimelineFields * (size_t)slots) != hipSuccess) return PARO_EHIP;
    int dev = 0, khz = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess) return PARO_EHIP;
    return khz;
}
#endif
