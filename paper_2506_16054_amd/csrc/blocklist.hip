// Device-side expansion of per-head block bitmasks into the compacted live-block list that
// paro_sparse_attn walks (paper Sec. 4.2 (1): masks are kept as bitmasks, 9.2 KB per head, and
// prefetched per transformer block and timestep; App. C "Overhead of Prefetch": the load of the
// next mask overlaps the attention of the current one through two buffers).  The caller copies the
// next bitmask to the GPU on a side stream and enqueues this expansion behind the copy; nothing
// here touches the host.
//
// Masks of up to kOneLaunchBytes in all go through ONE launch (blocklist_whole_kernel); larger ones through three:
//   1. count:  c[h][i] = live blocks of row block i of head h, c[h][k] = 0, stored in row_ptr;
//   2. scan:   in-place exclusive prefix sum over the flat [nh][k+1] array by one workgroup, which
//              yields exactly the offsets of the list (row_ptr[h][k] = end of head h = start of
//              head h+1), and the total;
//   3. fill:   one wavefront per row block writes its live columns in ascending order (ballot +
//              prefix popcount keeps the order without atomics).
#include "common.h"

namespace paro {

// Number of set bits among bits [bit0, bit0 + nbits) of a little-endian bit string.
__device__ inline int count_bits(const uint8_t* bm, int bit0, int nbits) {
    int cnt = 0;
    int pos = bit0;
    const int end = bit0 + nbits;
    while (pos < end) {
        const int lo = pos & 7;
        const int take = min(8 - lo, end - pos);
        cnt += __popc(((unsigned)bm[pos >> 3] >> lo) & ((1u << take) - 1u));
        pos += take;
    }
    return cnt;
}

__global__ __launch_bounds__(256) void blocklist_count_kernel(int nh, int k, int nbytes, const uint8_t* __restrict__ bitmask,
                                                              int* __restrict__ row_ptr) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= nh * (k + 1)) return;
    const int h = e / (k + 1);
    const int i = e - h * (k + 1);
    row_ptr[e] = i < k ? count_bits(bitmask + (size_t)h * nbytes, i * k, k) : 0;
}

constexpr int kScanThreads = 1024;

__global__ __launch_bounds__(kScanThreads) void blocklist_scan_kernel(int n, int* __restrict__ row_ptr, int* __restrict__ nnz_out) {
    __shared__ int part[kScanThreads];
    const int t = threadIdx.x;
    const int per = (n + kScanThreads - 1) / kScanThreads;
    const int lo = min(t * per, n), hi = min(lo + per, n);
    int sum = 0;
    for (int e = lo; e < hi; ++e) sum += row_ptr[e];
    part[t] = sum;
    __syncthreads();
    // inclusive Hillis-Steele scan over the 1024 partial sums
    for (int off = 1; off < kScanThreads; off <<= 1) {
        const int add = t >= off ? part[t - off] : 0;
        __syncthreads();
        part[t] += add;
        __syncthreads();
    }
    int run = part[t] - sum;  // exclusive prefix of this thread's chunk
    for (int e = lo; e < hi; ++e) {
        const int c = row_ptr[e];
        row_ptr[e] = run;
        run += c;
    }
    if (nnz_out && t == kScanThreads - 1) *nnz_out = part[t];
}

__global__ __launch_bounds__(256) void blocklist_fill_kernel(int nh, int k, int nbytes, const uint8_t* __restrict__ bitmask,
                                                             const int* __restrict__ row_ptr, int* __restrict__ col_idx, int cap) {
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= nh * k) return;
    const int lane = threadIdx.x & 63;
    const int h = row / k;
    const int i = row - h * k;
    const uint8_t* bm = bitmask + (size_t)h * nbytes;
    int base = row_ptr[h * (k + 1) + i];
    for (int j0 = 0; j0 < k; j0 += 64) {
        const int j = j0 + lane;
        const int bit = i * k + j;
        const bool live = j < k && ((bm[bit >> 3] >> (bit & 7)) & 1);
        const unsigned long long b = __ballot(live);
        const int pos = base + __popcll(b & ((1ull << lane) - 1ull));
        if (live && (unsigned)pos < (unsigned)cap) col_idx[pos] = j;  // entries outside [0, cap) are dropped, never written
        base += __popcll(b);
    }
}

// The whole expansion in one launch.  A workgroup owns `per_wg` consecutive row blocks of the flat [nh][k] array.  Where its part of
// the list starts is the number of live blocks in front of it, which it counts itself, straight from the masks: they
// are a few hundred KB that every XCD's L2 holds, and reading on average half of them (16 bytes per lane and load) takes less than
// a launch that waits for the one before it.  Bound by the last workgroup's counting (at the size below 454 KB through one
// compute unit, 3.4 us at 64 bytes a cycle, in four rounds of seven loads per thread) and by what stands before and behind
// it: 48 masks of 275 x 275 blocks take 10.0 us a call, against 13.1 with half as many threads and 14 rounds of four loads, and
// 24.6 us for the three launches (a thread per row reading single bytes, a scan by one workgroup, the fill).  The first
// round's loads travel while the workgroup's own rows are staged.  4, 10 and 14 loads in flight: 10.3, 10.4, 10.4; a
// wavefront per row in the staging: 10.4.
constexpr int kWholeThreads = 1024;
constexpr int kWholeMaxRows = kWholeThreads;  // a thread per row in the scan
constexpr int kWholeGroups = 256;             // one workgroup per compute unit
constexpr int kWholeFlight = 7;               // pieces of 16 bytes that a thread has in flight
// Counting what lies in front grows with the square of the masks' size, the three launches with the size.  At 1 MB the one
// launch is still ahead (30 heads of 512 x 512 blocks: 17.5 against 41.8 us; 1 of 2896 x 2896: 21.4 against 65.7; 256 of
// 181 x 181: 20.7 against 94.3); beyond it the rows of a workgroup outgrow their 8 KB of LDS.
constexpr int64_t kOneLaunchBytes = 1 << 20;
constexpr int kWholeStage = 8192;             // bytes of a workgroup's own rows, see launch_whole

__global__ __launch_bounds__(kWholeThreads) void blocklist_whole_kernel(int nh, int k, int nbytes, int per_wg, const uint8_t* __restrict__ bitmask,
                                                                        int* __restrict__ row_ptr, int* __restrict__ col_idx, int cap,
                                                                        int* __restrict__ nnz_out) {
    __shared__ unsigned stage[kWholeStage / 4 + 2];  // the bytes of this workgroup's rows, row after row, each from a word of its own
    __shared__ int start[kWholeMaxRows + 1];
    __shared__ int part[2][kWholeThreads / 64];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int rows = nh * k;
    const int r0 = blockIdx.x * per_wg, r1 = min(r0 + per_wg, rows);
    if (r0 >= r1) return;
    const int words = (k + 31) / 32 + 1;  // words that a row's bits can touch, counted from the byte its first bit is in

    // ---- live blocks in front of row r0: whole bytes [0, whole) of the masks, minus the bits behind every finished
    // head's last block, plus the bits of the byte that row r0 starts in
    const int h0 = r0 / k, bit0 = (r0 - h0 * k) * k;
    const int whole = h0 * nbytes + (bit0 >> 3);
    const int head = min(whole, (int)(-(uintptr_t)bitmask & 15u));  // bytes in front of the first aligned piece
    const int pieces = (whole - head) >> 4;
    const uint4* src16 = (const uint4*)(bitmask + head);
    uint4 x[kWholeFlight];
    auto request = [&](int p0) {  // a piece past the last one is read as the first one (there is one) and not counted
#pragma unroll
        for (int u = 0; u < kWholeFlight; ++u) {
            const int p = p0 + u * kWholeThreads;
            x[u] = src16[p < pieces ? p : 0];
        }
    };
    int before = 0;
    auto count = [&](int p0) {
#pragma unroll
        for (int u = 0; u < kWholeFlight; ++u) {
            const int n = __popc(x[u].x) + __popc(x[u].y) + __popc(x[u].z) + __popc(x[u].w);
            before += p0 + u * kWholeThreads < pieces ? n : 0;
        }
    };
    if (pieces > 0) request(t);

    // ---- while those travel, this workgroup's rows: bits i k .. i k + k - 1 of head h, from the byte that holds the first of them
    uint8_t* bytes = (uint8_t*)stage;
    const int row_bytes = 4 * words;
    for (int e = t; e < (r1 - r0) * row_bytes; e += kWholeThreads) {
        const int r = r0 + e / row_bytes, b = e % row_bytes;
        const int h = r / k, i = r - h * k;
        const int at = ((i * k) >> 3) + b;
        bytes[e] = at < nbytes ? bitmask[(size_t)h * nbytes + at] : (uint8_t)0;
    }

    if (pieces > 0) {
        count(t);
        for (int p0 = t + kWholeFlight * kWholeThreads; p0 - t < pieces; p0 += kWholeFlight * kWholeThreads) {
            request(p0);
            count(p0);
        }
    }
    {
        const int rest = head + 16 * pieces;  // at most 15 bytes on either side of the pieces
        if (t < head) before += __popc((unsigned)bitmask[t]);
        if (t < whole - rest) before += __popc((unsigned)bitmask[rest + t]);
        const int unused = 8 * nbytes - k * k;
        if (t < h0 && unused) before -= __popc((unsigned)bitmask[(size_t)(t + 1) * nbytes - 1] >> (8 - unused));
        if (t == 0 && (bit0 & 7)) before += __popc((unsigned)bitmask[whole] & ((1u << (bit0 & 7)) - 1u));
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) before += __shfl_xor(before, off);
    if (lane == 0) part[0][w] = before;
    __syncthreads();  // and the rows are staged

    // ---- live blocks of every own row, and their running sum
    int own = 0;
    if (r0 + t < r1) {
        const int i = (r0 + t) % k;
        const unsigned* src = stage + t * words;
        const int shift = (i * k) & 7;
        for (int b = 0; b < k; b += 32) {
            const unsigned x = __builtin_amdgcn_alignbit(src[b / 32 + 1], src[b / 32], shift);
            own += __popc(k - b >= 32 ? x : x & ((1u << (k - b)) - 1u));
        }
    }
    int run = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(run, off);
        run += lane >= off ? up : 0;
    }
    if (lane == 63) part[1][w] = run;
    __syncthreads();
    int base = 0;
#pragma unroll
    for (int v = 0; v < kWholeThreads / 64; ++v) base += part[0][v] + (v < w ? part[1][v] : 0);
    if (r0 + t < r1) {
        const int r = r0 + t, h = r / k, i = r - h * k;
        start[t] = base + run - own;
        row_ptr[r + h] = base + run - own;
        if (i == k - 1) row_ptr[r + h + 1] = base + run;
        if (r == rows - 1 && nnz_out) *nnz_out = base + run;
    }
    __syncthreads();

    // ---- the columns: a wavefront per row, 64 columns at a time in ascending order
    if (cap == 0) return;
    for (int r = w; r < r1 - r0; r += kWholeThreads / 64) {
        const int i = (r0 + r) % k;
        const unsigned* src = stage + r * words;
        const int shift = (i * k) & 7;
        int pos0 = start[r];
        for (int j0 = 0; j0 < k; j0 += 64) {
            const int j = j0 + lane;
            const int bit = j + shift;
            const bool live = j < k && ((src[bit >> 5] >> (bit & 31)) & 1u);
            const unsigned long long b = __ballot(live);
            const int pos = pos0 + __popcll(b & ((1ull << lane) - 1ull));
            if (live && (unsigned)pos < (unsigned)cap) col_idx[pos] = j;  // entries outside [0, cap) are dropped, never written
            pos0 += __popcll(b);
        }
    }
}

// Rows per workgroup of the one-launch form, or 0 where it does not apply.
static int whole_rows_per_group(int nh, int k, int nbytes) {
    if ((int64_t)nh * nbytes > kOneLaunchBytes) return 0;
    const int64_t per = ((int64_t)nh * k + kWholeGroups - 1) / kWholeGroups;
    const int64_t row_bytes = 4 * ((k + 31) / 32 + 1);
    return per <= kWholeMaxRows && per * row_bytes <= kWholeStage ? (int)per : 0;
}

}  // namespace paro

extern "C" int paro_mask_to_blocklist_device(int nh, int k, const uint8_t* bitmask, int32_t* row_ptr, int32_t* col_idx,
                                             int64_t cap, int32_t* nnz_out, void* stream) {
    using namespace paro;
    if (nh < 1 || nh > kMaxHeads) return fail(PARO_EINVAL, "nh=%d out of range [1, %d]", nh, kMaxHeads);
    if (k < 1 || k > 32768) return fail(PARO_EINVAL, "k=%d out of range [1, 32768]", k);
    if (!bitmask || !row_ptr) return fail(PARO_EINVAL, "bitmask and row_ptr must not be NULL");
    if (cap < 0 || cap > 0x7fffffffLL) return fail(PARO_EINVAL, "cap=%lld out of range", (long long)cap);
    if (cap > 0 && !col_idx) return fail(PARO_EINVAL, "col_idx is NULL but cap=%lld", (long long)cap);
    if ((int64_t)nh * k * k > 0x7fffffffLL) return fail(PARO_EINVAL, "nh*k*k = %lld live blocks cannot be indexed with int32", (long long)nh * k * k);
    const int nbytes = (int)(((int64_t)k * k + 7) / 8);
    const int n = nh * (k + 1);
    hipStream_t st = (hipStream_t)stream;
    if (const int per = whole_rows_per_group(nh, k, nbytes)) {
        hipLaunchKernelGGL(blocklist_whole_kernel, dim3((unsigned)((nh * k + per - 1) / per)), dim3(kWholeThreads), 0, st, nh, k, nbytes, per, bitmask,
                           row_ptr, col_idx, (int)cap, nnz_out);
        return check_launch("paro_mask_to_blocklist_device");
    }
    hipLaunchKernelGGL(blocklist_count_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, nh, k, nbytes, bitmask, row_ptr);
    hipLaunchKernelGGL(blocklist_scan_kernel, dim3(1), dim3(kScanThreads), 0, st, n, row_ptr, nnz_out);
    if (cap > 0)
        hipLaunchKernelGGL(blocklist_fill_kernel, dim3((unsigned)((nh * k + 3) / 4)), dim3(256), 0, st, nh, k, nbytes, bitmask, row_ptr,
                           col_idx, (int)cap);
    return check_launch("paro_mask_to_blocklist_device");
}

extern "C" int paro_blocklist_cols_device(int nh, int k, const uint8_t* bitmask, const int32_t* row_ptr, int32_t* col_idx,
                                          int64_t cap, void* stream) {
    using namespace paro;
    if (nh < 1 || nh > kMaxHeads) return fail(PARO_EINVAL, "nh=%d out of range [1, %d]", nh, kMaxHeads);
    if (k < 1 || k > 32768) return fail(PARO_EINVAL, "k=%d out of range [1, 32768]", k);
    if (!bitmask || !row_ptr || !col_idx) return fail(PARO_EINVAL, "bitmask, row_ptr and col_idx must not be NULL");
    if (cap < 1 || cap > 0x7fffffffLL) return fail(PARO_EINVAL, "cap=%lld out of range", (long long)cap);
    if ((int64_t)nh * k * k > 0x7fffffffLL) return fail(PARO_EINVAL, "nh*k*k = %lld live blocks cannot be indexed with int32", (long long)nh * k * k);
    const int nbytes = (int)(((int64_t)k * k + 7) / 8);
    hipLaunchKernelGGL(blocklist_fill_kernel, dim3((unsigned)((nh * k + 3) / 4)), dim3(256), 0, (hipStream_t)stream, nh, k, nbytes, bitmask,
                       row_ptr, col_idx, (int)cap);
    return check_launch("paro_blocklist_cols_device");
}
