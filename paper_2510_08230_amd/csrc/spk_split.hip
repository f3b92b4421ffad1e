// Plan-time construction of the split gathers (SplitDev in spk_internal.h;
// the product's kernels are in spk_spmv.h).
//   k_split_count: every tile's entries per column block (an LDS histogram),
//     counts[block][tile].
//   k_split_scan_sums / _scan_tops / _scan: exclusive scan of the counts in
//     that order, i.e. every segment's first stream position.
//   k_split_fill: per tile, the segment table, then every entry's stream
//     position (its column goes there) and its place in the tile's segments.
//     Entries of one segment take their places in any order: the stream and
//     perm agree, and the products sum in storage order.
// Both walks over the entries read the column indices once: 2 x 4 bytes per
// entry and 6 bytes written.
#include "spk_launch.h"
#include "spk_spmv.h"

namespace spk {
namespace {

using namespace dev;
using namespace tile;

constexpr int kScanItems = 4096;   // counts per workgroup of the scan (16 per thread)

template <typename P, typename I>
__global__ __launch_bounds__(kBlock) void k_split_count(int64_t n, const P *__restrict__ rp, const I *__restrict__ ci,
                                                        int blocks, int shift, int64_t T, uint32_t *counts) {
    __shared__ uint32_t hist[kSplitBlocks];
    for (int64_t tile = blockIdx.x; tile < T; tile += gridDim.x) {
        const int64_t r0 = tile * kTileRows, r1 = min(r0 + kTileRows, n);
        const int64_t s = static_cast<int64_t>(rp[r0]), e = static_cast<int64_t>(rp[r1]);
        if (threadIdx.x < kSplitBlocks) hist[threadIdx.x] = 0;
        __syncthreads();
        if (e - s <= kStreamCap)
            for (int64_t k = s + threadIdx.x; k < e; k += kBlock) atomicAdd(&hist[static_cast<int64_t>(ci[k]) >> shift], 1u);
        __syncthreads();
        if (static_cast<int>(threadIdx.x) < blocks) counts[threadIdx.x * T + tile] = hist[threadIdx.x];
        __syncthreads();
    }
}

// Inclusive scan over the workgroup; *total receives the sum.
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t *total) {
    __shared__ uint32_t wave[kBlock / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t u = __shfl_up(v, off, 64);
        if (lane >= off) v += u;
    }
    if (lane == 63) wave[wid] = v;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) {
        if (w < wid) before += wave[w];
        all += wave[w];
    }
    __syncthreads();
    *total = all;
    return v + before;
}

__global__ __launch_bounds__(kBlock) void k_split_scan_sums(int64_t m, const uint32_t *__restrict__ counts, uint32_t *sums) {
    uint32_t v = 0, total;
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanItems;
    for (int i = threadIdx.x; i < kScanItems; i += kBlock)
        if (base + i < m) v += counts[base + i];
    block_scan(v, &total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// One workgroup: exclusive scan of the nb sums; sums[nb] = the total.
__global__ __launch_bounds__(kBlock) void k_split_scan_tops(int nb, uint32_t *sums) {
    uint32_t carry = 0;
    for (int b0 = 0; b0 < nb; b0 += kBlock) {
        const int i = b0 + threadIdx.x;
        const uint32_t v = i < nb ? sums[i] : 0;
        uint32_t total;
        const uint32_t inc = block_scan(v, &total);
        if (i < nb) sums[i] = carry + inc - v;
        carry += total;
    }
    if (threadIdx.x == 0) sums[nb] = carry;
}

__global__ __launch_bounds__(kBlock) void k_split_scan(int64_t m, uint32_t *counts, const uint32_t *__restrict__ sums) {
    uint32_t carry = sums[blockIdx.x];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanItems;
    for (int i0 = 0; i0 < kScanItems; i0 += kBlock) {
        const int64_t i = base + i0 + threadIdx.x;
        const uint32_t v = i < m ? counts[i] : 0;
        uint32_t total;
        const uint32_t inc = block_scan(v, &total);
        if (i < m) counts[i] = carry + inc - v;
        carry += total;
    }
}

template <typename P, typename I>
__global__ __launch_bounds__(kBlock) void k_split_fill(int64_t n, const P *__restrict__ rp, const I *__restrict__ ci,
                                                       int blocks, int shift, int64_t T,
                                                       const uint32_t *__restrict__ starts, int32_t *cols,
                                                       uint16_t *perm, uint32_t *seg, uint16_t *off,
                                                       const uint32_t *__restrict__ end) {
    __shared__ uint32_t first[kSplitBlocks], place[kSplitBlocks], taken[kSplitBlocks];
    for (int64_t tile = blockIdx.x; tile < T; tile += gridDim.x) {
        const int64_t r0 = tile * kTileRows, r1 = min(r0 + kTileRows, n);
        const int64_t s = static_cast<int64_t>(rp[r0]), e = static_cast<int64_t>(rp[r1]);
        const int c = threadIdx.x;
        uint32_t g = 0, len = 0, all;
        if (c < blocks) {   // a thread per block
            const int64_t at = static_cast<int64_t>(c) * T + tile;
            g = starts[at];
            len = (at + 1 < static_cast<int64_t>(blocks) * T ? starts[at + 1] : *end) - g;
        }
        const uint32_t inc = block_scan(len, &all);
        if (c < kSplitBlocks) {
            first[c] = g;
            place[c] = inc - len;
            taken[c] = 0;
            if (c < blocks) {
                seg[tile * blocks + c] = g;
                off[tile * (blocks + 1) + c] = static_cast<uint16_t>(inc - len);
                if (c == blocks - 1) off[tile * (blocks + 1) + blocks] = static_cast<uint16_t>(inc);
            }
        }
        __syncthreads();
        if (e - s <= kStreamCap)
            for (int64_t k = s + threadIdx.x; k < e; k += kBlock) {
                const int64_t c = static_cast<int64_t>(ci[k]);
                const int b = static_cast<int>(c >> shift);
                const uint32_t r = atomicAdd(&taken[b], 1u);
                cols[first[b] + r] = static_cast<int32_t>(c);
                perm[k] = static_cast<uint16_t>(place[b] + r);
            }
        __syncthreads();
    }
}

size_t up256(size_t v) { return (v + 255) & ~size_t(255); }

struct Layout {
    size_t xg, cols, perm, seg, off, rows, starts, sums, total;
};

Layout layout(int64_t n, int64_t nnz, int blocks) {
    const size_t T = static_cast<size_t>((n + kTileRows - 1) / kTileRows), m = T * blocks;
    Layout l{};
    size_t at = 0;
    auto take = [&](size_t bytes) {
        const size_t p = at;
        at += up256(bytes);
        return p;
    };
    l.xg = take(sizeof(double) * nnz);
    l.cols = take(sizeof(int32_t) * nnz);
    l.perm = take(sizeof(uint16_t) * nnz);
    l.seg = take(sizeof(uint32_t) * m);
    l.off = take(sizeof(uint16_t) * T * (blocks + 1));
    l.rows = take(rowpack_bytes(n));
    l.starts = take(sizeof(uint32_t) * m);
    l.sums = take(sizeof(uint32_t) * ((m + kScanItems - 1) / kScanItems + 1));
    l.total = at;
    return l;
}

}  // namespace

size_t split_buffer_bytes(int64_t n_rows, int64_t nnz, int blocks) { return layout(n_rows, nnz, blocks).total; }

hipError_t launch_split_build(const CsrDev &A, int blocks, int shift, void *buf, unsigned *words, int grid, SplitDev *out,
                              const uint32_t **count, hipStream_t s) {
    if (blocks < 1 || blocks > kSplitBlocks || shift < 0 || A.nnz > INT32_MAX || A.n_rows < 1 ||
        ((A.n_cols - 1) >> shift) >= blocks)
        return hipErrorInvalidValue;
    const Layout l = layout(A.n_rows, A.nnz, blocks);
    char *p = static_cast<char *>(buf);
    const int64_t T = (A.n_rows + kTileRows - 1) / kTileRows, m = T * blocks;
    const int nb = static_cast<int>((m + kScanItems - 1) / kScanItems);
    uint32_t *starts = reinterpret_cast<uint32_t *>(p + l.starts), *sums = reinterpret_cast<uint32_t *>(p + l.sums);
    SplitDev d;
    d.xg = p + l.xg;
    d.cols = reinterpret_cast<int32_t *>(p + l.cols);
    d.perm = reinterpret_cast<uint16_t *>(p + l.perm);
    d.seg = reinterpret_cast<uint32_t *>(p + l.seg);
    d.off = reinterpret_cast<uint16_t *>(p + l.off);
    d.rows = p + l.rows;
    d.blocks = blocks;
    d.shift = shift;
    const hipError_t e = dispatch_idx(A, [&](auto rp, auto ci) {
        using P = pointee_t<decltype(rp)>;
        using I = pointee_t<decltype(ci)>;
        hipLaunchKernelGGL((k_split_count<P, I>), dim3(grid), dim3(kBlock), 0, s, A.n_rows, rp, ci, blocks, shift, T, starts);
        hipLaunchKernelGGL(k_split_scan_sums, dim3(nb), dim3(kBlock), 0, s, m, starts, sums);
        hipLaunchKernelGGL(k_split_scan_tops, dim3(1), dim3(kBlock), 0, s, nb, sums);
        hipLaunchKernelGGL(k_split_scan, dim3(nb), dim3(kBlock), 0, s, m, starts, sums);
        hipLaunchKernelGGL((k_split_fill<P, I>), dim3(grid), dim3(kBlock), 0, s, A.n_rows, rp, ci, blocks, shift, T, starts,
                           const_cast<int32_t *>(d.cols), const_cast<uint16_t *>(d.perm), const_cast<uint32_t *>(d.seg),
                           const_cast<uint16_t *>(d.off), sums + nb);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    *out = d;
    *count = sums + nb;
    return launch_rowpack(A, const_cast<void *>(d.rows), words, grid, s);
}

}  // namespace spk
