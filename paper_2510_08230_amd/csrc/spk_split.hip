// Plan-time construction of the split gathers (SplitDev in spk_internal.h;
// the product's kernels are in spk_spmv.h).
//   k_split_count: every tile group's entries per column block (an LDS
//     histogram), counts[block][group].
//   k_split_scan_sums / _scan_tops / _scan: exclusive scan of the counts in
//     that order, i.e. where a group's entries of a block begin in the stream.
//   k_split_fill: per group and tile, every entry's stream position (its column
//     goes there) and its place in the tile, in block order.
// Entries of one block within a group, and within a tile, take their
// positions and places in any order: cols, src and perm agree, and the
// products sum in storage order.
#include "spk_launch.h"
#include "spk_spmv.h"

namespace spk {
namespace {

using namespace dev;
using namespace tile;

constexpr int kScanItems = 4096;   // counts per workgroup of the scan (16 per thread)

// f(entry range of every tile of the group that takes part).
template <typename P, class F>
__device__ __forceinline__ void group_tiles(int64_t n, const P *__restrict__ rp, int64_t group, F &&f) {
    for (int t = 0; t < kSplitGroup; ++t) {
        const int64_t r0 = (group * kSplitGroup + t) * kTileRows;
        if (r0 >= n) break;
        const int64_t s = static_cast<int64_t>(rp[r0]), e = static_cast<int64_t>(rp[min(r0 + kTileRows, n)]);
        if (e > s && e - s <= kStreamCap) f(s, e);   // uniform
    }
}

template <typename P, typename I>
__global__ __launch_bounds__(kBlock) void k_split_count(int64_t n, const P *__restrict__ rp, const I *__restrict__ ci,
                                                        int blocks, int shift, int64_t groups, uint32_t *counts) {
    __shared__ uint32_t hist[kSplitBlocks];
    for (int64_t g = blockIdx.x; g < groups; g += gridDim.x) {
        for (int c = threadIdx.x; c < blocks; c += kBlock) hist[c] = 0;
        __syncthreads();
        group_tiles(n, rp, g, [&](int64_t s, int64_t e) {
            for (int64_t k = s + threadIdx.x; k < e; k += kBlock) atomicAdd(&hist[static_cast<int64_t>(ci[k]) >> shift], 1u);
        });
        __syncthreads();
        for (int c = threadIdx.x; c < blocks; c += kBlock) counts[c * groups + g] = hist[c];
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

template <typename C, typename P, typename I>
__global__ __launch_bounds__(kBlock) void k_split_fill(int64_t n, const P *__restrict__ rp, const I *__restrict__ ci,
                                                       int blocks, int shift, int64_t groups,
                                                       const uint32_t *__restrict__ starts, C *cols,
                                                       uint32_t *src, uint16_t *perm) {
    __shared__ uint32_t next[kSplitBlocks], place[kSplitBlocks];
    constexpr int U = kStreamCap / kBlock, B = kSplitBlocks / kBlock;
    const int64_t within = sizeof(C) == 2 ? (int64_t(1) << shift) - 1 : -1;
    for (int64_t g = blockIdx.x; g < groups; g += gridDim.x) {
        for (int c = threadIdx.x; c < blocks; c += kBlock) next[c] = starts[c * groups + g];
        group_tiles(n, rp, g, [&](int64_t s, int64_t e) {
            for (int c = threadIdx.x; c < kSplitBlocks; c += kBlock) place[c] = 0;
            __syncthreads();
            int64_t col[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t k = s + threadIdx.x + u * kBlock;
                col[u] = static_cast<int64_t>(ci[k < e ? k : e - 1]);
                if (k < e) atomicAdd(&place[col[u] >> shift], 1u);
            }
            __syncthreads();
            // exclusive scan over the blocks, B of them per thread
            uint32_t own[B], sum = 0, all;
#pragma unroll
            for (int i = 0; i < B; ++i) {
                own[i] = place[threadIdx.x * B + i];
                sum += own[i];
            }
            uint32_t before = block_scan(sum, &all) - sum;
#pragma unroll
            for (int i = 0; i < B; ++i) {
                place[threadIdx.x * B + i] = before;
                before += own[i];
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t k = s + threadIdx.x + u * kBlock;
                if (k >= e) continue;
                const int c = static_cast<int>(col[u] >> shift);
                const uint32_t at = atomicAdd(&next[c], 1u), p = atomicAdd(&place[c], 1u);
                cols[at] = static_cast<C>(col[u] & within);
                src[s + p] = at;
                perm[k] = static_cast<uint16_t>(p);
            }
            __syncthreads();
        });
        __syncthreads();
    }
}

// The blocks' first stream positions, and the end.
__global__ __launch_bounds__(kBlock) void k_split_starts(int blocks, int64_t groups, const uint32_t *__restrict__ starts,
                                                         const uint32_t *__restrict__ end, uint32_t *out) {
    for (int c = threadIdx.x; c <= blocks; c += kBlock) out[c] = c < blocks ? starts[c * groups] : *end;
}

size_t up256(size_t v) { return (v + 255) & ~size_t(255); }

struct Layout {
    size_t xg, cols, src, perm, start, rows, starts, sums, total;
};

int64_t groups_of(int64_t n) { return (n + int64_t(kTileRows) * kSplitGroup - 1) / (int64_t(kTileRows) * kSplitGroup); }

Layout layout(int64_t n, int64_t nnz, int blocks, int shift) {
    const size_t m = static_cast<size_t>(groups_of(n)) * blocks;
    Layout l{};
    size_t at = 0;
    auto take = [&](size_t bytes) {
        const size_t p = at;
        at += up256(bytes);
        return p;
    };
    l.xg = take(sizeof(double) * nnz);
    l.cols = take((shift <= kSplitLocal ? sizeof(uint16_t) : sizeof(int32_t)) * nnz);
    l.src = take(sizeof(uint32_t) * nnz);
    l.perm = take(sizeof(uint16_t) * nnz);
    l.start = take(sizeof(uint32_t) * (blocks + 1));
    l.rows = take(rowpack_bytes(n));
    l.starts = take(sizeof(uint32_t) * m);
    l.sums = take(sizeof(uint32_t) * ((m + kScanItems - 1) / kScanItems + 1));
    l.total = at;
    return l;
}

}  // namespace

size_t split_buffer_bytes(int64_t n_rows, int64_t nnz, int blocks, int shift) {
    return layout(n_rows, nnz, blocks, shift).total;
}

hipError_t launch_split_build(const CsrDev &A, int blocks, int shift, void *buf, unsigned *words, int grid, SplitDev *out,
                              const uint32_t **count, hipStream_t s) {
    if (blocks < 1 || blocks > kSplitBlocks || shift < 0 || A.nnz > INT32_MAX || A.n_rows < 1 ||
        ((A.n_cols - 1) >> shift) >= blocks)
        return hipErrorInvalidValue;
    const Layout l = layout(A.n_rows, A.nnz, blocks, shift);
    char *p = static_cast<char *>(buf);
    const int64_t groups = groups_of(A.n_rows), m = groups * blocks;
    const int nb = static_cast<int>((m + kScanItems - 1) / kScanItems);
    uint32_t *starts = reinterpret_cast<uint32_t *>(p + l.starts), *sums = reinterpret_cast<uint32_t *>(p + l.sums);
    uint32_t *src = reinterpret_cast<uint32_t *>(p + l.src), *start = reinterpret_cast<uint32_t *>(p + l.start);
    uint16_t *perm = reinterpret_cast<uint16_t *>(p + l.perm);
    SplitDev d;
    d.xg = p + l.xg;
    d.cols = p + l.cols;
    d.src = src;
    d.perm = perm;
    d.start = start;
    d.rows = p + l.rows;
    d.blocks = blocks;
    d.shift = shift;
    const hipError_t e = dispatch_idx(A, [&](auto rp, auto ci) {
        using P = pointee_t<decltype(rp)>;
        using I = pointee_t<decltype(ci)>;
        hipLaunchKernelGGL((k_split_count<P, I>), dim3(grid), dim3(kBlock), 0, s, A.n_rows, rp, ci, blocks, shift, groups,
                           starts);
        hipLaunchKernelGGL(k_split_scan_sums, dim3(nb), dim3(kBlock), 0, s, m, starts, sums);
        hipLaunchKernelGGL(k_split_scan_tops, dim3(1), dim3(kBlock), 0, s, nb, sums);
        hipLaunchKernelGGL(k_split_scan, dim3(nb), dim3(kBlock), 0, s, m, starts, sums);
        hipLaunchKernelGGL(k_split_starts, dim3(1), dim3(kBlock), 0, s, blocks, groups, starts, sums + nb, start);
        auto fill = [&](auto cols) {
            using C = std::remove_pointer_t<decltype(cols)>;
            hipLaunchKernelGGL((k_split_fill<C, P, I>), dim3(grid), dim3(kBlock), 0, s, A.n_rows, rp, ci, blocks, shift,
                               groups, starts, cols, src, perm);
        };
        if (shift <= kSplitLocal) fill(reinterpret_cast<uint16_t *>(p + l.cols));
        else fill(reinterpret_cast<int32_t *>(p + l.cols));
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    *out = d;
    *count = sums + nb;
    return launch_rowpack(A, const_cast<void *>(d.rows), words, grid, s);
}

}  // namespace spk
