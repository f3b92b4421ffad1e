// The SpMV tilings and their launch helper, shared by the kernel sources.
//
//   * LDS-staged row tiles: a workgroup owns 256 consecutive rows; it streams
//     the tile's values and column indices from HBM into LDS with fully
//     coalesced loads (one contiguous nnz range per tile), then each thread
//     reduces one row from LDS while gathering x.  Tiles whose nnz exceed the
//     LDS capacity fall back to direct loads.
//   * lanes-per-row vector kernel: 2^k lanes of a wave64 share a row.
// Both hand each row sum to an epilogue object (row(i, s), finish()), which is
// where the solvers fuse their elementwise work and dot-product partials.
// The LDS tiles also read a plan's compressed index arrays: one-byte column
// codes (I = Code8: column = row + offset table[code], the table in LDS) and
// packed row pointers (P = RowPack: an int64 per tile, a uint16 per row);
// row sums keep their order, so the products equal the plain ones bit for bit.
#pragma once

#include "spk_device.h"

#include <algorithm>
#include <type_traits>
#include <utility>

namespace spk {
namespace tile {

using namespace dev;

// Partial-sum slab k of the workspace.
inline double *site(double *partials, int k) { return partials + static_cast<size_t>(k) * kSiteWidth * kMaxGrid; }

template <typename T>
struct Vec16 {
    static constexpr int W = 16 / sizeof(T);
    typedef T type __attribute__((ext_vector_type(W)));
};

// Entry range [a, b) of one row (long-row pass: the bounds are loaded again
// rather than kept live through the per-lane row loop).
template <typename P>
__device__ __forceinline__ void row_range(const P *__restrict__ rp, int64_t n, int64_t row, int64_t &a, int64_t &b) {
    a = static_cast<int64_t>(rp[row]);
    b = static_cast<int64_t>(rp[row + 1]);
}

template <>
__device__ __forceinline__ void row_range<RowPack>(const RowPack *__restrict__ rp, int64_t n, int64_t row, int64_t &a,
                                                   int64_t &b) {
    const int64_t *tb = reinterpret_cast<const int64_t *>(rp);
    const uint16_t *ro = reinterpret_cast<const uint16_t *>(tb + (n + kTileRows - 1) / kTileRows + 1);
    const int64_t tile = row / kTileRows;
    const int64_t r1 = min((tile + 1) * static_cast<int64_t>(kTileRows), n);
    a = tb[tile] + ro[row];
    b = row + 1 < r1 ? tb[tile] + ro[row + 1] : tb[tile + 1];
}

// Sum of entries [a, b) of one row (b - a <= kLongPiece) by the whole
// workgroup, the same in every thread: each thread its strided share in
// storage order with every load in flight before the first use, then the wave
// sums and the four wave totals in a fixed order.  val(k) / cix(k): entry k's
// value and stored column.  Every thread of the workgroup calls this.
template <typename C, class Gx, class D, class Val, class Cix>
__device__ __forceinline__ C piece_sum(int64_t a, int64_t b, int64_t row, const Gx &gx, const D &col, const Val &val,
                                       const Cix &cix) {
    __shared__ C s_red[kBlock / 64];
    constexpr int U = kLongPiece / kBlock;
    C av[U], xv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t k = a + threadIdx.x + u * kBlock;
        const int64_t kc = k < b ? k : b - 1;   // every lane loads
        av[u] = static_cast<C>(widen(val(kc)));
        xv[u] = static_cast<C>(gx(col(cix(kc), row)));
    }
    C acc = 0;
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (a + threadIdx.x + u * kBlock < b) acc = fma(av[u], xv[u], acc);
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = acc;
    __syncthreads();
    C t = s_red[0];
#pragma unroll
    for (int v = 1; v < kBlock / 64; ++v) t += s_red[v];
    __syncthreads();   // s_red is reused by the next piece
    return t;
}

// The rows of the tile at r0 whose flag lng is set (rows longer than the
// long-row limit), summed one at a time by the whole workgroup in ascending
// row order, piece by piece, and handed to epi.row by the row's own thread
// (for products that form their input vector on the fly; the others have
// their pieces summed ahead, k_long_pieces, in the same order).  Every thread
// of the workgroup calls this (it synchronises); the flags go through LDS as
// one ballot per wave, so nothing of the per-lane row loop stays live for it.
// val(k) / cix(k) read global memory, also for a tile staged in LDS: one call
// site keeps the kernel's register count down.
template <typename C, typename P, class Gx, class D, class Epi, class Val, class Cix>
__device__ __forceinline__ void long_rows(bool lng, const P *__restrict__ rp, int64_t n, int64_t r0, const Gx &gx,
                                          const D &col, Epi &epi, const Val &val, const Cix &cix) {
    __shared__ unsigned long long s_mask[kBlock / 64];
    const unsigned long long m = __ballot(lng);
    if ((threadIdx.x & 63) == 0) s_mask[threadIdx.x >> 6] = m;
    __syncthreads();
#pragma unroll 1
    for (int w = 0; w < kBlock / 64; ++w) {
        unsigned long long left = s_mask[w];
        while (left != 0) {   // the same in every thread
            const int i = w * 64 + __builtin_ctzll(left);
            left &= left - 1;
            const int64_t row = r0 + i;
            int64_t ra, rb;
            row_range(rp, n, row, ra, rb);
            C acc = 0;
#pragma unroll 1
            for (int64_t k = ra; k < rb; k += kLongPiece)
                acc += piece_sum<C>(k, k + kLongPiece < rb ? k + kLongPiece : rb, row, gx, col, val, cix);
            if (static_cast<int>(threadIdx.x) == i) epi.row(row, acc);
        }
    }
    __syncthreads();           // s_mask is rewritten by the next tile
}

// What a kernel needs of the long rows' pieces: nothing unless its LR is 2.
template <int LR>
struct LongArg {};
template <>
struct LongArg<2> {
    const int32_t *base;
    const double *sums;
    // a long row's sum, from its pieces in order
    template <typename C>
    __device__ __forceinline__ C sum(int64_t row, int64_t len) const {
        const int32_t at = base[row];
        const int np = static_cast<int>((len + kLongPiece - 1) / kLongPiece);
        C t = 0;
        for (int p = 0; p < np; ++p) t += static_cast<C>(sums[at + p]);
        return t;
    }
};

// Epilogue operands loaded with the tile: an epilogue that reads a vector at
// its row (p_i for p.q, b_i for a residual) may provide pre(i), returning
// that value, and row(i, sum, value).  The tile loop then issues the load
// beside the tile's DMA, whose wait covers it, instead of after the row sum,
// where it would add a memory round trip to every tile.
template <class Epi, class = void>
struct HasPre : std::false_type {};
template <class Epi>
struct HasPre<Epi, std::void_t<decltype(std::declval<const Epi &>().pre(int64_t(0)))>> : std::true_type {};

struct NoPre {};

template <class Epi>
__device__ __forceinline__ auto pre_of(const Epi &epi, int64_t i) {
    if constexpr (HasPre<Epi>::value) return epi.pre(i);
    else return NoPre{};
}

template <class Epi, class C, class Pv>
__device__ __forceinline__ void emit_row(Epi &epi, int64_t i, C sum, const Pv &pv) {
    if constexpr (std::is_same_v<Pv, NoPre>) epi.row(i, sum);
    else epi.row(i, sum, pv);
}

// LDS-staged row tiles: DMA the tile's values and columns into LDS, then one
// thread per row reduces from LDS while gathering x.  Occupancy (several
// workgroups per CU) overlaps one workgroup's DMA with another's gathers.
// The tile loop of the LDS-staged SpMV, shared by the per-launch kernel and the
// persistent CG kernel: calls epi.row(row, sum) for every row of the tiles
// this workgroup visits.  lv / lc: the workgroup's LDS staging buffers.
// LR (the matrix has rows longer than kLongRow entries): 1: those rows are
// summed by the whole workgroup (long_rows), so a hub row does not serialise
// its tile on one lane; 2: their pieces have been summed by an earlier launch
// (lra), so a tile with a hub row is not the launch's tail either.  A
// compile-time switch: the passes cost registers, and with one in every
// instance the kernels without hub rows lost a workgroup per CU.
template <typename V, typename P, typename I, typename C, int LR, class Gx, class Epi, class D = ColPlain>
__device__ __forceinline__ void spmv_tiles_lds(int64_t n, int64_t nnz, const P *__restrict__ rp,
                                               const I *__restrict__ ci, const V *__restrict__ va, const Gx &gx,
                                               int remap, int nt, int pf, Epi &epi, u32x4 *lv, u32x4 *lc,
                                               const D &col = D{}, uint32_t walkers = 0,
                                               const LongArg<LR> &lra = LongArg<LR>{}) {
    const V *sv = reinterpret_cast<const V *>(lv);
    const I *sc = reinterpret_cast<const I *>(lc);
    const int64_t T = (n + kTileRows - 1) / kTileRows;
    TileIter it(T, remap, walkers ? walkers : gridDim.x);
    if (!it.valid()) return;
    // pf = 1: the row pointers of the next tile are loaded while the current
    // tile's entries stream in, so each tile starts with its bounds at hand.
    TileMeta<P> cur, nxt;
    cur.load(rp, n, it.tile());
    while (true) {
        TileIter after = it;
        after.next();
        const bool more = after.valid();
        const int64_t r1 = min(cur.r0 + static_cast<int64_t>(kTileRows), n);
        const int64_t row = cur.r0 + threadIdx.x;
        const int64_t s = cur.first(), e = cur.end();
        const int64_t a = cur.lo(), b = cur.hi();
        const bool lng = LR != 0 && row < r1 && b - a > kLongRow;
        if (e - s <= kStreamCap) {
            dma_chunks<V>(va, s, e, nnz, lv, nt);
            dma_chunks<I>(ci, s, e, nnz, lc, nt);
            if (more && pf) nxt.load(rp, n, after.tile());
            const auto pv = pre_of(epi, row < r1 ? row : r1 - 1);   // every lane loads
            __builtin_amdgcn_s_waitcnt(0);   // this wave's DMA (and the prefetches) has landed
            __syncthreads();                 // ... and every other wave's
            // The row sums run at raised wave priority, so on a SIMD shared
            // with workgroups that are issuing or awaiting their next tile's
            // DMA they finish first and free their LDS sooner.
            __builtin_amdgcn_s_setprio(2);
            const int64_t s0v = s & ~static_cast<int64_t>(Chunks<V>::EPC - 1);
            const int64_t s0c = s & ~static_cast<int64_t>(Chunks<I>::EPC - 1);
            if (row < r1 && !lng) emit_row(epi, row, row_from_lds<V, I, C>(sv, sc, a, b, s0v, s0c, gx, col, row), pv);
            __builtin_amdgcn_s_setprio(0);
            lds_barrier();                   // LDS free for the next tile (the row's stores stay in flight)
        } else {
            if (more && pf) nxt.load(rp, n, after.tile());
            const auto pv = pre_of(epi, row < r1 ? row : r1 - 1);
            if (row < r1 && !lng)
                emit_row(epi, row, row_from_global<V, I, C, LR == 2 ? kRowUnroll : 1>(va, ci, a, b, gx, nt, col, row), pv);
        }
        if constexpr (LR == 2) {
            if (lng) epi.row(row, lra.template sum<C>(row, b - a));
        }
        if constexpr (LR == 1)
            long_rows<C>(lng, rp, n, cur.r0, gx, col, epi, [&](int64_t k) { return ldv(va + k, nt); },
                         [&](int64_t k) { return ci[k]; });
        if (!more) break;
        if (!pf) nxt.load(rp, n, after.tile());
        it = after;
        cur = nxt;
    }
}

// The gather of the product's input vector: x[c] itself, unless the epilogue
// forms the vector on the fly (it then provides gather(), e.g. the fused CG
// step, whose direction p_k = r_{k-1} - alpha q_{k-1} + beta p_{k-1} is
// formed at every gathered column).
template <class Epi, class = void>
struct HasGather : std::false_type {};
template <class Epi>
struct HasGather<Epi, std::void_t<decltype(std::declval<const Epi &>().gather())>> : std::true_type {};

template <typename X, typename C, class Epi>
__device__ __forceinline__ auto gather_of(const Epi &epi, const X *x) {
    if constexpr (HasGather<Epi>::value) return epi.gather();
    else return PlainGather<X, C>{x};
}

// Register budget of the row-tile kernel, as waves per SIMD it must fit: the
// CG loop's product on coded FP64 tiles with packed rows (an epilogue that
// declares kHotLoop) is held to seven, where it otherwise lands one
// register above the budget and loses a workgroup per CU to it; every other
// instance is left to the compiler.
template <class Epi, class = void>
struct HotLoop : std::false_type {};
template <class Epi>
struct HotLoop<Epi, std::void_t<decltype(Epi::kHotLoop)>> : std::bool_constant<Epi::kHotLoop> {};

template <typename V, typename P, class Epi>
constexpr int spmv_min_waves() {
    return std::is_same_v<V, double> && std::is_same_v<P, RowPack> && HotLoop<Epi>::value ? 7 : 1;
}

// walkers: the workgroups that walk the tiles (0 = all).  A grid sized for
// the autotuned kernel can exceed what another epilogue's kernel holds
// resident; the workgroups past the resident count would then start only
// when the first ones finish and walk their tiles alone.  They take no
// tiles instead and store zero partials, so a consumer still sums one
// partial per launched workgroup and gets the same total.
template <typename V, typename P, typename I, typename X, typename C, class Epi, int LR = 0>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(spmv_min_waves<V, P, Epi>()))) void k_spmv_stream(int64_t n, int64_t nnz, const P *__restrict__ rp,
                                                        const I *__restrict__ ci, const V *__restrict__ va,
                                                        const X *__restrict__ x, int remap, int nt, int pf,
                                                        int walkers, Epi epi_in, LongArg<LR> lra) {
    Epi epi = epi_in;
    if (epi.skip()) return;
    const uint32_t W = walkers > 0 && static_cast<uint32_t>(walkers) < gridDim.x ? walkers : gridDim.x;
    if (blockIdx.x >= W) {   // uniform
        epi.finish();
        return;
    }
    __shared__ u32x4 lv[Chunks<V>::LDS];
    __shared__ u32x4 lc[Chunks<I>::LDS];
    if constexpr (std::is_same_v<I, Code8>) {
        // the offset table sits in the kCodeDict * 8 bytes before the codes
        __shared__ int64_t dict[kCodeDict];
        const int64_t *g = reinterpret_cast<const int64_t *>(ci) - kCodeDict;
        for (int i = threadIdx.x; i < kCodeDict; i += kBlock) dict[i] = g[i];
        __syncthreads();
        spmv_tiles_lds<V, P, I, C, LR>(n, nnz, rp, ci, va, gather_of<X, C>(epi, x), remap, nt, pf, epi, lv, lc,
                                       ColCoded{dict}, W);
    } else {
        spmv_tiles_lds<V, P, I, C, LR>(n, nnz, rp, ci, va, gather_of<X, C>(epi, x), remap, nt, pf, epi, lv, lc,
                                       ColPlain{}, W, lra);
    }
    epi.finish();
}

// Sums of the long rows' pieces, one workgroup each, ahead of the row tiles.
// A hub row of 10^4 entries otherwise holds up its tile's workgroup (or, in
// the lanes-per-row kernel, its lanes) long after the rest of the matrix is
// done: 205-250 us for a product of 7.1e6 FP16 entries with 16 hubs, now 54, of
// which the other rows take 38.
template <typename V, typename I, typename X, typename C, class Epi>
__global__ __launch_bounds__(kBlock) void k_long_pieces(const LongPiece *__restrict__ pieces, int np,
                                                        const I *__restrict__ ci, const V *__restrict__ va,
                                                        const X *__restrict__ x, int nt, double *__restrict__ sums,
                                                        Epi epi) {
    if (epi.skip()) return;
    const PlainGather<X, C> gx{x};
    for (int p = blockIdx.x; p < np; p += gridDim.x) {
        const LongPiece pc = pieces[p];
        const C t = piece_sum<C>(pc.first, pc.first + pc.len, pc.row, gx, ColPlain{},
                                 [&](int64_t k) { return ldv(va + k, nt); }, [&](int64_t k) { return ci[k]; });
        if (threadIdx.x == 0) sums[p] = static_cast<double>(t);
    }
}

template <typename V, typename P, typename I, typename C, class Gx, class Epi>
__device__ __forceinline__ void spmv_tiles_vector(int64_t n, const P *__restrict__ rp, const I *__restrict__ ci,
                                                  const V *__restrict__ va, const Gx &gx, int lanes_log2, int remap,
                                                  int nt, Epi &epi) {
    const int L = 1 << lanes_log2;
    const int lane = threadIdx.x & (L - 1);
    const int group = threadIdx.x >> lanes_log2;
    const int groups = kBlock >> lanes_log2;
    const int64_t T = (n + kTileRows - 1) / kTileRows;
    for (TileIter it(T, remap); it.valid(); it.next()) {
        const int64_t r0 = it.tile() * kTileRows;
        const int64_t r1 = min(r0 + (int64_t)kTileRows, n);
        for (int pass = 0; pass < L; ++pass) {
            const int64_t row = r0 + static_cast<int64_t>(pass) * groups + group;
            C sum = 0;
            if (row < r1) {
                const int64_t a = static_cast<int64_t>(rp[row]), b = static_cast<int64_t>(rp[row + 1]);
                for (int64_t k = a + lane; k < b; k += L)
                    sum = fma(static_cast<C>(widen(ldv(va + k, nt))), static_cast<C>(gx(static_cast<int64_t>(ci[k]))),
                              sum);
            }
            for (int off = L >> 1; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
            if (row < r1 && lane == 0) epi.row(row, sum);
        }
    }
}

template <typename V, typename P, typename I, typename X, typename C, class Epi>
__global__ __launch_bounds__(kBlock) void k_spmv_vector(int64_t n, const P *__restrict__ rp,
                                                        const I *__restrict__ ci, const V *__restrict__ va,
                                                        const X *__restrict__ x, int lanes_log2, int remap,
                                                        int nt, Epi epi_in) {
    Epi epi = epi_in;
    if (epi.skip()) return;
    spmv_tiles_vector<V, P, I, C>(n, rp, ci, va, gather_of<X, C>(epi, x), lanes_log2, remap, nt, epi);
    epi.finish();
}

// ---- row patterns (RowPatterns) ---------------------------------------------------
// A structured grid's rows repeat a few sequences of column offsets (a 7-point
// stencil's 27), so one byte per row names them all, and in a wave whose rows
// share one sequence the offsets are scalars: an entry costs one LDS read (its
// value) and one load at a scalar base, where a column code costs three LDS
// reads and 64-bit address arithmetic per lane.  That row work, not the
// stream, is what the coded tiles wait for (stencil7 N = 215 FP64: tiles
// streamed into LDS alone 97 us, with the row sums 150).  us per product, codes
// / patterns: stencil7 N = 215 FP64 in the CG loop 153 / 147.5 (134 since the
// loop leaves it its vectors in the Infinity Cache), FP32 plain 82 / 71; N =
// 512 FP32 in the loop 1,264 / 1,082.  Rows sum in storage order: products
// equal the coded ones bit for bit.
struct PatMeta {
    TileMeta<RowPack> rows;
    uint8_t id;
    __device__ __forceinline__ void load(const RowPack *__restrict__ rp, const uint8_t *__restrict__ pat, int64_t n,
                                         int64_t tile) {
        rows.load(rp, n, tile);
        const int64_t row = tile * kTileRows + threadIdx.x;
        id = pat[row < n ? row : n - 1];
    }
};

// Waves per SIMD the kernel is held to (without spills): FP64 vectors seven
// (the LDS of a CU holds seven workgroups too), FP32 eight; the loop's product
// lands at four to six when left to the compiler.
template <typename C>
constexpr int pattern_min_waves() {
    return std::is_same_v<C, double> ? 7 : 8;
}

template <typename V, typename X, typename C, class Epi>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(pattern_min_waves<C>()))) void
k_spmv_pattern(int64_t n, int64_t nnz, const RowPack *__restrict__ rp, const uint8_t *__restrict__ pat,
               const V *__restrict__ va, const X *__restrict__ x, int remap, int nt, int walkers, Epi epi_in) {
    Epi epi = epi_in;
    if (epi.skip()) return;
    const uint32_t W = walkers > 0 && static_cast<uint32_t>(walkers) < gridDim.x ? walkers : gridDim.x;
    if (blockIdx.x >= W) {   // uniform
        epi.finish();
        return;
    }
    __shared__ u32x4 lv[Chunks<V>::LDS];
    __shared__ uint32_t info[kPatterns];
    __shared__ int32_t offs[kPatternOffs];
    const RowPatterns *tab = reinterpret_cast<const RowPatterns *>(pat) - 1;
    for (int i = threadIdx.x; i < kPatterns; i += kBlock) info[i] = tab->info[i];
    for (int i = threadIdx.x; i < kPatternOffs; i += kBlock) offs[i] = tab->offs[i];
    __syncthreads();
    const V *sv = reinterpret_cast<const V *>(lv);
    const int64_t T = (n + kTileRows - 1) / kTileRows;
    TileIter it(T, remap, W);
    if (it.valid()) {
        PatMeta cur, nxt;
        cur.load(rp, pat, n, it.tile());
        while (true) {
            TileIter after = it;
            after.next();
            const bool more = after.valid();
            const int64_t r0 = cur.rows.r0;
            const int64_t r1 = min(r0 + static_cast<int64_t>(kTileRows), n);
            const int64_t row = r0 + threadIdx.x;
            const int64_t s = cur.rows.first(), e = cur.rows.end();
            const bool staged = e - s <= kStreamCap;   // uniform
            if (staged) dma_chunks<V>(va, s, e, nnz, lv, nt);
            if (more) nxt.load(rp, pat, n, after.tile());
            const auto pv = pre_of(epi, row < r1 ? row : r1 - 1);
            if (staged) {
                __builtin_amdgcn_s_waitcnt(0);
                __syncthreads();
                __builtin_amdgcn_s_setprio(2);   // (as in spmv_tiles_lds)
                if (row < r1) {
                    // this row's values, from its first one on
                    const V *v = sv + (cur.rows.lo() - (s & ~static_cast<int64_t>(Chunks<V>::EPC - 1)));
                    const int id = __builtin_amdgcn_readfirstlane(cur.id);
                    C sum = 0;
                    constexpr int U = 8;
                    if (__all(cur.id == id)) {
                        const uint32_t w = __builtin_amdgcn_readfirstlane(tab->info[id]);
                        const int32_t *o = tab->offs + (w & 0xffffu);
                        const int len = static_cast<int>(w >> 16);
                        const X *xr = x + r0;
                        for (int j0 = 0; j0 < len; j0 += U) {
                            C xv[U];
#pragma unroll
                            for (int u = 0; u < U; ++u) {
                                xv[u] = 0;
                                if (j0 + u < len) xv[u] = static_cast<C>((xr + o[j0 + u])[threadIdx.x]);
                            }
#pragma unroll
                            for (int u = 0; u < U; ++u)
                                if (j0 + u < len) sum = fma(static_cast<C>(widen(v[j0 + u])), xv[u], sum);
                        }
                    } else {
                        const uint32_t w = info[cur.id];
                        const int32_t *o = offs + (w & 0xffffu);
                        const int len = static_cast<int>(w >> 16);
                        for (int j0 = 0; j0 < len; j0 += kRowUnroll) {
                            C av[kRowUnroll], xv[kRowUnroll];
#pragma unroll
                            for (int u = 0; u < kRowUnroll; ++u) {
                                av[u] = 0;
                                xv[u] = 0;
                                if (j0 + u < len) {
                                    av[u] = static_cast<C>(widen(v[j0 + u]));
                                    xv[u] = static_cast<C>(x[row + o[j0 + u]]);
                                }
                            }
#pragma unroll
                            for (int u = 0; u < kRowUnroll; ++u) sum = fma(av[u], xv[u], sum);
                        }
                    }
                    emit_row(epi, row, sum, pv);
                }
                __builtin_amdgcn_s_setprio(0);
                lds_barrier();
            } else if (row < r1) {
                const uint32_t w = info[cur.id];
                const int32_t *o = offs + (w & 0xffffu);
                const int len = static_cast<int>(w >> 16);
                const V *v = va + cur.rows.lo();
                C sum = 0;
                for (int j = 0; j < len; ++j)
                    sum = fma(static_cast<C>(widen(ldv(v + j, nt))), static_cast<C>(x[row + o[j]]), sum);
                emit_row(epi, row, sum, pv);
            }
            if (!more) break;
            it = after;
            cur = nxt;
        }
    }
    epi.finish();
}

// ---- split gathers (SplitDev) ----------------------------------------------------
// A random pattern's product is bound by the lines its gathers fill: at 1e7
// columns nearly every 8-byte read brings a 128-byte line through the fabric
// (8.4 GB per product of 7e7 entries), at 1e6 from the L2 (170e9 reads/s).
// Taken block by block of 2^shift columns, the gathers find their slice of x
// in LDS (blocks of 128 KB) or in the XCD's L2 (larger ones, past 1,024 such
// blocks); what is added is streamed: 2 bytes of local column and 8 of value
// per entry out of the first launch, 8 of value, 4 of position and 2 of place
// into the second.  A tile reads its values in block order, so that the runs
// of one block (some 3 of a tile's 1,792 entries at 611 blocks, 12 of a group
// of four tiles') share lines: 1.9 GB fetched where 1.5 are needed, at 4.4
// TB/s.  Groups of 2, 8 and 16 tiles measure the same.  Row sums run in
// storage order on the caller's values, and rows longer than kLongRow from
// their pieces, so products equal the plain ones bit for bit.  Random pattern, 7 entries per row, us per call, plain / split (the
// two launches): FP64 n = 1e6 68 / 58 (17 + 32), n = 2e6 180 / 98, n = 1e7
// 1,186 / 587 (145 + 430; with the slices of 128 blocks gathered from L2,
// 795: 474 + 322); FP32 n = 3e6 228 / 102.
constexpr int kSplitDepth = 8;   // gathers in flight per thread

template <typename X, class Epi>
__global__ __launch_bounds__(kBlock) void k_split_gather(const int32_t *__restrict__ cols, int64_t count,
                                                         const X *__restrict__ x, X *__restrict__ xg, Epi epi) {
    if (epi.skip()) return;
    // each XCD walks its own eighth of the stream, so the slices of x that its
    // L2 holds are its own
    const int64_t span = static_cast<int64_t>(kBlock) * kSplitDepth;
    for (TileIter it((count + span - 1) / span, 1); it.valid(); it.next()) {
        const int64_t base = it.tile() * span + threadIdx.x;
        int32_t c[kSplitDepth];
        X v[kSplitDepth];
#pragma unroll
        for (int u = 0; u < kSplitDepth; ++u) {
            const int64_t j = base + u * kBlock;
            c[u] = __builtin_nontemporal_load(cols + (j < count ? j : count - 1));
        }
#pragma unroll
        for (int u = 0; u < kSplitDepth; ++u) v[u] = x[c[u]];
#pragma unroll
        for (int u = 0; u < kSplitDepth; ++u) {
            const int64_t j = base + u * kBlock;
            if (j < count) __builtin_nontemporal_store(v[u], xg + j);
        }
    }
}

// The same with the block's slice of x in LDS: a workgroup loads it and takes
// its part (of `parts`) of the block's stream.
constexpr int kSplitLdsThreads = 1024;
constexpr size_t kSplitLds = size_t(128) << 10;

template <typename X, class Epi>
__global__ __launch_bounds__(kSplitLdsThreads) void k_split_gather_lds(SplitDev sp, int parts, int64_t n_cols,
                                                                       const X *__restrict__ x, Epi epi) {
    if (epi.skip()) return;
    __shared__ X lx[kSplitLds / sizeof(X)];
    const int c = blockIdx.x / parts, part = blockIdx.x % parts;
    const int64_t first = static_cast<int64_t>(c) << sp.shift;
    const int width = static_cast<int>(min(n_cols - first, static_cast<int64_t>(1) << sp.shift));
    const int64_t b0 = sp.start[c], b1 = sp.start[c + 1];
    const int64_t j0 = b0 + (b1 - b0) * part / parts, j1 = b0 + (b1 - b0) * (part + 1) / parts;
    const X *xs = x + first;
    constexpr int U = 8;
    for (int i = threadIdx.x; i < width; i += U * kSplitLdsThreads) {
        X v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = xs[i + u * kSplitLdsThreads < width ? i + u * kSplitLdsThreads : i];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + u * kSplitLdsThreads < width) lx[i + u * kSplitLdsThreads] = v[u];
    }
    __syncthreads();
    // 16 bytes of values per thread and store: W places of the stream at a
    // time, aligned (those of a neighbouring part are left to it); a place at
    // a time n = 1e7 takes 201 us, so 145
    constexpr int W = 16 / sizeof(X), D = 16 / W;
    using KV = uint16_t __attribute__((ext_vector_type(W)));
    using XV = X __attribute__((ext_vector_type(W)));
    X *xg = static_cast<X *>(sp.xg);
    const KV *cols = static_cast<const KV *>(sp.cols);
    const int64_t w1 = (j1 + W - 1) / W;
    for (int64_t base = j0 / W + threadIdx.x; base < w1; base += D * kSplitLdsThreads) {
        KV k[D];
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int64_t w = base + u * kSplitLdsThreads;
            k[u] = cols[w < w1 ? w : w1 - 1];
        }
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int64_t w = base + u * kSplitLdsThreads, j = w * W;
            if (w >= w1) continue;
            if (j >= j0 && j + W <= j1) {
                XV v;
#pragma unroll
                for (int i = 0; i < W; ++i) v[i] = lx[k[u][i]];
                reinterpret_cast<XV *>(xg)[w] = v;
            } else {
#pragma unroll
                for (int i = 0; i < W; ++i)
                    if (j + i >= j0 && j + i < j1) xg[j + i] = lx[k[u][i]];
            }
        }
    }
}

// The row tiles of a product whose gathers have run.  Tiles of more than
// kStreamCap entries gather from x themselves (ci: the plain indices, 64-bit
// ones when ci64).
template <typename V, typename X, typename C, class Epi>
__global__ __launch_bounds__(kBlock) void k_spmv_split(int64_t n, int64_t nnz, const void *__restrict__ ci, int ci64,
                                                       const V *__restrict__ va, const X *__restrict__ x, SplitDev sp,
                                                       int remap, int nt, int walkers, Epi epi_in, LongArg<2> lra) {
    Epi epi = epi_in;
    if (epi.skip()) return;
    const uint32_t W = walkers > 0 && static_cast<uint32_t>(walkers) < gridDim.x ? walkers : gridDim.x;
    if (blockIdx.x >= W) {   // uniform
        epi.finish();
        return;
    }
    __shared__ u32x4 lv[Chunks<V>::LDS];
    __shared__ u32x4 lp[Chunks<uint16_t>::LDS];
    __shared__ X lx[kStreamCap];
    const RowPack *rp = static_cast<const RowPack *>(sp.rows);
    const X *xg = static_cast<const X *>(sp.xg);
    const int64_t T = (n + kTileRows - 1) / kTileRows;
    TileIter it(T, remap, W);
    if (it.valid()) {
        TileMeta<RowPack> cur, nxt;
        cur.load(rp, n, it.tile());
        while (true) {
            TileIter after = it;
            after.next();
            const bool more = after.valid();
            const int64_t r1 = min(cur.r0 + static_cast<int64_t>(kTileRows), n);
            const int64_t row = cur.r0 + threadIdx.x;
            const int64_t s = cur.first(), e = cur.end();
            const int64_t a = cur.lo(), b = cur.hi();
            const bool lng = lra.base && row < r1 && b - a > kLongRow;   // its pieces have been summed
            if (e - s <= kStreamCap) {
                dma_chunks<V>(va, s, e, nnz, lv, nt);
                dma_chunks<uint16_t>(sp.perm, s, e, nnz, lp, nt);
                // the tile's values of x: both rounds of loads whole before
                // the first use (places past the end re-read the last one)
                constexpr int U = kStreamCap / kBlock;
                const int m = static_cast<int>(e - s);
                uint32_t at[U];
                X xv[U];
                if (m > 0) {   // uniform
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int p = threadIdx.x + u * kBlock;
                        at[u] = __builtin_nontemporal_load(sp.src + s + (p < m ? p : m - 1));
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) xv[u] = xg[at[u]];
                }
                if (more) nxt.load(rp, n, after.tile());
                if (m > 0) {
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (static_cast<int>(threadIdx.x) + u * kBlock < m) lx[threadIdx.x + u * kBlock] = xv[u];
                }
                const auto pv = pre_of(epi, row < r1 ? row : r1 - 1);
                __builtin_amdgcn_s_waitcnt(0);   // this wave's DMA has landed
                __syncthreads();                 // ... and every other wave's
                __builtin_amdgcn_s_setprio(2);   // (as in spmv_tiles_lds)
                if (row < r1 && !lng)
                    emit_row(epi, row,
                             row_from_lds<V, uint16_t, C>(reinterpret_cast<const V *>(lv),
                                                          reinterpret_cast<const uint16_t *>(lp), a, b,
                                                          s & ~static_cast<int64_t>(Chunks<V>::EPC - 1),
                                                          s & ~static_cast<int64_t>(Chunks<uint16_t>::EPC - 1),
                                                          LdsGather<X, C>{lx}),
                             pv);
                __builtin_amdgcn_s_setprio(0);
                lds_barrier();
            } else {
                if (more) nxt.load(rp, n, after.tile());
                const PlainGather<X, C> gx{x};
                if (row < r1 && !lng)
                    epi.row(row, ci64 ? row_from_global<V, int64_t, C, kRowUnroll>(va, static_cast<const int64_t *>(ci), a,
                                                                                   b, gx, nt)
                                      : row_from_global<V, int32_t, C, kRowUnroll>(va, static_cast<const int32_t *>(ci), a,
                                                                                   b, gx, nt));
            }
            if (lng) epi.row(row, lra.template sum<C>(row, b - a));
            if (!more) break;
            it = after;
            cur = nxt;
        }
    }
    epi.finish();
}

// Parts of a block's stream in k_split_gather_lds, one workgroup and slice load
// each: about one workgroup per CU for few blocks, two parts when the blocks
// alone are one to four per CU (their last round is then half as long).
inline int split_parts(int cus, int blocks) {
    return blocks <= cus ? std::max(1, cus / blocks) : blocks < 4 * cus ? 2 : 1;
}

template <class F>
hipError_t dispatch_idx(const CsrDev &A, F &&f) {
    if (A.ptr_t == 0) {
        if (A.idx_t == 0) return f(static_cast<const int32_t *>(A.rp), static_cast<const int32_t *>(A.ci));
        return f(static_cast<const int32_t *>(A.rp), static_cast<const int64_t *>(A.ci));
    }
    if (A.idx_t == 0) return f(static_cast<const int64_t *>(A.rp), static_cast<const int32_t *>(A.ci));
    return f(static_cast<const int64_t *>(A.rp), static_cast<const int64_t *>(A.ci));
}

template <class Ptr>
using pointee_t = std::remove_const_t<std::remove_pointer_t<Ptr>>;

// Workgroups of kernel Kern resident on one CU at once (asked once per
// kernel; 0 if the runtime cannot tell).
template <auto Kern>
int resident_per_cu() {
    static const int blocks = [] {
        int b = 0;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, Kern, kBlock, 0) == hipSuccess ? b : 0;
    }();
    return blocks;
}

template <typename V, typename X, typename C, class Epi>
hipError_t launch_family(const CsrDev &A, const SpmvTune &t, const X *x, const Epi &epi, hipStream_t s) {
    if (A.n_rows == 0) return hipSuccess;
    if constexpr (!HasGather<Epi>::value) {
        // local columns want their block's slice in LDS: not split where X is too wide for that
        const bool local = A.split.shift <= kSplitLocal;
        if (t.kind == 0 && t.split && A.split.xg && (reinterpret_cast<uintptr_t>(A.va) & 15) == 0 &&
            (!local || (sizeof(X) << A.split.shift) <= kSplitLds)) {
            constexpr auto K = k_spmv_split<V, X, C, Epi>;
            const int per_cu = resident_per_cu<K>();
            const int walk = t.cus > 0 && per_cu > 0 ? std::min(t.grid, t.cus * per_cu) : 0;
            if (A.pieces) {
                auto pieces = [&](auto ci) {
                    hipLaunchKernelGGL((k_long_pieces<V, pointee_t<decltype(ci)>, X, C, Epi>),
                                       dim3(std::min(A.n_pieces, kMaxGrid)), dim3(kBlock), 0, s, A.pieces, A.n_pieces, ci,
                                       static_cast<const V *>(A.va), x, t.nt, A.piece_sums, epi);
                };
                if (A.idx_t == 0) pieces(static_cast<const int32_t *>(A.ci));
                else pieces(static_cast<const int64_t *>(A.ci));
            }
            if (A.split.count > 0 && local)
                hipLaunchKernelGGL((k_split_gather_lds<X, Epi>),
                                   dim3(A.split.blocks * split_parts(t.cus, A.split.blocks)), dim3(kSplitLdsThreads), 0, s,
                                   A.split, split_parts(t.cus, A.split.blocks), A.n_cols, x, epi);
            else if (A.split.count > 0)
                hipLaunchKernelGGL((k_split_gather<X, Epi>), dim3(t.cus > 0 ? std::min(t.cus * 8, kMaxGrid) : t.grid),
                                   dim3(kBlock), 0, s, static_cast<const int32_t *>(A.split.cols), A.split.count, x,
                                   static_cast<X *>(A.split.xg), epi);
            hipLaunchKernelGGL(K, dim3(t.grid), dim3(kBlock), 0, s, A.n_rows, A.nnz, A.ci, A.idx_t, static_cast<const V *>(A.va),
                               x, A.split, t.xcd_remap, t.nt, walk, epi,
                               LongArg<2>{A.pieces ? A.long_base : nullptr, A.piece_sums});
            return hipGetLastError();
        }
    }
    if constexpr (!HasGather<Epi>::value) {
        if (t.kind == 0 && t.pats && A.patterns && (reinterpret_cast<uintptr_t>(A.va) & 15) == 0) {
            constexpr auto K = k_spmv_pattern<V, X, C, Epi>;
            const int per_cu = resident_per_cu<K>();
            const int walk = t.cus > 0 && per_cu > 0 ? std::min(t.grid, t.cus * per_cu) : 0;
            hipLaunchKernelGGL(K, dim3(t.grid), dim3(kBlock), 0, s, A.n_rows, A.nnz,
                               static_cast<const RowPack *>(A.rowpack), static_cast<const uint8_t *>(A.patterns),
                               static_cast<const V *>(A.va), x, t.xcd_remap, t.nt, walk, epi);
            return hipGetLastError();
        }
    }
    // tile walkers of a row-tile kernel: the grid, or as many workgroups as
    // that kernel holds resident on the device if fewer
    auto walkers = [&](int per_cu) { return t.cus > 0 && per_cu > 0 ? std::min(t.grid, t.cus * per_cu) : 0; };
    return dispatch_idx(A, [&](auto rp, auto ci) {
        using P = pointee_t<decltype(rp)>;
        using I = pointee_t<decltype(ci)>;
        const V *va = static_cast<const V *>(A.va);
        const dim3 grid(t.grid), block(kBlock);
        // the LDS tiles DMA the values (and the plain column indices) in
        // 16-byte chunks; arrays without that alignment take one lane per
        // row, which sums each row in the same order
        auto al16 = [](const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
        // column codes exist only for matrices without rows longer than
        // kLongRow (the plan's rule), so only the plain-index kernel has a
        // long-row instance
        const bool coded = t.kind == 0 && t.codes && A.codes;
        const bool lr = A.max_row > kLongRow;
        if (t.kind == 0 && !(al16(A.va) && (coded || al16(A.ci)))) {
            hipLaunchKernelGGL((k_spmv_vector<V, P, I, X, C, Epi>), grid, block, 0, s, A.n_rows, rp, ci, va, x, 0,
                               t.xcd_remap, t.nt, epi);
        } else if (coded && t.pack && A.rowpack) {
            constexpr auto K = k_spmv_stream<V, RowPack, Code8, X, C, Epi>;
            hipLaunchKernelGGL(K, grid, block, 0, s, A.n_rows, A.nnz, static_cast<const RowPack *>(A.rowpack),
                               static_cast<const Code8 *>(A.codes), va, x, t.xcd_remap, t.nt, t.pf, walkers(resident_per_cu<K>()), epi, LongArg<0>{});
        } else if (coded) {
            constexpr auto K = k_spmv_stream<V, P, Code8, X, C, Epi>;
            hipLaunchKernelGGL(K, grid, block, 0, s, A.n_rows, A.nnz, rp, static_cast<const Code8 *>(A.codes), va, x,
                               t.xcd_remap, t.nt, t.pf, walkers(resident_per_cu<K>()), epi, LongArg<0>{});
        } else if (t.kind == 0 && lr) {
            if constexpr (!HasGather<Epi>::value) {
                if (A.pieces) {
                    hipLaunchKernelGGL((k_long_pieces<V, I, X, C, Epi>), dim3(std::min(A.n_pieces, kMaxGrid)), block, 0,
                                       s, A.pieces, A.n_pieces, ci, va, x, t.nt, A.piece_sums, epi);
                    constexpr auto K2 = k_spmv_stream<V, P, I, X, C, Epi, 2>;
                    hipLaunchKernelGGL(K2, grid, block, 0, s, A.n_rows, A.nnz, rp, ci, va, x, t.xcd_remap, t.nt, t.pf,
                                       walkers(resident_per_cu<K2>()), epi, LongArg<2>{A.long_base, A.piece_sums});
                    return hipGetLastError();
                }
            }
            constexpr auto K = k_spmv_stream<V, P, I, X, C, Epi, 1>;
            hipLaunchKernelGGL(K, grid, block, 0, s, A.n_rows, A.nnz, rp, ci, va, x, t.xcd_remap, t.nt, t.pf,
                               walkers(resident_per_cu<K>()), epi, LongArg<1>{});
        } else if (t.kind == 0) {
            constexpr auto K = k_spmv_stream<V, P, I, X, C, Epi>;
            hipLaunchKernelGGL(K, grid, block, 0, s, A.n_rows, A.nnz, rp, ci, va, x, t.xcd_remap, t.nt, t.pf,
                               walkers(resident_per_cu<K>()), epi, LongArg<0>{});
        } else {
            hipLaunchKernelGGL((k_spmv_vector<V, P, I, X, C, Epi>), grid, block, 0, s, A.n_rows, rp, ci, va, x,
                               t.lanes_log2, t.xcd_remap, t.nt, epi);
        }
        return hipGetLastError();
    });
}

}  // namespace tile
}  // namespace spk
