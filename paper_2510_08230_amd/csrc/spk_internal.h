// Internal types and constants shared by the host runtime (spk_api.cpp,
// spk_server.cpp) and the gfx950 kernels.  The launchers that start the
// kernels are declared in spk_launch.h.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

struct spk_ctx_s;

namespace spk {

constexpr int kBlock = 256;        // threads per workgroup (4 wave64s)
constexpr int kTileRows = 256;     // rows per SpMV tile
constexpr int kMaxGrid = 8192;     // cap on workgroups of any grid-stride launch
constexpr int kNumXcd = 8;         // MI355X: 8 XCDs, workgroups dispatched round-robin
// Device scratch of the allocation-free solve (one array per GPU, held until
// the process ends): solve state, reduction partials and three FP64 vectors.
constexpr size_t kNoallocScratchBytes = size_t(64) << 20;

enum Stop : int32_t {
    STOP_RUNNING = 0,
    STOP_CONVERGED = 1,
    STOP_MAX_ITERS = 2,
    STOP_BREAKDOWN = 3,
    STOP_NON_FINITE = 4
};

// Reduction sites: each owns an arrival counter and a partials slab.
// SITE_FCG: the fused CG step's two partial sets (p.q, r.q, q.q, r.r; one set
// per iteration parity), slabs 4 * parity + j from the site's start.
enum Site : int { SITE_INIT = 0, SITE_PQ = 1, SITE_RR = 2, SITE_TRUE = 3, SITE_FCG = 4, SITE_COUNT = 7 };
constexpr int kSiteWidth = 3;      // values reduced at once per site (max)

// Device-resident scalars of one CG solve.  Loop kernels read only fields
// written by earlier launches; workgroup 0 of a launch writes the results.
struct SolveState {
    double rho[4];        // ring: rho[k & 3] = r_k . r_k
    double pq, alpha;     // last p.q and alpha (diagnostics)
    double bnorm;         // ||b||
    double thresh;        // reduction_factor * ||b||
    double resnorm;       // sqrt(rho) at the last check
    double true_resnorm;  // ||b - A x|| at exit (NaN if not computed)
    int64_t base;         // absolute index of the current chunk's first iteration
    int64_t iter;         // completed updates
    int64_t max_iters;
    int32_t stop;         // Stop
    int32_t zero_x;       // b == 0: the finaliser sets x = 0
    void *x;              // solution vector of this solve (FP64 x, or FP32 d of an inner solve)
    double *hist;         // optional ||r_k|| history
    int64_t hist_cap;
};

// Vector pairs of the fused CG loop: step k reads buffer (k + 1) & 1 of each
// pair and writes buffer k & 1; the initial residual goes to buffer 1.
template <typename T>
struct FcgBufs {
    T *r[2], *p[2], *q[2];
};

// Result of a persistent mixed-precision solve (written by workgroup 0).
struct PersistResult {
    int64_t inner, outer;   // inner iterations in all, refinement steps
    double rnorm, bnorm;    // last ||b - A x|| (FP64) and ||b||
    int32_t stop;
};

// Resident solves (one launch per solve, the matrix held on the chip).
constexpr int kResidentRows = 512;      // most rows of a workgroup (one thread each)
constexpr int kResidentGrid = 256;      // most workgroups (16 groups of 16)
constexpr int kResidentRegs = 8;        // entries of a row held in registers
constexpr int kResidentRowMax = 32;     // longest row: one thread works through it
constexpr size_t kResidentLds = size_t(152) << 10;   // LDS for the rows' other entries (of 160 KB per CU)
constexpr int kResidentTurns = 4;       // sets of exchange words used in turn
constexpr int kResidentSlots = kResidentTurns * (8 + 16) * 4 * 16;   // words of the grid sums
constexpr int kResidentCtl = 16;        // control words

// What the host reads back after a resident launch.  A launch that leaves
// early writes neither st, res nor launch.
struct ResidentState {
    SolveState st;             // FP64 solve
    PersistResult res;         // mixed solve
    uint32_t launch, failed;   // the launch that wrote the result; nonzero: a wait timed out
};
constexpr size_t kResidentStateBytes = 4096;
static_assert(sizeof(ResidentState) <= kResidentStateBytes);
// The device block of a plan's resident launches, zero before the first one:
// the state, the control words, the words of the grid sums.  (Where the sums'
// words lie is worth 1% of a solve: us for 36 steps with 256 B / 4 KB for the
// state: stencil7 n = 97,336: 213.2 / 211.4, random n = 20,011: 264.7 / 262.9.)
constexpr size_t kResidentBlockBytes =
    kResidentStateBytes + sizeof(unsigned) * kResidentCtl + sizeof(unsigned long long) * kResidentSlots;

// Arguments of a resident solve (the launcher fills in the matrix, xd, x0 and
// the pointers into the plan's block).
struct ResidentSolve {
    int64_t n;
    const void *rp, *ci, *va, *va64;
    int ptr_t, idx_t;
    int rows;                 // consecutive rows per workgroup
    int lds_entries;          // most entries of a workgroup, 0 when no row is longer than the registers hold
    const double *b;
    double *x;
    void *xch;                // exchange buffers (resident_exchange_bytes), zero before the first launch
    double *xd;
    double *x0;               // x as it was, for the loop that follows a time-out
    unsigned long long *slots;
    unsigned *ctl;
    unsigned epoch;           // 1, 2, ... per launch on this block
    unsigned long long gate_ticks, spin_ticks;   // wall-clock limits of the start and of one wait
    ResidentState *state;     // the plan's block: the state, the control words, the words of the sums
    double tau, tau_in;
    int64_t max_iters, max_outer;
    double *hist;
    int64_t hist_cap;
    int true_residual;
};

// Arguments of a persistent solve (matrix fields filled by the launcher).
struct PersistSolve {
    int64_t n, nnz;
    const void *rp, *ci, *va, *va64;
    const double *b;
    double *x;
    FcgBufs<double> f64;   // FP64 solve
    FcgBufs<float> f32;    // mixed: inner vectors
    float *d32;            // mixed: inner correction
    SolveState *st;        // FP64 solve: the state the host reads
    PersistResult *res;    // mixed: the result
    double *partials;
    unsigned *bar;
    uint64_t spin_ticks;
    double tau, tau_in;
    int64_t max_iters, max_outer;
    double *hist;
    int64_t hist_cap;
    int remap, nt, true_residual;
};

// Whether the vectors of a CG loop (x, p, r and q of n values of T) outgrow the
// 256 MB Infinity Cache, and the passes over them go past it with those that
// they do not share (k_cg_pupdate).  Plain / past it, us per FP64 solve: 45 MB
// per vector 5,940 / 5,985, 64 MB 8,180 / 7,980.
template <typename T>
constexpr bool stream_vectors(int64_t n) {
    return n >= (int64_t(60) << 20) / static_cast<int64_t>(sizeof(T));
}

// Restarted GMRES: the small per-solve arrays (device memory, one per plan).
constexpr int kMaxKrylov = 32;   // largest restart length m
struct GmresState {
    double H[(kMaxKrylov + 1) * kMaxKrylov];   // rotated Hessenberg, H[i * kMaxKrylov + j]
    double Hu[(kMaxKrylov + 1) * kMaxKrylov];  // the same columns unrotated (A Q = Q Hu)
    double cs[kMaxKrylov], sn[kMaxKrylov];     // Givens rotations
    double g[kMaxKrylov + 1];                  // rotated right-hand side beta e_0
    double y[kMaxKrylov];                      // solution of R y = g
    double b[kMaxKrylov + 1];                  // first pass: q_t . w (t < j), u_j . w
    double a[kMaxKrylov + 1];                  // candidate u_j = Q_j a + nu q_j: its components along Q_j
    double h[kMaxKrylov + 1];                  // column j before the delayed correction
    double d[kMaxKrylov + 1];                  // u_{j+1} = w / nu - sum d_t q_t
    double nu;                                 // norm of the candidate's part orthogonal to Q_j
    int32_t used;                              // columns built in this cycle
    int32_t cycle_done;                        // nonzero: later kernels of the cycle return at once
};

// Launch shape of the SpMV family (shared by every SpMV-based kernel).
struct SpmvTune {
    int kind;        // 0 = LDS-staged row tiles, 1 = lanes-per-row vector kernel
    int lanes_log2;  // vector kernel: log2(lanes per row)
    int grid;        // workgroups
    int xcd_remap;   // 1 = contiguous tile ranges per XCD
    int nt;          // 1 = non-temporal loads for the matrix value stream
    int pf;          // LDS tiles: 1 = the next tile's row pointers load while this tile's entries stream in
    int bpc;         // workgroups per CU the grid was sized for
    int codes = 0;   // LDS tiles: 1 = read the matrix's one-byte column codes (CsrDev::codes)
    int pack = 0;    // with codes: 1 = read the packed row pointers (CsrDev::rowpack)
    int pats = 0;    // LDS tiles: 1 = read the matrix's row patterns (CsrDev::patterns)
    int split = 0;   // LDS tiles: 1 = the gathers run ahead in column order (CsrDev::split)
    int cus = 0;     // compute units of the device (0 = unknown: every workgroup walks tiles)
};

// The gathers of an irregular product, taken in an order of their own.  The
// entries of the row tiles (those of at most kStreamCap entries) are listed by
// column block (2^shift columns), within a block by group of kSplitGroup
// tiles: the stream.  A first launch reads x[cols[j]] for every stream
// position j into xg[j], a block's slice of x at a time.  A row tile then
// reads its values of xg into LDS, place p of the tile that starts at entry s
// from xg[src[s + p]] (in block order, so neighbouring places read
// neighbouring words), and takes entry k's from place perm[k].
struct SplitDev {
    void *xg = nullptr;              // one value of x per stream position (8 bytes each)
    const void *cols = nullptr;      // stream position -> column: uint16 within its block up to
                                     // kSplitLocal, else int32
    const uint32_t *src = nullptr;   // tile place -> stream position
    const uint16_t *perm = nullptr;  // entry -> tile place
    const uint32_t *start = nullptr; // block -> its first stream position (blocks + 1)
    const void *rows = nullptr;      // packed row pointers (as CsrDev::rowpack)
    int64_t count = 0;               // stream positions
    int blocks = 0, shift = 0;
};

constexpr int kSplitBlocks = 1024;   // most column blocks
constexpr int kSplitLocal = 15;      // largest shift of the blocks gathered from LDS
constexpr int kSplitGroup = 4;       // row tiles whose entries of a block are listed together

// Device CSR view with runtime-typed arrays.
struct CsrDev {
    int64_t n_rows, n_cols, nnz;
    int ptr_t, idx_t, val_t;   // spk_itype / spk_dtype codes
    const void *rp, *ci, *va;
    // Optional one-byte column codes (null when absent): byte k names entry k's
    // column offset from its row, c - i, in a table of kCodeDict int64 offsets
    // stored in the kCodeDict * 8 bytes just before the codes.
    const void *codes = nullptr;
    // Optional packed row pointers (null when absent; only with codes): the
    // int64 first entry of every 256-row tile (tiles + 1 values), followed
    // directly by one uint16 per row, its first entry less its tile's.
    const void *rowpack = nullptr;
    // Optional row patterns (null when absent; only with codes and rowpack):
    // byte i names row i's whole sequence of column offsets in the pattern
    // table (RowPatterns) stored just before the bytes.
    const void *patterns = nullptr;
    // The longest row's entry count (measured when the plan validates A; 0 =
    // unknown).  Above kLongRow the row tiles sum such rows with the whole
    // workgroup (host side only: it sets the kernels' long-row argument).
    int64_t max_row = 0;
    // Optional pieces of the rows longer than kLongRow (null when absent): at
    // most kLongPiece entries each, summed by a launch of their own ahead of
    // the row tiles (sums[p] = piece p's); a long row's pieces are consecutive
    // from long_base[row] on.
    const struct LongPiece *pieces = nullptr;
    int n_pieces = 0;
    const int32_t *long_base = nullptr;
    double *piece_sums = nullptr;
    // Optional split of the gathers (xg null when absent): see SplitDev.
    SplitDev split;
};

constexpr int kLongRow = 256;   // rows longer than this are summed by whole workgroups
// Entries of a long row that one workgroup sums at once: 4 per thread, all of
// their loads in flight together.
constexpr int kLongPiece = 1024;

struct LongPiece {
    int64_t first;   // entry
    int32_t len;
    int32_t row;
};

// The distinct rows of a coded matrix, as sequences of column offsets c - i.
constexpr int kPatterns = 256;      // distinct rows
constexpr int kPatternOffs = 1024;  // offsets of all of them together
constexpr int kPatternRow = 64;     // longest row
struct RowPatterns {
    uint32_t info[kPatterns];       // first offset | entries << 16
    int32_t offs[kPatternOffs];
};

constexpr int kCodeDict = 256;    // distinct column offsets a code table holds
constexpr int kCodeSlots = 1024;  // plan-time hash table of distinct offsets (power of two)

// Byte sizes of the plan's code buffer: the offset table, the codes (rounded
// to 16 bytes), then the packed row pointers (tiles + 1 int64, n uint16).
inline size_t code_bytes(int64_t nnz) { return (static_cast<size_t>(nnz) + 15) & ~size_t(15); }
// Bytes of the packed row pointers of n rows: tiles + 1 int64, n uint16.
inline size_t rowpack_bytes(int64_t n_rows) {
    const size_t tiles = static_cast<size_t>((n_rows + kTileRows - 1) / kTileRows);
    return sizeof(int64_t) * (tiles + 1) + ((sizeof(uint16_t) * static_cast<size_t>(n_rows) + 15) & ~size_t(15));
}
inline size_t code_buffer_bytes(int64_t n_rows, int64_t nnz) {
    return sizeof(int64_t) * kCodeDict + code_bytes(nnz) + rowpack_bytes(n_rows);
}

// Validation flag bits (set by the GPU check, order resolved on the host).
enum : unsigned { VFLAG_BAD_FIRST = 1u, VFLAG_DECREASING = 2u, VFLAG_BAD_LAST = 4u, VFLAG_BAD_COLUMN = 8u,
                  VFLAG_UNSORTED = 16u };

}  // namespace spk

// ==== batched serving ==========================================================
namespace spk {

// Per-slot life cycle, advanced on the device once per tick.
enum Phase : int32_t {
    PH_FREE = 0,     // slot unused
    PH_OUTER = 1,    // refinement residual r = b - A x (FP64) this tick
    PH_INNER = 2,    // CG iterations on A d = r (FP32 with FP64 dots, or FP64)
    PH_CORRECT = 3,  // x += d this tick
    PH_ZEROX = 4,    // b == 0: x = 0 this tick
    PH_DONE = 5      // finished; waiting for the host to retire it
};

// Per-slot partial-sum sites (kPartSites doubles per tile).
enum : int { PART_PQ = 0, PART_RR = 1, PART_OUT = 2 /* 3 sites: r.r, r32.r32, b.b */, kPartSites = 5 };

// Written by the host at admission; read-only on the device.
struct SlotDesc {
    int64_t n, nnz, tiles;
    const int32_t *rp, *ci;
    const double *va64;     // the request's FP64 values
    const float *va32;      // rounded copy (slot workspace)
    const double *b;
    double *x;
    float *r, *p, *q, *d;          // slot workspace of an FP32-inner request
    double *r64, *p64, *q64, *d64; // slot workspace of an FP64 request
    double *part;                  // slot workspace: kPartSites * tiles
    double tau, tau_in;
    int64_t max_iters, max_outer;
    int32_t stage;          // 1: values and columns 16-byte aligned, tiles staged in LDS by DMA
    int32_t fp64;           // 1: the inner CG runs in FP64 on the caller's values (no FP32 copy)
};

// Device-resident per-slot scalars.
struct SlotState {
    double rho[4];
    double thresh_in, bnorm, rnorm, alpha, beta;
    int64_t iter_in, iters, outer;
    int32_t phase, next_phase, stop_in, stop;
};

// Compact per-slot record the host polls after each batch of ticks.
struct SlotStatus {
    int32_t phase, stop;
    int64_t iters, outer;
    double rnorm, bnorm;
};

// Workgroups per CU of the tick's vector launches: all that a CU holds, since a
// tile's few loads wait behind those of its table entry, descriptor and state.
// 64 requests of 1e3 to 1e6 rows, us per tick and ms in all, with the four of
// the product's launch / with eight: update 87 / 54, p 30 / 20, 29.3 / 27.0 ms
// (sixteen 26.9).  The product keeps its own figure: 5 or 6 per CU gather
// through the same L2s in 434 us, 4 in 339.
constexpr int kTickVecBlocks = 8;

// Device tables of one server: counts plus tile and slot lists.
struct BatchDev {
    const int32_t *counts;   // [0] live tiles, [1] live slots
    const int2 *tiles;       // (slot, local tile)
    const int32_t *slots;    // live slot ids
    const SlotDesc *desc;
    SlotState *state;
    SlotStatus *status;
    int tile_grid, vec_grid, slot_grid;   // workgroups: products, vector passes, per-slot sums
    int remap;   // tile order of the tile launches (TileIter: 0 round-robin, 1 contiguous eighths per XCD)
    int nt;      // 1: non-temporal loads of the matrix stream
};

}  // namespace spk
