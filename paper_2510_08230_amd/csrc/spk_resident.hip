// Resident solves: a small system's whole CG solve (FP64, or FP64 refinement
// around the FP32 inner CG) in one launch, with the matrix held on the chip.
//
// What bounds a small solve is neither bytes nor arithmetic but the chain of
// dependent memory round trips: a kernel boundary, the stop flag, the partial
// sums, the row pointers, the tile, the gathers.  Here every workgroup keeps
// its rows for the whole solve, one thread per row: the row's first kRegs
// entries in registers (value, column and, for the entry's column, the
// thread's own copy of r and p), the rest in LDS.  An iteration is then
//
//   alpha, beta from the grid's sums of step k-1; update x, r, p of the row
//     and the copies of r and p held for its columns; q_k = A p_k
//   store q_k and the workgroup's sums
//   read q_k at the row's columns and the grid's sums
//
// with the arithmetic of the fused step (spk_fcg.h).  The copies are updated
// by the same expressions from the same q as the rows they copy, so they stay
// equal to them bit for bit and only q travels between workgroups.
//
// Measured (us per FP64 solve, plan kept; one launch per iteration before,
// this now): stencil7 n = 1,000: 430 / 142, n = 15,625: 444 / 196,
// n = 97,336: 515 / 228 (39 iterations: 12.9 -> 5.3 us each); random pattern
// n = 1,000: 490 / 201, n = 20,011: 697 / 338, n = 100,000 (three launches
// per iteration before): 905 / 443.  Of 4.9 us per step at n = 97,336 the row
// work takes 1.0, the workgroup's sums 0.4, and the exchange the rest.
//
// Exchange between workgroups (they run on eight XCDs with separate L2
// caches): agent-scope relaxed atomic stores and loads, which go to the
// memory side, so no cache is written back or invalidated (an agent-scope
// release costs 25 ns per workgroup in the barrier of spk_persist.hip).  The
// words carry their own arrival flag: a word holds 0 until its writer stores
// it (a value of +0 is written as -0), so a workgroup waits neither for its
// stores to be acknowledged nor for a counter, and polls the sums and its q
// words at the same time.  Words are used in four turns: in step m a writer
// stores turn m mod 4 and, at its start, empties turn m + 2 (= m - 2).  Every
// workgroup has read turn m - 2 by then, because it contributed to sum m - 1
// after that, and nobody polls turn m + 2 before sum m + 1 is complete, to
// which the writer contributes only after the loads of step m, which it
// waits for behind the emptying stores, have returned.
//
// No workgroup may wait for one that is not running: the launch begins with a
// rendezvous.  If not every workgroup has started within a short time (the
// device is shared with other streams' or processes' kernels), all of them
// leave and the caller runs the launch-per-iteration loop instead; once all
// have started, all stay until the solve ends.  Every wait is bounded, by the
// wall clock or by a count of polls: a workgroup whose wait ran out says so
// (failed) and leaves, so the others finish, or run out of their waits and
// leave too.  The caller then puts x back (x0) and runs the loop, whatever
// they stored.
#include "spk_fcg.h"
#include "spk_launch.h"

#include <algorithm>
#include <type_traits>

namespace spk {
namespace {

using namespace dev;

constexpr int kRegs = kResidentRegs;
constexpr int kBatch = 4;   // further entries whose words are read together
constexpr unsigned kTurns = kResidentTurns;
constexpr unsigned kMaxSpins = 1u << 20;   // polls of a word that must be on its way (about a second)

template <typename T>
using bits_t = std::conditional_t<sizeof(T) == 8, unsigned long long, unsigned int>;

template <typename T>
__device__ __forceinline__ void put(T *p, T v) {
    bits_t<T> u;
    __builtin_memcpy(&u, &v, sizeof(T));
    __hip_atomic_store(reinterpret_cast<bits_t<T> *>(p), u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T>
__device__ __forceinline__ T get(const T *p) {
    const bits_t<T> u = __hip_atomic_load(reinterpret_cast<const bits_t<T> *>(p), __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
    T v;
    __builtin_memcpy(&v, &u, sizeof(T));
    return v;
}

// The element at a byte offset.
template <typename T>
__device__ __forceinline__ const T *at(const T *p, unsigned off) {
    return reinterpret_cast<const T *>(reinterpret_cast<const char *>(p) + off);
}

__device__ __forceinline__ int64_t index_at(const void *p, int type, int64_t k) {
    return type == 0 ? static_cast<int64_t>(static_cast<const int32_t *>(p)[k]) : static_cast<const int64_t *>(p)[k];
}

// Sum over the 16 lanes of a DPP row, the same in each.
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    unsigned u[2];
    __builtin_memcpy(u, &v, 8);
    u[0] = __builtin_amdgcn_update_dpp(0, u[0], CTRL, 0xf, 0xf, true);
    u[1] = __builtin_amdgcn_update_dpp(0, u[1], CTRL, 0xf, 0xf, true);
    __builtin_memcpy(&v, u, 8);
    return v;
}

__device__ __forceinline__ double row_total(double v) {
    v += dpp<0xB1>(v);    // quad_perm [1, 0, 3, 2]
    v += dpp<0x4E>(v);    // quad_perm [2, 3, 0, 1]
    v += dpp<0x141>(v);   // row_half_mirror
    v += dpp<0x140>(v);   // row_mirror
    return v;
}

// Control words of a plan's resident launches.
enum : int { CTL_ARRIVED = 0, CTL_GATE = 1, CTL_SYNCS = 2, CTL_PUBS = 4 };

// 0 marks a word that its writer has not reached yet: a value of +0 goes out as -0.
template <typename T>
__device__ __forceinline__ T marked(T v) {
    return v == T(0) ? -T(0) : v;
}

template <typename T>
__device__ __forceinline__ bool empty(T v) {
    bits_t<T> u;
    __builtin_memcpy(&u, &v, sizeof(T));
    return u == 0;
}

// Sums over the grid, in two levels: workgroup g's sums go to slot g mod 16 of
// group g / 16, the group's first workgroup adds them, and every workgroup
// adds the groups' sums.  (Every workgroup reading every workgroup's slots
// takes 256 x 256 x 4 words per poll; the same few cache lines then serve all
// of them, which took 4.5 us at 254 workgroups against 0.8 us at 4.)
constexpr int kGroup = 16;
constexpr size_t kSlotsAt = kResidentStateBytes + sizeof(unsigned) * kResidentCtl;   // in the plan's block
constexpr int kCopies = 8;

struct GridSum {
    // [kTurns][kCopies + kGroup][4][kGroup]: the groups' sums (in kCopies
    // copies, each polled by an eighth of the workgroups), then each group's
    // members' sums
    unsigned long long *slots;
    unsigned syncs;              // sums taken so far, over all launches of the plan
    unsigned long long ticks;
    int *late;                   // LDS: a thread's words did not come

    // (The word found from slots: a pointer to it costs registers in every step.)
    __device__ __forceinline__ void fail() const {
        ResidentState *state = reinterpret_cast<ResidentState *>(reinterpret_cast<char *>(slots) - kSlotsAt);
        __hip_atomic_store(&state->failed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    __device__ __forceinline__ unsigned long long *set(unsigned turn, int which) const {
        return slots + (static_cast<size_t>(turn % kTurns) * (kCopies + kGroup) + which) * 4 * kGroup;
    }

    // Empties this workgroup's slots of the sum two turns on (once before
    // every sum).
    __device__ __forceinline__ void empty_ahead() const {
        const int tid = threadIdx.x, g = blockIdx.x, group = g / kGroup, member = g % kGroup;
        if (tid < 4)
            __hip_atomic_store(set(syncs + 2u, kCopies + group) + tid * kGroup + member, 0ull, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        if (tid < 4 * kCopies && member == 0)
            __hip_atomic_store(set(syncs + 2u, tid % kCopies) + (tid / kCopies) * kGroup + group, 0ull,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    // Lane l of a wave: the word l of 4 x 16 slots once it is there (lanes
    // with want false: 0), then the sum over each row of 16 lanes.  One read
    // in flight: more of them see a word sooner but hold up its store.
    __device__ __forceinline__ double collect(const unsigned long long *words, int lane, bool want, int &bad) const {
        const double *word = reinterpret_cast<const double *>(words) + lane;
        double w = 0.0;
        const unsigned long long t0 = wall_clock64();
        for (unsigned spins = 1; want; ++spins) {
            w = get(word);
            want = empty(w);
            if ((spins & 63u) == 0 && wall_clock64() - t0 > ticks) {
                fail();
                bad = 1;
                break;
            }
        }
        return row_total(w);
    }

    // tot[j] = the sum over the grid of v[j] (one fixed order, the same in
    // every thread).  gather() is called until it returns true, first while
    // the sums are on their way.  ACK: stores made before the call are visible
    // to every workgroup after it.  False after a time-out (then every
    // workgroup leaves).
    template <int NV, bool ACK, class F>
    __device__ __forceinline__ bool sum(double (&v)[NV], double (&tot)[NV], F &&gather) {
        __shared__ double s_part[4][kResidentRows / 16];   // each DPP row's sums
        __shared__ double s_tot[4];
        __shared__ int s_bad;
        static_assert(kResidentRows / 16 == 2 * kGroup, "a wave adds two DPP rows' sums per lane");
        const int G = gridDim.x, tid = threadIdx.x, lane = tid & 63;
        const int g = blockIdx.x, group = g / kGroup, member = g % kGroup, groups = (G + kGroup - 1) / kGroup;
        const int rows = blockDim.x >> 4, j = lane / kGroup, i = lane % kGroup;
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const double t = row_total(v[u]);
            if ((tid & 15) == 0) s_part[u][tid >> 4] = t;
        }
        if (tid == 0) s_bad = 0;
        if constexpr (ACK) {
            __builtin_amdgcn_s_waitcnt(0);   // this wave's stores have been acknowledged
            __syncthreads();
        } else {
            lds_barrier();
        }
        if (tid < 64) {   // lane 16 j + i: value j
            double t = j < NV && i < rows ? s_part[j][i] : 0.0;
            if (j < NV && i + kGroup < rows) t += s_part[j][i + kGroup];
            t = row_total(t);
            if (i == 0 && j < NV)
                put(reinterpret_cast<double *>(set(syncs, kCopies + group)) + j * kGroup + member, marked(t));
        }
        bool there = gather();   // the words of workgroups that are ahead are there already
        if (tid < 64) {
            int bad = *late;   // set before the barrier of this sum, if at all
            const bool one = groups == 1;   // its members' slots are read directly
            if (member == 0 && !one) {
                const double t = collect(set(syncs, kCopies + group), lane, j < NV && group * kGroup + i < G, bad);
                if (i < kCopies && j < NV)
                    put(reinterpret_cast<double *>(set(syncs, i)) + j * kGroup + group, marked(t));
            }
            const double t = collect(set(syncs, one ? kCopies : g % kCopies), lane, j < NV && i < (one ? G : groups), bad);
            if (i == 0) s_tot[j] = t;
            if (bad) s_bad = 1;
        }
        __syncthreads();
        // the vector was stored before the sums: it is there or about to be
        for (unsigned spins = 0; !there; ++spins) {
            there = gather();
            if (spins > kMaxSpins) {
                fail();
                *late = 1;   // the workgroup leaves at the next sum
                break;
            }
        }
#pragma unroll
        for (int u = 0; u < NV; ++u) tot[u] = s_tot[u];
        ++syncs;
        return s_bad == 0;
    }
};

// True once every workgroup of the launch has started, false if they did not
// within the time limit (the same answer in every workgroup).
__device__ __forceinline__ bool rendezvous(unsigned *ctl, unsigned epoch, unsigned long long ticks) {
    __shared__ int s_go;
    if (threadIdx.x == 0) {
        const unsigned mine = epoch << 1;
        auto settle = [&](unsigned verdict) {   // the first verdict of the epoch stands
            unsigned cur = __hip_atomic_load(ctl + CTL_GATE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((cur & ~1u) != mine)
                __hip_atomic_compare_exchange_strong(ctl + CTL_GATE, &cur, verdict, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
        };
        if (ticks == 0) settle(mine | 1u);
        const unsigned prev = __hip_atomic_fetch_add(ctl + CTL_ARRIVED, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (prev + 1u == epoch * gridDim.x) settle(mine);
        const unsigned long long t0 = wall_clock64();
        unsigned g;
        while (((g = __hip_atomic_load(ctl + CTL_GATE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) & ~1u) != mine)
            if (wall_clock64() - t0 > ticks) settle(mine | 1u);
        s_go = (g & 1u) == 0;
    }
    __syncthreads();
    return s_go != 0;
}

// T: the iterations' type (double: FP64 CG; float: the inner solve of
// refinement); V, V64: value types of the iterations' and of the
// refinement's matrix.
template <typename T, typename V, typename V64>
__global__ __launch_bounds__(kResidentRows) void k_resident(ResidentSolve a) {
    extern __shared__ __attribute__((aligned(8))) char smem[];   // doubles first
    __shared__ int s_late;
    if (threadIdx.x == 0) s_late = 0;
    if (!rendezvous(a.ctl, a.epoch, a.gate_ticks)) return;
    GridSum grid{a.slots, a.ctl[CTL_SYNCS], a.spin_ticks, &s_late};
    unsigned pubs = a.ctl[CTL_PUBS];   // vectors exchanged so far, over all launches of the plan
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * a.rows;
    const int64_t r1 = min(r0 + a.rows, a.n);
    const int64_t row = r0 + threadIdx.x;
    const bool has = threadIdx.x < a.rows && row < r1;

    // this row's entries: the first kRegs in registers, the rest in LDS at
    // their place in the workgroup's entry range
    const int64_t s = index_at(a.rp, a.ptr_t, r0 < a.n ? r0 : a.n);
    const int64_t ka = has ? index_at(a.rp, a.ptr_t, row) : 0;
    const int len = has ? static_cast<int>(index_at(a.rp, a.ptr_t, row + 1) - ka) : 0;
    const int rest = len > kRegs ? len - kRegs : 0;
    T *lv = reinterpret_cast<T *>(smem), *lr = lv + a.lds_entries, *lp = lr + a.lds_entries;
    T *lg = lp + a.lds_entries;
    unsigned *lc = reinterpret_cast<unsigned *>(lg + a.lds_entries);
    const int base = static_cast<int>(ka - s) + kRegs;
    // Slots past the row's end hold a zero value and the row's own column:
    // they add 0 to the row's sum (or NaN when the row's own direction is not
    // finite, which stops the solve anyway), so the loops need no masks.
    T av[kRegs], rn[kRegs], pn[kRegs];
    unsigned cl[kRegs];   // byte offsets of the entries' columns in an exchange buffer
    auto fill = [&](const auto *ci) {
        const V *va = static_cast<const V *>(a.va);
#pragma unroll
        for (int u = 0; u < kRegs; ++u) {
            const unsigned c = u < len ? static_cast<unsigned>(ci[ka + u]) : has ? static_cast<unsigned>(row) : 0u;
            cl[u] = c * static_cast<unsigned>(sizeof(T));
            av[u] = u < len ? static_cast<T>(widen(va[ka + u])) : T(0);
        }
#pragma unroll 1
        for (int u = 0; u < rest; ++u) {
            lv[base + u] = static_cast<T>(widen(va[ka + kRegs + u]));
            lc[base + u] = static_cast<unsigned>(ci[ka + kRegs + u]) * static_cast<unsigned>(sizeof(T));
        }
    };
    if (a.idx_t == 0) fill(static_cast<const int32_t *>(a.ci));
    else fill(static_cast<const int64_t *>(a.ci));

    // Vectors travel through kTurns exchange buffers in turn.
    T *const xch = static_cast<T *>(a.xch);
    const T *from = xch;
    auto empty_ahead = [&]() {
        if (has) put(xch + ((pubs + 2u) % kTurns) * static_cast<size_t>(a.n) + row, T(0));
        grid.empty_ahead();
    };
    // The published vector at the row's columns: the words not read yet are
    // read again; false while some are missing.
    T g[kRegs];
    auto expect = [&]() {
#pragma unroll
        for (int u = 0; u < kRegs; ++u) g[u] = T(0);
#pragma unroll 1
        for (int e = base; e < base + rest; ++e) lg[e] = T(0);
    };
    auto gather = [&]() {
        bool all = true;
#pragma unroll
        for (int u = 0; u < kRegs; ++u)
            if (empty(g[u])) g[u] = get(at(from, cl[u]));
        for (int e0 = base; e0 < base + rest; e0 += kBatch) {   // the further ones, a batch at a time
            T h[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) h[u] = e0 + u < base + rest ? lg[e0 + u] : T(1);
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                if (empty(h[u])) h[u] = get(at(from, lc[e0 + u]));
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                all = all && !empty(h[u]);
                if (e0 + u < base + rest) lg[e0 + u] = h[u];
            }
        }
#pragma unroll
        for (int u = 0; u < kRegs; ++u) all = all && !empty(g[u]);
        return all || !has;
    };
    auto publish = [&](T v) {
        T *to = xch + (pubs % kTurns) * static_cast<size_t>(a.n);
        if (has) put(to + row, marked(v));
        from = to;
        ++pubs;
        expect();
    };
    auto nothing = []() { return true; };

    // the row of the FP64 product A x (of the refinement's matrix), x read by
    // load at a column's byte offset in an FP64 vector
    auto product64 = [&](auto &&load) {
        constexpr unsigned W = sizeof(double) / sizeof(T);
        const V64 *va = static_cast<const V64 *>(a.va64);
        double sum = 0.0;
#pragma unroll
        for (int u = 0; u < kRegs; ++u) {
            if (u >= len) continue;
            if constexpr (std::is_same_v<T, double>) sum = fma(av[u], load(cl[u] * W), sum);
            else sum = fma(static_cast<double>(va[ka + u]), load(cl[u] * W), sum);
        }
#pragma unroll 1
        for (int u = 0; u < rest; ++u) sum = fma(static_cast<double>(va[ka + kRegs + u]), load(lc[base + u] * W), sum);
        return sum;
    };

    // The fused steps from r (already published, its grid sum taken) until a
    // decision stops them: x += the combination.  Returns the stop reason
    // (-1 after a time-out) and the completed iterations.
    auto steps = [&](T r, T &x, double thresh, int64_t max_it, SolveState *st, int64_t &done_out) -> int {
        T p = r, q = T(0);
        double acc[4], tot[4];
#pragma unroll
        for (int u = 0; u < kRegs; ++u) rn[u] = pn[u] = T(0);
#pragma unroll 1
        for (int u = 0; u < rest; ++u) lr[base + u] = lp[base + u] = T(0);
        for (int64_t k = 0;; ++k) {
            // here g holds q_{k-1} at the row's columns (k = 0: r)
            // k = 0: r of the columns is 0 - (-1) r, p = r + 0
            T al = T(0), be = T(0), an = T(-1);
            if (k >= 1) {
                double ald = 0.0, bed = 0.0;
                const int stop = fcg::decide(tot, k - 1, thresh, max_it, ald, bed);
                if (lead && st) {
                    fcg::record(st, tot, k - 1);
                    if (stop == STOP_RUNNING) st->alpha = ald;
                }
                if (stop != STOP_RUNNING) {
                    done_out = k - 1;
                    return stop;
                }
                al = an = static_cast<T>(ald);
                be = static_cast<T>(bed);
            }
            empty_ahead();
            x = fma(al, p, x);
            r = fma(-al, q, r);
            p = fma(be, p, r);
            T sum = T(0);
#pragma unroll
            for (int u = 0; u < kRegs; ++u) {
                rn[u] = fma(-an, g[u], rn[u]);
                pn[u] = fma(be, pn[u], rn[u]);
                sum = fma(av[u], pn[u], sum);
            }
#pragma unroll 1
            for (int e = base; e < base + rest; ++e) {
                const T rv = fma(-an, lg[e], lr[e]);
                const T pv = fma(be, lp[e], rv);
                lr[e] = rv;
                lp[e] = pv;
                sum = fma(lv[e], pv, sum);
            }
            q = marked(sum);
            publish(q);
            const double qd = static_cast<double>(q), rd = static_cast<double>(r);
            acc[0] = has ? static_cast<double>(p) * qd : 0.0;
            acc[1] = has ? rd * qd : 0.0;
            acc[2] = has ? qd * qd : 0.0;
            acc[3] = has ? rd * rd : 0.0;
            if (!(grid.template sum<4, false>(acc, tot, gather))) return -1;
        }
    };

    const double bi = has ? a.b[row] : 0.0;
    double xi = has ? a.x[row] : 0.0;
    if (has) a.x0[row] = xi;
    auto caller_x = [&](unsigned off) { return *at(a.x, off); };
    auto shared_x = [&](unsigned off) { return get(at(a.xd, off)); };
    if constexpr (std::is_same_v<T, double>) {
        const double r = marked(has ? bi - product64(caller_x) : 0.0);
        empty_ahead();
        publish(r);
        double v2[2] = {r * r, bi * bi}, t2[2];
        if (!(grid.template sum<2, true>(v2, t2, gather))) return;
        const double bn = sqrt(t2[1]), rho = t2[0], res = sqrt(rho);
        int stop = STOP_RUNNING, zero_x = 0;
        if (!isfinite(bn)) stop = STOP_NON_FINITE;
        else if (bn == 0.0) {
            stop = STOP_CONVERGED;
            zero_x = 1;
        } else if (!isfinite(rho)) stop = STOP_NON_FINITE;
        else if (res <= a.tau * bn) stop = STOP_CONVERGED;
        else if (a.max_iters <= 0) stop = STOP_MAX_ITERS;
        SolveState *S = &a.state->st;
        if (lead) {
            S->x = a.x;
            S->hist = a.hist;
            S->hist_cap = a.hist_cap;
            S->max_iters = a.max_iters;
            S->iter = 0;
            S->zero_x = zero_x;
            S->alpha = 0.0;
            S->pq = 0.0;
            S->bnorm = bn;
            S->thresh = a.tau * bn;
            S->rho[0] = zero_x ? 0.0 : rho;
            S->resnorm = zero_x ? 0.0 : (isfinite(bn) ? res : bn);
            S->true_resnorm = zero_x ? 0.0 : __builtin_nan("");
            if (a.hist && a.hist_cap > 0) a.hist[0] = S->resnorm;
        }
        int64_t done = 0;
        if (stop == STOP_RUNNING) {
            stop = steps(r, xi, a.tau * bn, a.max_iters, S, done);
            if (stop < 0) return;
        }
        if (zero_x) xi = 0.0;
        if (has && (zero_x || done > 0)) a.x[row] = xi;
        if (!zero_x && a.true_residual && stop != STOP_NON_FINITE) {
            if (has) put(a.xd + row, xi);
            double v1[1] = {0.0}, t1[1];
            grid.empty_ahead();
            if (!(grid.template sum<1, true>(v1, t1, nothing))) return;
            const double ri = has ? bi - product64(shared_x) : 0.0;
            v1[0] = ri * ri;
            grid.empty_ahead();
            if (!(grid.template sum<1, true>(v1, t1, nothing))) return;
            if (lead) S->true_resnorm = sqrt(t1[0]);
        }
        if (lead) {
            S->iter = done;
            S->stop = stop;
        }
    } else {
        int64_t inner = 0, outer = 0;
        double rnorm = 0.0, bn = 0.0;
        int stop = STOP_RUNNING;
        while (true) {
            const double r = has ? bi - (outer == 0 ? product64(caller_x) : product64(shared_x)) : 0.0;
            const float r32 = marked(static_cast<float>(r));
            empty_ahead();
            publish(r32);
            double v3[3] = {r * r, static_cast<double>(r32) * static_cast<double>(r32), bi * bi}, t3[3];
            if (!(grid.template sum<3, true>(v3, t3, gather))) return;
            rnorm = sqrt(t3[0]);
            bn = sqrt(t3[2]);
            const double r32n = sqrt(t3[1]);
            if (!isfinite(bn) || !isfinite(rnorm)) {
                stop = STOP_NON_FINITE;
                break;
            }
            if (bn == 0.0) {
                xi = 0.0;
                rnorm = 0.0;
                stop = STOP_CONVERGED;
                break;
            }
            if (rnorm <= a.tau * bn) {
                stop = STOP_CONVERGED;
                break;
            }
            if (outer >= a.max_outer || inner >= a.max_iters) {
                stop = STOP_MAX_ITERS;
                break;
            }
            int64_t kin = 0;
            int in_stop = STOP_CONVERGED;   // r32 = 0: nothing to solve
            float d = 0.0f;
            if (!isfinite(t3[1])) in_stop = STOP_NON_FINITE;
            else if (r32n != 0.0) {
                in_stop = steps(r32, d, a.tau_in * r32n, a.max_iters - inner, nullptr, kin);
                if (in_stop < 0) return;
            }
            inner += kin;
            if ((in_stop == STOP_BREAKDOWN || in_stop == STOP_NON_FINITE) && kin == 0) {
                stop = in_stop;
                break;
            }
            xi += static_cast<double>(d);
            ++outer;
            if (has) put(a.xd + row, xi);
            double v1[1] = {0.0}, t1[1];
            grid.empty_ahead();
            if (!(grid.template sum<1, true>(v1, t1, nothing))) return;
        }
        if (has && (outer > 0 || bn == 0.0)) a.x[row] = xi;
        if (lead) {
            a.state->res.inner = inner;
            a.state->res.outer = outer;
            a.state->res.rnorm = rnorm;
            a.state->res.bnorm = bn;
            a.state->res.stop = stop;
        }
    }
    if (lead) {
        a.state->launch = a.epoch;   // tells the host that the launch went through
        a.ctl[CTL_SYNCS] = grid.syncs;
        a.ctl[CTL_PUBS] = pubs;
    }
}

const void *kernel_for(const CsrDev &A, const CsrDev *outer) {
    auto k = [](auto t, auto v, auto w) {
        return reinterpret_cast<const void *>(&k_resident<decltype(t), decltype(v), decltype(w)>);
    };
    if (!outer) return A.val_t == 0 ? k(0.0, 0.0, 0.0) : nullptr;
    if (A.val_t == 1 && outer->val_t == 0) return k(0.0f, 0.0f, 0.0);
    if (A.val_t == 1 && outer->val_t == 1) return k(0.0f, 0.0f, 0.0f);
    if (A.val_t == 2 && outer->val_t == 0) return k(0.0f, _Float16(0), 0.0);
    if (A.val_t == 3 && outer->val_t == 0) return k(0.0f, bf16s{}, 0.0);
    return nullptr;
}

}  // namespace

size_t resident_lds_bytes(int64_t entries, bool mixed) {
    const size_t t = mixed ? sizeof(float) : sizeof(double);
    return static_cast<size_t>(entries) * (4 * t + sizeof(int));
}

// The exchange buffers: kTurns vectors of the iterations' type, then xd and x0.
static size_t resident_xd_at(int64_t n, bool mixed) {
    const size_t t = mixed ? sizeof(float) : sizeof(double);
    return (kTurns * t * static_cast<size_t>(n) + 255) & ~size_t(255);
}

size_t resident_exchange_bytes(int64_t n, bool mixed) {
    return resident_xd_at(n, mixed) + 2 * sizeof(double) * static_cast<size_t>(n);
}

const double *resident_x0(const void *xch, int64_t n, bool mixed) {
    return reinterpret_cast<const double *>(static_cast<const char *>(xch) + resident_xd_at(n, mixed)) + n;
}

hipError_t launch_resident(const CsrDev &A, const CsrDev *outer, ResidentSolve a, void *block, int grid, hipStream_t s) {
    const bool mixed = outer != nullptr;
    if (a.rows < 1 || a.rows > kResidentRows || grid < 1 || grid > kResidentGrid || static_cast<int64_t>(grid) * a.rows < A.n_rows ||
        A.n_rows > INT32_MAX)
        return hipErrorInvalidValue;
    a.n = A.n_rows;
    a.rp = A.rp;
    a.ci = A.ci;
    a.va = A.va;
    a.ptr_t = A.ptr_t;
    a.idx_t = A.idx_t;
    a.va64 = outer ? outer->va : A.va;
    a.xd = reinterpret_cast<double *>(static_cast<char *>(a.xch) + resident_xd_at(a.n, mixed));
    a.x0 = a.xd + a.n;
    a.ctl = reinterpret_cast<unsigned *>(static_cast<char *>(block) + kResidentStateBytes);
    a.slots = reinterpret_cast<unsigned long long *>(static_cast<char *>(block) + kSlotsAt);
    a.state = static_cast<ResidentState *>(block);
    const int threads = (a.rows + 63) & ~63;   // one per row
    const void *k = kernel_for(A, outer);
    if (threads > kResidentRows || !k) return hipErrorInvalidValue;
    const size_t lds = resident_lds_bytes(a.lds_entries, mixed);
    if (lds > size_t(64) << 10) {
        const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
        if (e != hipSuccess) return e;
    }
    void *args[] = {&a};
    return hipLaunchKernel(k, dim3(grid), dim3(threads), args, lds, s);
}

}  // namespace spk
