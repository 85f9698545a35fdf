// Grouped form (coarse levels and small finest levels): G = 4 .. 64 lanes per
// block row, 64 / G rows per wavefront; a slot holds the next G blocks of every
// row of the slice, its values stored as in the sliced form (one 64-lane group
// per nonzero entry), so a row of L blocks is ceil(L / G) slots deep.
#include "solve_device.h"
#include "dpp.h"

#include <algorithm>
#include <climits>
#include <cmath>

namespace mbamg {


// A row's D values as other workgroups of the running launch may be writing
// them: relaxed loads at device scope (past the L1, coherent across the XCDs),
// 8 bytes at a time where rows are 8-byte aligned.
template <class T, int D>
__device__ __forceinline__ void load_shared_vec(const T* p, T (&v)[D]) {
    if constexpr (sizeof(T) == 4 && D % 2 == 0) {
#pragma unroll
        for (int c = 0; c < D; c += 2) {
            const unsigned long long u = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p + c),
                                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            v[c] = __uint_as_float((unsigned)u);
            v[c + 1] = __uint_as_float((unsigned)(u >> 32));
        }
    } else {
#pragma unroll
        for (int c = 0; c < D; ++c) v[c] = __hip_atomic_load(p + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}
template <class T, int D>
__device__ __forceinline__ bool any_unwritten(const T (&v)[D]) {
    bool m = false;
#pragma unroll
    for (int c = 0; c < D; ++c) m = m || unwritten(v[c]);
    return m;
}

// data that no running launch writes, at an address all lanes share: a scalar load
template <class U>
__device__ __forceinline__ U uniform_load(const U* p) {
    typedef const U __attribute__((address_space(4))) * ConstPtr;
    return *(ConstPtr)(uintptr_t)p;
}

// The damped update of one value; written by a sweep and recomputed by the blocks
// that follow in the same launch.
template <class T>
__device__ __forceinline__ T damped(T x, T w, T t) { return x + w * (t - x); }

// x_j of a coupling operand whose block is relaxed in this launch, from the awaited t_j
template <class T, int D>
__device__ __forceinline__ void operand_value(const SweepOperand<T>& o, int j, const T (&xo)[D], T (&v)[D]) {
    const T w = o.w_row ? o.w_row[j] : o.omega;
#pragma unroll
    for (int c = 0; c < D; ++c) v[c] = o.x ? damped(xo[c], w, v[c]) : w * v[c];
}

// acc -= sum over the slice's slots of one part.  MODE 0: x_j from xa.  MODE 1:
// columns below cstart from ta (awaited), others from xa.  MODE 2: columns below
// cstart from ta (awaited), others contribute 0.  MODE 3: the coupling operand op,
// every column awaited.
template <class T, int D, int MODE, int S, class TX = T>
__device__ __forceinline__ void group_sub(const GroupView<T>& A, int w, int cb, int lane, const TX* __restrict__ xa,
                                          const T* ta, int cstart, T (&acc)[D],
                                          SweepWait wait = {}, const SweepOperand<T>* op = nullptr) {
    constexpr int CH = 2;
    for (int t0 = 0; t0 < w; t0 += CH) {
        int j[CH];
        uint32_t m[CH];
        int64_t vg[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const bool live = t0 + u < w;
            const int64_t sl = (int64_t)cb + t0 + u;
            m[u] = live ? uniform_load(A.mask + sl) : 0u;
            vg[u] = live ? uniform_load(A.voff + sl) : 0;
            j[u] = live ? A.col[sl * WAVE + lane] : -1;
        }
        constexpr int NE = shape_entries<D, S>();
        T v[CH][NE], xj[CH][D], xo[MODE == 3 ? CH : 1][D];
#pragma unroll
        for (int u = 0; u < CH; ++u) load_masked<T, NE>(A.val + vg[u] * WAVE + lane, m[u], v[u]);
        // every load of the chunk is issued before the first value is looked at
        bool await[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u) {
#pragma unroll
            for (int c = 0; c < D; ++c) xj[u][c] = T(0);
            await[u] = MODE != 0 && j[u] >= 0 && (MODE == 3 || j[u] < cstart);
            if (MODE == 3) {
#pragma unroll
                for (int c = 0; c < D; ++c) xo[u][c] = T(0);
                if (xa && j[u] >= 0) load_vec_from<T, D>(xa + (int64_t)j[u] * D, xo[u]);
            }
            if (await[u]) load_shared_vec<T, D>(ta + (int64_t)j[u] * D, xj[u]);
            else if (MODE < 2 && j[u] >= 0) load_vec_from<T, D>(xa + (int64_t)j[u] * D, xj[u]);
        }
        if (MODE != 0) {
            for (int round = 0;; ++round) {
                bool more = false;
#pragma unroll
                for (int u = 0; u < CH; ++u) {
                    await[u] = await[u] && any_unwritten<T, D>(xj[u]);
                    more = more || await[u];
                }
                if (!__any(more)) break;
                if (round >= wait.rounds) {
                    __hip_atomic_store(wait.late, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                    break;
                }
                pause_after(round);
#pragma unroll
                for (int u = 0; u < CH; ++u)
                    if (await[u]) load_shared_vec<T, D>(ta + (int64_t)j[u] * D, xj[u]);
            }
        }
        if (MODE == 3) {
#pragma unroll
            for (int u = 0; u < CH; ++u)
                if (j[u] >= 0) operand_value<T, D>(*op, j[u], xo[u], xj[u]);
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) block_sub<T, D, S>(v[u], xj[u], acc);
    }
}

__device__ __forceinline__ SweepRec load_rec(const SweepRec* p) {
    typedef int v8i __attribute__((ext_vector_type(8)));
    static_assert(sizeof(SweepRec) == sizeof(v8i), "one 32-byte record");
    return __builtin_bit_cast(SweepRec, uniform_load(reinterpret_cast<const v8i*>(p)));
}

template <int CTRL>
__device__ __forceinline__ float dpp_get(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp_get(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// the sum over each aligned group of 2^lg lanes (4 .. 64), in every lane of the
// group, per component; lg is the same for the whole wavefront
template <class T, int D>
__device__ __forceinline__ void group_all_sum(T (&acc)[D], int lg) {
#pragma unroll
    for (int r = 0; r < D; ++r) {
        acc[r] += dpp_get<0xB1>(acc[r]);    // quad_perm [1,0,3,2]
        acc[r] += dpp_get<0x4E>(acc[r]);    // quad_perm [2,3,0,1]
    }
    if (lg >= 3)
#pragma unroll
        for (int r = 0; r < D; ++r) acc[r] += dpp_get<0x141>(acc[r]);   // row_half_mirror
    if (lg >= 4)
#pragma unroll
        for (int r = 0; r < D; ++r) acc[r] += dpp_get<0x140>(acc[r]);   // row_mirror
    if (lg >= 5)
#pragma unroll
        for (int r = 0; r < D; ++r) acc[r] += __shfl_xor(acc[r], 16, WAVE);
    if (lg >= 6)
#pragma unroll
        for (int r = 0; r < D; ++r) acc[r] += __shfl_xor(acc[r], 32, WAVE);
}

// Algorithm 1's Gauss-Seidel sub-solves in one launch, all colours of block 0, then
// all of block 1 (the arithmetic of k_gs).  A colour pass on a coarse level is a few
// microseconds of launch and dependent loads whatever its size, and one such pass
// per colour was most of a small system's cycle.  Here the rows wait for their own
// neighbours instead: a row of colour c reads t_j of its neighbours of earlier
// colours with device-scope loads and repeats them until the values are there
// ("unwritten" before); a row of block 1 does the same for the rows of block 0 it is
// coupled to and applies their damping itself.  The hop from one workgroup's store
// to another's load is 0.5 us, against 4.0 - 5.0 us per launched colour pass.
//
// Every wait ends: a workgroup takes its positions of the record lists by an atomic
// ticket, the lists are ordered by block and colour, and a position waits only for
// positions of earlier colours or blocks, whose tickets were taken before by
// workgroups that are already running.  The tickets are one counter (11 ns each),
// so a workgroup takes SWEEP_WAVES slices per ticket.
//
// A launch takes both blocks on small levels and one on larger ones (see
// BOTH_BLOCKS_MAX).
//
// The two undamped buffers of a level take turns: a launch writes t and sets its
// rows of the other buffer to "unwritten" for the next launch.

// LDS asked for by the workgroups of a sweep, and not used, so that a compute unit
// (160 KiB) takes one of them, or two.
// One, where a colour has few workgroups (spread): a colour's rows then spread over
// the chip.  Without it the dispatcher put several on some units and none on others
// (13,945 rows in 9 colours, 49 workgroups per colour: 31 us a sweep instead of 20;
// 164 per colour: 112 us instead of 110).
// Two otherwise: with more than half the units' number per colour they spread by
// themselves, and a second workgroup per unit hides latency (four blocks of 64,000
// rows, 250 per colour: 505 us per V-cycle with one, 468 with two); more only poll
// (see pause_after; a 30-iteration solve on 1,000,000 2D nodes 35.3 ms with four,
// 33.9 with three, 33.2 with two).
static unsigned sweep_lds(int spread) { return (spread ? 84 : 56) * 1024; }

// This wavefront's position of the launch (all of a workgroup call it).
__device__ __forceinline__ int sweep_position(uint32_t* ticket, uint32_t* ticket_next) {
    __shared__ int tick;
    if (threadIdx.x == 0) {
        const uint32_t k = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (k == 0) *ticket_next = 0u;
        tick = (int)k;
    }
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(tick) * SWEEP_WAVES + wave_id();
}

// One slice of a sweep; couplings(acc) subtracts the coupling terms.
template <class T, int D, bool ZX, int S, class Cpl>
__device__ __forceinline__ void sweep_slice(const SweepArgs<T>& a, const SweepWait& wait, const SweepRec& rec, int lane,
                                            Cpl&& couplings) {
    const int q = lane & ((1 << a.lg) - 1), rr = lane >> a.lg;
    const bool act = rr < rec.nrow && q < D;   // lane q of a row's group finishes component q
    const int row = rec.row0 + (rr < rec.nrow ? rr : 0);
    const int64_t at = (int64_t)row * D + (q < D ? q : 0);
    // the row's own data: fetched before the sums, whose latency it overlaps
    T bb[D], dv[D], xo = T(0);
    load_vec<T, D>(a.b + (int64_t)row * D, bb);
    load_vec<T, D>(a.dinv + at * D, dv);
    if (!ZX) xo = a.x[at];
    const T wgt = a.w_row ? a.w_row[row] : a.omega;
    T acc[D];
#pragma unroll
    for (int r = 0; r < D; ++r) acc[r] = T(0);
    couplings(acc);
    const int cstart = a.inplace ? INT_MAX : rec.cstart;
    if (ZX) {
        if (cstart > 0) group_sub<T, D, 2, S, T>(a.off, rec.off_w, rec.off_c, lane, nullptr, a.t, cstart, acc, wait);
    } else {
        group_sub<T, D, 1, S>(a.off, rec.off_w, rec.off_c, lane, a.x, a.t, cstart, acc, wait);
    }
    group_all_sum<T, D>(acc, a.lg);
    if (!act) return;
    T tn = T(0);
#pragma unroll
    for (int c = 0; c < D; ++c) tn += dv[c] * (bb[c] + acc[c]);
    const T xn = ZX ? wgt * tn : damped(xo, wgt, tn);
    a.xn[at] = xn;
    if (a.t_reset) a.t_reset[at] = unwritten_value<T>();
    if (unwritten(tn)) tn = T(NAN);
    __hip_atomic_store(a.t + at, tn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// BOTH: positions of both blocks, block 1's coupling operand awaited; otherwise those
// of one block, in the arguments' first places, with every operand complete.
template <class T, int D, bool ZX, int S, bool BOTH>
__global__ __launch_bounds__(SWEEP_WAVES * WAVE) void k_sweep(Sweep2Args<T> a) {
    int pos = sweep_position(a.ticket, a.ticket_next);
    const int f = BOTH && pos >= a.s[0].count ? 1 : 0;
    if (f) pos -= a.s[0].count;
    const SweepArgs<T>& s = a.s[f];
    if (pos >= s.count) return;   // whole wavefronts; no barrier follows
    const SweepRec rec = load_rec(s.rec + s.begin + pos);
    if (rec.nrow == 0) return;
    const int lane = threadIdx.x & (WAVE - 1);
    sweep_slice<T, D, ZX, S>(s, a.wait, rec, lane, [&](T (&acc)[D]) {
        const SweepOperand<T>& o = a.xg[f];
        if (BOTH && o.t) group_sub<T, D, 3, S>(a.cpl[f], rec.cpl_w, rec.cpl_c, lane, o.x, o.t, 0, acc, a.wait, &o);
        else if (o.x) group_sub<T, D, 0, S>(a.cpl[f], rec.cpl_w, rec.cpl_c, lane, o.x, nullptr, 0, acc);
    });
}

// acc -= one slice's A_fg x_g with BR x BC blocks
template <int BR, int BC>
__device__ __forceinline__ void group_sub_rect(const GroupPart& P, int slice, int lane, double (&acc)[BR]) {
    constexpr int CH = 2;
    const int w = uniform_load(P.width + slice);
    const int64_t cb = uniform_load(P.coff + slice);
    for (int t0 = 0; t0 < w; t0 += CH) {
        double v[CH][BR * BC], xj[CH][BC];
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const bool live = t0 + u < w;
            const int64_t sl = cb + t0 + u;
            const uint32_t m = live ? uniform_load(P.a.mask + sl) : 0u;
            const int64_t vg = live ? uniform_load(P.a.voff + sl) : 0;
            const int j = live ? P.a.col[sl * WAVE + lane] : -1;
            load_masked<double, BR * BC>(P.a.val + vg * WAVE + lane, m, v[u]);
#pragma unroll
            for (int c = 0; c < BC; ++c) xj[u][c] = 0.0;
            if (j >= 0) load_vec<double, BC>(P.x + (int64_t)j * BC, xj[u]);
        }
#pragma unroll
        for (int u = 0; u < CH; ++u)
#pragma unroll
            for (int r = 0; r < BR; ++r)
#pragma unroll
                for (int c = 0; c < BC; ++c) acc[r] -= v[u][r * BC + c] * xj[u][c];
    }
}

template <int D>
__device__ __forceinline__ void group_sub_parts(const GroupPart* parts, int n, int slice, int lane, double (&acc)[D]) {
    for (int k = 0; k < n; ++k) {
        const GroupPart& P = parts[k];
        switch (P.bc) {
            case 1: group_sub_rect<D, 1>(P, slice, lane, acc); break;
            case 2: group_sub_rect<D, 2>(P, slice, lane, acc); break;
            case 3: group_sub_rect<D, 3>(P, slice, lane, acc); break;
            default: group_sub_rect<D, 4>(P, slice, lane, acc); break;
        }
    }
}

// The sweep of one block among more than two: its couplings with every other
// block are summed with the row instead of being folded into a right-hand side
// beforehand (a launch per coupling, one thread per row: 33 us each on the 40^3
// system of 4 blocks, 1266 of 2080 us per V-cycle; that cycle takes 456 us now).
template <int D, bool ZX>
__global__ __launch_bounds__(SWEEP_WAVES * WAVE) void k_sweep_n(SweepNArgs a) {
    const int pos = sweep_position(a.ticket, a.ticket_next);
    if (pos >= a.s.count) return;   // whole wavefronts; no barrier follows
    const SweepRec rec = load_rec(a.s.rec + a.s.begin + pos);
    if (rec.nrow == 0) return;
    const int lane = threadIdx.x & (WAVE - 1);
    sweep_slice<double, D, ZX, SHAPE_FULL>(a.s, a.wait, rec, lane,
                               [&](double (&acc)[D]) { group_sub_parts<D>(a.cpl, a.n_cpl, rec.slice, lane, acc); });
}

template <int D>
__device__ __forceinline__ void resid_slice_n(const ResidNArgs& a, int f, const SweepRec& rec, int lane) {
    const int lg = a.lg[f];
    const int q = lane & ((1 << lg) - 1), rr = lane >> lg;
    const bool act = rr < rec.nrow && q < D;
    const int row = rec.row0 + (rr < rec.nrow ? rr : 0);
    const int64_t at = (int64_t)row * D + (q < D ? q : 0);
    double dg[D], xr[D], bq = 0.0;
    load_vec<double, D>(a.diag[f] + at * D, dg);
    load_vec<double, D>(a.x[f] + (int64_t)row * D, xr);
    if (a.b[f]) bq = a.b[f][at];
    double acc[D];
#pragma unroll
    for (int r = 0; r < D; ++r) acc[r] = 0.0;
    group_sub<double, D, 0, SHAPE_FULL>(a.off[f], rec.off_w, rec.off_c, lane, a.x[f], nullptr, 0, acc);
    group_sub_parts<D>(a.cpl[f], a.n_cpl[f], rec.slice, lane, acc);
    group_all_sum<double, D>(acc, lg);
    if (!act) return;
    double own = 0.0, sum = 0.0;
#pragma unroll
    for (int c = 0; c < D; ++c) {
        own += dg[c] * xr[c];
        sum = c == q ? acc[c] : sum;
    }
    const double ax = own - sum;
    a.r[f][at] = a.b[f] ? bq - ax : ax;
}

__global__ __launch_bounds__(256) void k_resid_n(ResidNArgs a, int padded_blocks) {
    int pos = xcd_block(padded_blocks) * WPB + wave_id();
    int f = 0;
    while (f < a.nb && pos >= a.count[f]) pos -= a.count[f++];
    if (f >= a.nb) return;   // whole wavefront
    const SweepRec rec = load_rec(a.rec[f] + pos);
    if (rec.nrow == 0) return;
    const int lane = threadIdx.x & (WAVE - 1);
    switch (a.d[f]) {
        case 1: resid_slice_n<1>(a, f, rec, lane); break;
        case 2: resid_slice_n<2>(a, f, rec, lane); break;
        case 3: resid_slice_n<3>(a, f, rec, lane); break;
        default: resid_slice_n<4>(a, f, rec, lane); break;
    }
}

// r = b - A x (or w = A x when b is NULL) in grouped form, block 0's record
// list, then block 1's
template <class T, class TX, int D, int S>
__global__ __launch_bounds__(256) void k_resid_group(ResidGroupArgs<T, TX> a) {
    // the positions a sweep's workgroup k takes go to two blocks here, both of them on
    // the XCD that k comes to there (blocks are dispatched in turn over the 8 XCDs).
    // With contiguous launch ranges per XCD instead, each XCD had slices from all over a
    // colour: operator on 256^2 nodes 19.6 us against 17.6, on 32^3 20.0 against 18.4
    const int b = blockIdx.x, k = (b >> 4) * 8 + (b & 7), half = (b >> 3) & 1;
    static_assert(SWEEP_WAVES == 2 * WPB, "two blocks per sweep workgroup");
    int pos = k * SWEEP_WAVES + half * WPB + wave_id();
    int f = 0;
    if (pos >= a.count[0]) {
        pos -= a.count[0];
        f = 1;
        if (pos >= a.count[1]) return;   // whole wavefront
    }
    const SweepRec rec = load_rec(a.rec[f] + pos);
    if (rec.nrow == 0) return;
    const int lane = threadIdx.x & (WAVE - 1), lg = a.lg[f];
    const int q = lane & ((1 << lg) - 1), rr = lane >> lg;
    const bool act = rr < rec.nrow && q < D;
    const int row = rec.row0 + (rr < rec.nrow ? rr : 0);
    const int64_t at = (int64_t)row * D + (q < D ? q : 0);
    T dg[D], xr[D], bq = T(0);
    load_vec<T, D>(a.diag[f] + at * D, dg);
    load_vec_from<T, D>(a.x[f] + (int64_t)row * D, xr);
    if (a.b[f]) bq = a.b[f][at];
    T acc[D];
#pragma unroll
    for (int r = 0; r < D; ++r) acc[r] = T(0);
    group_sub<T, D, 0, S>(a.off[f], rec.off_w, rec.off_c, lane, a.x[f], nullptr, 0, acc);
    group_sub<T, D, 0, S>(a.cpl[f], rec.cpl_w, rec.cpl_c, lane, a.x[1 - f], nullptr, 0, acc);
    group_all_sum<T, D>(acc, lg);
    if (!act) return;
    T own = T(0);
#pragma unroll
    for (int c = 0; c < D; ++c) own += dg[c] * xr[c];
    T sum = T(0);
#pragma unroll
    for (int c = 0; c < D; ++c) sum = c == q ? acc[c] : sum;
    const T ax = own - sum;
    a.r[f][at] = a.b[f] ? bq - ax : ax;
}

template <class T, int D, int S>
static void sweep_dispatch_s(bool zx, unsigned grid, const Sweep2Args<T>& a, hipStream_t s) {
    constexpr int TPB = SWEEP_WAVES * WAVE;
    const unsigned lds = sweep_lds(a.spread);
    if (a.s[1].count > 0) {
        if (zx) k_sweep<T, D, true, S, true><<<grid, TPB, lds, s>>>(a);
        else k_sweep<T, D, false, S, true><<<grid, TPB, lds, s>>>(a);
    } else {
        if (zx) k_sweep<T, D, true, S, false><<<grid, TPB, lds, s>>>(a);
        else k_sweep<T, D, false, S, false><<<grid, TPB, lds, s>>>(a);
    }
}

template <class T, int D>
static void sweep_dispatch(bool zx, unsigned grid, const Sweep2Args<T>& a, hipStream_t s) {
    if constexpr (D > 1) {
        if (a.shape == SHAPE_SCALED) return sweep_dispatch_s<T, D, SHAPE_SCALED>(zx, grid, a, s);
        if (a.shape == SHAPE_SYMMETRIC) return sweep_dispatch_s<T, D, SHAPE_SYMMETRIC>(zx, grid, a, s);
    }
    sweep_dispatch_s<T, D, SHAPE_FULL>(zx, grid, a, s);
}

template <class T, class TX, int D>
static void resid_group_dispatch(unsigned grid, const ResidGroupArgs<T, TX>& a, hipStream_t s) {
    if constexpr (D > 1) {
        if (a.shape == SHAPE_SCALED) {
            k_resid_group<T, TX, D, SHAPE_SCALED><<<grid, 256, 0, s>>>(a);
            return;
        }
        if (a.shape == SHAPE_SYMMETRIC) {
            k_resid_group<T, TX, D, SHAPE_SYMMETRIC><<<grid, 256, 0, s>>>(a);
            return;
        }
    }
    k_resid_group<T, TX, D, SHAPE_FULL><<<grid, 256, 0, s>>>(a);
}

// a block's positions come in whole workgroups, so no workgroup takes two blocks'
static void check_sweep_block(int count, int lg) {
    MB_CHECK(count >= 0 && count % SWEEP_WAVES == 0, MBAMG_E_INVALID, "whole workgroups per block");
    MB_CHECK(count == 0 || (lg >= 2 && lg <= 6), MBAMG_E_INVALID, "4 to 64 lanes per row");
}

template <class T>
void launch_sweep(int d, bool zero_x, const Sweep2Args<T>& a, hipStream_t s) {
    for (const SweepArgs<T>& f : a.s) check_sweep_block(f.count, f.lg);
    MB_CHECK(a.wait.late, MBAMG_E_INVALID, "a place for late waits");
    const unsigned grid = (unsigned)((a.s[0].count + a.s[1].count) / SWEEP_WAVES);
    if (grid == 0) return;
    switch (d) {
        case 1: sweep_dispatch<T, 1>(zero_x, grid, a, s); break;
        case 2: sweep_dispatch<T, 2>(zero_x, grid, a, s); break;
        case 3: sweep_dispatch<T, 3>(zero_x, grid, a, s); break;
        case 4: sweep_dispatch<T, 4>(zero_x, grid, a, s); break;
        default: throw Error(MBAMG_E_INVALID, "dofs per node must be 1..4");
    }
    MB_LAUNCH_CHECK();
}
template void launch_sweep<double>(int, bool, const Sweep2Args<double>&, hipStream_t);
template void launch_sweep<float>(int, bool, const Sweep2Args<float>&, hipStream_t);

template <int D>
static void sweep_n_dispatch(bool zx, const SweepNArgs& a, hipStream_t s) {
    const unsigned grid = (unsigned)(a.s.count / SWEEP_WAVES);
    constexpr int TPB = SWEEP_WAVES * WAVE;
    if (zx) k_sweep_n<D, true><<<grid, TPB, sweep_lds(a.spread), s>>>(a);
    else k_sweep_n<D, false><<<grid, TPB, sweep_lds(a.spread), s>>>(a);
}

void launch_sweep_n(int d, bool zero_x, const SweepNArgs& a, hipStream_t s) {
    check_sweep_block(a.s.count, a.s.lg);
    MB_CHECK(a.wait.late, MBAMG_E_INVALID, "a place for late waits");
    if (a.s.count == 0) return;
    MB_CHECK(a.n_cpl >= 0 && a.n_cpl < SWEEP_MAX_BLOCKS, MBAMG_E_INVALID, "at most 4 blocks");
    for (int k = 0; k < a.n_cpl; ++k)
        MB_CHECK(a.cpl[k].bc >= 1 && a.cpl[k].bc <= 4, MBAMG_E_INVALID, "row blocks of at most 4 x 4");
    switch (d) {
        case 1: sweep_n_dispatch<1>(zero_x, a, s); break;
        case 2: sweep_n_dispatch<2>(zero_x, a, s); break;
        case 3: sweep_n_dispatch<3>(zero_x, a, s); break;
        case 4: sweep_n_dispatch<4>(zero_x, a, s); break;
        default: throw Error(MBAMG_E_INVALID, "dofs per node must be 1..4");
    }
    MB_LAUNCH_CHECK();
}

void launch_resid_n(const ResidNArgs& a, hipStream_t s) {
    MB_CHECK(a.nb >= 1 && a.nb <= SWEEP_MAX_BLOCKS, MBAMG_E_INVALID, "at most 4 blocks");
    int total = 0;
    for (int f = 0; f < a.nb; ++f) {
        total += a.count[f];
        MB_CHECK(a.lg[f] >= 2 && a.lg[f] <= 6 && a.d[f] >= 1 && a.d[f] <= 4, MBAMG_E_INVALID,
                 "4 to 64 lanes per row, 1..4 dofs per node");
        for (int k = 0; k < a.n_cpl[f]; ++k)
            MB_CHECK(a.cpl[f][k].bc >= 1 && a.cpl[f][k].bc <= 4, MBAMG_E_INVALID, "row blocks of at most 4 x 4");
    }
    if (total <= 0) return;
    const unsigned grid = xcd_grid(total, 1);
    k_resid_n<<<grid, 256, 0, s>>>(a, (int)grid);
    MB_LAUNCH_CHECK();
}

template <class T, class TX>
void launch_resid_group(int d, const ResidGroupArgs<T, TX>& a, hipStream_t s) {
    const int total = a.count[0] + a.count[1];
    if (total <= 0) return;
    MB_CHECK(a.lg[0] >= 2 && a.lg[0] <= 6 && a.lg[1] >= 2 && a.lg[1] <= 6, MBAMG_E_INVALID, "4 to 64 lanes per row");
    const unsigned grid = (unsigned)ceil_div(ceil_div(total, SWEEP_WAVES), 8) * 16;
    switch (d) {
        case 1: resid_group_dispatch<T, TX, 1>(grid, a, s); break;
        case 2: resid_group_dispatch<T, TX, 2>(grid, a, s); break;
        case 3: resid_group_dispatch<T, TX, 3>(grid, a, s); break;
        case 4: resid_group_dispatch<T, TX, 4>(grid, a, s); break;
        default: throw Error(MBAMG_E_INVALID, "dofs per node must be 1..4");
    }
    MB_LAUNCH_CHECK();
}
template void launch_resid_group<double, double>(int, const ResidGroupArgs<double>&, hipStream_t);
template void launch_resid_group<float, float>(int, const ResidGroupArgs<float>&, hipStream_t);
template void launch_resid_group<double, float>(int, const ResidGroupArgs<double, float>&, hipStream_t);

}  // namespace mbamg
