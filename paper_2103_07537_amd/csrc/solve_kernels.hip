// Solve-phase kernels for gfx950: one 64-lane wavefront per slice of 64
// block rows, one lane per block row.  Matrix values are stored slot-major and
// lane-contiguous, so every value load of a wavefront is one contiguous
// 256 B (FP32) or 512 B (FP64) segment; only block entries that are nonzero
// somewhere in the slice are stored, which keeps the streamed bytes close to
// the structural nonzeros.  All loops over slots and mask bits are
// wave-uniform (scalar branches).
#include "solve_device.h"
#include "dpp.h"

#include <algorithm>
#include <climits>
#include <cstdint>
#include <cmath>
#include <utility>

namespace mbamg {

// acc[r] -= sum_c A[r,c] * x_col(c) over the slots part, part+P, part+2P, ...
// of one slice.  MODE 0: x from xa.  MODE 1: columns below cstart from xa
// (already updated this sweep), others from xb.  MODE 2: columns below cstart
// from xa, others contribute 0.
// When P waves share a slice (coarse levels: few wide slices, so each wave's
// chain of dependent loads is what the launch waits for), the column indices,
// masks and value offsets of the next chunk are fetched while the current
// chunk's values and gathers are in flight, and FP32 chunks are 4 slots wide.
template <class T, int P>
constexpr int sell_chunk() { return P >= 4 && sizeof(T) == 4 ? 4 : CHUNK; }

// Column indices, masks and value offsets of one chunk of slots.
template <int CH>
struct SlotChunk {
    int j[CH];
    uint32_t m[CH];
    int64_t vg[CH];
};

// The chunk of slots t0, t0 + P, ... of a slice of w slots from cb (slots past the
// width: empty); C16: columns in 16 bits.
template <class T, int P, int CH, bool C16 = false>
__device__ __forceinline__ void fetch_slots(const SellView<T>& A, int w, int64_t cb, int lane, int t0, int (&j)[CH],
                                            uint32_t (&m)[CH], int64_t (&vg)[CH]) {
#pragma unroll
    for (int u = 0; u < CH; ++u) {
        const int tt = t0 + u * P;
        const bool live = tt < w;
        m[u] = live ? A.mask[cb + tt] : 0u;
        vg[u] = live ? A.voff[cb + tt] : 0;
    }
    if constexpr (C16) {
        uint16_t c[CH];
        int base[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int tt = t0 + u * P;
            const bool live = tt < w;
            base[u] = live ? A.cbase[cb + tt] : 0;
            c[u] = live ? A.col16[(cb + tt) * WAVE + lane] : (uint16_t)COL16_NONE;
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) j[u] = c[u] == COL16_NONE ? -1 : base[u] + c[u];
    } else {
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int tt = t0 + u * P;
            j[u] = tt < w ? A.col[(cb + tt) * WAVE + lane] : -1;
        }
    }
}

// the same of slice s
template <class T, int P, int CH>
__device__ __forceinline__ void fetch_chunk(const SellView<T>& A, int s, int lane, int t0, SlotChunk<CH>& c) {
    const int w = A.width[s];
    const int64_t cb = A.coff[s];
    fetch_slots<T, P, CH>(A, w, cb, lane, t0, c.j, c.m, c.vg);
}

// SKIPD: the slot holding column `self` (the row's own node) is left out.
// pre (split slices only): the first chunk, fetched by the caller ahead of time.
template <class T, int D, int MODE, int P, int S = SHAPE_FULL, bool SKIPD = false, bool C16 = false, class TX = T>
__device__ __forceinline__ void sell_sub(const SellView<T>& A, int s, int lane, int part, const TX* __restrict__ xa,
                                         const std::common_type_t<TX>* __restrict__ xb, int cstart, T (&acc)[D], int self = -1,
                                         const SlotChunk<sell_chunk<T, P>()>* pre = nullptr) {
    constexpr int CH = sell_chunk<T, P>();
    constexpr bool PF = P >= 4;
    const int w = A.width[s];
    const int64_t cb = A.coff[s];
    int j[CH];
    uint32_t m[CH];
    int64_t vg[CH];
    auto fetch = [&](int t0) { fetch_slots<T, P, CH, C16>(A, w, cb, lane, t0, j, m, vg); };
    if (PF) {
        if (pre) {
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                j[u] = pre->j[u];
                m[u] = pre->m[u];
                vg[u] = pre->vg[u];
            }
        } else {
            fetch(part);
        }
    }
    for (int t = part; t < w; t += P * CH) {
        if (!PF) fetch(t);
        int jc[CH];
        uint32_t mc[CH];
        int64_t gc[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            jc[u] = j[u];
            mc[u] = m[u];
            gc[u] = vg[u];
        }
        if (PF) fetch(t + P * CH);
        constexpr int NE = shape_entries<D, S>();
        T v[CH][NE];
#pragma unroll
        for (int u = 0; u < CH; ++u) load_masked<T, NE>(A.val + gc[u] * WAVE + lane, mc[u], v[u]);
        T xj[CH][D];
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int jj = jc[u];
            const TX* src = nullptr;
            if (MODE == 0) src = xa;
            else if (MODE == 1) src = jj < cstart ? xa : xb;
            else src = jj < cstart ? xa : nullptr;
            if (jj >= 0 && src && !(SKIPD && jj == self)) load_vec_from<T, D>(src + (int64_t)jj * D, xj[u]);
            else {
#pragma unroll
                for (int c = 0; c < D; ++c) xj[u][c] = T(0);
            }
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) block_sub<T, D, S>(v[u], xj[u], acc);
    }
}

// Sum the P partial accumulators of one slice through LDS in a fixed order;
// the result is valid in the slice's part-0 wave.
template <class T, int D, int P>
__device__ __forceinline__ void combine_parts(T (&acc)[D], int wave, int part, int lane) {
    if constexpr (P > 1) {
        __shared__ T red[waves_per_block<P>()][WAVE][D];
#pragma unroll
        for (int r = 0; r < D; ++r) red[wave][lane][r] = acc[r];
        __syncthreads();
        if (part == 0) {
#pragma unroll
            for (int p = 1; p < P; ++p)
#pragma unroll
                for (int r = 0; r < D; ++r) acc[r] += red[wave + p][lane][r];
        }
    }
}

// One colour of the multicolour nodal-block Gauss-Seidel sub-solve of block f
// inside Algorithm 1: for each row i of the colour
//   t_i  = D_i^-1 (b_i - sum_{j != i} A_ff[i,j] t_j - (A_fg x_g)_i)
//   xn_i = x_i + omega (t_i - x_i)
// where t_j is the updated value for rows of earlier colours and x_j otherwise;
// t_i - x_i is the sub-solve's correction e_i for the residual b - A x.
template <class T, int D, bool ZX, bool CPL, int P, int S, bool C16>
__global__ __launch_bounds__(waves_per_block<P>() * WAVE) void k_gs(GsArgs<T> a, int padded_blocks) {
    const int wave = wave_id();
    const int part = wave % P;
    const int sidx = xcd_block(padded_blocks) * (waves_per_block<P>() / P) + wave / P;
    const bool valid = sidx < a.s_count;
    if (P == 1 && !valid) return;
    const int s = a.s_begin + (valid ? sidx : 0);
    const int lane = threadIdx.x & (WAVE - 1);
    const int row0 = a.sl.row0[s], nrow = a.sl.nrow[s];
    const bool act = valid && lane < nrow;
    const int row = row0 + (lane < nrow ? lane : 0);
    T acc[D];
    if (part == 0) load_vec<T, D>(a.b + (int64_t)row * D, acc);
    else {
#pragma unroll
        for (int r = 0; r < D; ++r) acc[r] = T(0);
    }
    // small levels (split slices): the row's own data, and the coupling part's first slots,
    // are fetched before the sums, so their latency overlaps the sums' instead of following
    T dv[D * D], xo[D];
    T w = a.omega;
    constexpr int CH = sell_chunk<T, P>();
    SlotChunk<CH> cpre;
    if (P > 1 && valid) {
        if (part == 0) {
            load_masked<T, D * D>(a.dinv.val + a.dinv.voff[a.dinv.coff[s]] * WAVE + lane,
                                  a.dinv.mask[a.dinv.coff[s]], dv);
            if (!ZX) load_vec<T, D>(a.x + (int64_t)row * D, xo);
            if (a.w_row) w = a.w_row[row];
        }
        if (CPL && P >= 4) fetch_chunk<T, P, CH>(a.cpl, s, lane, part, cpre);
    }
    if (valid) {
        if (!a.skip_off) {
            if (ZX) sell_sub<T, D, 2, P, S, false, C16>(a.off, s, lane, part, a.t, nullptr, a.cstart, acc);
            else sell_sub<T, D, 1, P, S, false, C16>(a.off, s, lane, part, a.t, a.x, a.cstart, acc);
        }
        if (CPL) sell_sub<T, D, 0, P, S, false, C16>(a.cpl, s, lane, part, a.xg, nullptr, 0, acc, -1, P >= 4 ? &cpre : nullptr);
    }
    combine_parts<T, D, P>(acc, wave, part, lane);
    if (part != 0 || !valid) return;
    if (P == 1)
        load_masked<T, D * D>(a.dinv.val + a.dinv.voff[a.dinv.coff[s]] * WAVE + lane, a.dinv.mask[a.dinv.coff[s]],
                              dv);
    T tn[D];
#pragma unroll
    for (int r = 0; r < D; ++r) {
        T sum = T(0);
#pragma unroll
        for (int c = 0; c < D; ++c) sum += dv[r * D + c] * acc[c];
        tn[r] = sum;
    }
    if (!act) return;
    if (P == 1 && a.w_row) w = a.w_row[row];
    T xn[D];
    if (ZX) {
#pragma unroll
        for (int r = 0; r < D; ++r) xn[r] = w * tn[r];
    } else {
        if (P == 1) load_vec<T, D>(a.x + (int64_t)row * D, xo);
#pragma unroll
        for (int r = 0; r < D; ++r) xn[r] = xo[r] + w * (tn[r] - xo[r]);
    }
    if (a.keep_t) store_vec<T, D>(a.t + (int64_t)row * D, tn);
    store_vec<T, D>(a.xn + (int64_t)row * D, xn);
}

// One colour of the nodal-block Gauss-Seidel over the full node blocks (the
// FC-AMG comparison smoother): for each node i of the colour, both blocks' rows
//   t_i  = D_i^-1 (b_i - sum_{j != i} A[i,j] t_j / x_j)   (D_i: the full node block)
//   xn_i = x_i + omega (t_i - x_i)
// with the sums over A_ff's off-diagonal blocks and A_fg's blocks other than
// the node's own, t_j for rows of earlier colours and x_j otherwise.
template <class T, int D, bool ZX, int P>
__global__ __launch_bounds__(waves_per_block<P>() * WAVE) void k_gs_fc(GsFcArgs<T> a, int padded_blocks) {
    constexpr int M = 2 * D;
    const int wave = wave_id();
    const int part = wave % P;
    const int sidx = xcd_block(padded_blocks) * (waves_per_block<P>() / P) + wave / P;
    const bool valid = sidx < a.s_count;
    if (P == 1 && !valid) return;
    const int s = a.s_begin + (valid ? sidx : 0);
    const int lane = threadIdx.x & (WAVE - 1);
    const int row0 = a.sl.row0[s], nrow = a.sl.nrow[s];
    const bool act = valid && lane < nrow;
    const int row = row0 + (lane < nrow ? lane : 0);
    T acc0[D], acc1[D];
    if (part == 0) {
        load_vec<T, D>(a.b[0] + (int64_t)row * D, acc0);
        load_vec<T, D>(a.b[1] + (int64_t)row * D, acc1);
    } else {
#pragma unroll
        for (int r = 0; r < D; ++r) acc0[r] = acc1[r] = T(0);
    }
    if (valid && !a.skip_off) {
        constexpr int MODE = ZX ? 2 : 1;
        sell_sub<T, D, MODE, P>(a.off[0], s, lane, part, a.t[0], a.x[0], a.cstart, acc0);
        sell_sub<T, D, MODE, P, SHAPE_FULL, true>(a.cpl[0], s, lane, part, a.t[1], a.x[1], a.cstart, acc0, row);
        sell_sub<T, D, MODE, P>(a.off[1], s, lane, part, a.t[1], a.x[1], a.cstart, acc1);
        sell_sub<T, D, MODE, P, SHAPE_FULL, true>(a.cpl[1], s, lane, part, a.t[0], a.x[0], a.cstart, acc1, row);
    }
    T acc[M];
#pragma unroll
    for (int r = 0; r < D; ++r) {
        acc[r] = acc0[r];
        acc[D + r] = acc1[r];
    }
    combine_parts<T, M, P>(acc, wave, part, lane);
    if (part != 0 || !valid) return;
    // the node inverse: only the slice's nonzero entries are stored
    const uint64_t dm = a.dmask[s];
    const T* dv = a.dinv + (int64_t)a.doff[s] * WAVE + lane;
    T inv[M * M];
    int g = 0;
#pragma unroll
    for (int k = 0; k < M * M; ++k) {
        if ((dm >> k) & 1) {
            inv[k] = dv[(int64_t)g * WAVE];
            ++g;
        } else {
            inv[k] = T(0);
        }
    }
    T tn[M];
#pragma unroll
    for (int r = 0; r < M; ++r) {
        T sum = T(0);
#pragma unroll
        for (int c = 0; c < M; ++c) sum += inv[r * M + c] * acc[c];
        tn[r] = sum;
    }
    if (!act) return;
    const T w = a.w_row ? a.w_row[row] : a.omega;
#pragma unroll
    for (int f = 0; f < 2; ++f) {
        T tf[D], xn[D];
#pragma unroll
        for (int r = 0; r < D; ++r) tf[r] = tn[f * D + r];
        if (ZX) {
#pragma unroll
            for (int r = 0; r < D; ++r) xn[r] = w * tf[r];
        } else {
            T xo[D];
            load_vec<T, D>(a.x[f] + (int64_t)row * D, xo);
#pragma unroll
            for (int r = 0; r < D; ++r) xn[r] = xo[r] + w * (tf[r] - xo[r]);
        }
        store_vec<T, D>(a.t[f] + (int64_t)row * D, tf);
        store_vec<T, D>(a.xn[f] + (int64_t)row * D, xn);
    }
}

// ---------------------------------------------------------------------------
// Row form (transfers to small levels): one wavefront per row, its lanes over
// the row's blocks, partial sums combined across the wavefront.
// ---------------------------------------------------------------------------
// a dense block of N values, with 16-byte loads where the size allows (blocks
// are stored back to back, so a block of 4 or 16 entries is 16-byte aligned)
template <class T, int N>
__device__ __forceinline__ void load_block(const T* __restrict__ p, T (&v)[N]) {
    if constexpr (sizeof(T) == 4 && N % 4 == 0) {
#pragma unroll
        for (int k = 0; k < N / 4; ++k) {
            const float4 q = reinterpret_cast<const float4*>(p)[k];
            v[4 * k] = q.x; v[4 * k + 1] = q.y; v[4 * k + 2] = q.z; v[4 * k + 3] = q.w;
        }
    } else if constexpr (sizeof(T) == 8 && N % 2 == 0) {
#pragma unroll
        for (int k = 0; k < N / 2; ++k) {
            const double2 q = reinterpret_cast<const double2*>(p)[k];
            v[2 * k] = q.x; v[2 * k + 1] = q.y;
        }
    } else {
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = p[k];
    }
}

template <class T, int D>
__device__ __forceinline__ void row_sub(const RowView<T>& A, int row, int lane, const T* __restrict__ x, T (&acc)[D]) {
    const int e = A.rp[row + 1];
    for (int p = A.rp[row] + lane; p < e; p += WAVE) {
        T xj[D];
        load_vec<T, D>(x + (int64_t)A.col[p] * D, xj);
        T blk[D * D];
        load_block<T, D * D>(A.val + (int64_t)p * D * D, blk);
#pragma unroll
        for (int r = 0; r < D; ++r)
#pragma unroll
            for (int c = 0; c < D; ++c) acc[r] -= blk[r * D + c] * xj[c];
    }
}

// The same sums with the row's values read back to back: in a pass over the
// row, lane u reads the u-th 16-byte piece (one block row of a float block,
// half of a double one), so one load instruction covers 1 KiB with no gaps.
// Every lane keeps one block-row position (the row's first block starts a
// piece group), so its partial sum belongs to one component r.
template <class T, int D>
__device__ __forceinline__ void row_sub_c(const RowView<T>& A, int row, int lane, const T* __restrict__ x,
                                          T (&acc)[D]) {
    constexpr int V = 16 / (int)sizeof(T);   // values per piece
    static_assert(D % V == 0, "block rows split into 16-byte pieces");
    constexpr int LR = D / V;                // pieces per block row
    constexpr int LB = D * LR;               // pieces per block
    static_assert(WAVE % LB == 0, "a pass keeps every lane on one block-row position");
    constexpr int UNROLL = 4;
    const int part = lane % LB;
    const int r = part / LR, c0 = (part % LR) * V;
    const int64_t u0 = (int64_t)A.rp[row] * LB, u1 = (int64_t)A.rp[row + 1] * LB;
    T sum = T(0);
    for (int64_t ub = u0; ub < u1; ub += UNROLL * WAVE) {
        T av[UNROLL][V], xv[UNROLL][V];
        bool ok[UNROLL];
#pragma unroll
        for (int h = 0; h < UNROLL; ++h) {
            const int64_t u = ub + (int64_t)h * WAVE + lane;
            ok[h] = u < u1;
            const int64_t uc = ok[h] ? u : u0 + part;   // in range: the row's first block
            load_vec<T, V>(A.val + uc * V, av[h]);
            load_vec<T, V>(x + (int64_t)A.col[uc / LB] * D + c0, xv[h]);
        }
#pragma unroll
        for (int h = 0; h < UNROLL; ++h) {
            T s = T(0);
#pragma unroll
            for (int c = 0; c < V; ++c) s += av[h][c] * xv[h][c];
            sum += ok[h] ? s : T(0);
        }
    }
#pragma unroll
    for (int rr = 0; rr < D; ++rr) acc[rr] -= rr == r ? sum : T(0);
}

// Sum over the wavefront, valid in lane WAVE - 1, per component.
template <class T, int D>
__device__ __forceinline__ void wave_sum_vec(T (&acc)[D]) {
#pragma unroll
    for (int r = 0; r < D; ++r) acc[r] = group_sum<64>(acc[r]);
}

// y = A x (or y += A x when accumulating) for a transfer in row form: one
// wavefront per row, the row's blocks read as in the row-form smoother.
template <class T, int D>
__global__ __launch_bounds__(256) void k_xfer_rows(XferRowArgs<T> a) {
    const int lane = threadIdx.x & (WAVE - 1);
    int row = blockIdx.x * WPB + wave_id();
    int f = 0;
    if (row >= a.n[0]) {
        row -= a.n[0];
        f = 1;
        if (row >= a.n[1]) return;   // whole wavefront
    }
    T acc[D];
#pragma unroll
    for (int r = 0; r < D; ++r) acc[r] = T(0);
    if constexpr (D == 4) row_sub_c<T, D>(a.A[f], row, lane, a.x[f], acc);
    else row_sub<T, D>(a.A[f], row, lane, a.x[f], acc);
    wave_sum_vec<T, D>(acc);
    if (lane != WAVE - 1) return;
    const int orow = a.out_row[f] ? a.out_row[f][row] : row;
    T out[D];
    if (a.accumulate) {
        T y[D];
        load_vec<T, D>(a.y[f] + (int64_t)orow * D, y);
#pragma unroll
        for (int r = 0; r < D; ++r) out[r] = y[r] - acc[r];
    } else {
#pragma unroll
        for (int r = 0; r < D; ++r) out[r] = -acc[r];
    }
    store_vec<T, D>(a.y[f] + (int64_t)orow * D, out);
}

template <class T>
void launch_xfer_rows(int d, const XferRowArgs<T>& a, hipStream_t s) {
    const int64_t total = (int64_t)a.n[0] + a.n[1];
    if (total <= 0) return;
    const unsigned grid = (unsigned)ceil_div(total, WPB);
    switch (d) {
        case 1: k_xfer_rows<T, 1><<<grid, 256, 0, s>>>(a); break;
        case 2: k_xfer_rows<T, 2><<<grid, 256, 0, s>>>(a); break;
        case 3: k_xfer_rows<T, 3><<<grid, 256, 0, s>>>(a); break;
        case 4: k_xfer_rows<T, 4><<<grid, 256, 0, s>>>(a); break;
        default: throw Error(MBAMG_E_INVALID, "dofs per node must be 1..4");
    }
    MB_LAUNCH_CHECK();
}
template void launch_xfer_rows<double>(int, const XferRowArgs<double>&, hipStream_t);
template void launch_xfer_rows<float>(int, const XferRowArgs<float>&, hipStream_t);

// r = b - A x (or w = A x when b is NULL) for both block rows in one launch.
template <class T, class TX, int D, int P, int S, bool C16>
__global__ __launch_bounds__(waves_per_block<P>() * WAVE) void k_resid(ResidArgs<T, TX> a, int padded_blocks) {
    const int wave = wave_id();
    const int part = wave % P;
    int sidx = xcd_block(padded_blocks) * (waves_per_block<P>() / P) + wave / P;
    int f = 0;
    bool valid = true;
    if (sidx >= a.s_count[0]) {
        sidx -= a.s_count[0];
        f = 1;
        if (sidx >= a.s_count[1]) valid = false;
    }
    if (P == 1 && !valid) return;
    if (!valid) {   // padding wave of a split slice: read any existing slice, write nothing
        f = a.s_count[0] > 0 ? 0 : 1;
        sidx = 0;
    } else if (a.order[f]) {
        sidx = a.order[f][sidx];
    }
    const int g = 1 - f;
    const int lane = threadIdx.x & (WAVE - 1);
    const int row0 = a.sl[f].row0[sidx], nrow = a.sl[f].nrow[sidx];
    const bool act = valid && lane < nrow;
    const int row = row0 + (lane < nrow ? lane : 0);
    T acc[D];
#pragma unroll
    for (int r = 0; r < D; ++r) acc[r] = T(0);
    if (valid) {
        sell_sub<T, D, 0, P, S, false, C16>(a.diag[f], sidx, lane, part, a.x[f], nullptr, 0, acc);
        sell_sub<T, D, 0, P, S, false, C16>(a.off[f], sidx, lane, part, a.x[f], nullptr, 0, acc);
        sell_sub<T, D, 0, P, S, false, C16>(a.cpl[f], sidx, lane, part, a.x[g], nullptr, 0, acc);
    }
    combine_parts<T, D, P>(acc, wave, part, lane);
    if (part != 0 || !act) return;
    T out[D];
    if (a.b[f]) {
        T bb[D];
        load_vec<T, D>(a.b[f] + (int64_t)row * D, bb);
#pragma unroll
        for (int r = 0; r < D; ++r) out[r] = bb[r] + acc[r];
    } else {
#pragma unroll
        for (int r = 0; r < D; ++r) out[r] = -acc[r];
    }
    store_vec<T, D>(a.r[f] + (int64_t)row * D, out);
}

// y = A x (or y += A x) for both blocks in one launch: the smoothed
// prolongator (rows of the fine level) and its transpose (rows of the coarse
// level) in masked sliced-ELL form.
template <class T, int D, int P>
__global__ __launch_bounds__(waves_per_block<P>() * WAVE) void k_xfer(XferArgs<T> a, int padded_blocks) {
    const int wave = wave_id();
    const int part = wave % P;
    int sidx = xcd_block(padded_blocks) * (waves_per_block<P>() / P) + wave / P;
    int f = 0;
    bool valid = true;
    if (sidx >= a.s_count[0]) {
        sidx -= a.s_count[0];
        f = 1;
        if (sidx >= a.s_count[1]) valid = false;
    }
    if (P == 1 && !valid) return;
    if (!valid) {   // padding wave of a split slice: read any existing slice, write nothing
        f = a.s_count[0] > 0 ? 0 : 1;
        sidx = 0;
    }
    const int lane = threadIdx.x & (WAVE - 1);
    const int row0 = a.sl[f].row0[sidx], nrow = a.sl[f].nrow[sidx];
    const int row = row0 + (lane < nrow ? lane : 0);
    T acc[D];
#pragma unroll
    for (int r = 0; r < D; ++r) acc[r] = T(0);
    if (valid) sell_sub<T, D, 0, P>(a.A[f], sidx, lane, part, a.x[f], nullptr, 0, acc);
    combine_parts<T, D, P>(acc, wave, part, lane);
    if (part != 0 || !valid || lane >= nrow) return;
    const int orow = a.out_row[f] ? a.out_row[f][row] : row;
    T out[D];
    if (a.accumulate) {
        T y[D];
        load_vec<T, D>(a.y[f] + (int64_t)orow * D, y);
#pragma unroll
        for (int r = 0; r < D; ++r) out[r] = y[r] - acc[r];
    } else {
#pragma unroll
        for (int r = 0; r < D; ++r) out[r] = -acc[r];
    }
    store_vec<T, D>(a.y[f] + (int64_t)orow * D, out);
}

// Sum over aligned groups of G lanes, valid in each group's last lane, per component.
template <class T, int D, int G>
__device__ __forceinline__ void group_sum_vec(T (&acc)[D]) {
#pragma unroll
    for (int r = 0; r < D; ++r) acc[r] = group_sum<G>(acc[r]);
}

// coarse b_k = sum over members i of aggregate k of q_i .* r_i (per component):
// G lanes per coarse row, the members strided over them (their rows are
// scattered over the fine vector, so many are fetched at once; the weights q
// are stored in member-list order, so only r is gathered)
template <class T, int D, int G>
__global__ __launch_bounds__(256) void k_restrict(TransferArgs<T> a, int padded_blocks) {
    // consecutive coarse rows (neighbouring aggregates, which share fine rows' cache lines)
    // go to the same XCD
    const int64_t t = (int64_t)xcd_block(padded_blocks) * blockDim.x + threadIdx.x;
    int k = (int)(t / G);
    const int gl = (int)(t % G);
    int f = 0;
    if (k >= a.n_rows[0]) {
        k -= a.n_rows[0];
        f = 1;
        if (k >= a.n_rows[1]) return;   // whole groups
    }
    if (a.order[f]) k = a.order[f][k];
    const int32_t* mp = a.map[f];
    const int32_t* mi = a.idx[f];
    T acc[D];
#pragma unroll
    for (int c = 0; c < D; ++c) acc[c] = T(0);
    for (int m = mp[k] + gl; m < mp[k + 1]; m += G) {
        const int64_t i = mi[m];
        const T q = a.q[f][m];
        T r[D];
        load_vec<T, D>(a.in[f] + i * D, r);
#pragma unroll
        for (int c = 0; c < D; ++c) acc[c] += q * r[c];
    }
    group_sum_vec<T, D, G>(acc);
    if (gl == G - 1) store_vec<T, D>(a.out[f] + (int64_t)k * D, acc);
}

// x_i += q_i x_c[agg(i)]
template <class T, int D>
__global__ void k_prolong(TransferArgs<T> a) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    int f = 0;
    if (i >= a.n_rows[0]) {
        i -= a.n_rows[0];
        f = 1;
        if (i >= a.n_rows[1]) return;
    }
    const int64_t k = a.map[f][i];
    const T q = a.q[f][i];
    T xc[D], x[D];
    load_vec<T, D>(a.in[f] + k * D, xc);
    load_vec<T, D>(a.out[f] + (int64_t)i * D, x);
#pragma unroll
    for (int c = 0; c < D; ++c) x[c] += q * xc[c];
    store_vec<T, D>(a.out[f] + (int64_t)i * D, x);
}

// y = inv * x with the inverse in FP64 (one wavefront per row).  A row's loads are a
// chain when they are waited for one by one: COARSE_CH of them go out together
// (2,152 unknowns 19.4 -> 13.5 us, 930 unknowns 6.0 -> 3.9 us; 16 together, 15.6 and 4.1).
constexpr int COARSE_CH = 8;
template <class T>
__global__ __launch_bounds__(256) void k_coarse(int n, const double* __restrict__ inv, const T* __restrict__ x,
                                                T* __restrict__ y) {
    const int row = blockIdx.x * WPB + (threadIdx.x >> 6);
    const int lane = threadIdx.x & (WAVE - 1);
    if (row >= n) return;
    const double* a = inv + (int64_t)row * n;
    double s = 0.0;
    for (int c0 = lane; c0 < n; c0 += COARSE_CH * WAVE) {
        double av[COARSE_CH], xv[COARSE_CH];
#pragma unroll
        for (int u = 0; u < COARSE_CH; ++u) {
            const int c = min(c0 + u * WAVE, n - 1);
            av[u] = a[c];
            xv[u] = (double)x[c];
        }
#pragma unroll
        for (int u = 0; u < COARSE_CH; ++u)
            if (c0 + u * WAVE < n) s += av[u] * xv[u];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, WAVE);
    if (lane == 0) y[row] = (T)s;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <class T, int D, int P, int S, bool C16>
static void gs_dispatch_c(bool zx, bool cpl, const GsArgs<T>& a, hipStream_t s) {
    unsigned grid = xcd_grid(a.s_count, P);
    int pb = (int)grid;
    constexpr int TPB = waves_per_block<P>() * WAVE;
    if (zx) {
        if (cpl) k_gs<T, D, true, true, P, S, C16><<<grid, TPB, 0, s>>>(a, pb);
        else k_gs<T, D, true, false, P, S, C16><<<grid, TPB, 0, s>>>(a, pb);
    } else {
        if (cpl) k_gs<T, D, false, true, P, S, C16><<<grid, TPB, 0, s>>>(a, pb);
        else k_gs<T, D, false, false, P, S, C16><<<grid, TPB, 0, s>>>(a, pb);
    }
}

template <class T, int D, int P, int S>
static void gs_dispatch(bool zx, bool cpl, const GsArgs<T>& a, hipStream_t s) {
    if constexpr (P == 1) {
        if (a.off.col16) return gs_dispatch_c<T, D, P, S, true>(zx, cpl, a, s);
    }
    MB_CHECK(!a.off.col16, MBAMG_E_INVALID, "split slices have 32-bit columns");
    gs_dispatch_c<T, D, P, S, false>(zx, cpl, a, s);
}

template <class T, int D>
static void gs_dispatch_p(int P, bool zx, bool cpl, const GsArgs<T>& a, hipStream_t s) {
    if constexpr (D > 1) {
        if (a.shape != SHAPE_FULL) {
            MB_CHECK(P <= SHAPE_MAX_SPLIT, MBAMG_E_INVALID, "slot split too large for this block shape");
            if (a.shape == SHAPE_SCALED) {
                if (P == 1) gs_dispatch<T, D, 1, SHAPE_SCALED>(zx, cpl, a, s);
                else gs_dispatch<T, D, 2, SHAPE_SCALED>(zx, cpl, a, s);
            } else {
                if (P == 1) gs_dispatch<T, D, 1, SHAPE_SYMMETRIC>(zx, cpl, a, s);
                else gs_dispatch<T, D, 2, SHAPE_SYMMETRIC>(zx, cpl, a, s);
            }
            return;
        }
    }
    switch (P) {
        case 1: gs_dispatch<T, D, 1, SHAPE_FULL>(zx, cpl, a, s); break;
        case 2: gs_dispatch<T, D, 2, SHAPE_FULL>(zx, cpl, a, s); break;
        case 4: gs_dispatch<T, D, 4, SHAPE_FULL>(zx, cpl, a, s); break;
        case 8: gs_dispatch<T, D, 8, SHAPE_FULL>(zx, cpl, a, s); break;
        case 16: gs_dispatch<T, D, 16, SHAPE_FULL>(zx, cpl, a, s); break;
        default: throw Error(MBAMG_E_INVALID, "slot split must be 1, 2, 4, 8 or 16");
    }
}

template <class T>
void launch_gs(int d, int P, bool zero_x, bool has_cpl, const GsArgs<T>& a, hipStream_t s) {
    if (a.s_count <= 0) return;
    switch (d) {
        case 1: gs_dispatch_p<T, 1>(P, zero_x, has_cpl, a, s); break;
        case 2: gs_dispatch_p<T, 2>(P, zero_x, has_cpl, a, s); break;
        case 3: gs_dispatch_p<T, 3>(P, zero_x, has_cpl, a, s); break;
        case 4: gs_dispatch_p<T, 4>(P, zero_x, has_cpl, a, s); break;
        default: throw Error(MBAMG_E_INVALID, "dofs per node must be 1..4");
    }
    MB_LAUNCH_CHECK();
}

template <class T, int D, int P>
static void gs_fc_dispatch(bool zx, const GsFcArgs<T>& a, hipStream_t s) {
    const unsigned grid = xcd_grid(a.s_count, P);
    constexpr int TPB = waves_per_block<P>() * WAVE;
    if (zx) k_gs_fc<T, D, true, P><<<grid, TPB, 0, s>>>(a, (int)grid);
    else k_gs_fc<T, D, false, P><<<grid, TPB, 0, s>>>(a, (int)grid);
}

template <class T, int D>
static void gs_fc_dispatch_p(int P, bool zx, const GsFcArgs<T>& a, hipStream_t s) {
    switch (P) {
        case 1: gs_fc_dispatch<T, D, 1>(zx, a, s); break;
        case 2: gs_fc_dispatch<T, D, 2>(zx, a, s); break;
        case 4: gs_fc_dispatch<T, D, 4>(zx, a, s); break;
        case 8: gs_fc_dispatch<T, D, 8>(zx, a, s); break;
        case 16: gs_fc_dispatch<T, D, 16>(zx, a, s); break;
        default: throw Error(MBAMG_E_INVALID, "slot split must be 1, 2, 4, 8 or 16");
    }
}

template <class T>
void launch_gs_fc(int d, int P, bool zero_x, const GsFcArgs<T>& a, hipStream_t s) {
    if (a.s_count <= 0) return;
    switch (d) {
        case 1: gs_fc_dispatch_p<T, 1>(P, zero_x, a, s); break;
        case 2: gs_fc_dispatch_p<T, 2>(P, zero_x, a, s); break;
        case 3: gs_fc_dispatch_p<T, 3>(P, zero_x, a, s); break;
        case 4: gs_fc_dispatch_p<T, 4>(P, zero_x, a, s); break;
        default: throw Error(MBAMG_E_INVALID, "dofs per node must be 1..4");
    }
    MB_LAUNCH_CHECK();
}

template <class T, class TX, int D, int P, int S>
static void resid_dispatch_p(unsigned grid, const ResidArgs<T, TX>& a, hipStream_t s) {
    constexpr int TPB = waves_per_block<P>() * WAVE;
    if constexpr (P == 1) {
        if (a.off[0].col16) {
            k_resid<T, TX, D, P, S, true><<<grid, TPB, 0, s>>>(a, (int)grid);
            return;
        }
    }
    MB_CHECK(!a.off[0].col16, MBAMG_E_INVALID, "split slices have 32-bit columns");
    k_resid<T, TX, D, P, S, false><<<grid, TPB, 0, s>>>(a, (int)grid);
}

template <class T, class TX, int D>
static void resid_dispatch(int P, const ResidArgs<T, TX>& a, hipStream_t s) {
    const int total = a.s_count[0] + a.s_count[1];
    unsigned grid = xcd_grid(total, P);
    MB_CHECK(!a.off[0].col16 == !a.off[1].col16, MBAMG_E_INVALID, "both blocks' columns in one width");
    if constexpr (D > 1) {
        if (a.shape != SHAPE_FULL) {
            MB_CHECK(P <= SHAPE_MAX_SPLIT, MBAMG_E_INVALID, "slot split too large for this block shape");
            if (a.shape == SHAPE_SCALED) {
                if (P == 1) resid_dispatch_p<T, TX, D, 1, SHAPE_SCALED>(grid, a, s);
                else resid_dispatch_p<T, TX, D, 2, SHAPE_SCALED>(grid, a, s);
            } else {
                if (P == 1) resid_dispatch_p<T, TX, D, 1, SHAPE_SYMMETRIC>(grid, a, s);
                else resid_dispatch_p<T, TX, D, 2, SHAPE_SYMMETRIC>(grid, a, s);
            }
            return;
        }
    }
    switch (P) {
        case 1: resid_dispatch_p<T, TX, D, 1, SHAPE_FULL>(grid, a, s); break;
        case 2: resid_dispatch_p<T, TX, D, 2, SHAPE_FULL>(grid, a, s); break;
        case 4: resid_dispatch_p<T, TX, D, 4, SHAPE_FULL>(grid, a, s); break;
        case 8: resid_dispatch_p<T, TX, D, 8, SHAPE_FULL>(grid, a, s); break;
        case 16: resid_dispatch_p<T, TX, D, 16, SHAPE_FULL>(grid, a, s); break;
        default: throw Error(MBAMG_E_INVALID, "slot split must be 1, 2, 4, 8 or 16");
    }
}

template <class T, class TX>
void launch_resid(int d, int P, const ResidArgs<T, TX>& a, hipStream_t s) {
    if (a.s_count[0] + a.s_count[1] <= 0) return;
    switch (d) {
        case 1: resid_dispatch<T, TX, 1>(P, a, s); break;
        case 2: resid_dispatch<T, TX, 2>(P, a, s); break;
        case 3: resid_dispatch<T, TX, 3>(P, a, s); break;
        case 4: resid_dispatch<T, TX, 4>(P, a, s); break;
        default: throw Error(MBAMG_E_INVALID, "dofs per node must be 1..4");
    }
    MB_LAUNCH_CHECK();
}

template <class T, int D>
static void xfer_dispatch(int P, const XferArgs<T>& a, hipStream_t s) {
    const int total = a.s_count[0] + a.s_count[1];
    unsigned grid = xcd_grid(total, P);
    int pb = (int)grid;
    switch (P) {
        case 1: k_xfer<T, D, 1><<<grid, 256, 0, s>>>(a, pb); break;
        case 2: k_xfer<T, D, 2><<<grid, 256, 0, s>>>(a, pb); break;
        case 4: k_xfer<T, D, 4><<<grid, 256, 0, s>>>(a, pb); break;
        case 8: k_xfer<T, D, 8><<<grid, 512, 0, s>>>(a, pb); break;
        case 16: k_xfer<T, D, 16><<<grid, 1024, 0, s>>>(a, pb); break;
        default: throw Error(MBAMG_E_INVALID, "slot split must be 1, 2, 4, 8 or 16");
    }
}

template <class T>
void launch_xfer(int d, int P, const XferArgs<T>& a, hipStream_t s) {
    if (a.s_count[0] + a.s_count[1] <= 0) return;
    switch (d) {
        case 1: xfer_dispatch<T, 1>(P, a, s); break;
        case 2: xfer_dispatch<T, 2>(P, a, s); break;
        case 3: xfer_dispatch<T, 3>(P, a, s); break;
        case 4: xfer_dispatch<T, 4>(P, a, s); break;
        default: throw Error(MBAMG_E_INVALID, "dofs per node must be 1..4");
    }
    MB_LAUNCH_CHECK();
}
template void launch_xfer<double>(int, int, const XferArgs<double>&, hipStream_t);
template void launch_xfer<float>(int, int, const XferArgs<float>&, hipStream_t);

template <class T, int D>
static void restrict_dispatch(int64_t total, int G, const TransferArgs<T>& a, hipStream_t s) {
    const unsigned grid = (unsigned)(ceil_div(ceil_div(total * G, 256), 8) * 8);
    const int pb = (int)grid;
    switch (G) {
        case 4: k_restrict<T, D, 4><<<grid, 256, 0, s>>>(a, pb); break;
        case 8: k_restrict<T, D, 8><<<grid, 256, 0, s>>>(a, pb); break;
        case 16: k_restrict<T, D, 16><<<grid, 256, 0, s>>>(a, pb); break;
        default: k_restrict<T, D, 64><<<grid, 256, 0, s>>>(a, pb); break;
    }
}

template <class T>
void launch_restrict(int d, const TransferArgs<T>& a, int G, hipStream_t s) {
    const int64_t total = (int64_t)a.n_rows[0] + a.n_rows[1];
    if (total <= 0) return;
    MB_CHECK(G == 4 || G == 8 || G == 16 || G == 64, MBAMG_E_INVALID, "restriction group of 4, 8, 16 or 64 lanes");
    switch (d) {
        case 1: restrict_dispatch<T, 1>(total, G, a, s); break;
        case 2: restrict_dispatch<T, 2>(total, G, a, s); break;
        case 3: restrict_dispatch<T, 3>(total, G, a, s); break;
        case 4: restrict_dispatch<T, 4>(total, G, a, s); break;
        default: throw Error(MBAMG_E_INVALID, "dofs per node must be 1..4");
    }
    MB_LAUNCH_CHECK();
}

template <class T>
void launch_prolong(int d, const TransferArgs<T>& a, hipStream_t s) {
    const int total = a.n_rows[0] + a.n_rows[1];
    if (total <= 0) return;
    unsigned grid = (unsigned)ceil_div(total, 256);
    switch (d) {
        case 1: k_prolong<T, 1><<<grid, 256, 0, s>>>(a); break;
        case 2: k_prolong<T, 2><<<grid, 256, 0, s>>>(a); break;
        case 3: k_prolong<T, 3><<<grid, 256, 0, s>>>(a); break;
        case 4: k_prolong<T, 4><<<grid, 256, 0, s>>>(a); break;
        default: throw Error(MBAMG_E_INVALID, "dofs per node must be 1..4");
    }
    MB_LAUNCH_CHECK();
}

template <class T>
void launch_coarse(int n, const double* inv, const T* x, T* y, hipStream_t s) {
    if (n <= 0) return;
    k_coarse<T><<<(unsigned)ceil_div(n, WPB), 256, 0, s>>>(n, inv, x, y);
    MB_LAUNCH_CHECK();
}

template void launch_gs<double>(int, int, bool, bool, const GsArgs<double>&, hipStream_t);
template void launch_gs_fc<double>(int, int, bool, const GsFcArgs<double>&, hipStream_t);
template void launch_gs_fc<float>(int, int, bool, const GsFcArgs<float>&, hipStream_t);
template void launch_gs<float>(int, int, bool, bool, const GsArgs<float>&, hipStream_t);
template void launch_resid<double, double>(int, int, const ResidArgs<double>&, hipStream_t);
template void launch_resid<float, float>(int, int, const ResidArgs<float>&, hipStream_t);
template void launch_resid<double, float>(int, int, const ResidArgs<double, float>&, hipStream_t);
template void launch_restrict<double>(int, const TransferArgs<double>&, int, hipStream_t);
template void launch_restrict<float>(int, const TransferArgs<float>&, int, hipStream_t);
template void launch_prolong<double>(int, const TransferArgs<double>&, hipStream_t);
template void launch_prolong<float>(int, const TransferArgs<float>&, hipStream_t);
template void launch_coarse<double>(int, const double*, const double*, double*, hipStream_t);
template void launch_coarse<float>(int, const double*, const float*, float*, hipStream_t);

// ---------------------------------------------------------------------------
// Krylov kernels: fixed grid, per-block partial sums; the block that finishes
// last adds them up in a fixed order
// ---------------------------------------------------------------------------
constexpr int KT = 256, KW = KT / WAVE;   // threads and wavefronts per block

// This block's sums of N per-thread values, left in the first N threads' return
// values: wavefront sums by DPP moves (no barrier per value), one pass through LDS.
template <int N>
__device__ __forceinline__ double block_sums(double (&v)[N], double (*sh)[KMAXQ]) {
    const int t = threadIdx.x, lane = t & (WAVE - 1), w = t / WAVE;
#pragma unroll
    for (int q = 0; q < N; ++q) {
        v[q] = group_sum<WAVE>(v[q]);
        if (lane == WAVE - 1) sh[w][q] = v[q];
    }
    __syncthreads();
    double r = 0.0;
    if (t < N) {
        r = sh[0][t];
#pragma unroll
        for (int k = 1; k < KW; ++k) r += sh[k][t];
    }
    return r;
}

// Publishes this block's N sums (thread q < N holds sum q) and tells whether it is
// the last block to do so; that block gets the totals in res (all threads, after
// the return) and leaves the counters at zero for the next launch.  The counters say
// who is last, not that the others' partials can be seen yet: a partial is its own
// signal ("unwritten" before) and is loaded until it is there, which it nearly always
// is.  (A release at device scope before the increment would write back the XCD's
// whole L2, once per block.)  The two sets of partials take turns: a launch sets what
// the one before it used of the other set to "unwritten".
template <int N>
__device__ __forceinline__ bool last_block_totals(double mine, const KrylovBufs& kb, double* res) {
    __shared__ int last;
    const int t = threadIdx.x, nb = gridDim.x;
    static_assert(KMAXQ <= KT, "a thread per partial");
    if (t < kb.n_next)
        __hip_atomic_store(kb.partial_next + (int64_t)t * KBLOCKS + blockIdx.x, unwritten_value<double>(),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (t < N)
        __hip_atomic_store(kb.partial + (int64_t)t * KBLOCKS + blockIdx.x, unwritten(mine) ? (double)NAN : mine,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    // increments of one address take 11 ns each (1024 blocks: 12 us at the end of a short
    // pass), so the blocks count in KCOUNTERS groups, and the groups' last ones in one more
    if (t == 0) {
        const int k = blockIdx.x % KCOUNTERS, members = (nb - k + KCOUNTERS - 1) / KCOUNTERS;
        uint32_t* sub = kb.counter + (1 + k) * KCOUNTER_STRIDE;
        last = 0;
        if (__hip_atomic_fetch_add(sub, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)members - 1u) {
            __hip_atomic_store(sub, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int groups = nb < KCOUNTERS ? nb : KCOUNTERS;
            last = __hip_atomic_fetch_add(kb.counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                   (uint32_t)groups - 1u;
            if (last) __hip_atomic_store(kb.counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
    if (!last) return false;
    // 8 lanes per sum, all sums at once: lane l adds the blocks l, l + 8, ... in turn (32
    // loads in flight, 16 where that covers the blocks), then the group (a wavefront per sum
    // took the sums one after the other)
    constexpr int G = 8;
    static_assert(N <= 2 * (KT / G), "two sums per group at most");
    const int l = t % G;
    auto partial_at = [&](int q, int b) {
        return __hip_atomic_load(kb.partial + (int64_t)q * KBLOCKS + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto add_all = [&](auto in_flight) {
        constexpr int U = decltype(in_flight)::value;
        for (int q = t / G; q < N; q += KT / G) {
            double v = 0.0;
            for (int b0 = l; b0 < nb; b0 += U * G) {
                double x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) x[u] = b0 + u * G < nb ? partial_at(q, b0 + u * G) : 0.0;
                for (int round = 0;; ++round) {
                    bool more = false;
#pragma unroll
                    for (int u = 0; u < U; ++u) more = more || unwritten(x[u]);
                    if (!__any(more)) break;
                    if (round >= kb.wait.rounds) {
                        __hip_atomic_store(kb.wait.late, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                        break;
                    }
                    pause_after(round);
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (unwritten(x[u])) x[u] = partial_at(q, b0 + u * G);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) v += x[u];
            }
            v = group_sum<G>(v);
            if (l == G - 1) res[q] = v;
        }
    };
    if (nb <= 16 * G) add_all(std::integral_constant<int, 16>{});
    else add_all(std::integral_constant<int, 32>{});
    __syncthreads();
    return true;
}

// Dot pass: r_q = V_q . w (q < NQ) and, WITH_NORM, r_NQ = w . w.  NQ is the exact
// count (one instance per count: guarded loads would cost a branch each and
// registers for the predicates); all loads of one element are issued before any
// use.  The last block writes kb.d1[q] = r_q (q < NQ), or *kb.nu2 = r_0 for a norm, and
// the delayed reorthogonalisation's coefficients b_q = r_q (q < NQ - 1) and
// c_j = (r_{NQ-1} - sum_q a_q r_q) / nu.  At 16.8M unknowns the pass streams 5.9 TB/s
// (27 vectors 640 us); four wavefronts per unit are all the grid has, and without the
// attribute the compiler kept some counts' loads back to fit eight (24 - 26, 29 and 30
// vectors 800 - 880 us).
template <int NQ, bool NORM>
__global__ __launch_bounds__(KT) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_orth(int64_t n, const double* __restrict__ V, int64_t ldv,
                                             const double* __restrict__ w, KrylovBufs kb) {
    constexpr int N = NORM ? 1 : NQ;
    __shared__ double sh[KW][KMAXQ];
    __shared__ double res[KMAXQ];
    double acc[N];
#pragma unroll
    for (int q = 0; q < N; ++q) acc[q] = 0.0;
    const int64_t stride = (int64_t)gridDim.x * KT;
    for (int64_t e = (int64_t)blockIdx.x * KT + threadIdx.x; e < n; e += stride) {
        const double u = w[e];
        if constexpr (NORM) {
            acc[0] += u * u;
        } else {
            double v[N];
#pragma unroll
            for (int q = 0; q < N; ++q) v[q] = V[q * ldv + e];
#pragma unroll
            for (int q = 0; q < N; ++q) acc[q] += v[q] * u;
        }
    }
    const double mine = block_sums<N>(acc, sh);
    if (!last_block_totals<N>(mine, kb, res)) return;
    const int t = threadIdx.x;
    if constexpr (NORM) {
        if (t == 0) *kb.nu2 = res[0];
    } else {
        if (t < NQ) kb.d1[t] = res[t];
        if (t < NQ - 1) kb.coef[KC_B + t] = res[t];
        if (t == 0) {
            double ab = 0.0;
            for (int k = 0; k < NQ - 1; ++k) ab += kb.coef[KC_A + k] * res[k];
            kb.coef[KC_CJ] = (res[NQ - 1] - ab) * kb.coef[KC_INV_NU];
        }
    }
}

// Update pass of classical Gram-Schmidt with delayed reorthogonalisation
// (DCGS2: Swirydowicz, Langou, Ananthan, Yang & Thomas 2020; Bielich et al.
// 2022).  Q_0..Q_{NQ-1} are final orthonormal basis vectors, u the candidate for
// Q_NQ (projected once), w the operator applied to the preconditioned u, and
// coef holds a = Q^T u (found by the previous update pass), b = Q^T w, 1/nu with
// nu = |u - Q a|, and c_j = (u . w - a . b) / nu.  Per element:
//   q  = (u - sum_k a_k Q_k) / nu            (the reorthogonalised candidate, over u)
//   un = (w - sum_k b_k Q_k - c_j q) / nu     (the next candidate, projected once)
// and the dots a' = [Q q]^T un and |un|^2 for the next step.  The last block
// writes them out (d2, nu2), the next candidate's nu' = sqrt(|un|^2 - |a'|^2) (nu;
// 0 when the candidate lies in the basis) and the next step's coefficients a' and
// 1/nu', so the next step needs nothing from the host.  out32 (may be null): un in
// FP32, for a preconditioner that runs in it.  NQ is the exact count.
template <int NQ>
__global__ __launch_bounds__(KT) void k_dcgs_update(int64_t n, const double* __restrict__ V, int64_t ldv, double* u,
                                                    const double* __restrict__ w, double* __restrict__ out,
                                                    float* __restrict__ out32, KrylovBufs kb) {
    constexpr int NV = NQ > 0 ? NQ : 1;
    __shared__ double sh[KW][KMAXQ];
    __shared__ double res[KMAXQ];
    __shared__ double cab[2 * NV];
    if (threadIdx.x < NQ) {
        cab[threadIdx.x] = kb.coef[KC_A + threadIdx.x];
        cab[NQ + threadIdx.x] = kb.coef[KC_B + threadIdx.x];
    }
    const double inv_nu = kb.coef[KC_INV_NU];
    const double cj = kb.coef[KC_CJ];
    __syncthreads();
    double acc[NQ + 2];   // Q_k . un, q . un, un . un
#pragma unroll
    for (int k = 0; k < NQ + 2; ++k) acc[k] = 0.0;
    const int64_t stride = (int64_t)gridDim.x * KT;
    for (int64_t e = (int64_t)blockIdx.x * KT + threadIdx.x; e < n; e += stride) {
        double v[NV];
#pragma unroll
        for (int k = 0; k < NQ; ++k) v[k] = V[k * ldv + e];
        double q = u[e];
        double un = w[e];
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
            q -= cab[k] * v[k];
            un -= cab[NQ + k] * v[k];
        }
        q *= inv_nu;
        un = (un - cj * q) * inv_nu;
        u[e] = q;
        out[e] = un;
        if (out32) out32[e] = (float)un;
#pragma unroll
        for (int k = 0; k < NQ; ++k) acc[k] += v[k] * un;
        acc[NQ] += q * un;
        acc[NQ + 1] += un * un;
    }
    const double mine = block_sums<NQ + 2>(acc, sh);
    if (!last_block_totals<NQ + 2>(mine, kb, res)) return;
    const int t = threadIdx.x;
    // every block has read its coefficients: its sums, which have arrived, depend on them
    if (t <= NQ) {
        kb.d2[t] = res[t];
        kb.coef[KC_A + t] = res[t];
    }
    if (t == 0) {
        double nu2 = res[NQ + 1];
        for (int k = 0; k <= NQ; ++k) nu2 -= res[k] * res[k];
        const double nu = nu2 > 0.0 && nu2 <= 1.7976931348623157e308 ? sqrt(nu2) : 0.0;
        *kb.nu = nu;
        kb.coef[KC_INV_NU] = nu > 0.0 ? 1.0 / nu : 0.0;
    }
}

template <class TZ>
__global__ void k_combine(int64_t n, int k, const TZ* __restrict__ Z, int64_t ldz, const double* __restrict__ y,
                          double* __restrict__ x) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        double s = x[e];
        for (int q = 0; q < k; ++q) s += y[q] * (double)Z[q * ldz + e];
        x[e] = s;
    }
}

__global__ void k_axpby(int64_t n, double a, const double* __restrict__ x, double b, double* __restrict__ y) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
        y[e] = a * x[e] + b * y[e];
}

// Between the interface's order and the colour order, all blocks in one launch:
// block f's rows i in natural order, iperm[i] their colour positions.  The natural
// side is read or written straight through; the colour side is as many sequential
// streams as there are colours.  (One launch per block, in colour order, read or
// wrote the natural side in 32-byte pieces of every line, once per colour, and
// divided 64-bit indices by the block size: 76 us in and 88 us out for 16.8M
// unknowns.  The V-cycle of that size 2023 -> 1953 us, the operator on 8.1M unknowns
// 237 -> 208 us.)
constexpr int REORDER_PER_THREAD = 4, REORDER_PER_BLOCK = REORDER_PER_THREAD * 256;
template <int D, bool TO_COLOUR>
__device__ __forceinline__ void reorder_elements(int64_t first, int64_t len, const int32_t* __restrict__ iperm,
                                                 const double* __restrict__ src, double* __restrict__ dst) {
#pragma unroll
    for (int u = 0; u < REORDER_PER_THREAD; ++u) {
        const int64_t t = first + u * 256 + threadIdx.x;
        if (t >= len) continue;
        const uint32_t e = (uint32_t)t, i = e / D;   // at most 2^31 rows of D: see the launcher
        const int64_t c = (int64_t)iperm[i] * D + (e - i * D);
        if (TO_COLOUR) dst[c] = src[t];
        else dst[t] = src[c];
    }
}

template <bool TO_COLOUR>
__global__ __launch_bounds__(256) void k_reorder(ReorderArgs a, const double* __restrict__ src,
                                                 double* __restrict__ dst) {
    int64_t blk = blockIdx.x;
    int f = 0;
    while (f + 1 < a.nb && blk >= a.blocks[f]) blk -= a.blocks[f++];
    const int64_t first = blk * REORDER_PER_BLOCK, len = (int64_t)a.n[f] * a.d[f];
    const double* s = src + a.off[f];
    double* t = dst + a.off[f];
    switch (a.d[f]) {
        case 1: reorder_elements<1, TO_COLOUR>(first, len, a.iperm[f], s, t); break;
        case 2: reorder_elements<2, TO_COLOUR>(first, len, a.iperm[f], s, t); break;
        case 3: reorder_elements<3, TO_COLOUR>(first, len, a.iperm[f], s, t); break;
        default: reorder_elements<4, TO_COLOUR>(first, len, a.iperm[f], s, t); break;
    }
}

__global__ void k_c64to32(int64_t n, const double* __restrict__ a, float* __restrict__ b) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
        b[e] = (float)a[e];
}

__global__ void k_c32to64(int64_t n, const float* __restrict__ a, double* __restrict__ b) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
        b[e] = (double)a[e];
}

// seeded start vector in [-1, 1): SplitMix64 output finaliser of (i + seed * golden ratio)
__global__ void k_seeded(int64_t n, uint64_t seed, double* v) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        uint64_t z = (uint64_t)e + 0x9E3779B97F4A7C15ull * (seed + 1);
        z ^= z >> 30;
        z *= 0xBF58476D1CE4E5B9ull;
        z ^= z >> 27;
        z *= 0x94D049BB133111EBull;
        z ^= z >> 31;
        v[e] = 2.0 * ((double)(z >> 11) * 0x1.0p-53) - 1.0;
    }
}

// one element per thread up to 262,144 unknowns: a small system's pass is a chain of
// latencies, and fewer, longer blocks only lengthen it (24,576 unknowns, 27 vectors, with
// the final sums: 24 blocks and a launch for the sums 26 us, 96 blocks 8 us)
int krylov_blocks(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>(KBLOCKS, ceil_div(n, KT))); }

static unsigned stream_grid(int64_t n) {
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(4096, ceil_div(n, 256)));
}

// one instance per basis size 0..32
template <template <int> class L, int... Q>
static void by_count(int nq, std::integer_sequence<int, Q...>, const typename L<0>::Args& a) {
    ((nq == Q ? (L<Q>::run(a), 0) : 0), ...);
}

struct OrthArgs {
    int64_t n;
    const double* V;
    int64_t ldv;
    const double* w;
    const KrylovBufs& kb;
    hipStream_t s;
};
template <int Q>
struct OrthLaunch {
    using Args = OrthArgs;
    static void run(const OrthArgs& a) {
        if constexpr (Q > 0) k_orth<Q, false><<<krylov_blocks(a.n), KT, 0, a.s>>>(a.n, a.V, a.ldv, a.w, a.kb);
    }
};

struct DcgsArgs {
    int64_t n;
    const double* V;
    int64_t ldv;
    double* u;
    const double* w;
    double* out;
    float* out32;
    const KrylovBufs& kb;
    hipStream_t s;
};
template <int Q>
struct DcgsLaunch {
    using Args = DcgsArgs;
    static void run(const DcgsArgs& a) {
        k_dcgs_update<Q><<<krylov_blocks(a.n), KT, 0, a.s>>>(a.n, a.V, a.ldv, a.u, a.w, a.out, a.out32, a.kb);
    }
};

void launch_norm2(int64_t n, const double* w, const KrylovBufs& kb, hipStream_t s) {
    k_orth<1, true><<<krylov_blocks(n), KT, 0, s>>>(n, nullptr, 0, w, kb);
    MB_LAUNCH_CHECK();
}

void launch_orth(int64_t n, int nq, const double* V, int64_t ldv, const double* w, const KrylovBufs& kb,
                 hipStream_t s) {
    MB_CHECK(nq >= 1 && nq <= KMAXQ - 1 && nq <= 32, MBAMG_E_INVALID, "too many Krylov vectors");
    by_count<OrthLaunch>(nq, std::make_integer_sequence<int, 33>{}, OrthArgs{n, V, ldv, w, kb, s});
    MB_LAUNCH_CHECK();
}

void launch_dcgs_update(int64_t n, int nq, const double* V, int64_t ldv, double* u, const double* w, double* out,
                        float* out32, const KrylovBufs& kb, hipStream_t s) {
    MB_CHECK(nq >= 0 && nq <= KMAXQ - 2 && nq <= 31, MBAMG_E_INVALID, "too many Krylov vectors");
    by_count<DcgsLaunch>(nq, std::make_integer_sequence<int, 32>{}, DcgsArgs{n, V, ldv, u, w, out, out32, kb, s});
    MB_LAUNCH_CHECK();
}

void launch_combine(int64_t n, int k, const double* Z, int64_t ldz, const double* y, double* x, hipStream_t s) {
    if (k <= 0) return;
    k_combine<double><<<stream_grid(n), 256, 0, s>>>(n, k, Z, ldz, y, x);
    MB_LAUNCH_CHECK();
}

void launch_combine32(int64_t n, int k, const float* Z, int64_t ldz, const double* y, double* x, hipStream_t s) {
    if (k <= 0) return;
    k_combine<float><<<stream_grid(n), 256, 0, s>>>(n, k, Z, ldz, y, x);
    MB_LAUNCH_CHECK();
}

void launch_seeded(int64_t n, uint64_t seed, double* v, hipStream_t s) {
    k_seeded<<<stream_grid(n), 256, 0, s>>>(n, seed, v);
    MB_LAUNCH_CHECK();
}

void launch_axpby(int64_t n, double a, const double* x, double b, double* y, hipStream_t s) {
    k_axpby<<<stream_grid(n), 256, 0, s>>>(n, a, x, b, y);
    MB_LAUNCH_CHECK();
}

void launch_reorder(bool to_colour, ReorderArgs a, const double* src, double* dst, hipStream_t s) {
    int64_t total = 0;
    MB_CHECK(a.nb >= 1 && a.nb <= SWEEP_MAX_BLOCKS && src && dst, MBAMG_E_INVALID, "reorder: invalid argument");
    for (int f = 0; f < a.nb; ++f) {
        const int64_t len = (int64_t)a.n[f] * a.d[f];
        MB_CHECK(a.iperm[f] && a.d[f] >= 1 && a.d[f] <= 4 && a.n[f] >= 0 && len <= (int64_t)UINT32_MAX,
                 MBAMG_E_INVALID, "reorder: invalid argument");
        a.blocks[f] = (int)ceil_div(len, REORDER_PER_BLOCK);
        total += a.blocks[f];
    }
    if (total == 0) return;
    if (to_colour) k_reorder<true><<<(unsigned)total, 256, 0, s>>>(a, src, dst);
    else k_reorder<false><<<(unsigned)total, 256, 0, s>>>(a, src, dst);
    MB_LAUNCH_CHECK();
}

void launch_cast64to32(int64_t n, const double* a, float* b, hipStream_t s) {
    if (n == 0) return;
    k_c64to32<<<stream_grid(n), 256, 0, s>>>(n, a, b);
    MB_LAUNCH_CHECK();
}

void launch_cast32to64(int64_t n, const float* a, double* b, hipStream_t s) {
    if (n == 0) return;
    k_c32to64<<<stream_grid(n), 256, 0, s>>>(n, a, b);
    MB_LAUNCH_CHECK();
}

}  // namespace mbamg
