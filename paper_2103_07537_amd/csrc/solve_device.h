// Device helpers shared by the solve-phase kernel files.
#pragma once

#include "solve_kernels.h"

namespace mbamg {

// "not yet written" where other workgroups of the running launch wait for a value:
// all bits set, a NaN that is never stored as a value.  Each value is its own signal,
// so no order between different addresses is needed.
__device__ __forceinline__ bool unwritten(double v) { return __double_as_longlong(v) == -1ll; }
__device__ __forceinline__ bool unwritten(float v) { return __float_as_uint(v) == 0xFFFFFFFFu; }
template <class T>
__device__ __forceinline__ T unwritten_value() {
    if constexpr (sizeof(T) == 8) return __longlong_as_double(-1ll);
    else return __uint_as_float(0xFFFFFFFFu);
}

// The polls of a wait must not hold up what they wait for.  Every wavefront of later
// colours that is resident polls past the L1; with four workgroups per compute unit
// doing so without a pause, the memory path was kept so busy that an awaited store
// was now and then not seen for 10^4 - 10^6 rounds (139,897 rows of 3 x 3 blocks in
// FP64: a wait ran out about once in 240 solver iterations, and the solve ended in
// NaN).  So a wavefront pauses between its polls, longer the longer it has waited
// (4 clocks per round past the first few), and at most two workgroups share a unit
// (see sweep_lds): there no wait was longer than 63 rounds in 4,500 iterations.
__device__ __forceinline__ void pause_after(int round) {
    for (int k = 0; k < round >> 4; ++k) __builtin_amdgcn_s_sleep(1);   // 64 clocks
}

constexpr int WPB = 4;          // waves per block when a slice has at most 4 waves

// P waves share each slice; a block holds max(P, WPB) waves
template <int P>
constexpr int waves_per_block() { return P > WPB ? P : WPB; }
constexpr int CHUNK = 2;        // slots whose loads are issued together

// Blocks are dispatched round-robin over the 8 XCDs; give each XCD a
// contiguous range of slices so neighbour gathers stay in its own L2.
__device__ __forceinline__ int xcd_block(int padded_blocks) {
    const int per = padded_blocks >> 3;
    const int bid = blockIdx.x;
    return (bid & 7) * per + (bid >> 3);
}

__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

// grid for nslices slices with P waves per slice (4/P slices per 256-thread block)
static inline unsigned xcd_grid(int nslices, int P) {
    int blocks = (int)ceil_div(nslices, std::max(WPB, P) / P);
    return (unsigned)(ceil_div(blocks, 8) * 8);
}

template <class T, int BS>
__device__ __forceinline__ void load_masked(const T* __restrict__ p, uint32_t m, T (&v)[BS]) {
    int g = 0;
#pragma unroll
    for (int k = 0; k < BS; ++k) {
        if (m & (1u << k)) {
            v[k] = p[(int64_t)g * WAVE];
            ++g;
        } else {
            v[k] = T(0);
        }
    }
}

template <class T, int D>
__device__ __forceinline__ void load_vec(const T* __restrict__ p, T (&v)[D]) {
#pragma unroll
    for (int c = 0; c < D; ++c) v[c] = p[c];
}

template <>
__device__ __forceinline__ void load_vec<double, 4>(const double* __restrict__ p, double (&v)[4]) {
    const double2* q = reinterpret_cast<const double2*>(p);
    double2 a = q[0], b = q[1];
    v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
}

template <>
__device__ __forceinline__ void load_vec<float, 4>(const float* __restrict__ p, float (&v)[4]) {
    float4 a = *reinterpret_cast<const float4*>(p);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
}

template <>
__device__ __forceinline__ void load_vec<double, 2>(const double* __restrict__ p, double (&v)[2]) {
    const double2 a = *reinterpret_cast<const double2*>(p);
    v[0] = a.x; v[1] = a.y;
}

// a vector stored as TX, in T
template <class T, int D, class TX>
__device__ __forceinline__ void load_vec_from(const TX* __restrict__ p, T (&v)[D]) {
    if constexpr (std::is_same_v<T, TX>) {
        load_vec<T, D>(p, v);
    } else {
        TX x[D];
        load_vec<TX, D>(p, x);
#pragma unroll
        for (int c = 0; c < D; ++c) v[c] = (T)x[c];
    }
}

template <class T, int D>
__device__ __forceinline__ void store_vec(T* __restrict__ p, const T (&v)[D]) {
#pragma unroll
    for (int c = 0; c < D; ++c) p[c] = v[c];
}

template <>
__device__ __forceinline__ void store_vec<double, 4>(double* __restrict__ p, const double (&v)[4]) {
    double2* q = reinterpret_cast<double2*>(p);
    q[0] = make_double2(v[0], v[1]);
    q[1] = make_double2(v[2], v[3]);
}

template <>
__device__ __forceinline__ void store_vec<float, 4>(float* __restrict__ p, const float (&v)[4]) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}

// The entries a stored block keeps, by its part's shape (see BlockShape): all
// D x D of them, or those that determine the block.
template <int D, int S>
constexpr int shape_entries() { return S == SHAPE_FULL ? D * D : S == SHAPE_SCALED ? 2 * D : D + 1; }

// acc -= block * x for a block of shape S given by its kept entries
template <class T, int D, int S>
__device__ __forceinline__ void block_sub(const T (&v)[shape_entries<D, S>()], const T (&x)[D], T (&acc)[D]) {
    if constexpr (S == SHAPE_FULL) {
#pragma unroll
        for (int r = 0; r < D; ++r)
#pragma unroll
            for (int c = 0; c < D; ++c) acc[r] -= v[r * D + c] * x[c];
    } else {
        constexpr int L = D - 1, ROW = S == SHAPE_SYMMETRIC ? 1 : D;   // first entry of the last row
#pragma unroll
        for (int r = 0; r < L; ++r) {
            acc[r] -= v[0] * x[r];
            acc[r] -= v[1 + r] * x[L];
            acc[L] -= v[ROW + r] * x[r];
        }
        acc[L] -= v[shape_entries<D, S>() - 1] * x[L];
    }
}

}  // namespace mbamg
