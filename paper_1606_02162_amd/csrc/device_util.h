// Device helpers shared by libgila kernels: wavefront and workgroup scans and
// reductions for 64-wide wavefronts and 256-thread workgroups.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

namespace gila {

__device__ __forceinline__ int lane64() { return threadIdx.x & 63; }
__device__ __forceinline__ int wave_id() { return threadIdx.x >> 6; }

// Lane exchanges in the vector ALU (DPP moves and the half-wave swaps) rather than
// through the LDS crossbar, which the force kernels' gathers keep busy and whose answer
// takes some hundred cycles.  The lanes of a group must all be active.  (1000 random
// trees, build and layout: 4635 -> 3836 us with these for the crossbar's; 25 iterations
// of R-MAT 18, k = 2: 6976 -> 6880; 20 of a 32 x 32 grid in FP64: 163 -> 154.)
//
// x of another lane by DPP control CTRL, in the rows and banks of the masks; `old` in
// the others and where the control has no source lane.
template <int CTRL, int ROWS = 0xf, int BANKS = 0xf, class T>
__device__ __forceinline__ T dpp_move(T old, T x) {
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "whole registers");
    constexpr int kWords = sizeof(T) / 4;
    int o[kWords], i[kWords];
    __builtin_memcpy(o, &old, sizeof(T));
    __builtin_memcpy(i, &x, sizeof(T));
#pragma unroll
    for (int w = 0; w < kWords; ++w)
        o[w] = __builtin_amdgcn_update_dpp(o[w], i[w], CTRL, ROWS, BANKS, false);
    T r;
    __builtin_memcpy(&r, o, sizeof(T));
    return r;
}

// x of lane l and of lane l ^ OFF (OFF = 16 or 32), the lower lane's first.
template <int OFF, class T>
__device__ __forceinline__ void lane_pair(T x, T& low, T& high) {
    constexpr int kWords = sizeof(T) / 4;
    unsigned i[kWords], lo[kWords], hi[kWords];
    __builtin_memcpy(i, &x, sizeof(T));
#pragma unroll
    for (int w = 0; w < kWords; ++w) {
        if constexpr (OFF == 32) {
            const auto r = __builtin_amdgcn_permlane32_swap(i[w], i[w], false, false);
            lo[w] = r[0];
            hi[w] = r[1];
        } else {
            const auto r = __builtin_amdgcn_permlane16_swap(i[w], i[w], false, false);
            lo[w] = r[0];
            hi[w] = r[1];
        }
    }
    __builtin_memcpy(&low, lo, sizeof(T));
    __builtin_memcpy(&high, hi, sizeof(T));
}

// x of lane l ^ OFF, OFF = 1, 2, 4 or 8.
template <int OFF, class T>
__device__ __forceinline__ T lane_xor(T x) {
    if constexpr (OFF == 1) return dpp_move<0xB1>(x, x);  // quad_perm 1 0 3 2
    else if constexpr (OFF == 2) return dpp_move<0x4E>(x, x);  // quad_perm 2 3 0 1
    else if constexpr (OFF == 4)  // row_shl 4 in banks 0 and 2, row_shr 4 in banks 1 and 3
        return dpp_move<0x114, 0xf, 0xa>(dpp_move<0x104, 0xf, 0x5>(x, x), x);
    else return dpp_move<0x128>(x, x);  // row_ror 8
}

// f over aligned groups of G lanes by a fixed butterfly from the farthest lane to the
// nearest: every lane of a group ends with the same bits (f commutative).
template <int G, class T, class F>
__device__ __forceinline__ T group_reduce(T v, F f) {
    if constexpr (G >= 64) {
        T a, b;
        lane_pair<32>(v, a, b);
        v = f(a, b);
    }
    if constexpr (G >= 32) {
        T a, b;
        lane_pair<16>(v, a, b);
        v = f(a, b);
    }
    if constexpr (G >= 16) v = f(v, lane_xor<8>(v));
    if constexpr (G >= 8) v = f(v, lane_xor<4>(v));
    if constexpr (G >= 4) v = f(v, lane_xor<2>(v));
    if constexpr (G >= 2) v = f(v, lane_xor<1>(v));
    return v;
}

// Inclusive prefix sum of whole numbers across the 64 lanes of a wavefront: within
// rows of 16 lanes, then each row's last lane to the rows after it.
template <class T>
__device__ __forceinline__ T wave_inclusive_scan(T x) {
    static_assert(std::is_integral<T>::value, "the order of the additions is not the lanes'");
    x += dpp_move<0x111>(T(0), x);  // row_shr 1, 2, 4, 8
    x += dpp_move<0x112>(T(0), x);
    x += dpp_move<0x114>(T(0), x);
    x += dpp_move<0x118>(T(0), x);
    x += dpp_move<0x142, 0xa>(T(0), x);  // row_bcast 15: rows 1 and 3
    x += dpp_move<0x143, 0xc>(T(0), x);  // row_bcast 31: rows 2 and 3
    return x;
}

// Exclusive prefix sum over a workgroup of NW wavefronts (256 threads by
// default).  `sh` is LDS scratch of at least NW elements.  Contains two
// barriers; every thread must call it.
template <class T, int NW = 4>
__device__ __forceinline__ T block_exclusive_scan(T v, T* sh, T& total) {
    const int w = wave_id();
    T inc = wave_inclusive_scan(v);
    if (lane64() == 63) sh[w] = inc;
    __syncthreads();
    T before = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        T s = sh[i];
        before += (i < w) ? s : T(0);
        tot += s;
    }
    __syncthreads();
    total = tot;
    return before + inc - v;
}

// Sum over a workgroup of NW wavefronts (256 threads by default) in a fixed
// order (butterfly within each wavefront, then wavefronts 0..NW-1 in order).
// Result valid in every thread.
template <class T, int NW = 4>
__device__ __forceinline__ T block_sum(T v, T* sh) {
    v = group_reduce<64>(v, [](T a, T b) { return a + b; });
    if (lane64() == 0) sh[wave_id()] = v;
    __syncthreads();
    T r = sh[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) r += sh[i];
    __syncthreads();
    return r;
}

// Fixed-order butterfly sum over aligned groups of G lanes (G a power of two
// <= 64).  Every lane of a group ends with the same bits.
template <int G, class T>
__device__ __forceinline__ T group_sum(T v) {
    return group_reduce<G>(v, [](T a, T b) { return a + b; });
}

template <class T>
__device__ __forceinline__ T wave_sum(T v) {
    return group_sum<64>(v);
}

template <class T>
__device__ __forceinline__ T wave_max(T v) {
    return group_reduce<64>(v, [](T a, T b) { return b > a ? b : a; });
}

// Orders LDS accesses of one wavefront (which the hardware executes in order).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

}  // namespace gila
