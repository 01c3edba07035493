// Device-side helpers shared by the tiled kernels: address-space views,
// uniform job lookup and a wave-wide float64 sum.
//
// Plan descriptors (jobs, passes, phases, ops, op matrices) are the same for
// every lane of a wave.  Reading them through generic pointers makes the
// compiler treat the loaded values as per-lane (a generic pointer may point
// into per-lane scratch), so every branch on an op field becomes an
// exec-masked branch and every gate's register block is copied at the join.
// Reading them through constant-address-space pointers yields scalar loads,
// uniform values in scalar registers and scalar branches.
#pragma once

#include "kernels.h"

namespace tcng {

// (the host pass of a HIP compile only sees the kernels' signatures; plain
// pointers keep it from checking device-only address-space conversions)
#if defined(__HIP_DEVICE_COMPILE__)
template <typename T>
using cptr = const __attribute__((address_space(4))) T*;
template <typename T>
using gptr = __attribute__((address_space(1))) T*;
#else
template <typename T>
using cptr = const T*;
template <typename T>
using gptr = T*;
#endif

template <typename T>
__device__ __forceinline__ cptr<T> as_const(const T* p) {
    return (cptr<T>)(p);
}
template <typename T>
__device__ __forceinline__ gptr<T> as_global(T* p) {
    return (gptr<T>)(p);
}
template <typename T>
__device__ __forceinline__ gptr<const T> as_global(const T* p) {
    return (gptr<const T>)(p);
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// block -> (job, block index inside the job); a single job travels by value
__device__ __forceinline__ Job load_job(const JobList& jl, const Job& single, int64_t blk, int64_t& local) {
    if (!jl.jobs) {
        local = blk;
        return single;
    }
    cptr<int64_t> prefix = as_const(jl.prefix);
    int lo = 0, hi = jl.njobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (prefix[mid] <= blk) lo = mid;
        else hi = mid - 1;
    }
    local = blk - prefix[lo];
    return as_const(jl.jobs)[lo];
}

// v + (v of the DPP source lane); lanes of rows outside ROWMASK add zero
template <int CTRL, int ROWMASK>
__device__ __forceinline__ double dpp_add(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, int(b), CTRL, ROWMASK, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, int(b >> 32), CTRL, ROWMASK, 0xF, false);
    return v + __longlong_as_double((long long)(unsigned)lo | ((long long)hi << 32));
}

// sum over the 64 lanes of a wave, returned uniformly (fixed order, so the
// result does not depend on scheduling): pairs and quads by quad
// permutations, 8 and 16 lanes by half-row and row mirrors, then rows 0+1 and
// 2+3 by the row-15 broadcast and all four rows by the lane-31 broadcast,
// which leaves the total in lane 63.
__device__ __forceinline__ double wave_sum(double v) {
    v = dpp_add<0xB1, 0xF>(v);    // quad_perm [1, 0, 3, 2]
    v = dpp_add<0x4E, 0xF>(v);    // quad_perm [2, 3, 0, 1]
    v = dpp_add<0x141, 0xF>(v);   // row_half_mirror
    v = dpp_add<0x140, 0xF>(v);   // row_mirror
    v = dpp_add<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane(int(b), 63);
    const int hi = __builtin_amdgcn_readlane(int(b >> 32), 63);
    return __longlong_as_double((long long)(unsigned)lo | ((long long)hi << 32));
}

// the same for float: v + (v of the DPP source lane)
template <int CTRL, int ROWMASK>
__device__ __forceinline__ float dpp_add(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWMASK, 0xF, false));
}

// float sum over the 64 lanes of a wave in the same fixed order, returned uniformly
__device__ __forceinline__ float wave_sum(float v) {
    v = dpp_add<0xB1, 0xF>(v);
    v = dpp_add<0x4E, 0xF>(v);
    v = dpp_add<0x141, 0xF>(v);
    v = dpp_add<0x140, 0xF>(v);
    v = dpp_add<0x142, 0xA>(v);
    v = dpp_add<0x143, 0xC>(v);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// ---------------------------------------------------------------------------
// wave sums of N values at once (N a power of two up to 16): lane l of the
// result holds the sum of v[l % N] over the 64 lanes.  The additions pair lanes
// in the order of wave_sum (1, 2, 4, 8, 16, 32 apart), so every sum is the same
// to the last bit; while lanes still hold several values each level halves
// them (a lane keeps one of a pair and sends the other), so N = 8 sums take
// about 30 instructions instead of 8 butterflies (rotation rounds, 28 qubits and 12
// layers: 73.6 -> 70.9 ms).
// ---------------------------------------------------------------------------
template <int CTRL, int BANKS>
__device__ __forceinline__ int dpp_get(int old, int v) {
    return __builtin_amdgcn_update_dpp(old, v, CTRL, 0xF, BANKS, false);
}
// the value of lane l ^ D (D = 1, 2, 4 or 8)
template <int D>
__device__ __forceinline__ int xor_lane(int v) {
    if constexpr (D == 1) return dpp_get<0xB1, 0xF>(0, v);        // quad_perm [1, 0, 3, 2]
    else if constexpr (D == 2) return dpp_get<0x4E, 0xF>(0, v);   // quad_perm [2, 3, 0, 1]
    else if constexpr (D == 4) return dpp_get<0x114, 0xA>(dpp_get<0x104, 0x5>(0, v), v);   // row_shl:4 | row_shr:4
    else return dpp_get<0x128, 0xF>(0, v);                        // row_ror:8
}
template <int D>
__device__ __forceinline__ float xor_lane(float v) { return __int_as_float(xor_lane<D>(__float_as_int(v))); }
template <int D>
__device__ __forceinline__ double xor_lane(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = xor_lane<D>(int(b)), hi = xor_lane<D>(int(b >> 32));
    return __longlong_as_double((long long)(unsigned)lo | ((long long)hi << 32));
}
// v of this lane + v of lane l ^ 16 (l ^ 32)
template <bool ROWS32>
__device__ __forceinline__ float add_rows(float v) {
    const unsigned u = __float_as_uint(v);
    const auto r = ROWS32 ? __builtin_amdgcn_permlane32_swap(u, u, false, false)
                          : __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
template <bool ROWS32>
__device__ __forceinline__ double add_rows(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = unsigned(b), hi = unsigned(b >> 32);
    const auto rl = ROWS32 ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                           : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto rh = ROWS32 ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                           : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __longlong_as_double((long long)(((unsigned long long)rh[0] << 32) | rl[0])) +
           __longlong_as_double((long long)(((unsigned long long)rh[1] << 32) | rl[1]));
}

template <int D, int N, typename R>
__device__ __forceinline__ R multi_level(const R* v, int lane) {
    if constexpr (N == 1) {   // one value a lane: plain additions
        if constexpr (D == 16) return add_rows<true>(add_rows<false>(v[0]));
        else {
            const R s = v[0] + xor_lane<D>(v[0]);
            return multi_level<2 * D, 1>(&s, lane);
        }
    } else {
        R w[N / 2];
        const bool odd = (lane & D) != 0;
#pragma unroll
        for (int i = 0; i < N / 2; ++i) {
            const R keep = odd ? v[2 * i + 1] : v[2 * i], send = odd ? v[2 * i] : v[2 * i + 1];
            w[i] = keep + xor_lane<D>(send);
        }
        return multi_level<2 * D, N / 2>(w, lane);
    }
}
template <int N, typename R>
__device__ __forceinline__ R multi_wave_sum(const R* v, int lane) {
    static_assert(N == 8 || N == 16, "8 or 16 values");
    return multi_level<1, N>(v, lane);
}

// base offset of a tile: its index's bits in the qubits outside it (four runs
// without a branch, as brick walls and ladders have at most; the rest in a loop).
// A walk over the qubits before it: 70.9 -> 67.8 ms at 28 qubits and 12 layers.
__device__ __forceinline__ uint64_t runs_base(uint64_t tile, cptr<TileRuns> R) {
    uint64_t base = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) base |= uint64_t(uint32_t(tile) & R->mask[k]) << R->shift[k];
    for (int k = 4; k < R->n; ++k) base |= uint64_t(uint32_t(tile) & R->mask[k]) << R->shift[k];
    return base;
}

}  // namespace tcng
