// device_util.h -- wavefront/block reductions and small dense helpers for the
// gfx950 kernels. Reductions run in a fixed tree order (64-lane shuffles,
// then one wave over the per-wave results) so every result is a function of
// the input order only: two runs, or the same scene alone and in a batch,
// produce bit-identical sums.
#pragma once
#include <hip/hip_runtime.h>

#include "ipc_internal.h"

namespace ipcg {

// Global-memory views of device pointers. The arrays of a scene's view are
// reached through generic pointers, so plain accesses compile to flat
// instructions, which also count against the LDS counter: every LDS wait and
// block barrier after them waits for them too. Through these views they are
// global loads and stores, which the latency-bound PCG update kernel keeps in
// flight across its LDS work and barriers.
template <class T>
using gptr = __attribute__((address_space(1))) T *;
template <class T>
__device__ __forceinline__ gptr<T> glob(T *p)
{
    return (gptr<T>)p;
}

// A value the optimiser cannot trace back: addresses made from it are formed
// where they are used. Hoisted out of a resident solve's iteration loop they
// would take the registers of its matrix rows.
template <class T>
__device__ __forceinline__ T here(T v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// One 32-bit step of a 64-lane butterfly: lanes exchange over distance O
// without the LDS crossbar (a __shfl of a double is two ds_bpermute of about
// 130 cycles each; these are VALU moves). For O <= 8 the row rotation reads
// lane i - O, which after the wider steps holds lane i + O's value.
template <int O>
__device__ __forceinline__ void lane_pair(uint32_t x, uint32_t &a, uint32_t &b)
{
    if constexpr (O == 32) {
        auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        a = r[0];
        b = r[1];
    } else if constexpr (O == 16) {
        auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        a = r[0];
        b = r[1];
    } else {
        a = x;
        b = (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x120 + O, 0xf, 0xf, true);
    }
}
template <int O>
__device__ __forceinline__ double lane_add(double v)
{
    const uint64_t x = (uint64_t)__double_as_longlong(v);
    uint32_t a0, b0, a1, b1;
    lane_pair<O>((uint32_t)x, a0, b0);
    lane_pair<O>((uint32_t)(x >> 32), a1, b1);
    return __longlong_as_double((long long)((uint64_t)a1 << 32 | a0)) +
           __longlong_as_double((long long)((uint64_t)b1 << 32 | b0));
}

// the value of another lane of the quad (CTRL 0xb1: lane ^ 1, 0x4e: lane ^ 2) or
// row of 16 lanes (0x141: 7 - lane of each eight, 0x140: 15 - lane)
template <int CTRL>
__device__ __forceinline__ double quad_other(double v)
{
    const uint64_t x = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)x, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(x >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// a value that every lane holds, as a wavefront-uniform (scalar) one
__device__ __forceinline__ double wave_first(double v)
{
    const uint64_t x = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// lane i's value (i the same in every lane)
__device__ __forceinline__ double lane_value(double v, int i)
{
    const uint64_t x = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, i);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), i);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// orders a wavefront's LDS writes before its other lanes' reads
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Sum over the wavefront, the same value in every lane: the tree of
// distances 32, 16, ..., 1.
__device__ __forceinline__ double wave_sum(double v)
{
    return lane_add<1>(lane_add<2>(lane_add<4>(lane_add<8>(lane_add<16>(lane_add<32>(v))))));
}
__device__ __forceinline__ double wave_max(double v)
{
    for (int o = kWave / 2; o > 0; o >>= 1) v = fmax(v, __shfl_down(v, o, kWave));
    return v;
}
__device__ __forceinline__ double wave_min(double v)
{
    for (int o = kWave / 2; o > 0; o >>= 1) v = fmin(v, __shfl_down(v, o, kWave));
    return v;
}
__device__ __forceinline__ int wave_isum(int v)
{
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_down(v, o, kWave);
    return v;
}

// Block-wide reductions; blockDim.x must be a multiple of 64 and <= 1024.
// The result is valid in thread 0 (and broadcast through shared memory to
// all threads by the *_all variants).
template <int OP>
__device__ __forceinline__ double wave_op(double v)
{
    return OP == 0 ? wave_sum(v) : (OP == 1 ? wave_max(v) : wave_min(v));
}

template <int OP>
__device__ double block_reduce_all(double v, double ident)
{
    __shared__ double sh[16];
    __shared__ double result;
    int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    int nw = (blockDim.x + kWave - 1) / kWave;
    v = wave_op<OP>(v);
    if (lane == 0) sh[w] = v;
    __syncthreads();
    if (w == 0) {
        double t = lane < nw ? sh[lane] : ident;
        t = wave_op<OP>(t);
        if (lane == 0) result = t;
    }
    __syncthreads();
    double r = result;
    __syncthreads();
    return r;
}

__device__ inline double block_sum_all(double v) { return block_reduce_all<0>(v, 0.0); }
__device__ inline double block_max_all(double v) { return block_reduce_all<1>(v, -INFINITY); }
__device__ inline double block_min_all(double v) { return block_reduce_all<2>(v, INFINITY); }

// Vector sum over the block (blockDim.x a multiple of 64, at most kBlock) in
// a fixed order; every thread gets the result.
template <int NC>
__device__ __forceinline__ void block_sum_vec(double v[NC])
{
    __shared__ double sh[kBlock / kWave][NC];
    int lane = threadIdx.x % kWave, w = threadIdx.x / kWave, nw = blockDim.x / kWave;
#pragma unroll
    for (int c = 0; c < NC; ++c) v[c] = wave_sum(v[c]);
    if (nw == 1) {
#pragma unroll
        for (int c = 0; c < NC; ++c) v[c] = __shfl(v[c], 0, kWave);
        return;
    }
    if (lane == 0)
#pragma unroll
        for (int c = 0; c < NC; ++c) sh[w][c] = v[c];
    __syncthreads();
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        double t = 0.0;
        for (int k = 0; k < nw; ++k) t += sh[k][c];
        v[c] = t;
    }
    __syncthreads();
}

// ---- compensated (double-double style) sums for energies ----------------
struct CSum {
    double s, c;
};
__device__ __forceinline__ CSum csum_add(CSum a, CSum b)
{
    // TwoSum of the leading parts; errors accumulate in c
    double s = a.s + b.s;
    double bp = s - a.s;
    double e = (a.s - (s - bp)) + (b.s - bp);
    CSum r;
    r.s = s;
    r.c = a.c + b.c + e;
    return r;
}
__device__ __forceinline__ CSum wave_csum(CSum v)
{
    for (int o = kWave / 2; o > 0; o >>= 1) {
        CSum w;
        w.s = __shfl_down(v.s, o, kWave);
        w.c = __shfl_down(v.c, o, kWave);
        v = csum_add(v, w);
    }
    return v;
}
__device__ inline CSum block_csum(CSum v)
{
    __shared__ double shs[16], shc[16];
    __shared__ CSum result;
    int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    int nw = (blockDim.x + kWave - 1) / kWave;
    v = wave_csum(v);
    if (lane == 0) {
        shs[w] = v.s;
        shc[w] = v.c;
    }
    __syncthreads();
    if (w == 0) {
        CSum t;
        t.s = lane < nw ? shs[lane] : 0.0;
        t.c = lane < nw ? shc[lane] : 0.0;
        t = wave_csum(t);
        if (lane == 0) result = t;
    }
    __syncthreads();
    CSum r = result;
    __syncthreads();
    return r;
}

// ---- 3x3 helpers (row-major) ----------------------------------------------
__device__ __forceinline__ double det3(const double *M)
{
    return M[0] * (M[4] * M[8] - M[5] * M[7]) - M[1] * (M[3] * M[8] - M[5] * M[6]) +
           M[2] * (M[3] * M[7] - M[4] * M[6]);
}
// inverse by the adjugate; returns the determinant
__device__ __forceinline__ double inverse3(const double *M, double *O)
{
    double c00 = M[4] * M[8] - M[5] * M[7];
    double c01 = M[5] * M[6] - M[3] * M[8];
    double c02 = M[3] * M[7] - M[4] * M[6];
    double d = M[0] * c00 + M[1] * c01 + M[2] * c02;
    double id = 1.0 / d;
    O[0] = c00 * id;
    O[1] = (M[2] * M[7] - M[1] * M[8]) * id;
    O[2] = (M[1] * M[5] - M[2] * M[4]) * id;
    O[3] = c01 * id;
    O[4] = (M[0] * M[8] - M[2] * M[6]) * id;
    O[5] = (M[2] * M[3] - M[0] * M[5]) * id;
    O[6] = c02 * id;
    O[7] = (M[1] * M[6] - M[0] * M[7]) * id;
    O[8] = (M[0] * M[4] - M[1] * M[3]) * id;
    return d;
}

}  // namespace ipcg
