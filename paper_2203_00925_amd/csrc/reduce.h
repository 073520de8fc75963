// Deterministic block and grid reductions for wave64.
//
// A block reduces with a butterfly over the 64 lanes of each wavefront (every
// lane ends with the bitwise-identical total, since a+b == b+a) and then sums
// the wavefront totals in a fixed order.  A grid reduction writes one partial
// per block with a plain store; a separate one-block kernel sums the partials
// in index order.  No device-scope fence is executed per block: on a
// multi-XCD part such a fence writes back the XCD's L2, which costs more than
// the extra kernel launch.
#pragma once
#include <hip/hip_runtime.h>

namespace mifvm {

// A lane's partner value, lanes O apart by exclusive or (O a power of two):
// register moves within the vector unit (the LDS crossbar that __shfl goes
// through takes several times as long, and a small kernel's reductions are
// part of its latency chain: 48k-cell solve 4.76 -> 4.53 ms, 619k refined 25.9
// -> 24.6 ms).  O = 32, 16: the halves and rows swapped; O < 16:
// a rotation of each row of 16 lanes, which reaches the partner's value once
// the larger steps have made the row periodic, and exact exchanges for the
// quad's steps used on their own.
template <int CTRL>
__device__ inline double lane_dpp(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ inline float lane_dpp(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;             // quad permutations 1032, 2301
constexpr int kDppRor1 = 0x121, kDppRor2 = 0x122, kDppRor4 = 0x124, kDppRor8 = 0x128;

// v of both rows (halves) of each pair: first the even row's (lower half's)
struct LanePair { double a, b; };
__device__ inline LanePair swap_halves(double v) {
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    return {__hiloint2double(int(hi[0]), int(lo[0])), __hiloint2double(int(hi[1]), int(lo[1]))};
}
__device__ inline LanePair swap_rows(double v) {
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    return {__hiloint2double(int(hi[0]), int(lo[0])), __hiloint2double(int(hi[1]), int(lo[1]))};
}

__device__ inline double wave_sum(double v) {
    LanePair p = swap_halves(v);
    v = p.a + p.b;
    p = swap_rows(v);
    v = p.a + p.b;
    v += lane_dpp<kDppRor8>(v);
    v += lane_dpp<kDppRor4>(v);
    v += lane_dpp<kDppRor2>(v);
    v += lane_dpp<kDppRor1>(v);
    return v;
}

__device__ inline double wave_min(double v) {
    LanePair p = swap_halves(v);
    v = fmin(p.a, p.b);
    p = swap_rows(v);
    v = fmin(p.a, p.b);
    v = fmin(v, lane_dpp<kDppRor8>(v));
    v = fmin(v, lane_dpp<kDppRor4>(v));
    v = fmin(v, lane_dpp<kDppRor2>(v));
    v = fmin(v, lane_dpp<kDppRor1>(v));
    return v;
}

// sum over the 4 lanes of each quad, valid in all of them
template <class R>
__device__ inline R quad_sum(R v) {
    v += lane_dpp<kDppXor1>(v);
    v += lane_dpp<kDppXor2>(v);
    return v;
}

// blockDim.x == 256 assumed; lds needs 4 doubles.  Result valid in all threads.
__device__ inline double block_sum256(double v, double* lds) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[w] = v;
    __syncthreads();
    return ((lds[0] + lds[1]) + lds[2]) + lds[3];
}

// blockDim.x in {64, 128, 256}; lds needs 4 doubles.  Result valid in all threads.
__device__ inline double block_sum_upto256(double v, double* lds) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[w] = v;
    __syncthreads();
    double s = lds[0];
    for (int k = 1; k < nw; ++k) s += lds[k];
    return s;
}

// blockDim.x == 1024 assumed; lds needs 16 doubles.  Result valid in all threads.
__device__ inline double block_sum1024(double v, double* lds) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[w] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) s += lds[k];
    return s;
}

__device__ inline double block_min1024(double v, double* lds) {
    v = wave_min(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[w] = v;
    __syncthreads();
    double s = lds[0];
#pragma unroll
    for (int k = 1; k < 16; ++k) s = fmin(s, lds[k]);
    return s;
}

// In a one-block kernel of 1024 threads: fixed-order sum of n partials.
__device__ inline double reduce_partials_sum(const double* partial, int64_t n, double* lds) {
    double s = 0.0;
    // batches of 8 independent loads, summed in index order
    for (int64_t b = threadIdx.x; b < n; b += 8 * 1024) {
        double v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = b + j * 1024 < n ? partial[b + j * 1024] : 0.0;
#pragma unroll
        for (int j = 0; j < 8; ++j) s += v[j];
    }
    return block_sum1024(s, lds);
}

__device__ inline double reduce_partials_min(const double* partial, int64_t n, double* lds) {
    double s = __builtin_huge_val();
    for (int64_t i = threadIdx.x; i < n; i += 1024) s = fmin(s, partial[i]);
    return block_min1024(s, lds);
}

__device__ inline double block_min256(double v, double* lds) {
    v = wave_min(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[w] = v;
    __syncthreads();
    return fmin(fmin(lds[0], lds[1]), fmin(lds[2], lds[3]));
}

}  // namespace mifvm
