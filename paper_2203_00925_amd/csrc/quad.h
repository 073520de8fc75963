// Four values per cell, laid out so that a wavefront reads them with 16-byte
// loads of whole lines: FP32 as one float4 per cell, FP64 as two planes of
// double2 ((0, 1), then (2, 3)).  One array per value ([4][n]) takes twice as
// many loads, each with its own address work, and a gathered cell's values
// then lie in four lines instead of two.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace mifvm {

__device__ inline void load_quad(const double* __restrict__ p, int64_t n, int64_t i, double (&v)[4]) {
    const double2 a = reinterpret_cast<const double2*>(p)[i], b = reinterpret_cast<const double2*>(p)[n + i];
    v[0] = a.x;
    v[1] = a.y;
    v[2] = b.x;
    v[3] = b.y;
}
__device__ inline void load_quad(const float* __restrict__ p, int64_t, int64_t i, float (&v)[4]) {
    const float4 a = reinterpret_cast<const float4*>(p)[i];
    v[0] = a.x;
    v[1] = a.y;
    v[2] = a.z;
    v[3] = a.w;
}
__device__ inline void load_quad(const int32_t* __restrict__ p, int64_t, int64_t i, int (&v)[4]) {
    const int4 a = reinterpret_cast<const int4*>(p)[i];
    v[0] = a.x;
    v[1] = a.y;
    v[2] = a.z;
    v[3] = a.w;
}
__device__ inline void store_quad(double* p, int64_t n, int64_t i, const double (&v)[4]) {
    reinterpret_cast<double2*>(p)[i] = make_double2(v[0], v[1]);
    reinterpret_cast<double2*>(p)[n + i] = make_double2(v[2], v[3]);
}
__device__ inline void store_quad(float* p, int64_t, int64_t i, const float (&v)[4]) {
    reinterpret_cast<float4*>(p)[i] = make_float4(v[0], v[1], v[2], v[3]);
}
__device__ inline void store_quad(int32_t* p, int64_t, int64_t i, const int (&v)[4]) {
    reinterpret_cast<int4*>(p)[i] = make_int4(v[0], v[1], v[2], v[3]);
}
// value k of cell i
__device__ inline double quad_value(const double* __restrict__ p, int64_t n, int64_t i, int k) {
    return p[(k >> 1) * 2 * n + 2 * i + (k & 1)];
}
__device__ inline float quad_value(const float* __restrict__ p, int64_t, int64_t i, int k) { return p[4 * i + k]; }

}  // namespace mifvm
