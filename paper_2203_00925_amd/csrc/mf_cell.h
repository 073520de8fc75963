// Row i of the matrix-free Poisson operator from the per-cell tables that
// k_mf_cell_setup (mf_kernels.hip) builds:
//     (K x)_i = -(sum_k w_k x_v[vid_k] + sum_k r_k t_k)
// over the cell's 4 vertices (vertex values x_v of the current x) and its 4
// faces: t_k = x[n_k] - x_i across an interior face (n_k the cell there), t_k =
// x_i on a boundary face (r_k = -2 kRL on a Dirichlet face, 0 on the others).
// A face's vertex weights kAC, kBC, -(kAC + kBC) add up to zero, so the cell's
// do and three are stored: sum_k w_k x_v[vid_k] = sum_{k<3} w_k (x_v[vid_k] -
// x_v[vid_3]).  The tables are read 16 bytes a load (quad.h).
// Shared by the per-launch product and the persistent batch solver.
#pragma once
#include "quad.h"
#include "state.h"

namespace mifvm {

template <class R> struct MfCell;
template <> struct MfCell<double> {
    __device__ static const double* w(const Dev& d) { return d.mfc_w; }
    __device__ static const double* r(const Dev& d) { return d.mfc_r; }
};
template <> struct MfCell<float> {
    __device__ static const float* w(const Dev& d) { return d.mfc_w32; }
    __device__ static const float* r(const Dev& d) { return d.mfc_r32; }
};

// where weight k < 3 of cell i lies: FP64 a double2 and a double per cell, FP32
// three floats of a float4
template <class R> __host__ __device__ inline int64_t mfc_weight(int64_t nc, int64_t i, int k);
template <> __host__ __device__ inline int64_t mfc_weight<double>(int64_t nc, int64_t i, int k) {
    return k < 2 ? 2 * i + k : 2 * nc + i;
}
template <> __host__ __device__ inline int64_t mfc_weight<float>(int64_t, int64_t i, int k) { return 4 * i + k; }

__device__ inline void load_weights(const double* __restrict__ p, int64_t nc, int64_t i, double (&w)[3]) {
    const double2 a = reinterpret_cast<const double2*>(p)[i];
    w[0] = a.x;
    w[1] = a.y;
    w[2] = p[2 * nc + i];
}
__device__ inline void load_weights(const float* __restrict__ p, int64_t, int64_t i, float (&w)[3]) {
    const float4 a = reinterpret_cast<const float4*>(p)[i];
    w[0] = a.x;
    w[1] = a.y;
    w[2] = a.z;
}

// (K x)_i from the tables: the row's table loads go out together, then its
// 4 vertex values and 4 neighbour values (a boundary face reads x_i)
template <class R>
__device__ inline R cell_row(const Dev& d, const R* __restrict__ x, const R* __restrict__ xv, int64_t i) {
    const int64_t nc = d.nc;
    int vid[4], nb[4];
    R w[3], r[4];
    load_quad(d.mfc_vid, nc, i, vid);
    load_quad(d.cell_nb, nc, i, nb);
    load_weights(MfCell<R>::w(d), nc, i, w);
    load_quad(MfCell<R>::r(d), nc, i, r);
    const R xi = x[i];
    R xvv[4], xn[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        xvv[k] = xv[vid[k]];
        xn[k] = x[nb[k] < nc ? nb[k] : i];
    }
    R acc = R(0);
#pragma unroll
    for (int k = 0; k < 3; ++k) acc += w[k] * (xvv[k] - xvv[3]);
#pragma unroll
    for (int k = 0; k < 4; ++k) acc += r[k] * (nb[k] < nc ? xn[k] - xi : xn[k]);
    return -acc;
}

}  // namespace mifvm
