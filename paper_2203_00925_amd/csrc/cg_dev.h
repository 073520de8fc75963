// Device parts of the CG iterations' kernels (cg_iter.hip, amg_kernels.hip):
// which rows a block takes, the sums of partials every block forms itself,
// and a vertex value summed by four lanes.
#pragma once
#include "cg_iter.h"
#include "reduce.h"
#include "seg.h"
#include "state.h"
#include "xcd.h"

namespace mifvm {

constexpr int kMaxWaves = 8;              // 512 threads

template <class R> struct CgVec;
template <> struct CgVec<double> {
    __device__ static double *x(const Dev& d) { return d.x; }
    __device__ static double *r(const Dev& d) { return d.r; }
    __device__ static double *p(const Dev& d) { return d.p; }
    __device__ static double *q(const Dev& d) { return d.q; }
    __device__ static const double *dinv(const Dev& d) { return d.k_dinv; }
    __device__ static const double *diag(const Dev& d) { return d.k_diag; }
    __device__ static const double *val(const Dev& d) { return d.k_val; }
    __device__ static const double *alpha(const Dev& d) { return d.n_alpha; }
};
template <> struct CgVec<float> {
    __device__ static float *x(const Dev& d) { return d.d32; }
    __device__ static float *r(const Dev& d) { return d.r32; }
    __device__ static float *p(const Dev& d) { return d.p32; }
    __device__ static float *q(const Dev& d) { return d.q32; }
    __device__ static const float *dinv(const Dev& d) { return d.k_dinv32; }
    __device__ static const float *diag(const Dev& d) { return d.k_diag32; }
    __device__ static const float *val(const Dev& d) { return d.k_val32; }
    __device__ static const float *alpha(const Dev& d) { return d.n_alpha32; }
};

// a block's rows, its mesh's scalars and the partials it adds (the mesh's)
struct Seg {
    int64_t r0, r1;
    double* sc;
    int p0, np, pp0, pnp;                 // first and count: the vector kernels', the product's
    bool lead;                            // the mesh's first block
};

__device__ inline Seg cg_seg(const Dev& d, int64_t lb) {
    if (d.nm == 1) {
        const int64_t r0 = lb * d.cg_rows, r1 = r0 + d.cg_rows;
        return {r0, r1 < d.nc ? r1 : d.nc, d.scal, 0, d.cg_nblk, 0, d.cg_pblk, lb == 0};
    }
    const int4 t = d.cg_blk[lb], pr = d.cg_parts[t.x];
    return {t.y, t.z, msc(d, t.x), pr.x, pr.y, pr.z, pr.w, lb == pr.x};
}

// Sum of K values over the block, in a fixed order; valid in every thread.
// `lds`: K * kMaxWaves doubles, not in use by an earlier call.
template <int K>
__device__ inline void block_sums(double (&v)[K], double* lds) {
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = wave_sum(v[k]);
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) lds[k * kMaxWaves + w] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        v[k] = lds[k * kMaxWaves];
        for (int j = 1; j < nw; ++j) v[k] += lds[k * kMaxWaves + j];
    }
}

// The K sums of a mesh's partials (part[k * stride + b]), added by every
// block of a kernel; a thread's four loads of a round go out together.
template <int K>
__device__ inline void sum_parts(const double* __restrict__ part, int64_t stride, int np, double* lds,
                                 double (&out)[K]) {
    const int T = blockDim.x;
#pragma unroll
    for (int k = 0; k < K; ++k) out[k] = 0.0;
    for (int b0 = threadIdx.x; b0 < np; b0 += 4 * T) {
        double v[K][4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int b = b0 + j * T;
            const bool in = b < np;
#pragma unroll
            for (int k = 0; k < K; ++k) v[k][j] = in ? part[k * stride + b] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < K; ++k) out[k] += (v[k][0] + v[k][1]) + (v[k][2] + v[k][3]);
    }
    block_sums<K>(out, lds);
}

// The vertex value A z of one vertex, summed by kCgVertexLanes neighbouring
// lanes: lane q takes the entries q, q + 4, ..., up to 6 at a time (an
// interior vertex of the 6-tetrahedra cube has 24 cells, one round).  With
// one lane per vertex (24 loads, then 24 gathers a lane) a small mesh has
// too few wavefronts to cover the chain: 5.9 us at 9,261 vertices.
template <class R>
__device__ inline R vertex_sum(const Dev& d, const R* __restrict__ z, int64_t v, int q) {
    constexpr int L = kCgVertexLanes, B = 6;
    const R* __restrict__ alpha = CgVec<R>::alpha(d);
    const int64_t sl = v >> 6;
    const int64_t base = d.n_off[sl] + (v & 63);
    const int w = d.n_w[sl];
    R s = R(0);
    for (int k0 = q; k0 < w; k0 += B * L) {
        int e[B];
        R al[B];
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const int k = k0 + j * L;
            const bool in = k < w;
            const int64_t at = base + int64_t(in ? k : 0) * 64;
            e[j] = d.mf_nidx[at];
            al[j] = in ? alpha[at] : R(0);
        }
        R xe[B];
#pragma unroll
        for (int j = 0; j < B; ++j) xe[j] = z[e[j] >= 0 ? e[j] : ~e[j]];
#pragma unroll
        for (int j = 0; j < B; ++j) s += al[j] * (e[j] >= 0 ? xe[j] : -xe[j]);
    }
    return quad_sum(s);
}

// the vertex values of p that block b of a grid writes when a matrix-free loop opens
template <class R>
__device__ inline void open_vertices(const Dev& d, int64_t b) {
    const int64_t v = b * (blockDim.x / kCgVertexLanes) + threadIdx.x / kCgVertexLanes;
    const int q = threadIdx.x & (kCgVertexLanes - 1);
    const R s = vertex_sum<R>(d, CgVec<R>::p(d), v < d.nv ? v : d.nv - 1, q);
    if (q == 0 && v < d.nv) reinterpret_cast<R*>(d.mf_xv)[v] = s;
}
inline unsigned vertex_blocks(const Dev& d, int threads) {
    return unsigned((d.nv * kCgVertexLanes + threads - 1) / threads);
}

}  // namespace mifvm
