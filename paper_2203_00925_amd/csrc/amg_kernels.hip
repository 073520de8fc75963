// Aggregation multigrid cycle (V(1,1) or W(1,1), damped Jacobi) and the
// flexible CG around it (the setup and the cycle's definition are in amg.h).
// Level 0 is the state's system: its product is the matrix-free one, its
// diagonal K's; coarser levels store their off-diagonal entries in slices of
// at most 64 rows beside the diagonal.  Every kernel takes the solve's done
// flag and returns at once when it is set (a captured chunk of iterations
// then runs to its end without work).
//
// A visit of a coarse level is a chain of small kernels (a W-cycle of five
// levels visits level l 2^(l-1) times), so their number is its time, each 1.6
// us from the launch before it plus a few us of latency.  A cycle of a level
// is two: k_amg_down (residual of the pre-smoothed iterate, restricted to the
// next level and pre-smoothed there) and k_amg_up (post-smoothing, the result
// added to the next finer iterate); between the two visits of a W-cycle one
// more, k_amg_mid (the remaining residual, pre-smoothed).  The kernels of one
// step each (smoothing, product, restriction, prolongation, subtraction,
// addition) were 15 launches for the two visits.
#include "amg_dev.h"
#include "cg_dev.h"
#include "mf_cell.h"

namespace mifvm {
namespace {

__device__ inline int64_t tid_a() { return int64_t(blockIdx.x) * blockDim.x + threadIdx.x; }
inline unsigned grid_a(int64_t n) { return unsigned((n + kBlock - 1) / kBlock); }
__device__ inline bool done(const double* flag) { return flag && *flag != 0.0; }

constexpr int kShare = 4;                 // wavefronts that share a slice of coarse rows

// x = w D^-1 b
__global__ __launch_bounds__(kBlock) void k_amg_smooth0(int64_t n, double w, const double* __restrict__ dinv,
                                                        const double* __restrict__ b, double* __restrict__ x,
                                                        const double* flag) {
    if (done(flag)) return;
    const int64_t i = tid_a();
    if (i < n) x[i] = w * dinv[i] * b[i];
}

// b_c[I] = sum of the finest level's residual over the members of aggregate I;
// x_c = w D_c^-1 b_c (xc null: the coarsest level needs no start)
__global__ __launch_bounds__(kBlock) void k_amg_restrict0(int64_t nco, const int32_t* __restrict__ mptr,
                                                          const int32_t* __restrict__ midx,
                                                          const double* __restrict__ res, double w,
                                                          const double* __restrict__ dinv, double* __restrict__ bc,
                                                          double* __restrict__ xc, const double* flag) {
    if (done(flag)) return;
    const int64_t I = tid_a();
    if (I >= nco) return;
    // members in batches of 8: their indices in flight together, then their
    // values, then the sums in member order (a slot past the aggregate
    // re-reads its first member and is not added; aggregates are non-empty)
    const int m0 = mptr[I], cnt = mptr[I + 1] - m0;
    const double di = dinv[I];
    double s = 0.0;
    for (int k0 = 0; k0 < cnt; k0 += 8) {
        int id[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) id[j] = midx[m0 + (k0 + j < cnt ? k0 + j : 0)];
        double rv[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) rv[j] = res[id[j]];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (k0 + j < cnt) s += rv[j];
    }
    bc[I] = s;
    if (xc) xc[I] = w * di * s;
}

// (A x) of a slice's rows, lane j of every wavefront its row j: wavefront q of
// the block takes the entries q, q + 4, ... of all 64 rows, twelve at a time,
// and the four sums meet in LDS.  At 2,800 rows of 20 entries one wavefront a
// slice leaves 44, each a chain of three rounds; four neighbouring lanes a row
// would share the entries as well, but load a slice's columns and values in
// quarters of its lines.  Valid in every thread; `part` is free again after
// the next barrier.
__device__ inline double row_product(const AmgLevelDev& L, const double* __restrict__ x, int slice, int64_t row,
                                     double (*part)[64]) {
    constexpr int B = 12;
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int64_t base = L.off[slice] + lane;
    const int w = L.w[slice];
    const double dg = L.diag[row], xr = x[row];
    double y = 0.0;
    for (int k0 = q; k0 < w; k0 += B * kShare) {
        int c[B];
        double a[B];
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const int k = k0 + j * kShare;
            const bool in = k < w;
            const int64_t at = base + int64_t(in ? k : k0) * 64;
            c[j] = L.idx[at];
            a[j] = in ? L.val[at] : 0.0;
        }
        double xe[B];
#pragma unroll
        for (int j = 0; j < B; ++j) xe[j] = x[c[j]];
#pragma unroll
        for (int j = 0; j < B; ++j) y += a[j] * xe[j];
    }
    part[q][lane] = y;
    __syncthreads();
    return dg * xr + ((part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]));
}

// r = b - A x, restricted: b_c[I] = sum of r over I's members, and x_c = w
// D_c^-1 b_c (xc null: the coarsest level).  A block holds whole aggregates.
__global__ __launch_bounds__(kBlock) void k_amg_down(AmgLevelDev L, const double* __restrict__ b,
                                                     const double* __restrict__ x, double w,
                                                     const double* __restrict__ dinv_c, double* __restrict__ bc,
                                                     double* __restrict__ xc, const double* flag) {
    __shared__ double part[kShare][64], rs[64];
    const int64_t blk = xcd_block();
    if (blk >= L.nblk) return;
    const int lane = threadIdx.x & 63;
    const int s0 = L.bslice[blk], s1 = L.bslice[blk + 1], a0 = L.bagg[blk], a1 = L.bagg[blk + 1];
    if (done(flag)) return;
    double big = 0.0;                                     // an aggregate over several slices
    for (int s = s0; s < s1; ++s) {
        const int r0 = L.srow[s], n = L.srow[s + 1] - r0;
        const int64_t row = r0 + (lane < n ? lane : n - 1);
        const double br = b[row];
        const double t = row_product(L, x, s, row, part);
        if (int(threadIdx.x) < n) rs[threadIdx.x] = br - t;
        __syncthreads();
        if (s1 - s0 == 1) {
            const int I = a0 + int(threadIdx.x);
            if (I < a1) {
                double v = 0.0;
                for (int m = L.mptr[I] - r0; m < L.mptr[I + 1] - r0; ++m) v += rs[m];
                bc[I] = v;
                if (xc) xc[I] = w * dinv_c[I] * v;
            }
        } else {
            if (threadIdx.x == 0)
                for (int m = 0; m < n; ++m) big += rs[m];
            __syncthreads();
        }
    }
    if (s1 - s0 > 1 && threadIdx.x == 0) {
        bc[a0] = big;
        if (xc) xc[a0] = w * dinv_c[a0] * big;
    }
}

// z = x + w D^-1 (b - A x).  KEEP: stored (the first of two visits).  Else
// z, plus the first visit's result if there is one, is added to the iterate of
// the row's members on the finer level (midx: the finest level).
template <bool KEEP>
__global__ __launch_bounds__(kBlock) void k_amg_up(AmgLevelDev L, const double* __restrict__ b,
                                                   const double* __restrict__ x, double w, double* __restrict__ keep,
                                                   const double* __restrict__ first, const int32_t* __restrict__ mptr,
                                                   const int32_t* __restrict__ midx, double* __restrict__ fine,
                                                   const double* flag) {
    __shared__ double part[kShare][64];
    const int64_t s = xcd_block();
    if (s >= L.nslices) return;
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int r0 = L.srow[s], n = L.srow[s + 1] - r0;
    if (done(flag)) return;
    const int64_t row = r0 + (lane < n ? lane : n - 1);
    const double br = b[row], di = L.dinv[row], xr = x[row], f = first ? first[row] : 0.0;
    int m0 = 0, m1 = 0;
    if (!KEEP) {
        m0 = mptr[row];
        m1 = mptr[row + 1];
    }
    double z = xr + w * di * (br - row_product(L, x, int(s), row, part));
    if (lane >= n) return;
    if (KEEP) {
        if (q == 0) keep[row] = z;
        return;
    }
    if (first) z = f + z;
    for (int m = m0 + q; m < m1; m += kShare) {
        const int i = midx ? midx[m] : m;
        fine[i] = fine[i] + z;
    }
}

// r = b - A x, e = w D^-1 r (the second visit's start)
__global__ __launch_bounds__(kBlock) void k_amg_mid(AmgLevelDev L, const double* __restrict__ b,
                                                    const double* __restrict__ x, double w, double* __restrict__ r,
                                                    double* __restrict__ e, const double* flag) {
    __shared__ double part[kShare][64];
    const int64_t s = xcd_block();
    if (s >= L.nslices) return;
    const int lane = threadIdx.x & 63;
    const int r0 = L.srow[s], n = L.srow[s + 1] - r0;
    if (done(flag)) return;
    const int64_t row = r0 + (lane < n ? lane : n - 1);
    const double br = b[row], di = L.dinv[row];
    const double v = br - row_product(L, x, int(s), row, part);
    if (int(threadIdx.x) < n) {
        r[row] = v;
        e[row] = w * di * v;
    }
}

// x = C^-1 b on the coarsest level, one block per row; stored (out), or added
// to the members of the row on the finer level
__global__ __launch_bounds__(256) void k_amg_dense(int64_t n, const double* __restrict__ cinv,
                                                   const double* __restrict__ b, double* __restrict__ out,
                                                   const int32_t* __restrict__ mptr, const int32_t* __restrict__ midx,
                                                   double* __restrict__ fine, const double* flag) {
    __shared__ double lds[4];
    if (done(flag)) return;
    const int64_t r = blockIdx.x;
    double s = 0.0;
    for (int64_t c = threadIdx.x; c < n; c += 256) s += cinv[r * n + c] * b[c];
    s = block_sum256(s, lds);
    if (out) {
        if (threadIdx.x == 0) out[r] = s;
        return;
    }
    for (int m = mptr[r] + int(threadIdx.x); m < mptr[r + 1]; m += 256) {
        const int i = midx ? midx[m] : m;
        fine[i] = fine[i] + s;
    }
}

// ---- the finest level ------------------------------------------------------------
// vertex values of x
__global__ __launch_bounds__(kBlock) void k_amg_vertices(Dev d, const double* __restrict__ x, double* __restrict__ xv,
                                                         const double* flag) {
    if (done(flag)) return;
    const int64_t v = xcd_block() * (kBlock / kCgVertexLanes) + threadIdx.x / kCgVertexLanes;
    const int q = threadIdx.x & (kCgVertexLanes - 1);
    const double s = vertex_sum<double>(d, x, v < d.nv ? v : d.nv - 1, q);
    if (q == 0 && v < d.nv) xv[v] = s;
}

// res = b - K x
__global__ __launch_bounds__(kBlock) void k_amg_residual0(Dev d, const double* __restrict__ b,
                                                          const double* __restrict__ x, const double* __restrict__ xv,
                                                          double* __restrict__ res, const double* flag) {
    if (done(flag)) return;
    const int64_t i = gtid_m();
    if (i >= d.nc) return;
    const double bi = b[i];
    res[i] = bi - cell_row(d, x, xv, i);
}

// z = x + w D^-1 (b - K x); with r_old: partial z.b and z.r_old (b is the CG's r)
__global__ __launch_bounds__(kBlock) void k_amg_smooth_dots(Dev d, const double* __restrict__ b,
                                                            const double* __restrict__ x,
                                                            const double* __restrict__ xv, double w,
                                                            double* __restrict__ z, const double* __restrict__ r_old,
                                                            const double* flag) {
    __shared__ double lds[2 * kMaxWaves];
    if (done(flag)) return;
    const int64_t lb = xcd_block();
    if (lb >= d.cg_pblk) return;
    const int64_t r0 = lb * d.cg_prows, r1 = r0 + d.cg_prows < d.nc ? r0 + d.cg_prows : d.nc;
    double v[2] = {0.0, 0.0};
    for (int64_t i = r0 + threadIdx.x; i < r1; i += kBlock) {
        const double bi = b[i], ro = r_old ? r_old[i] : 0.0, xi = x[i], di = d.k_dinv[i];
        const double zi = xi + w * di * (bi - cell_row(d, x, xv, i));
        z[i] = zi;
        v[0] += zi * bi;
        v[1] += zi * ro;
    }
    if (!r_old) return;
    block_sums<2>(v, lds);
    if (threadIdx.x == 0) {
        double* __restrict__ out = d.partial + 2 * d.cg_stride;
        out[lb] = v[0];
        out[d.cg_stride + lb] = v[1];
    }
}

// the same dots of a z formed elsewhere (a learned smoother)
__global__ __launch_bounds__(kBlock) void k_amg_dots(Dev d, const double* __restrict__ r_old, const double* flag) {
    __shared__ double lds[2 * kMaxWaves];
    if (done(flag)) return;
    const int64_t lb = xcd_block();
    if (lb >= d.cg_pblk) return;
    const int64_t r0 = lb * d.cg_prows, r1 = r0 + d.cg_prows < d.nc ? r0 + d.cg_prows : d.nc;
    double v[2] = {0.0, 0.0};
    for (int64_t i = r0 + threadIdx.x; i < r1; i += kBlock) {
        const double zi = d.z[i];
        v[0] += zi * d.r[i];
        v[1] += zi * r_old[i];
    }
    block_sums<2>(v, lds);
    if (threadIdx.x == 0) {
        double* __restrict__ out = d.partial + 2 * d.cg_stride;
        out[lb] = v[0];
        out[d.cg_stride + lb] = v[1];
    }
}

// x += y
__global__ __launch_bounds__(kBlock) void k_amg_add(int64_t n, const double* __restrict__ y, double* __restrict__ x,
                                                    const double* flag) {
    if (done(flag)) return;
    const int64_t i = tid_a();
    if (i < n) x[i] = x[i] + y[i];
}

// ---- flexible CG (one mesh) -------------------------------------------------------
// r = b - t (t = K x); partial rr, bb
__global__ __launch_bounds__(kBlock) void k_amg_open(Dev d, const double* __restrict__ t) {
    __shared__ double lds[4];
    const int64_t i = tid_a();
    const BlockSeg g = block_seg(d, int64_t(blockIdx.x) * kBlock, kBlock);
    double v[2] = {0.0, 0.0};
    if (i < d.nc) {
        const double bi = d.b[i];
        const double ri = bi - t[i];
        d.r[i] = ri;
        v[0] = ri * ri;
        v[1] = bi * bi;
    }
    seg_publish<2>(d, g, v, i >= g.split, lds);
}

// what the next product takes over (the opening, or the tests of an iteration)
__device__ inline void stage(double* sc) {
    sc[SC_N_RR] = sc[SC_RR];
    sc[SC_N_IT] = sc[SC_IT];
    sc[SC_N_SINCE] = sc[SC_SINCE];
    sc[SC_N_DONE] = sc[SC_DONE];
}

__global__ __launch_bounds__(1024) void k_amg_open_fin(Dev d, int64_t nparts, double tol, int maxit, int restart,
                                                       int fresh) {
    __shared__ double lds[16];
    double t[2];
    seg_sums<2>(d, 0, 0, nparts, kBlock, lds, t);
    const double rr = t[0], bb = t[1];
    if (threadIdx.x == 0) {
        double* sc = d.scal;
        sc[SC_RR] = rr;
        sc[SC_TRUE_RR] = rr;
        sc[SC_BB] = bb;
        if (fresh) {
            sc[SC_TOL2BB] = tol * tol * bb;
            sc[SC_MAXIT] = double(maxit);
            sc[SC_RESTART] = double(restart);
            sc[SC_IT] = 0.0;
        }
        sc[SC_SINCE] = 0.0;
        sc[SC_DONE] = (rr <= sc[SC_TOL2BB] || bb == 0.0) ? 1.0 : (sc[SC_IT] >= sc[SC_MAXIT] ? 2.0 : 0.0);
        stage(sc);
    }
}

// after the cycle of the opening: p = z, partial z.r
__global__ __launch_bounds__(kBlock) void k_amg_p0(Dev d) {
    __shared__ double lds[4];
    if (d.scal[SC_DONE] != 0.0) return;
    const int64_t i = tid_a();
    const BlockSeg g = block_seg(d, int64_t(blockIdx.x) * kBlock, kBlock);
    double v[1] = {0.0};
    if (i < d.nc) {
        const double zi = d.z[i];
        d.p[i] = zi;
        v[0] = zi * d.r[i];
    }
    seg_publish<1>(d, g, v, i >= g.split, lds);
}

__global__ __launch_bounds__(1024) void k_amg_rz_fin(Dev d, int64_t nparts) {
    __shared__ double lds[16];
    if (d.scal[SC_DONE] != 0.0) return;
    const double zr = seg_sum(d, 0, 0, nparts, kBlock, lds);
    if (threadIdx.x == 0) d.scal[SC_RZ] = d.scal[SC_N_RZ] = zr;
}

// alpha from the product's partials; x += alpha p; r_old = r; r -= alpha q;
// the cycle's pre-smoothed start s = w D^-1 r; partial rr
__global__ __launch_bounds__(512) void k_amg_step(Dev d, int np, double w, double* __restrict__ r_old,
                                                  double* __restrict__ s0) {
    __shared__ double lds[2 * kMaxWaves];
    const int64_t lb = xcd_block();
    if (lb >= d.cg_nblk) return;
    double* sc = d.scal;
    if (sc[SC_DONE] != 0.0) return;
    const Seg s = cg_seg(d, lb);
    double pq[1];
    sum_parts<1>(d.partial, 0, np, lds, pq);
    const double alpha = sc[SC_RZ] / pq[0];
    if (s.lead && threadIdx.x == 0) {
        sc[SC_PQ] = pq[0];
        sc[SC_ALPHA] = alpha;
    }
    double v[1] = {0.0};
    for (int64_t i = s.r0 + threadIdx.x; i < s.r1; i += blockDim.x) {
        const double xi = d.x[i], pi = d.p[i], ro = d.r[i], qi = d.q[i], di = d.k_dinv[i];
        const double ri = ro - alpha * qi;
        d.x[i] = xi + alpha * pi;
        r_old[i] = ro;
        d.r[i] = ri;
        s0[i] = w * di * ri;
        v[0] += ri * ri;
    }
    block_sums<1>(v, lds + kMaxWaves);
    if (threadIdx.x == 0) d.partial[d.cg_stride + lb] = v[0];
}

// count; convergence (1), limit (2) or a scheduled restart (3)
__global__ __launch_bounds__(1024) void k_amg_rr_fin(Dev d) {
    __shared__ double lds[16];
    double* sc = d.scal;
    if (sc[SC_DONE] != 0.0) return;
    const double rr = reduce_partials_sum(d.partial + d.cg_stride, d.cg_nblk, lds);
    if (threadIdx.x == 0) {
        sc[SC_RR] = rr;
        sc[SC_IT] = sc[SC_IT] + 1.0;
        sc[SC_SINCE] = sc[SC_SINCE] + 1.0;
        if (rr <= sc[SC_TOL2BB]) sc[SC_DONE] = 1.0;
        else if (sc[SC_IT] >= sc[SC_MAXIT]) sc[SC_DONE] = 2.0;
        else if (sc[SC_RESTART] > 0.0 && sc[SC_SINCE] >= sc[SC_RESTART]) sc[SC_DONE] = 3.0;
        stage(sc);
    }
}

// Flexible (Polak-Ribiere) beta = z_new . (r_new - r_old) / (z_old . r_old), by
// every block; p = z + beta p, and with VERTS the first `nvert` blocks update
// the vertex values of p by the same recurrence (as cg_iter.hip's direction).
template <bool VERTS>
__global__ __launch_bounds__(512) void k_amg_direction(Dev d, int nvert) {
    __shared__ double lds[2 * kMaxWaves];
    double* sc = d.scal;
    if (sc[SC_DONE] != 0.0) return;
    const int T = blockDim.x;
    const bool vert = VERTS && int(blockIdx.x) < nvert;
    const int blk = vert ? int(blockIdx.x) : int(blockIdx.x) - nvert;
    const int per = (vert ? nvert : int(gridDim.x) - nvert) / kXcds;
    const int64_t lb = int64_t(blk % kXcds) * per + blk / kXcds;
    if (lb >= (vert ? d.cg_vblk : d.cg_nblk)) return;
    double zv = 0.0, old = 0.0;
    const int q = threadIdx.x & (kCgVertexLanes - 1);
    const int64_t v = lb * (T / kCgVertexLanes) + threadIdx.x / kCgVertexLanes;
    if (VERTS && vert) {
        const int64_t vc = v < d.nv ? v : d.nv - 1;
        old = d.mf_xv[vc];
        zv = vertex_sum<double>(d, d.z, vc, q);
    }
    double t[2];
    sum_parts<2>(d.partial + 2 * d.cg_stride, d.cg_stride, d.cg_pblk, lds, t);
    const double beta = (t[0] - t[1]) / sc[SC_RZ];
    if (VERTS && vert) {
        if (q == 0 && v < d.nv) d.mf_xv[v] = zv + beta * old;
        return;
    }
    const Seg s = cg_seg(d, lb);
    for (int64_t i = s.r0 + threadIdx.x; i < s.r1; i += T) d.p[i] = d.z[i] + beta * d.p[i];
    if (s.lead && threadIdx.x == 0) {
        sc[SC_BETA] = beta;
        sc[SC_N_RZ] = t[0];
    }
}

// Where a level's result goes: the rows of the finer level that make up each
// of its rows.
struct Fine {
    const int32_t *mptr, *midx;
    double* x;
};

// One cycle of coarse level l (>= 1) on b from x = w D^-1 b (level l not the
// coarsest; there x is unused): the result, plus `first`, is added to f.x, or
// stored in `keep`.
hipError_t coarse_cycle(const AmgDev& a, int l, const double* b, double* x, const double* first, double* keep,
                        const Fine& f, const double* flag, hipStream_t s) {
    const double w = a.omega;
    const AmgLevelDev& L = a.lv[l];
    if (l == a.nl - 1) {               // the coarsest level: its dense inverse
        hipLaunchKernelGGL(k_amg_dense, dim3(unsigned(L.n)), dim3(256), 0, s, L.n, a.cinv, b, (double*)nullptr, f.mptr,
                           f.midx, f.x, flag);
        return hipGetLastError();
    }
    const AmgLevelDev& N = a.lv[l + 1];
    const bool last = l + 1 == a.nl - 1;
    hipLaunchKernelGGL(k_amg_down, dim3(pad8(L.nblk)), dim3(kBlock), 0, s, L, b, (const double*)x, w,
                       (const double*)N.dinv, N.b, last ? nullptr : N.x, flag);
    const Fine here = {L.mptr, nullptr, x};
    hipError_t e;
    if (a.gamma < 2 || last) {
        e = coarse_cycle(a, l + 1, N.b, N.x, nullptr, nullptr, here, flag, s);
    } else {                           // a second cycle on the remaining residual
        e = coarse_cycle(a, l + 1, N.b, N.x, nullptr, N.t, here, flag, s);
        hipLaunchKernelGGL(k_amg_mid, dim3(pad8(N.nslices)), dim3(kBlock), 0, s, N, (const double*)N.b,
                           (const double*)N.t, w, N.r, N.e, flag);
        if (e == hipSuccess) e = coarse_cycle(a, l + 1, N.r, N.e, N.t, nullptr, here, flag, s);
    }
    if (e != hipSuccess) return e;
    if (keep)
        hipLaunchKernelGGL(k_amg_up<true>, dim3(pad8(L.nslices)), dim3(kBlock), 0, s, L, b, (const double*)x, w, keep,
                           first, f.mptr, f.midx, f.x, flag);
    else
        hipLaunchKernelGGL(k_amg_up<false>, dim3(pad8(L.nslices)), dim3(kBlock), 0, s, L, b, (const double*)x, w, keep,
                           first, f.mptr, f.midx, f.x, flag);
    return hipGetLastError();
}

// level 1's correction of the finest iterate x0 from the residual res
hipError_t coarse_levels(const AmgDev& a, const double* res, double* x0, const double* flag, hipStream_t s) {
    const double w = a.omega;
    const AmgLevelDev& N = a.lv[1];
    const bool last = a.nl == 2;
    hipLaunchKernelGGL(k_amg_restrict0, dim3(grid_a(N.n)), dim3(kBlock), 0, s, N.n, a.lv[0].mptr, a.lv[0].midx, res, w,
                       (const double*)N.dinv, N.b, last ? nullptr : N.x, flag);
    const Fine top = {a.lv[0].mptr, a.lv[0].midx, x0};
    if (a.gamma < 2 || last) return coarse_cycle(a, 1, N.b, N.x, nullptr, nullptr, top, flag, s);
    hipError_t e = coarse_cycle(a, 1, N.b, N.x, nullptr, N.t, top, flag, s);
    hipLaunchKernelGGL(k_amg_mid, dim3(pad8(N.nslices)), dim3(kBlock), 0, s, N, (const double*)N.b, (const double*)N.t, w,
                       N.r, N.e, flag);
    return e == hipSuccess ? coarse_cycle(a, 1, N.r, N.e, N.t, nullptr, top, flag, s) : e;
}

// x0 = cycle(b0); smoothed: a.s0 already holds w D^-1 b0; dots: partial x0.b0
// and x0.r_old
hipError_t cycle(const Dev& d, const AmgDev& a, const double* b0, double* x0, bool smoothed, bool dots,
                 const double* flag, hipStream_t s, const AmgSmoother* fine) {
    const double w = a.omega;
    const dim3 T(kBlock), rows(rows_m(d.nc, kBlock)), part(pad8(d.cg_pblk)), verts(rows_m(d.nv * kCgVertexLanes, kBlock));
    hipError_t e = hipSuccess;
    if (a.nl == 1) {                   // the system is small enough to invert densely
        hipLaunchKernelGGL(k_amg_dense, dim3(unsigned(d.nc)), T, 0, s, d.nc, a.cinv, b0, x0, (const int32_t*)nullptr,
                           (const int32_t*)nullptr, (double*)nullptr, flag);
        if (dots) hipLaunchKernelGGL(k_amg_dots, part, T, 0, s, d, (const double*)a.r_old, flag);
        return hipGetLastError();
    }
    // a.s1 or a.s0 = b - K v (the vertex values of the CG's p stay in mf_xv)
    auto residual = [&](const double* v, double* out) {
        hipLaunchKernelGGL(k_amg_vertices, verts, T, 0, s, d, v, a.zv, flag);
        hipLaunchKernelGGL(k_amg_residual0, rows, T, 0, s, d, b0, v, (const double*)a.zv, out, flag);
    };
    if (fine) {                        // x = M(b), the coarse correction, x += M(b - K x)
        e = (*fine)(b0, x0, s);
        if (e != hipSuccess) return e;
        residual(x0, a.s0);
        e = coarse_levels(a, a.s0, x0, flag, s);
        if (e != hipSuccess) return e;
        residual(x0, a.s0);
        e = (*fine)(a.s0, a.s1, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_amg_add, dim3(grid_a(d.nc)), T, 0, s, d.nc, a.s1, x0, flag);
        if (dots) hipLaunchKernelGGL(k_amg_dots, part, T, 0, s, d, (const double*)a.r_old, flag);
        return hipGetLastError();
    }
    double* x = a.s0;                  // pre-smoothed, then corrected
    if (!smoothed)
        hipLaunchKernelGGL(k_amg_smooth0, dim3(grid_a(d.nc)), T, 0, s, d.nc, w, d.k_dinv, b0, x, flag);
    residual(x, a.s1);
    e = coarse_levels(a, a.s1, x, flag, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_amg_vertices, verts, T, 0, s, d, (const double*)x, a.zv, flag);
    hipLaunchKernelGGL(k_amg_smooth_dots, part, T, 0, s, d, b0, (const double*)x, (const double*)a.zv, w, x0,
                       dots ? (const double*)a.r_old : nullptr, flag);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_amg_cycle(const Dev& d, const BcTable&, const AmgDev& a, const double* b0, double* x0,
                            const double* flag, hipStream_t s, const AmgSmoother* fine) {
    return cycle(d, a, b0, x0, false, false, flag, s, fine);
}

hipError_t launch_amg_open(const Dev& d, const BcTable& bc_pot, const AmgDev& a, double tol, int maxit,
                           int restart, bool fresh, bool matrix_free, hipStream_t s, const AmgSmoother* fine) {
    const int64_t nb = grid_a(d.nc);
    hipError_t e = launch_mf_apply(d, bc_pot, d.x, d.tmp, s);            // t = K x
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_amg_open, dim3(unsigned(nb)), dim3(kBlock), 0, s, d, d.tmp);
    hipLaunchKernelGGL(k_amg_open_fin, dim3(1), dim3(1024), 0, s, d, nb, tol, maxit, restart, fresh ? 1 : 0);
    e = cycle(d, a, d.r, d.z, false, false, d.scal + SC_DONE, s, fine);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_amg_p0, dim3(unsigned(nb)), dim3(kBlock), 0, s, d);
    hipLaunchKernelGGL(k_amg_rz_fin, dim3(1), dim3(1024), 0, s, d, nb);
    e = hipGetLastError();
    return e == hipSuccess && matrix_free ? launch_cg_open_vertices(d, s) : e;
}

hipError_t launch_amg_iteration(const Dev& d, const BcTable&, const AmgDev& a, bool matrix_free,
                                hipStream_t s, const AmgSmoother* fine) {
    hipError_t e = launch_cg_part(d, false, !matrix_free, 0, s);         // q = K p, partial p.q
    if (e != hipSuccess) return e;
    const dim3 T(d.cg_threads);
    const unsigned rows = pad8(d.cg_nblk), nv = matrix_free ? pad8(d.cg_vblk) : 0u;
    hipLaunchKernelGGL(k_amg_step, dim3(rows), T, 0, s, d, cg_product_parts(d, !matrix_free), a.omega, a.r_old, a.s0);
    hipLaunchKernelGGL(k_amg_rr_fin, dim3(1), dim3(1024), 0, s, d);
    e = cycle(d, a, d.r, d.z, true, true, d.scal + SC_DONE, s, fine);
    if (e != hipSuccess) return e;
    if (matrix_free) hipLaunchKernelGGL(k_amg_direction<true>, dim3(rows + nv), T, 0, s, d, int(nv));
    else hipLaunchKernelGGL(k_amg_direction<false>, dim3(rows), T, 0, s, d, 0);
    return hipGetLastError();
}

}  // namespace mifvm
