// One iteration of Jacobi-preconditioned CG in three kernels, matrix-free in
// FP64 or FP32 (the inner solve of the refined form):
//   k_cg_product   q = K p from the cells' tables and the vertex values of
//                  p; partial p.q;
//   k_cg_residual  alpha = rz / p.q (every block adds the partials), r -=
//                  alpha q, z = D^-1 r in q's place; partial rz, rr;
//   k_cg_direction beta and the convergence tests (every block), x += alpha
//                  p, p = z + beta p; its first blocks update the vertex
//                  values of p by the same recurrence, A p = A z + beta A p
//                  with A z summed over the vertex lists.
// On the stored matrix (one mesh) the product is k_cg_product_stored and
// there are no vertex values.
//
// Why three: the iteration is a chain of dependent kernels, each at least
// 1.6 us from the launch before it plus its own latency chain, so on small
// meshes their number is the time.  The vertex values need beta only for the
// recurrence, not for the gathers, so they share a launch with the direction;
// alpha and beta are formed by whoever needs them instead of in kernels of
// one block.  No block reads a scalar that another block of the same kernel
// writes: k_cg_direction leaves the new scalars in the SC_N_* slots and the
// next product (or k_cg_commit, after a chunk's last iteration) copies them.
#include <algorithm>

#include "cg_iter.h"
#include "cg_dev.h"
#include "halo_stage.h"
#include "mf_cell.h"

namespace mifvm {
namespace {

// the scalars the last direction kernel left for the next iteration
__device__ inline void commit(double* sc) {
    sc[SC_RZ] = sc[SC_N_RZ];
    sc[SC_RR] = sc[SC_N_RR];
    sc[SC_IT] = sc[SC_N_IT];
    sc[SC_SINCE] = sc[SC_N_SINCE];
    sc[SC_DONE] = sc[SC_N_DONE];
}

__global__ __launch_bounds__(256) void k_cg_commit(Dev d) {
    const int m = int(blockIdx.x) * 256 + threadIdx.x;
    if (m < d.nm) commit(msc(d, m));
}

// q = K p row by row; partial p.q
template <class R>
__global__ __launch_bounds__(kBlock) void k_cg_product(Dev d) {
    __shared__ double lds[kMaxWaves];
    const int64_t lb = xcd_block();
    if (lb >= d.cg_pblk) return;
    int64_t r0 = lb * d.cg_prows, r1 = r0 + d.cg_prows;
    if (r1 > d.nc) r1 = d.nc;
    double* sc = d.scal;
    bool lead = lb == 0;
    if (d.nm > 1) {
        const int4 t = d.cg_prod[lb];
        r0 = t.y;
        r1 = t.z;
        sc = msc(d, t.x);
        lead = t.w != 0;
    }
    if (lead && threadIdx.x == 0) commit(sc);
    if (sc[SC_N_DONE] != 0.0) return;
    const R* __restrict__ p = CgVec<R>::p(d);
    const R* __restrict__ pv = reinterpret_cast<const R*>(d.mf_xv);
    R* __restrict__ q = CgVec<R>::q(d);
    double v[1] = {0.0};
    for (int64_t i = r0 + threadIdx.x; i < r1; i += kBlock) {
        const R y = cell_row(d, p, pv, i);
        q[i] = y;
        v[0] += double(p[i]) * double(y);
    }
    block_sums<1>(v, lds);
    if (threadIdx.x == 0) d.partial[lb] = v[0];
}

// The same for one mesh in gradient tiles of 256 cells, FP64 and FP32: the
// tile's own p, which 85% of its cells' neighbours are, and the vertex values
// its cells touch (0.49 per cell instead of 4, named by 16-bit local numbers)
// go through LDS; a neighbour outside is gathered, and lanes without one read
// their own cell's line.
template <class R>
__global__ __launch_bounds__(kBlock) void k_cg_product_tiles(Dev d, BlockOrder order) {
    extern __shared__ __align__(16) unsigned char sp_raw[];
    __shared__ double lds[kMaxWaves];
    R* const sx = reinterpret_cast<R*>(sp_raw);            // [256] p
    R* const sv = sx + kBlock;                             // vertex values
    const int64_t lb = order.block();
    double* sc = d.scal;
    if (lb == 0 && threadIdx.x == 0) commit(sc);
    if (sc[SC_N_DONE] != 0.0) return;
    const int64_t nc = d.nc;
    const R* __restrict__ p = CgVec<R>::p(d);
    const R* __restrict__ pv = reinterpret_cast<const R*>(d.mf_xv);
    R* __restrict__ q = CgVec<R>::q(d);
    double v[1] = {0.0};
    for (int64_t t = lb; t < d.g_tiles; t += order.grid) {
        const int64_t t0 = t * kBlock, row = t0 + threadIdx.x, i = row < nc ? row : nc - 1;
        const int64_t w0 = d.gv_off[t];
        const int wn = int(d.gv_off[t + 1] - w0);
        const int wv = d.gv_idx[w0 + (int(threadIdx.x) < wn ? int(threadIdx.x) : 0)];
        int nb[4];
        R w[3], r[4];
        const uint2 cv = d.cell_cv[i];
        load_quad(d.cell_nb, nc, i, nb);
        load_weights(MfCell<R>::w(d), nc, i, w);
        load_quad(MfCell<R>::r(d), nc, i, r);
        const R xi = p[i], wval = pv[wv];
        R xn[4];
        int in_tile[4];                                    // the neighbour's place in the tile, or -1
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t l = nb[k] - t0;
            const bool bnd = nb[k] >= nc;                  // a boundary face takes x_i
            in_tile[k] = l >= 0 && l < kBlock && !bnd ? int(l) : -1;
            xn[k] = p[in_tile[k] < 0 && !bnd ? int64_t(nb[k]) : i];
        }
        if (t != lb) __syncthreads();        // the last tile's readers
        sx[threadIdx.x] = xi;
        if (int(threadIdx.x) < wn) sv[threadIdx.x] = wval;
        for (int u = kBlock + threadIdx.x; u < wn; u += kBlock) sv[u] = pv[d.gv_idx[w0 + u]];
        __syncthreads();
        const R x0 = sv[cv.x & 0xffff], x1 = sv[cv.x >> 16], x2 = sv[cv.y & 0xffff], x3 = sv[cv.y >> 16];
        R acc = w[0] * (x0 - x3);
        acc += w[1] * (x1 - x3);
        acc += w[2] * (x2 - x3);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const R xl = sx[in_tile[k] < 0 ? int(threadIdx.x) : in_tile[k]];
            const R x = in_tile[k] < 0 ? xn[k] : xl;
            acc += r[k] * (nb[k] < nc ? x - xi : x);
        }
        if (row < nc) {
            q[i] = -acc;
            v[0] -= double(xi) * double(acc);
        }
    }
    block_sums<1>(v, lds);
    if (threadIdx.x == 0) d.partial[lb] = v[0];
}

// The same on the stored matrix (one mesh): a block takes a cell tile a
// round over neighbouring tiles (in a run of tiles a block, their halos leave
// the L2: 10.4M cells 1.431 ms against 1.402), each tile's halo of p staged in
// LDS and addressed by 16-bit local indices; the entries of a row in stored order.
template <class R>
__global__ __launch_bounds__(kBlock) void k_cg_product_stored(Dev d) {
    extern __shared__ __align__(16) unsigned char sp_raw[];
    __shared__ double lds[kMaxWaves];
    R* sp = reinterpret_cast<R*>(sp_raw);
    double* sc = d.scal;
    if (blockIdx.x == 0 && threadIdx.x == 0) commit(sc);
    if (sc[SC_N_DONE] != 0.0) return;
    const R* __restrict__ val = CgVec<R>::val(d);
    const R* __restrict__ diag = CgVec<R>::diag(d);
    R* __restrict__ q = CgVec<R>::q(d);
    const int T = blockDim.x;
    double v[1] = {0.0};
    for (int64_t t = blockIdx.x; t < d.ntiles; t += gridDim.x) {
        if (t != blockIdx.x) __syncthreads();             // the last tile's readers
        stage_halo_values(d, t, CgVec<R>::p(d), sp);
        __syncthreads();
        const int64_t i = t * T + threadIdx.x;
        if (i < d.nc) {
            const R pi = sp[d.h_self[t] + threadIdx.x];
            const int64_t s = i >> 6;
            const int64_t base = d.k_off[s] + (i & 63);
            const int w = d.k_w[s];
            R y = diag[i] * pi;
            // 16 entries' loads in flight, then their sums in row order
            for (int k0 = 0; k0 < w; k0 += 16) {
                uint16_t l[16];
                R a[16];
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const bool in = k0 + j < w;
                    const int64_t at = base + int64_t(k0 + j) * 64;
                    l[j] = in ? d.k_lidx[at] : uint16_t(0);
                    a[j] = in ? val[at] : R(0);
                }
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    if (k0 + j < w) y += a[j] * sp[l[j]];   // w is one slice's: uniform over the wave
            }
            q[i] = y;
            v[0] += double(pi) * double(y);
        }
    }
    block_sums<1>(v, lds);
    if (threadIdx.x == 0) d.partial[blockIdx.x] = v[0];
}

// alpha; r -= alpha q; z = D^-1 r; partial rz, rr.  np: the product's partials
// of a single mesh (its blocks may differ from this kernel's).  z takes q's
// place, which nothing reads any more: one vector less for the cache to hold
// (1.3M cells 73.2 -> 67.8 ms, 4.4M 360 -> 352, refined 3.07M 160 -> 155).
template <class R>
__global__ __launch_bounds__(512) void k_cg_residual(Dev d, int np) {
    __shared__ double lds[3 * kMaxWaves];
    const int64_t lb = xcd_block();
    if (lb >= d.cg_nblk) return;
    const Seg s = cg_seg(d, lb);
    R* const qz = CgVec<R>::q(d);                          // q, replaced by z row by row
    const R* __restrict__ dinv = CgVec<R>::dinv(d);
    R* __restrict__ r = CgVec<R>::r(d);
    const int T = blockDim.x;
    // the first row's loads go out before the scalars are known
    int64_t i = s.r0 + threadIdx.x;
    const int64_t last = s.r1 - 1;
    int64_t c = i < last ? i : last;
    R ri = r[c], qi = qz[c], di = dinv[c];
    if (s.sc[SC_DONE] != 0.0) return;
    double pq[1];
    sum_parts<1>(d.partial + s.pp0, 0, d.nm == 1 ? np : s.pnp, lds, pq);
    const double alpha = s.sc[SC_RZ] / pq[0];
    if (s.lead && threadIdx.x == 0) {
        s.sc[SC_PQ] = pq[0];
        s.sc[SC_ALPHA] = alpha;
    }
    const R a = R(alpha);
    double v[2] = {0.0, 0.0};
    for (; i < s.r1; i += T) {
        const int64_t n = i + T;
        c = n < last ? n : last;
        const R rn = r[c], qn = qz[c], dn = dinv[c];       // the next row's, in flight
        const R rc = ri - a * qi;
        const R zc = di * rc;
        r[i] = rc;
        qz[i] = zc;
        v[0] += double(rc) * double(zc);
        v[1] += double(rc) * double(rc);
        ri = rn;
        qi = qn;
        di = dn;
    }
    block_sums<2>(v, lds + kMaxWaves);
    if (threadIdx.x == 0) {
        double* __restrict__ out = d.partial + d.cg_stride;
        out[lb] = v[0];
        out[d.cg_stride + lb] = v[1];
    }
}

// beta and the tests; x += alpha p; p = z + beta p; A p = A z + beta A p.
// VERTS: the first gridDim.x - nrow blocks take the vertices.
template <class R, bool VERTS>
__global__ __launch_bounds__(512) void k_cg_direction(Dev d, int nvert) {
    __shared__ double lds[2 * kMaxWaves];
    const int T = blockDim.x;
    const bool vert = VERTS && int(blockIdx.x) < nvert;
    const int blk = vert ? int(blockIdx.x) : int(blockIdx.x) - nvert;
    const int per = (vert ? nvert : int(gridDim.x) - nvert) / kXcds;
    const int64_t lb = int64_t(blk % kXcds) * per + blk / kXcds;
    if (lb >= (vert ? d.cg_vblk : d.cg_nblk)) return;
    if (VERTS && vert) {
        int64_t v0 = lb * (T / kCgVertexLanes), v1 = v0 + T / kCgVertexLanes;
        int m = 0, p0 = 0, np = d.cg_nblk;
        if (v1 > d.nv) v1 = d.nv;
        if (d.nm > 1) {
            const int4 t = d.cg_vert[lb];
            const int4 pr = d.cg_parts[t.x];
            m = t.x;
            v0 = t.y;
            v1 = t.z;
            p0 = pr.x;
            np = pr.y;
        }
        const double* sc = msc(d, m);
        if (sc[SC_DONE] != 0.0) return;
        R* __restrict__ pv = reinterpret_cast<R*>(d.mf_xv);
        const int q = threadIdx.x & (kCgVertexLanes - 1);
        const int64_t v = v0 + (threadIdx.x / kCgVertexLanes);
        const int64_t vc = v < v1 ? v : v1 - 1;
        const R old = pv[vc];
        const R zv = vertex_sum<R>(d, CgVec<R>::q(d), vc, q);     // z
        double t[1];
        sum_parts<1>(d.partial + d.cg_stride + p0, 0, np, lds, t);
        const R beta = R(t[0] / sc[SC_RZ]);
        if (q == 0 && v < v1) pv[v] = zv + beta * old;
        return;
    }
    const Seg s = cg_seg(d, lb);
    const R* __restrict__ z = CgVec<R>::q(d);              // left there by k_cg_residual
    R* __restrict__ x = CgVec<R>::x(d);
    R* __restrict__ p = CgVec<R>::p(d);
    int64_t i = s.r0 + threadIdx.x;
    const int64_t last = s.r1 - 1;
    int64_t c = i < last ? i : last;
    R xi = x[c], pi = p[c], zi = z[c];
    if (s.sc[SC_DONE] != 0.0) return;
    double t[2];
    sum_parts<2>(d.partial + d.cg_stride + s.p0, d.cg_stride, s.np, lds, t);
    const double beta = t[0] / s.sc[SC_RZ];
    const R a = R(s.sc[SC_ALPHA]), b = R(beta);
    for (; i < s.r1; i += T) {
        const int64_t n = i + T;
        c = n < last ? n : last;
        const R xn = x[c], pn = p[c], zn = z[c];
        x[i] = xi + a * pi;
        p[i] = zi + b * pi;
        xi = xn;
        pi = pn;
        zi = zn;
    }
    // count; convergence (1), iteration limit (2) or a scheduled restart (3)
    if (s.lead && threadIdx.x == 0) {
        double* sc = s.sc;
        const double it = sc[SC_IT] + 1.0, since = sc[SC_SINCE] + 1.0;
        sc[SC_BETA] = beta;
        sc[SC_N_RZ] = t[0];
        sc[SC_N_RR] = t[1];
        sc[SC_N_IT] = it;
        sc[SC_N_SINCE] = since;
        double done = 0.0;
        if (t[1] <= sc[SC_TOL2BB]) done = 1.0;
        else if (it >= sc[SC_MAXIT]) done = 2.0;
        else if (sc[SC_RESTART] > 0.0 && since >= sc[SC_RESTART]) done = 3.0;
        sc[SC_N_DONE] = done;
    }
}

// vertex values of p when the multigrid's loop opens
__global__ __launch_bounds__(256) void k_cg_open_vertices(Dev d) { open_vertices<double>(d, xcd_block()); }

}  // namespace

CgPlan cg_plan(const Mesh& m) {
    CgPlan c;
    const size_t nm = m.mesh_start.size() - 1;
    int64_t most = 0;
    for (size_t k = 0; k < nm; ++k) most = std::max(most, m.mesh_start[k + 1] - m.mesh_start[k]);
    // A block's rows: about kCgMaxBlocks blocks for the whole state, at least
    // 256 for its largest mesh (the last to finish) and no more than
    // kCgMaxBlocks for any mesh, whose partials every block of the next kernel
    // adds.  256 threads and more rows each: 384k cells in threads of one row
    // 20.7 ms, of two 19.6; 1.3M refined 49.4 and 47.6; eight meshes of 0.5M
    // cells 31.3 and 29.8, forty of 2.9M 106.6 and 99.8.  Above eight rows 512
    // threads: 4.4M 355 ms, with 256 360.  Of 512 blocks and 1,024 neither is
    // better; 2,048: 384k 21.0, 1.3M refined 52.4.
    const int64_t share = std::max((most + kCgMaxBlocks - 1) / kCgMaxBlocks,
                                   std::min((m.nc + kCgMaxBlocks - 1) / kCgMaxBlocks, (most + 255) / 256));
    if (share > 256) {                     // rows a thread, then threads in whole wavefronts
        const int64_t widest = share > 2048 ? 512 : 256, per = (share + widest - 1) / widest;
        c.threads = int32_t(((share + per - 1) / per + 63) / 64 * 64);
        c.rows = int32_t(c.threads * per);
    }
    c.prows = int32_t(256 * std::max<int64_t>(1, (most + 256 * kCgMaxProductBlocks - 1) / (256 * kCgMaxProductBlocks)));
    const int64_t vrows = c.threads / kCgVertexLanes;
    if (nm == 1) {
        c.nblk = int32_t((m.nc + c.rows - 1) / c.rows);
        c.pblk = int32_t((m.nc + c.prows - 1) / c.prows);
        c.vblk = int32_t((m.nv + vrows - 1) / vrows);
        return c;
    }
    // vertices are numbered by their lowest cell, so a mesh's are contiguous
    int64_t v = 0;
    for (size_t k = 0; k < nm; ++k) {
        const int64_t c0 = m.mesh_start[k], c1 = m.mesh_start[k + 1];
        auto split = [&](std::vector<CgPlan::Item>& out, int64_t from, int64_t to, int64_t step) {
            for (int64_t r = from; r < to; r += step)
                out.push_back({int32_t(k), int32_t(r), int32_t(std::min(r + step, to)), r == from ? 1 : 0});
        };
        const CgPlan::Range first = {int32_t(c.cells.size()), 0, int32_t(c.product.size()), 0};
        split(c.cells, c0, c1, c.rows);
        split(c.product, c0, c1, c.prows);
        c.parts.push_back({first.first, int32_t(c.cells.size()) - first.first, first.pfirst,
                           int32_t(c.product.size()) - first.pfirst});
        int64_t lo = v, hi = m.nv;
        while (lo < hi) {
            const int64_t mid = (lo + hi) / 2;
            if (m.nidx[m.nptr[mid]] < c1) lo = mid + 1;
            else hi = mid;
        }
        split(c.vertices, v, lo, vrows);
        v = lo;
    }
    c.nblk = int32_t(c.cells.size());
    c.pblk = int32_t(c.product.size());
    c.vblk = int32_t(c.vertices.size());
    return c;
}

bool cg_meshes_apart(const Mesh& m) {
    if (m.mesh_start.size() <= 2) return true;
    auto cell = [&](int32_t e) { return e < m.nc ? e : m.gowner[e - m.nc]; };
    size_t k = 0;
    for (int64_t v = 0; v < m.nv; ++v) {
        while (cell(m.nidx[m.nptr[v]]) >= m.mesh_start[k + 1]) ++k;
        for (int64_t e = m.nptr[v]; e < m.nptr[v + 1]; ++e)
            if (cell(m.nidx[e]) >= m.mesh_start[k + 1]) return false;
    }
    return true;
}

namespace {
// tiles per block of the stored product
int stored_tiles(const Dev& d) { return int((d.ntiles + kCgMaxProductBlocks - 1) / kCgMaxProductBlocks); }

// The product by tiles: 131k cells and more (two tiles a CU).  Below, its
// barrier costs more than its gathers save: 48k cells 4.50 ms against 4.39; above,
// 162k 9.84 against 10.04, 4.4M 361 against 372, refined 384k 16.4 against 17.2.
bool tiled_product(const Dev& d) { return d.nm == 1 && d.g_rows == kBlock && d.g_tiles >= 512; }
// Its blocks take a tile a round: one round and contiguous eighths to 8,192
// tiles, then as few rounds as that many partials allow, each over neighbouring
// tiles in the step kernels' windows.  (A block's tiles in sequence instead put
// the blocks at work so far apart that a neighbour outside the tile left the
// L2: 3.07M cells refined 159 ms against 154, 4.4M 354 against 349.  Windows in
// the one round: 1.3M 69 against 67 ms.)
BlockOrder tile_order(const Dev& d) {
    const int64_t rounds = (d.g_tiles + kCgMaxProductBlocks - 1) / kCgMaxProductBlocks;
    if (rounds > 1) return stream_order((d.g_tiles + rounds - 1) / rounds, 1);
    const unsigned g = pad8(d.g_tiles);
    return {g, 28u, g / kXcds};
}
}  // namespace

int cg_product_parts(const Dev& d, bool stored) {
    if (stored) return int((d.ntiles + stored_tiles(d) - 1) / stored_tiles(d));
    return tiled_product(d) ? int(tile_order(d).grid) : int(d.cg_pblk);
}

namespace {
template <class R>
hipError_t cg_part(const Dev& d, bool stored, int part, hipStream_t s) {
    const dim3 T(d.cg_threads);
    const unsigned rows = pad8(d.cg_nblk), verts = stored ? 0u : pad8(d.cg_vblk);
    const unsigned nst = unsigned(cg_product_parts(d, true));
    if (part == 0 && stored)
        hipLaunchKernelGGL(k_cg_product_stored<R>, dim3(nst), dim3(d.tile_rows), size_t(d.halo_max) * sizeof(R), s, d);
    else if (part == 0 && tiled_product(d))
        hipLaunchKernelGGL(k_cg_product_tiles<R>, dim3(tile_order(d).grid), dim3(kBlock),
                           size_t(kBlock + d.gv_max) * sizeof(R), s, d, tile_order(d));
    else if (part == 0)
        hipLaunchKernelGGL(k_cg_product<R>, dim3(pad8(d.cg_pblk)), dim3(kBlock), 0, s, d);
    else if (part == 1)
        hipLaunchKernelGGL(k_cg_residual<R>, dim3(rows), T, 0, s, d, cg_product_parts(d, stored));
    else if (stored)
        hipLaunchKernelGGL((k_cg_direction<R, false>), dim3(rows), T, 0, s, d, 0);
    else
        hipLaunchKernelGGL((k_cg_direction<R, true>), dim3(rows + verts), T, 0, s, d, int(verts));
    return hipGetLastError();
}
}  // namespace

hipError_t launch_cg_part(const Dev& d, bool fp32, bool stored, int part, hipStream_t s) {
    return fp32 ? cg_part<float>(d, stored, part, s) : cg_part<double>(d, stored, part, s);
}

hipError_t launch_cg_open_vertices(const Dev& d, hipStream_t s) {
    hipLaunchKernelGGL(k_cg_open_vertices, dim3(pad8(vertex_blocks(d, 256))), dim3(256), 0, s, d);
    return hipGetLastError();
}

hipError_t launch_cg_commit(const Dev& d, hipStream_t s) {
    hipLaunchKernelGGL(k_cg_commit, dim3((d.nm + 255) / 256), dim3(256), 0, s, d);
    return hipGetLastError();
}

}  // namespace mifvm
