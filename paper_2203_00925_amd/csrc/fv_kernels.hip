// Kernels of the explicit finite-volume residual (eq. (4) of the paper) and
// its Runge-Kutta update (eq. (6)), for CDNA4 wave64.
//
// A Runge-Kutta stage is three gather kernels, each owner-computes and free
// of atomics:
//   k_vertex_moments  per vertex: the moments of its list that the gradient
//                   needs, and the least-squares interpolation (Algorithm 2);
//   k_grad_cells    per tile of cells: least-squares gradient (Algorithm 1,
//                   in star-moment form), then the Barth-Jespersen limiter
//                   over the 4 face neighbours and the MUSCL values at the
//                   cell's face centroids;
//   k_cell_step     per cell: the upwind convective fluxes (eq. (15)) minus
//                   the diamond diffusive fluxes (eq. (diamond)) of its four
//                   faces, summed, and the stage update.
// The residual evaluation that returns the face fluxes runs the face kernel
// k_face_flux (one thread per face) after the gradient kernel instead.
// Ghost values (behind boundary faces) are materialised by k_step_begin
// before a run of steps (k_ghost_fill elsewhere) and by k_cell_step after every
// stage, so every gather is a plain indexed load.
//
// Every kernel is instantiated for FP64 (the method as stated) and FP32 (the
// reduced-precision form: state, gradients, fluxes and geometry copies in
// FP32; in LDS the FP32 form keeps positions relative to the tile's first
// cell, computed in FP64, so differences of nearby positions keep their
// digits).  Sums that must stay FP64 (conservation, the CFL bound) read the
// FP64 geometry.
//
// Per-row lists (stencil, vertex lists) are stored in 64-row slices with the
// entry index as the slow dimension, so the index/weight loads of a
// wavefront are one contiguous 128/256/512-byte segment.
#include <type_traits>

#include "quad.h"
#include "reduce.h"
#include "seg.h"
#include "state.h"
#include "xcd.h"

namespace mifvm {

__device__ inline int64_t gtid() { return int64_t(blockIdx.x) * blockDim.x + threadIdx.x; }

inline int grid_for(int64_t n) { return int((n + kBlock - 1) / kBlock); }

template <class R> struct Vec2T;
template <> struct Vec2T<double> { using T = double2; };
template <> struct Vec2T<float> { using T = float2; };

__device__ inline double4 mk4(double x, double y, double z, double w) { return make_double4(x, y, z, w); }
__device__ inline float4 mk4(float x, float y, float z, float w) { return make_float4(x, y, z, w); }
__device__ inline double2 mk2(double x, double y) { return make_double2(x, y); }
__device__ inline float2 mk2(float x, float y) { return make_float2(x, y); }

template <class R>
__device__ inline void fill_ghost(int64_t g, int64_t nc, const int32_t* __restrict__ gowner,
                                  const int32_t* __restrict__ gtag, const R* __restrict__ gdist, const BcTable& bc,
                                  R* u) {
    const int t = gtag[g];
    const int kind = bc.kind[t];
    const R val = bc_value<R>(bc, g);
    const R uo = u[gowner[g]];
    R ug;
    if (kind == kDirichlet) ug = R(2) * val - uo;
    else if (kind == kNeumann) ug = uo + val * gdist[g];
    else ug = uo;
    u[nc + g] = ug;
}

template <class R>
__global__ __launch_bounds__(kBlock) void k_ghost_fill(int64_t nc, int64_t nb,
                                                        const int32_t* __restrict__ gowner,
                                                        const int32_t* __restrict__ gtag,
                                                        const R* __restrict__ gdist, BcTable bc, R* u) {
    const int64_t g = gtid();
    if (g < nb) fill_ghost(g, nc, gowner, gtag, gdist, bc, u);
}

// ---- gradient in star-moment form ------------------------------------------
// The sum of Algorithm 1, J_i = sum_{j in N(i)} (x_j - x_i)(u_j - u_i) over
// the node-neighbour stencil N(i) (every cell and ghost sharing a vertex
// with i), rewritten exactly.  An entity sharing m vertices with i lies in m
// of i's 4 vertex lists, so with T_L(i) = sum_{j in L} (x_j - x_i)(u_j - u_i)
//   J_i = sum_{v of i} T_{L(v)}(i) - sum_{j sharing only an edge} (.) - 2 sum_{face nbrs} (.)
// (i itself adds zeros).  For a list L of n entities with mean position xb,
// mean value ub and centred moment C = sum (x_j - xb)(u_j - ub),
//   T_L(i) = C + n (xb - x_i)(ub - u_i).
// Every term is a product of differences of nearby values, so no large value
// cancels.
//
// k_vertex_moments forms (C, ub) of every vertex list once, and with it the
// least-squares vertex value of Algorithm 2: its weights are 1/n + b . (x_j -
// xb) with a slope b per vertex, so u_v = ub + b . C, and no weight per list
// entry is read.  k_grad_cells then needs, per cell, 4 vertex records, 4 face
// neighbours and ~14 edge-only neighbours instead of ~70 stencil entries.

// (C, ub) and u_v of one vertex, summed by 4 neighbouring lanes: lane q takes
// the entries q, q + 4, ..., six loads of each kind in flight.  Values are
// taken relative to the list's first entry's.
constexpr int kMomentLanes = 4, kMomentBatch = 6;

template <class R>
struct ListSums {                         // one lane's part
    R cx = R(0), cy = R(0), cz = R(0), su = R(0);

    __device__ void add(double x, double y, double z, R du, const double4& xb) {
        cx += R(x - xb.x) * du;
        cy += R(y - xb.y) * du;
        cz += R(z - xb.z) * du;
        su += du;
    }
    // The lanes' parts together; lane 0 of an existing vertex writes.  The
    // differences to the rounded xb add up to l, not to zero: C - l (ub - u0)
    // is the centred moment.
    __device__ void finish(const FvArrays<R>& a, int64_t v, bool write, R n, R u0, const double4& xb,
                           const double4& sb) {
#pragma unroll
        for (int o = 1; o < kMomentLanes; o <<= 1) {
            su += __shfl_xor(su, o, 64);
            cx += __shfl_xor(cx, o, 64);
            cy += __shfl_xor(cy, o, 64);
            cz += __shfl_xor(cz, o, 64);
        }
        if (!write) return;
        const R lx = R(__int_as_float(__double2loint(xb.w))), ly = R(__int_as_float(__double2hiint(xb.w)));
        const R lz = R(sb.w);
        const R bl = R(sb.x) * lx + R(sb.y) * ly + R(sb.z) * lz, bc = R(sb.x) * cx + R(sb.y) * cy + R(sb.z) * cz;
        const R mean = su / n, ub = u0 + mean;
        a.unode[v] = ub + (bc - bl * mean);
        a.vmom[v] = mk4(cx - lx * mean, cy - ly * mean, cz - lz * mean, ub);
    }
};

template <class R>
__global__ __launch_bounds__(kBlock) void k_vertex_moments(Dev d, FvArrays<R> a, BlockOrder order) {
    constexpr int L = kMomentLanes, B = kMomentBatch;
    const int64_t v = order.block() * (kBlock / L) + threadIdx.x / L;
    const int q = threadIdx.x & (L - 1);
    const int64_t vc = v < d.nv ? v : d.nv - 1;
    const int64_t sl = vc >> 6;
    const int64_t base = d.n_off[sl] + (vc & 63);
    const int n = d.n_len[vc];
    const double4 xb = d.vmean[vc], sb = d.vslope[vc];
    const double4* __restrict__ P = d.xyz4;
    const R* __restrict__ u = a.u;
    ListSums<R> sums;
    R u0 = R(0);
    for (int k0 = 0; k0 < n; k0 += B * L) {               // uniform over the 4 lanes
        int e[B];
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const int k = k0 + j * L + q;
            e[j] = d.n_idx[base + int64_t(k < n ? k : 0) * 64];
        }
        double4 pe[B];
        R ue[B];
#pragma unroll
        for (int j = 0; j < B; ++j) {
            pe[j] = P[e[j]];
            ue[j] = u[e[j]];
        }
        if (k0 == 0) u0 = __shfl(ue[0], int(threadIdx.x & 63 & ~(L - 1)), 64);
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const bool in = k0 + j * L + q < n;
            sums.add(pe[j].x, pe[j].y, pe[j].z, in ? ue[j] - u0 : R(0), xb);
        }
    }
    sums.finish(a, v, q == 0 && v < d.nv, R(n), u0, xb, sb);
}

// The same per slice of 64 vertices, one block each, with the entities their
// lists name staged in LDS: the direct gathers are bound by line accesses (24
// positions and values a vertex, two loads and one each), and a slice's
// entities, sorted, are half as many and mostly neighbours in memory.  The same
// sums in the same order.
template <class R>
__global__ __launch_bounds__(kBlock) void k_vertex_moments_tiles(Dev d, FvArrays<R> a, BlockOrder order) {
    constexpr int L = kMomentLanes, B = kMomentBatch, H = 4;
    extern __shared__ __align__(16) unsigned char sm_raw[];
    double2* const hxy = reinterpret_cast<double2*>(sm_raw);
    double* const hz = reinterpret_cast<double*>(hxy + d.nh_max);
    R* const hv = reinterpret_cast<R*>(hz + d.nh_max);
    const int64_t sl = order.block();
    if (sl * 64 >= d.nv) return;
    const int T = kBlock;
    const int64_t h0 = d.nh_off[sl];
    const int hn = int(d.nh_off[sl + 1] - h0);
    const int64_t v = sl * 64 + threadIdx.x / L;
    const int q = threadIdx.x & (L - 1);
    const int64_t vc = v < d.nv ? v : d.nv - 1;
    const int64_t base = d.n_off[sl] + (vc & 63);
    int he[H];
#pragma unroll
    for (int j = 0; j < H; ++j) {
        const int h = j * T + threadIdx.x;
        he[j] = d.nh_idx[h0 + (h < hn ? h : 0)];
    }
    const int n = d.n_len[vc];
    const double4* __restrict__ P = d.xyz4;
    const R* __restrict__ u = a.u;
    double4 hp[H];
    R hu[H];
#pragma unroll
    for (int j = 0; j < H; ++j) {
        hp[j] = P[he[j]];
        hu[j] = u[he[j]];
    }
    const double4 xb = d.vmean[vc], sb = d.vslope[vc];
    int l[B];
#pragma unroll
    for (int j = 0; j < B; ++j) {
        const int k = j * L + q;
        l[j] = d.nl_idx[base + int64_t(k < n ? k : 0) * 64];
    }
#pragma unroll
    for (int j = 0; j < H; ++j) {
        const int h = j * T + threadIdx.x;
        if (h < hn) {
            hxy[h] = make_double2(hp[j].x, hp[j].y);
            hz[h] = hp[j].z;
            hv[h] = hu[j];
        }
    }
    for (int h = H * T + threadIdx.x; h < hn; h += T) {
        const int e = d.nh_idx[h0 + h];
        const double4 p = P[e];
        hxy[h] = make_double2(p.x, p.y);
        hz[h] = p.z;
        hv[h] = u[e];
    }
    __syncthreads();
    ListSums<R> sums;
    R u0 = R(0);
    for (int k0 = 0; k0 < n; k0 += B * L) {               // uniform over the 4 lanes
        if (k0 > 0) {
#pragma unroll
            for (int j = 0; j < B; ++j) {
                const int k = k0 + j * L + q;
                l[j] = d.nl_idx[base + int64_t(k < n ? k : 0) * 64];
            }
        }
        if (k0 == 0) u0 = __shfl(hv[l[0]], int(threadIdx.x & 63 & ~(L - 1)), 64);
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const bool in = k0 + j * L + q < n;
            const double2 p = hxy[l[j]];
            sums.add(p.x, p.y, hz[l[j]], in ? hv[l[j]] - u0 : R(0), xb);
        }
    }
    sums.finish(a, v, q == 0 && v < d.nv, R(n), u0, xb, sb);
}

// One block per tile of d.g_rows cells.  The tile's halo (its cells and the
// entities sharing an edge or a face with one, 2.9 per cell) is staged in LDS
// as two arrays of 16-byte items, (x, y) and (z, u), and the records of the
// vertices its cells touch (0.49 per cell) as five and a half: random reads of
// 16-byte items spread over the bank groups.  39 KB a tile, so four tiles
// share a CU.  Loads go out in two waves before the one barrier: the indices
// and the cell's own tables (16 bytes a load: 8 local indices), then the
// gathers they address; out-of-range slots read a valid address and are
// discarded, so no load sits under a branch.
//
// The limiter's face centroids come from the cell's vertices: with x_i the
// mean of the four and x_f of three of them, x_f - x_i = (x_i - x_v)/3 for the
// vertex v across from the face.
template <class R, bool PARTS>
__global__ __launch_bounds__(kBlock, 4) void k_grad_cells(Dev d, FvArrays<R> a, BlockOrder order) {
    using V2 = typename Vec2T<R>::T;
    using V4 = typename Vec4T<R>::T;
    extern __shared__ __align__(16) unsigned char sm_raw[];
    const int hc = d.g_max, vcap = d.gv_max;
    V2* const xy = reinterpret_cast<V2*>(sm_raw);         // halo
    V2* const zu = xy + hc;
    V2* const va = zu + hc;                               // vertices: xb - x_v (x, y), (z, n),
    V2* const vb = va + vcap;
    V2* const vc = vb + vcap;                             // (C_x, C_y), (C_z, ub),
    V2* const vd = vc + vcap;
    V2* const ve = vd + vcap;                             // (x_v, y_v), z_v
    R* const vf = reinterpret_cast<R*>(ve + vcap);
    constexpr bool rel = std::is_same<R, float>::value;   // FP32: positions relative to the tile's first cell
    const int64_t nc = d.nc;
    const int64_t t = order.block();
    if (t >= d.g_tiles) return;
    const int T = blockDim.x;
    const int64_t i = t * T + threadIdx.x;
    const bool cell = i < nc;
    const int64_t ic = cell ? i : nc - 1;
    const int64_t h0 = d.g_off[t], w0 = d.gv_off[t];
    const int hn = int(d.g_off[t + 1] - h0), wn = int(d.gv_off[t + 1] - w0);
    const int self = d.g_self[t] + (cell ? int(threadIdx.x) : 0);
    const int64_t s = ic >> 6;
    const int64_t eb = d.ge_off[s];
    const int ew = int(d.ge_off[s + 1] - eb) >> 6;        // groups of 8 edge-only neighbours
    const uint4* __restrict__ ep = d.ge_idx + eb + (ic & 63);

    constexpr int HB = 4;
    int he[HB];
#pragma unroll
    for (int j = 0; j < HB; ++j) {
        const int h = j * T + threadIdx.x;
        he[j] = d.g_idx[h0 + (h < hn ? h : 0)];
    }
    int wv = d.gv_idx[w0 + (int(threadIdx.x) < wn ? int(threadIdx.x) : 0)];
    const uint4 cl = d.g_cell[ic];
    uint4 e0 = ew > 0 ? ep[0] : make_uint4(0, 0, 0, 0), e1 = ew > 1 ? ep[64] : make_uint4(0, 0, 0, 0);
    const double4* __restrict__ P = d.xyz4;
    const R* __restrict__ u = a.u;
    const double4 ref = rel ? P[t * T] : make_double4(0.0, 0.0, 0.0, 0.0);
    double4 hp[HB];
    R hu[HB];
#pragma unroll
    for (int j = 0; j < HB; ++j) {
        hp[j] = P[he[j]];
        hu[j] = u[he[j]];
    }
    auto put_vertex = [&](int w, const double4& off, const double4& xv, const V4& mo) {
        va[w] = mk2(R(off.x), R(off.y));
        vb[w] = mk2(R(off.z), R(off.w));
        vc[w] = mk2(mo.x, mo.y);
        vd[w] = mk2(mo.z, mo.w);
        ve[w] = mk2(R(xv.x - ref.x), R(xv.y - ref.y));
        vf[w] = R(xv.z - ref.z);
    };
    {
        const double4 off = d.voff[wv], xv = d.vpos[wv];
        const V4 mo = a.vmom[wv];
#pragma unroll
        for (int j = 0; j < HB; ++j) {
            const int h = j * T + threadIdx.x;
            if (h < hn) {
                xy[h] = mk2(R(hp[j].x - ref.x), R(hp[j].y - ref.y));
                zu[h] = mk2(R(hp[j].z - ref.z), hu[j]);
            }
        }
        if (int(threadIdx.x) < wn) put_vertex(threadIdx.x, off, xv, mo);
    }
    const R* __restrict__ m = a.minv;
    const R m0 = m[ic], m1 = m[nc + ic], m2 = m[2 * nc + ic];
    const R m3 = m[3 * nc + ic], m4 = m[4 * nc + ic], m5 = m[5 * nc + ic];
    for (int h = HB * T + threadIdx.x; h < hn; h += T) {
        const int e = d.g_idx[h0 + h];
        const double4 p = P[e];
        xy[h] = mk2(R(p.x - ref.x), R(p.y - ref.y));
        zu[h] = mk2(R(p.z - ref.z), u[e]);
    }
    for (int w = T + threadIdx.x; w < wn; w += T) {
        wv = d.gv_idx[w0 + w];
        put_vertex(w, d.voff[wv], d.vpos[wv], a.vmom[wv]);
    }
    __syncthreads();
    if (!cell) return;

    const V2 sxy = xy[self], szu = zu[self];
    const R xi = sxy.x, yi = sxy.y, zi = szu.x, ui = szu.y;
    const uint32_t fl[2] = {cl.x, cl.y}, vl[2] = {cl.z, cl.w};
    R jx = R(0), jy = R(0), jz = R(0);
    R ox[4], oy[4], oz[4];                                // x_i - x_v, formed ahead of the sums that wait for them
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int l = int(vl[k >> 1] >> (16 * (k & 1))) & 0xffff;
        const V2 E = ve[l];
        ox[k] = xi - E.x;
        oy[k] = yi - E.y;
        oz[k] = zi - vf[l];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int l = int(vl[k >> 1] >> (16 * (k & 1))) & 0xffff;
        const V2 A = va[l], Bv = vb[l], C = vc[l], Dv = vd[l];
        const R nd = Bv.y * (Dv.y - ui);
        jx += C.x + (A.x - ox[k]) * nd;                   // xb - x_i
        jy += C.y + (A.y - oy[k]) * nd;
        jz += Dv.x + (Bv.x - oz[k]) * nd;
    }
    R umax = ui, umin = ui;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int l = int(fl[k >> 1] >> (16 * (k & 1))) & 0xffff;
        const V2 p = xy[l], z = zu[l];
        const R du2 = R(2) * (z.y - ui);
        jx -= (p.x - xi) * du2;
        jy -= (p.y - yi) * du2;
        jz -= (z.x - zi) * du2;
        umax = fmax(umax, z.y);
        umin = fmin(umin, z.y);
    }
    auto edges = [&](const uint4& g) {                    // 8 edge-only neighbours (padding = the cell: adds zeros)
        const uint32_t w[4] = {g.x, g.y, g.z, g.w};
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int l = int(w[k >> 1] >> (16 * (k & 1))) & 0xffff;
            const V2 p = xy[l], z = zu[l];
            const R du = z.y - ui;
            jx -= (p.x - xi) * du;
            jy -= (p.y - yi) * du;
            jz -= (z.x - zi) * du;
        }
    };
    if (ew > 0) edges(e0);
    if (ew > 1) edges(e1);
    for (int g = 2; g < ew; ++g) edges(ep[int64_t(g) * 64]);
    const R gx = m0 * jx + m1 * jy + m2 * jz;
    const R gy = m1 * jx + m3 * jy + m4 * jz;
    const R gz = m2 * jx + m4 * jy + m5 * jz;
    R psi = R(1), dl[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        dl[k] = (gx * ox[k] + gy * oy[k] + gz * oz[k]) * (R(1) / R(3));
        R ph = R(1);
        if (dl[k] > R(0)) ph = fmin(R(1), (umax - ui) / dl[k]);
        else if (dl[k] < R(0)) ph = fmin(R(1), (umin - ui) / dl[k]);
        psi = fmin(psi, ph);
    }
    // The step: the MUSCL value u + psi g.(x_f - x_i) at each of the cell's
    // face centroids (in c2f order), which the cell step reads for both sides
    // of a face.  With parts: the gradient and limiter arrays, which the face
    // kernel reads.
    if constexpr (!PARTS) {
        const R face[4] = {ui + psi * dl[0], ui + psi * dl[1], ui + psi * dl[2], ui + psi * dl[3]};
        store_quad(a.uf, nc, i, face);
    } else {
        a.grad[i] = gx;
        a.grad[nc + i] = gy;
        a.grad[2 * nc + i] = gz;
        a.psi[i] = psi;
    }
}

// One thread per face (the residual evaluation; it reads
// the gradient and limiter arrays).  Every load of the face goes out before
// its first branch (boundary faces read a valid dummy where they need no
// data); the arithmetic of each kind of face is unchanged by that.
template <class R>
__global__ __launch_bounds__(kBlock) void k_face_flux(Dev d, FvArrays<R> a, BcTable bc) {
    const int64_t f = gtid();
    if (f >= d.nf) return;
    const int64_t nc = d.nc, NX = d.nc + d.nb, nf = d.nf;
    const R* __restrict__ u = a.u;
    const bool bnd = f >= d.nfi;
    const int64_t g = bnd ? f - d.nfi : 0;
    const int kind = bnd ? bc.kind[d.gtag[g]] : kDirichlet;
    const R val = bnd ? bc_value<R>(bc, g) : R(0);
    const R area = bnd ? a.area[f] : R(0);            // used on Neumann faces only
    const int L = d.fL[f], Rc = d.fR[f];
    const R D = R(d.mesh_D[mesh_of(d, L)]);
    const R ph = a.phi[f];
    const R fxx = a.fx[f], fxy = a.fx[nf + f], fxz = a.fx[2 * nf + f];
    const R cAC = a.kAC[f], cBC = a.kBC[f], cRL = a.kRL[f];
    const int iA = d.fA[f], iB = d.fB[f], iC = d.fC[f];
    const R uL = u[L], uR = u[Rc];
    const R uA = a.unode[iA], uB = a.unode[iB], uC = a.unode[iC];
    const int up = ph >= R(0) ? L : Rc;
    const bool cellside = up < nc;          // MUSCL on a cell side; a ghost side is first order
    const int uc = cellside ? up : L;
    const R rx = fxx - a.xc[uc];
    const R ry = fxy - a.xc[NX + uc];
    const R rz = fxz - a.xc[2 * NX + uc];
    const R gr = a.grad[uc] * rx + a.grad[nc + uc] * ry + a.grad[2 * nc + uc] * rz;
    const R uupc = up == L ? uL : uR;
    const R uup = cellside ? uupc + a.psi[uc] * gr : uupc;
    const R diff = kind == kNeumann ? val * area : cAC * (uA - uC) + cBC * (uB - uC) + cRL * (uR - uL);
    a.flux[f] = kind == kZeroFlux ? R(0) : uup * ph - D * diff;
}

// ---- the step: face fluxes and update in one pass per cell ------------------
// The residual of cell i is -(1/vol_i) sum_k s_k F_k + src_i over its four
// faces, s_k = +1 where the cell is the face's L side.  On the interior
// faces the diffusive parts are regrouped per cell as in the matrix-free
// product: a face of a tetrahedron holds three of the cell's four vertices,
// so sum_k s_k (kAC (u_A - u_C) + kBC (u_B - u_C)) = sum_v w_v u_node[v], and
// s_k kRL (u_R - u_L) = kRL (u_n - u_i) with n the cell across face k.  The
// convective part is (s_k phi_f) times the upwind side's MUSCL value at the
// face centroid, which the gradient kernel stores per cell and face: value k
// of cell i on the cell's side, value j of cell n across (j = the face's slot
// among n's faces).  A face's vertex weights add up to zero, so the cell's
// fourth follows from the other three, sum_v w_v u_v = sum_{k<3} w_k (u_k - u_3),
// and its place holds the cell's volume.  Both cells of a face take the same
// upwind value, so its convective parts cancel exactly in the sum over cells.
// Boundary faces (the cell is always their L side) are evaluated as in
// k_face_flux.

// the tables: geometry only, built once per state
__global__ __launch_bounds__(kBlock) void k_fv_cell_setup(Dev d) {
    const int64_t i = gtid();
    if (i >= d.nc) return;
    const int64_t nc = d.nc;
    // the cell's vertices, k across from face k
    const uint4 cl = d.g_cell[i];
    const int32_t* __restrict__ tv = d.gv_idx + d.gv_off[i / d.g_rows];
    const int vid[4] = {tv[cl.z & 0xffff], tv[cl.z >> 16], tv[cl.w & 0xffff], tv[cl.w >> 16]};
    double w[4] = {0.0, 0.0, 0.0, 0.0}, r[4] = {0.0, 0.0, 0.0, 0.0};
    auto add = [&](int v, double c) {
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] += vid[q] == v ? c : 0.0;
    };
    uint32_t slots = 0;
    int across[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        across[k] = d.c2n[k * nc + i];
        const int code = d.c2f[k * nc + i];
        const int f = code >= 0 ? code : ~code;
        const double sg = code >= 0 ? 1.0 : -1.0;
        const bool in = f < d.nfi;
        const double on = in ? sg : 0.0;
        const double kac = d.kAC[f], kbc = d.kBC[f];
        add(d.fA[f], on * kac);
        add(d.fB[f], on * kbc);
        add(d.fC[f], on * (-(kac + kbc)));
        r[k] = in ? d.kRL[f] : 0.0;
        const int n = in ? d.c2n[k * nc + i] : int(i);
        uint32_t j = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int cn = d.c2f[q * nc + n];
            if ((cn >= 0 ? cn : ~cn) == f) j = uint32_t(q);
        }
        slots |= (in ? j : 0u) << (2 * k);
    }
    w[3] = d.vol[i];
    const float w32[4] = {float(w[0]), float(w[1]), float(w[2]), float(w[3])};
    const float r32[4] = {float(r[0]), float(r[1]), float(r[2]), float(r[3])};
    store_quad(d.cell_nb, nc, i, across);
    d.cell_cv[i] = make_uint2(cl.z, cl.w);
    store_quad(d.fvc_w, nc, i, w);
    store_quad(d.fvc_r, nc, i, r);
    store_quad(d.fvc_w32, nc, i, w32);
    store_quad(d.fvc_r32, nc, i, r32);
    d.fvc_slot[i] = uint8_t(slots);
}

// u_out[i] = u[i] + alpha dt Res(u_in)_i (u holds u^n; u_in and u_out are
// other buffers, or u_out = u on the last stage, whose cell i alone reads
// u[i]); then the ghosts behind the cell's boundary faces, from the new value.
//
// One block per gradient tile.  The kernel is bound by its gathers' line
// accesses (with one gather per neighbour, vertex and upwind face value they
// were nine tenths of them), so the tile's own values, which 85% of its cells'
// neighbours are, and the vertex values its cells touch (0.49 per cell instead
// of 4) go through LDS; a neighbour outside the tile is gathered, and lanes
// without one read their own cell's line.
template <class R>
__global__ __launch_bounds__(kBlock) void k_cell_step(Dev d, FvArrays<R> a, BcTable bc, const R* __restrict__ uin,
                                                      R* uout, double alpha, BlockOrder order) {
    extern __shared__ __align__(16) unsigned char sm_raw[];
    const int T = d.g_rows;
    R* const su = reinterpret_cast<R*>(sm_raw);            // [T] u
    R* const sf = su + T;                                  // [4][T] face values
    R* const sv = sf + 4 * T;                              // vertex values
    const int64_t nc = d.nc;
    const int64_t t = order.block();
    if (t >= d.g_tiles) return;
    const int64_t t0 = t * T, row = t0 + threadIdx.x;
    const bool cell = row < nc;
    const int64_t i = cell ? row : nc - 1;
    const int64_t w0 = d.gv_off[t];
    const int wn = int(d.gv_off[t + 1] - w0);
    const int m = mesh_of(d, i);
    // the cell's tables go out first (coalesced), then the gathers they address
    int wv = d.gv_idx[w0 + (int(threadIdx.x) < wn ? int(threadIdx.x) : 0)];
    int nb[4];
    R w[4], r[4], uo[4], po[4];
    const uint32_t sl = d.fvc_slot[i];
    const uint2 cv = d.cell_cv[i];                         // its vertices
    load_quad(d.cell_nb, nc, i, nb);
    load_quad(a.uf, nc, i, uo);
    const R ui = uin[i];
    load_quad(a.cphi, nc, i, po);                          // outward
    load_quad(a.cw, nc, i, w);
    load_quad(a.cr, nc, i, r);
    const R base = a.u[i], vol = w[3], src = a.src[i];
    const R D = R(d.mesh_D[m]), a_dt = R(alpha * d.mesh_dt[m]);
    const R wval = a.unode[wv];
    R un[4], ux[4], uv[4];
    int in_tile[4];                                        // the neighbour's place in the tile, or -1
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int64_t l = nb[k] - t0;
        in_tile[k] = l >= 0 && l < T && nb[k] < nc ? int(l) : -1;
        const bool far = in_tile[k] < 0;
        un[k] = uin[far ? int64_t(nb[k]) : i];             // a ghost's value behind a boundary face
        const bool across = far && nb[k] < nc && po[k] < R(0);
        ux[k] = quad_value(a.uf, nc, across ? int64_t(nb[k]) : i, across ? int((sl >> (2 * k)) & 3u) : 0);
    }
    su[threadIdx.x] = ui;
#pragma unroll
    for (int k = 0; k < 4; ++k) sf[k * T + threadIdx.x] = uo[k];
    if (int(threadIdx.x) < wn) sv[threadIdx.x] = wval;
    for (int v = T + threadIdx.x; v < wn; v += T) {
        wv = d.gv_idx[w0 + v];
        sv[v] = a.unode[wv];
    }
    __syncthreads();
    if (!cell) return;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int l = in_tile[k] < 0 ? int(threadIdx.x) : in_tile[k];
        const R u_l = su[l], f_l = sf[int((sl >> (2 * k)) & 3u) * T + l];
        if (in_tile[k] >= 0) {
            un[k] = u_l;
            ux[k] = f_l;
        }
    }
    uv[0] = sv[cv.x & 0xffff];
    uv[1] = sv[cv.x >> 16];
    uv[2] = sv[cv.y & 0xffff];
    uv[3] = sv[cv.y >> 16];
    R dif = R(0);
#pragma unroll
    for (int k = 0; k < 3; ++k) dif += w[k] * (uv[k] - uv[3]);
#pragma unroll
    for (int k = 0; k < 4; ++k) dif += r[k] * (un[k] - ui);
    R conv = R(0);
    bool bnd = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool in = nb[k] < nc;
        bnd = bnd || !in;
        conv += in ? po[k] * (po[k] >= R(0) ? uo[k] : ux[k]) : R(0);
    }
    R acc = conv - D * dif;
    if (bnd) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (nb[k] < nc) continue;
            const int64_t g = nb[k] - nc;              // the cell is the L side of its boundary faces
            const int64_t f = d.nfi + g;
            const int kind = bc.kind[d.gtag[g]];
            if (kind == kZeroFlux) continue;
            // upwind: the cell's MUSCL value, or the ghost's value (first order)
            const R uup = po[k] >= R(0) ? uo[k] : un[k];
            R diff;
            if (kind == kNeumann) {
                diff = bc_value<R>(bc, g) * a.area[f];
            } else {
                const R uA = a.unode[d.fA[f]], uB = a.unode[d.fB[f]], uC = a.unode[d.fC[f]];
                diff = a.kAC[f] * (uA - uC) + a.kBC[f] * (uB - uC) + a.kRL[f] * (un[k] - ui);
            }
            acc += uup * po[k] - D * diff;
        }
    }
    const R unew = base + a_dt * (-acc / vol + src);
    uout[i] = unew;
    if (bnd) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (nb[k] < nc) continue;
            const int64_t g = nb[k] - nc;
            const int kind = bc.kind[d.gtag[g]];
            const R val = bc_value<R>(bc, g);
            R ug;
            if (kind == kDirichlet) ug = R(2) * val - unew;
            else if (kind == kNeumann) ug = unew + val * a.gdist[g];
            else ug = unew;
            uout[nc + g] = ug;
        }
    }
}

// The residual, the gradient and the limiter in the caller's cell order (each
// unless null), one launch for the three: with one to reorder each, a residual
// evaluation of 48,000 cells took 89 us, now 50.
template <class R>
__global__ __launch_bounds__(kBlock) void k_residual_out(Dev d, FvArrays<R> a, double* res, double* grad, double* psi) {
    const int64_t i = gtid();
    if (i >= d.nc) return;
    const int64_t nc = d.nc, o = d.cell_perm[i];
    if (grad)
        for (int c = 0; c < 3; ++c) grad[c * nc + o] = double(a.grad[c * nc + i]);
    if (psi) psi[o] = double(a.psi[i]);
    if (!res) return;
    R acc = R(0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int c = d.c2f[k * nc + i];
        if (c >= 0) acc += a.flux[c];
        else acc -= a.flux[~c];
    }
    res[o] = double(-acc / a.vol[i] + a.src[i]);
}

// phi_f = 1/2 (V_L + V_R) . S_f  (V_L . S_f on the boundary), with an FP32 copy
__global__ __launch_bounds__(kBlock) void k_face_phi(Dev d) {
    const int64_t f = gtid();
    if (f >= d.nf) return;
    const int64_t nc = d.nc, nf = d.nf;
    const int L = d.fL[f];
    const int R = f < d.nfi ? d.fR[f] : L;
    const double vx = 0.5 * (d.vel[L] + d.vel[R]);
    const double vy = 0.5 * (d.vel[nc + L] + d.vel[nc + R]);
    const double vz = 0.5 * (d.vel[2 * nc + L] + d.vel[2 * nc + R]);
    const double ph = vx * d.S[f] + vy * d.S[nf + f] + vz * d.S[2 * nf + f];
    d.phi[f] = ph;
    d.phi32[f] = float(ph);
}

// the FP64 cell step's copy of phi: per cell and face, outward from the cell
__global__ __launch_bounds__(kBlock) void k_cell_phi(Dev d) {
    const int64_t i = gtid();
    if (i >= d.nc) return;
    const int64_t nc = d.nc;
    double po[4];
    float po32[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int code = d.c2f[k * nc + i];
        po[k] = code >= 0 ? d.phi[code] : -d.phi[~code];
        po32[k] = float(po[k]);
    }
    store_quad(d.fvc_phi, nc, i, po);
    store_quad(d.fvc_phi32, nc, i, po32);
}

// FP32 copies of the static geometry the FP32 kernels read
__global__ __launch_bounds__(kBlock) void k_make_fp32_geometry(Dev d, int64_t node_padded) {
    const int64_t i = gtid();
    const int64_t nc = d.nc, nf = d.nf, NX = d.nc + d.nb;
    if (i < nc) {
        d.vol32[i] = float(d.vol[i]);
        for (int k = 0; k < 6; ++k) d.minv32[k * nc + i] = float(d.minv[k * nc + i]);
    }
    if (i < NX)
        for (int k = 0; k < 3; ++k) d.xc32[k * NX + i] = float(d.xc[k * NX + i]);
    if (i < nf) {
        d.kAC32[i] = float(d.kAC[i]);
        d.kBC32[i] = float(d.kBC[i]);
        d.kRL32[i] = float(d.kRL[i]);
        d.area32[i] = float(d.area[i]);
        for (int k = 0; k < 3; ++k) d.fx32[k * nf + i] = float(d.fx[k * nf + i]);
    }
    if (i < d.nb) d.gdist32[i] = float(d.gdist[i]);
    if (i < node_padded) d.n_alpha32[i] = float(d.n_alpha[i]);
}

__global__ __launch_bounds__(kBlock) void k_cast_to_f32(int64_t n, const double* __restrict__ src, float* dst) {
    const int64_t i = gtid();
    if (i < n) dst[i] = float(src[i]);
}

__global__ __launch_bounds__(kBlock) void k_cast_to_f64(int64_t n, const float* __restrict__ src, double* dst) {
    const int64_t i = gtid();
    if (i < n) dst[i] = double(src[i]);
}

// caller order <-> internal order (perm: internal -> caller), converting
// the element type on the way (FP64 <-> FP32 rounds to nearest)
template <class Tin, class Tout>
__global__ __launch_bounds__(kBlock) void k_to_internal(const int32_t* __restrict__ perm, int64_t n,
                                                         int64_t sin, int64_t sout, int comps,
                                                         const Tin* __restrict__ src, Tout* dst) {
    const int64_t i = gtid();
    if (i >= n) return;
    const int64_t o = perm[i];
    for (int c = 0; c < comps; ++c) dst[c * sout + i] = Tout(src[c * sin + o]);
}

template <class Tin, class Tout>
__global__ __launch_bounds__(kBlock) void k_to_user(const int32_t* __restrict__ perm, int64_t n,
                                                     int64_t sin, int64_t sout, int comps,
                                                     const Tin* __restrict__ src, Tout* dst) {
    const int64_t i = gtid();
    if (i >= n) return;
    const int64_t o = perm[i];
    for (int c = 0; c < comps; ++c) dst[c * sout + o] = Tout(src[c * sin + i]);
}

// boundary values of variable var at every ghost whose face carries `tag`:
// the constant `value`, or vals[the caller's boundary triangle of the ghost]
__global__ __launch_bounds__(kBlock) void k_set_bc_values(Dev d, int var, int tag, double value,
                                                           const double* __restrict__ vals) {
    const int64_t g = gtid();
    if (g >= d.nb || d.gtag[g] != tag) return;
    const double v = vals ? vals[d.gbtri[g]] : value;
    d.gval[var * d.nb + g] = v;
    if (var == 0) d.gval32[g] = float(v);
}

// dt bound of mesh m: min_i mu_i / sum_{active faces} (|phi_f| + D_m kRL_f),
// per block (FP64)
__global__ __launch_bounds__(kBlock) void k_cfl(Dev d, BcTable bc, int m) {
    __shared__ double lds[4];
    const int64_t nc = d.nc;
    const double D = d.mesh_D[m];
    double best = __builtin_huge_val();
    for (int64_t i = d.mesh_start[m] + gtid(); i < d.mesh_start[m + 1]; i += int64_t(gridDim.x) * blockDim.x) {
        double rate = 0.0;
        for (int k = 0; k < 4; ++k) {
            int f = d.c2f[k * nc + i];
            f = f < 0 ? ~f : f;
            if (f >= d.nfi && bc.kind[d.gtag[f - d.nfi]] == kZeroFlux) continue;
            rate += fabs(d.phi[f]) + D * d.kRL[f];
        }
        best = fmin(best, d.vol[i] / rate);
    }
    best = block_min256(best, lds);
    if (threadIdx.x == 0) d.partial[blockIdx.x] = best;
}

// sum_i mu_i u_i over mesh m in FP64 (FP64 volumes, the state widened to FP64)
template <class R>
__global__ __launch_bounds__(kBlock) void k_conservation(Dev d, const R* __restrict__ u, int m) {
    __shared__ double lds[4];
    double s = 0.0;
    for (int64_t i = d.mesh_start[m] + gtid(); i < d.mesh_start[m + 1]; i += int64_t(gridDim.x) * blockDim.x)
        s += d.vol[i] * double(u[i]);
    s = block_sum256(s, lds);
    if (threadIdx.x == 0) d.partial[blockIdx.x] = s;
}

// one block: reduce n partials into mesh m's scal[slot] (op 0 = sum, 1 = min),
// and into the host's mirror of it (pinned memory, read once the stream has
// been waited for: no copy behind the kernel)
__global__ __launch_bounds__(1024) void k_finalize(Dev d, int64_t n, int m, int slot, int op, double* host) {
    __shared__ double lds[16];
    const double v = op == 0 ? reduce_partials_sum(d.partial, n, lds) : reduce_partials_min(d.partial, n, lds);
    if (threadIdx.x == 0) {
        msc(d, m)[slot] = v;
        if (host) host[int64_t(m) * SC_COUNT_ + slot] = v;
    }
}

// What a run of steps starts from: the time step each mesh's update uses (dt
// if dt > 0, else its CFL bound times cfl, stored by the last CFL evaluation),
// and the ghosts of u
template <class R>
__global__ __launch_bounds__(kBlock) void k_step_begin(Dev d, const R* __restrict__ gdist, BcTable bc, R* u, double dt,
                                                        double cfl) {
    const int64_t g = gtid();
    if (g < d.nm) d.mesh_dt[g] = dt > 0.0 ? dt : cfl * msc(d, int(g))[SC_DT_INV];
    if (g < d.nb) fill_ghost(g, d.nc, d.gowner, d.gtag, gdist, bc, u);
}

// ---- launchers ---------------------------------------------------------------
FvArrays<double> fv64(const Dev& d) {
    return {d.u, d.grad, d.psi, d.unode, d.flux, d.phi, d.minv, d.kAC, d.kBC, d.kRL, d.area,
            d.vol, d.src, d.fx, d.xc, d.gdist, d.uf, d.fvc_w, d.fvc_r, d.fvc_phi, d.vmom};
}

FvArrays<float> fv32(const Dev& d) {
    return {d.u32, d.grad32, d.psi32, d.unode32, d.flux32, d.phi32, d.minv32, d.kAC32, d.kBC32,
            d.kRL32, d.area32, d.vol32, d.src32, d.fx32, d.xc32, d.gdist32,
            d.uf32, d.fvc_w32, d.fvc_r32, d.fvc_phi32, d.vmom32};
}

template <class R>
hipError_t launch_ghost_fill_t(const Dev& d, const FvArrays<R>& a, const BcTable& bc, hipStream_t s) {
    if (d.nb == 0) return hipSuccess;
    hipLaunchKernelGGL(k_ghost_fill<R>, dim3(grid_for(d.nb)), dim3(kBlock), 0, s, d.nc, d.nb, d.gowner,
                       d.gtag, a.gdist, bc, a.u);
    return hipGetLastError();
}

hipError_t launch_ghost_fill(const Dev& d, bool fp32, const BcTable& bc, hipStream_t s) {
    return fp32 ? launch_ghost_fill_t(d, fv32(d), bc, s) : launch_ghost_fill_t(d, fv64(d), bc, s);
}

// the gradient tiles' LDS: the halo's two 2-vectors, the vertices' five and z
template <class R>
size_t grad_lds_bytes(const Dev& d) {
    return (size_t(2 * d.g_max + 5 * d.gv_max) * 2 + d.gv_max) * sizeof(R);
}

// the cell step's: five values per cell of a tile, one per vertex (at most 18 KB)
template <class R>
size_t step_lds_bytes(const Dev& d) {
    return size_t(5 * d.g_rows + d.gv_max) * sizeof(R);
}

template <class R, bool PARTS>
hipError_t allow_lds(const Dev& d) {
    const size_t lds = grad_lds_bytes<R>(d);
    if (lds <= 65536) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_grad_cells<R, PARTS>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
}

hipError_t setup_fv_kernels(const Dev& d) {
    hipError_t e = allow_lds<double, false>(d);
    if (e == hipSuccess) e = allow_lds<double, true>(d);
    if (e == hipSuccess) e = allow_lds<float, true>(d);
    if (e == hipSuccess) e = allow_lds<float, false>(d);
    return e;
}

template <class R>
FvArrays<R> with_u(FvArrays<R> a, const void* u_in) {
    if (u_in) a.u = const_cast<R*>(static_cast<const R*>(u_in));   // read only
    return a;
}

hipError_t launch_vertex_moments(const Dev& d, bool fp32, hipStream_t s, const void* u_in) {
    const BlockOrder o = stream_order(d.nv * 4, kBlock);
    const dim3 g(o.grid), b(kBlock);
    // By slices from 512 of them (two a CU); on fewer the barrier costs more
    // than the gathers save.  27k vertices, six steps: 455 us by slices, 449
    // direct; 55k, four steps: 452 and 457; 531k, two steps: 1,802 and 1,921 (FP32
    // 1,351 and 1,444).  Lists that name more than 64 KB of entities a slice
    // stay with the direct form.
    const size_t lds = size_t(d.nh_max) * (24 + (fp32 ? 4 : 8));
    if (d.nh_max > 0 && lds <= 65536 && d.nv >= 64 * 512) {
        if (fp32) hipLaunchKernelGGL(k_vertex_moments_tiles<float>, g, b, lds, s, d, with_u(fv32(d), u_in), o);
        else hipLaunchKernelGGL(k_vertex_moments_tiles<double>, g, b, lds, s, d, with_u(fv64(d), u_in), o);
        return hipGetLastError();
    }
    if (fp32) hipLaunchKernelGGL(k_vertex_moments<float>, g, b, 0, s, d, with_u(fv32(d), u_in), o);
    else hipLaunchKernelGGL(k_vertex_moments<double>, g, b, 0, s, d, with_u(fv64(d), u_in), o);
    return hipGetLastError();
}

template <class R>
void launch_grad_t(const Dev& d, const FvArrays<R>& a, bool parts, hipStream_t s) {
    const dim3 b(d.g_rows);
    const BlockOrder o = stream_order(d.g_tiles, 1);
    const dim3 gx(o.grid);
    if (parts)
        hipLaunchKernelGGL((k_grad_cells<R, true>), gx, b, grad_lds_bytes<R>(d), s, d, a, o);
    else
        hipLaunchKernelGGL((k_grad_cells<R, false>), gx, b, grad_lds_bytes<R>(d), s, d, a, o);
}

hipError_t launch_grad_limiter(const Dev& d, bool fp32, hipStream_t s, bool parts, const void* u_in) {
    if (fp32) launch_grad_t(d, with_u(fv32(d), u_in), parts, s);
    else launch_grad_t(d, with_u(fv64(d), u_in), parts, s);
    return hipGetLastError();
}
hipError_t launch_face_flux(const Dev& d, bool fp32, const BcTable& bc, hipStream_t s) {
    if (fp32)
        hipLaunchKernelGGL(k_face_flux<float>, dim3(grid_for(d.nf)), dim3(kBlock), 0, s, d, fv32(d), bc);
    else
        hipLaunchKernelGGL(k_face_flux<double>, dim3(grid_for(d.nf)), dim3(kBlock), 0, s, d, fv64(d), bc);
    return hipGetLastError();
}

hipError_t launch_cell_step(const Dev& d, bool fp32, const BcTable& bc, const void* u_in, void* u_out,
                            double alpha, hipStream_t s) {
    const BlockOrder o = stream_order(d.g_tiles, 1);
    const dim3 g(o.grid), b(d.g_rows);
    if (fp32)
        hipLaunchKernelGGL(k_cell_step<float>, g, b, step_lds_bytes<float>(d), s, d, fv32(d), bc,
                           static_cast<const float*>(u_in), static_cast<float*>(u_out), alpha, o);
    else
        hipLaunchKernelGGL(k_cell_step<double>, g, b, step_lds_bytes<double>(d), s, d, fv64(d), bc,
                           static_cast<const double*>(u_in), static_cast<double*>(u_out), alpha, o);
    return hipGetLastError();
}

hipError_t launch_fv_cell_setup(const Dev& d, hipStream_t s) {
    if (d.nc == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fv_cell_setup, dim3(grid_for(d.nc)), dim3(kBlock), 0, s, d);
    return hipGetLastError();
}

hipError_t launch_step_begin(const Dev& d, bool fp32, const BcTable& bc, double dt, double cfl, hipStream_t s) {
    const dim3 g(grid_for(d.nb > d.nm ? d.nb : d.nm)), b(kBlock);
    if (fp32) hipLaunchKernelGGL(k_step_begin<float>, g, b, 0, s, d, (const float*)d.gdist32, bc, d.u32, dt, cfl);
    else hipLaunchKernelGGL(k_step_begin<double>, g, b, 0, s, d, (const double*)d.gdist, bc, d.u, dt, cfl);
    return hipGetLastError();
}

hipError_t launch_residual_out(const Dev& d, bool fp32, double* res, double* grad, double* psi, hipStream_t s) {
    if (fp32)
        hipLaunchKernelGGL(k_residual_out<float>, dim3(grid_for(d.nc)), dim3(kBlock), 0, s, d, fv32(d), res, grad, psi);
    else
        hipLaunchKernelGGL(k_residual_out<double>, dim3(grid_for(d.nc)), dim3(kBlock), 0, s, d, fv64(d), res, grad, psi);
    return hipGetLastError();
}

hipError_t launch_face_phi(const Dev& d, hipStream_t s) {
    hipLaunchKernelGGL(k_face_phi, dim3(grid_for(d.nf)), dim3(kBlock), 0, s, d);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || d.nc == 0) return e;
    hipLaunchKernelGGL(k_cell_phi, dim3(grid_for(d.nc)), dim3(kBlock), 0, s, d);
    return hipGetLastError();
}

hipError_t launch_make_fp32_geometry(const Dev& d, int64_t node_padded, hipStream_t s) {
    int64_t n = d.nc + d.nb;
    if (d.nf > n) n = d.nf;
    if (node_padded > n) n = node_padded;
    hipLaunchKernelGGL(k_make_fp32_geometry, dim3(grid_for(n)), dim3(kBlock), 0, s, d, node_padded);
    return hipGetLastError();
}

hipError_t launch_cast_to_f32(int64_t n, const double* src, float* dst, hipStream_t s) {
    hipLaunchKernelGGL(k_cast_to_f32, dim3(grid_for(n)), dim3(kBlock), 0, s, n, src, dst);
    return hipGetLastError();
}

hipError_t launch_cast_to_f64(int64_t n, const float* src, double* dst, hipStream_t s) {
    hipLaunchKernelGGL(k_cast_to_f64, dim3(grid_for(n)), dim3(kBlock), 0, s, n, src, dst);
    return hipGetLastError();
}

template <class Tin, class Tout>
hipError_t to_internal_t(const int32_t* perm, int64_t n, int64_t sin, int64_t sout, int comps, const Tin* src,
                         Tout* dst, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL((k_to_internal<Tin, Tout>), dim3(grid_for(n)), dim3(kBlock), 0, s, perm, n, sin, sout,
                       comps, src, dst);
    return hipGetLastError();
}

template <class Tin, class Tout>
hipError_t to_user_t(const int32_t* perm, int64_t n, int64_t sin, int64_t sout, int comps, const Tin* src,
                     Tout* dst, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL((k_to_user<Tin, Tout>), dim3(grid_for(n)), dim3(kBlock), 0, s, perm, n, sin, sout, comps,
                       src, dst);
    return hipGetLastError();
}

hipError_t launch_to_internal(const int32_t* perm, int64_t n, int64_t sin, int64_t sout, int comps,
                              const double* src, double* dst, hipStream_t s) {
    return to_internal_t(perm, n, sin, sout, comps, src, dst, s);
}

hipError_t launch_to_user(const int32_t* perm, int64_t n, int64_t sin, int64_t sout, int comps,
                          const double* src, double* dst, hipStream_t s) {
    return to_user_t(perm, n, sin, sout, comps, src, dst, s);
}

hipError_t launch_to_internal_typed(const int32_t* perm, int64_t n, int comps, const void* src, bool src_f32,
                                    void* dst, bool dst_f32, hipStream_t s) {
    if (src_f32)
        return dst_f32 ? to_internal_t(perm, n, n, n, comps, (const float*)src, (float*)dst, s)
                       : to_internal_t(perm, n, n, n, comps, (const float*)src, (double*)dst, s);
    return dst_f32 ? to_internal_t(perm, n, n, n, comps, (const double*)src, (float*)dst, s)
                   : to_internal_t(perm, n, n, n, comps, (const double*)src, (double*)dst, s);
}

hipError_t launch_to_user_typed(const int32_t* perm, int64_t n, int comps, const void* src, bool src_f32,
                                void* dst, bool dst_f32, hipStream_t s) {
    if (src_f32)
        return dst_f32 ? to_user_t(perm, n, n, n, comps, (const float*)src, (float*)dst, s)
                       : to_user_t(perm, n, n, n, comps, (const float*)src, (double*)dst, s);
    return dst_f32 ? to_user_t(perm, n, n, n, comps, (const double*)src, (float*)dst, s)
                   : to_user_t(perm, n, n, n, comps, (const double*)src, (double*)dst, s);
}

hipError_t launch_set_bc_values(const Dev& d, int var, int tag, double value, const double* vals, hipStream_t s) {
    if (d.nb == 0) return hipSuccess;
    hipLaunchKernelGGL(k_set_bc_values, dim3(grid_for(d.nb)), dim3(kBlock), 0, s, d, var, tag, value, vals);
    return hipGetLastError();
}

// per mesh: one grid-stride reduction over the mesh's cells, then a finalize
static int blocks_for_range(int64_t n) {
    const int64_t b = (n + kBlock - 1) / kBlock;
    return int(b < 1024 ? (b < 1 ? 1 : b) : 1024);
}

hipError_t launch_cfl(const Dev& d, const Mesh& mh, const BcTable& bc, double* host, hipStream_t s) {
    for (int m = 0; m < d.nm; ++m) {
        const int nblk = blocks_for_range(mh.mesh_start[m + 1] - mh.mesh_start[m]);
        hipLaunchKernelGGL(k_cfl, dim3(nblk), dim3(kBlock), 0, s, d, bc, m);
        hipLaunchKernelGGL(k_finalize, dim3(1), dim3(1024), 0, s, d, int64_t(nblk), m, int(SC_DT_INV), 1, host);
    }
    return hipGetLastError();
}

hipError_t launch_conservation(const Dev& d, const Mesh& mh, bool fp32, double* host, hipStream_t s) {
    for (int m = 0; m < d.nm; ++m) {
        const int nblk = blocks_for_range(mh.mesh_start[m + 1] - mh.mesh_start[m]);
        if (fp32)
            hipLaunchKernelGGL(k_conservation<float>, dim3(nblk), dim3(kBlock), 0, s, d, (const float*)d.u32, m);
        else
            hipLaunchKernelGGL(k_conservation<double>, dim3(nblk), dim3(kBlock), 0, s, d, (const double*)d.u, m);
        hipLaunchKernelGGL(k_finalize, dim3(1), dim3(1024), 0, s, d, int64_t(nblk), m, int(SC_CONS), 0, host);
    }
    return hipGetLastError();
}

}  // namespace mifvm
