// Host setup of the aggregation multigrid hierarchy (strength, aggregates,
// Galerkin coarse matrices, dense coarsest inverse).
#include "amg.h"

#include <algorithm>
#include <cmath>

#include "mifvm.h"

namespace mifvm {
namespace {

constexpr int E_ARG = MIFVM_E_ARG;

// strong neighbours of every row, in column order, with |a_ij|: counted,
// then written, row-parallel
void strength(const AmgCsr& A, double theta, std::vector<int64_t>& sptr, std::vector<int32_t>& sidx,
              std::vector<double>& sval) {
    sptr.assign(A.n + 1, 0);
    const int nt = setup_threads(A.n);
    auto row_max = [&](int64_t i) {
        double mx = 0.0;
        for (int64_t e = A.ptr[i]; e < A.ptr[i + 1]; ++e)
            if (A.col[e] != i) mx = std::max(mx, std::fabs(A.val[e]));
        return mx;
    };
    auto strong = [&](int64_t i, int64_t e, double mx) {
        return mx > 0.0 && A.col[e] != i && std::fabs(A.val[e]) >= theta * mx;
    };
    for_chunks(A.n, nt, [&](int, int64_t lo, int64_t hi) {
        for (int64_t i = lo; i < hi; ++i) {
            const double mx = row_max(i);
            int64_t c = 0;
            for (int64_t e = A.ptr[i]; e < A.ptr[i + 1]; ++e) c += strong(i, e, mx) ? 1 : 0;
            sptr[i + 1] = c;
        }
    });
    for (int64_t i = 0; i < A.n; ++i) sptr[i + 1] += sptr[i];
    sidx.assign(sptr[A.n], 0);
    sval.assign(sptr[A.n], 0.0);
    for_chunks(A.n, nt, [&](int, int64_t lo, int64_t hi) {
        for (int64_t i = lo; i < hi; ++i) {
            const double mx = row_max(i);
            int64_t at = sptr[i];
            for (int64_t e = A.ptr[i]; e < A.ptr[i + 1]; ++e)
                if (strong(i, e, mx)) {
                    sidx[at] = A.col[e];
                    sval[at] = std::fabs(A.val[e]);
                    ++at;
                }
        }
    });
}

int64_t aggregate(const AmgCsr& A, const std::vector<int64_t>& sptr, const std::vector<int32_t>& sidx,
                  const std::vector<double>& sval, std::vector<int32_t>& agg) {
    const int64_t n = A.n;
    agg.assign(n, -1);
    int64_t na = 0;
    // pass 1: a row whose strong neighbours are all free seeds an aggregate
    for (int64_t i = 0; i < n; ++i) {
        if (agg[i] >= 0) continue;
        bool free = true;
        for (int64_t e = sptr[i]; e < sptr[i + 1] && free; ++e) free = agg[sidx[e]] < 0;
        if (!free) continue;
        agg[i] = int32_t(na);
        for (int64_t e = sptr[i]; e < sptr[i + 1]; ++e) agg[sidx[e]] = int32_t(na);
        ++na;
    }
    // pass 2: join the aggregate of the strongest aggregated strong neighbour
    std::vector<int32_t> agg1 = agg;      // the aggregates of pass 1 only
    for (int64_t i = 0; i < n; ++i) {
        if (agg1[i] >= 0) continue;
        double best = -1.0;
        int32_t pick = -1;
        for (int64_t e = sptr[i]; e < sptr[i + 1]; ++e) {
            const int32_t j = sidx[e];
            if (agg1[j] < 0) continue;
            const double w = sval[e];
            if (w > best || (w == best && j < pick)) {
                best = w;
                pick = j;
            }
        }
        if (pick >= 0) agg[i] = agg1[pick];
    }
    // pass 3: what is left seeds aggregates with its free strong neighbours
    for (int64_t i = 0; i < n; ++i) {
        if (agg[i] >= 0) continue;
        agg[i] = int32_t(na);
        for (int64_t e = sptr[i]; e < sptr[i + 1]; ++e)
            if (agg[sidx[e]] < 0) agg[sidx[e]] = int32_t(na);
        ++na;
    }
    return na;
}

// A_c = P^T A P: coarse row I sums the rows of its members, columns mapped
// to aggregates; columns sorted
void galerkin(const AmgCsr& A, const std::vector<int32_t>& agg, int64_t na, AmgCsr& C) {
    std::vector<int64_t> mptr(na + 1, 0);
    for (int64_t i = 0; i < A.n; ++i) mptr[agg[i] + 1]++;
    for (int64_t a = 0; a < na; ++a) mptr[a + 1] += mptr[a];
    std::vector<int32_t> mem(A.n);
    {
        std::vector<int64_t> pos(mptr.begin(), mptr.end() - 1);
        for (int64_t i = 0; i < A.n; ++i) mem[pos[agg[i]]++] = int32_t(i);
    }
    C.n = na;
    C.ptr.assign(na + 1, 0);
    // coarse rows in contiguous chunks, one per thread, each into its own
    // buffers; then the chunks are concatenated in row order
    const int nt = setup_threads(A.n);
    std::vector<std::vector<int32_t>> pcol(nt);
    std::vector<std::vector<double>> pval(nt);
    for_chunks(na, nt, [&](int k, int64_t lo, int64_t hi) {
        std::vector<int32_t> slot(na, -1);
        std::vector<int32_t> cols, order;
        std::vector<double> acc;
        for (int64_t I = lo; I < hi; ++I) {
            cols.clear();
            acc.clear();
            for (int64_t m = mptr[I]; m < mptr[I + 1]; ++m) {
                const int64_t i = mem[m];
                for (int64_t e = A.ptr[i]; e < A.ptr[i + 1]; ++e) {
                    const int32_t J = agg[A.col[e]];
                    if (slot[J] < 0) {
                        slot[J] = int32_t(cols.size());
                        cols.push_back(J);
                        acc.push_back(0.0);
                    }
                    acc[slot[J]] += A.val[e];
                }
            }
            order.resize(cols.size());
            for (size_t q = 0; q < order.size(); ++q) order[q] = int32_t(q);
            std::sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return cols[a] < cols[b]; });
            for (int32_t q : order) {
                pcol[k].push_back(cols[q]);
                pval[k].push_back(acc[q]);
            }
            for (int32_t J : cols) slot[J] = -1;
            C.ptr[I + 1] = int64_t(cols.size());
        }
    });
    for (int64_t I = 0; I < na; ++I) C.ptr[I + 1] += C.ptr[I];
    C.col.resize(C.ptr[na]);
    C.val.resize(C.ptr[na]);
    for_chunks(na, nt, [&](int k, int64_t lo, int64_t) {
        std::copy(pcol[k].begin(), pcol[k].end(), C.col.begin() + C.ptr[lo]);
        std::copy(pval[k].begin(), pval[k].end(), C.val.begin() + C.ptr[lo]);
    });
}

// dense inverse by LU with partial pivoting (row-major, n x n)
bool dense_inverse(const AmgCsr& A, std::vector<double>& inv) {
    const int64_t n = A.n;
    std::vector<double> M(n * n, 0.0);
    for (int64_t i = 0; i < n; ++i)
        for (int64_t e = A.ptr[i]; e < A.ptr[i + 1]; ++e) M[i * n + A.col[e]] += A.val[e];
    std::vector<int64_t> piv(n);
    for (int64_t k = 0; k < n; ++k) {
        int64_t p = k;
        for (int64_t r = k + 1; r < n; ++r)
            if (std::fabs(M[r * n + k]) > std::fabs(M[p * n + k])) p = r;
        if (!(std::fabs(M[p * n + k]) > 0.0)) return false;
        piv[k] = p;
        if (p != k)
            for (int64_t c = 0; c < n; ++c) std::swap(M[k * n + c], M[p * n + c]);
        const double d = M[k * n + k];
        for (int64_t r = k + 1; r < n; ++r) {
            const double l = M[r * n + k] / d;
            M[r * n + k] = l;
            if (l != 0.0)
                for (int64_t c = k + 1; c < n; ++c) M[r * n + c] -= l * M[k * n + c];
        }
    }
    inv.assign(n * n, 0.0);
    std::vector<double> x(n);
    for (int64_t c = 0; c < n; ++c) {           // column c of the inverse: solve A x = e_c
        std::fill(x.begin(), x.end(), 0.0);
        x[c] = 1.0;
        for (int64_t k = 0; k < n; ++k) std::swap(x[k], x[piv[k]]);
        for (int64_t r = 0; r < n; ++r)
            for (int64_t k = 0; k < r; ++k) x[r] -= M[r * n + k] * x[k];
        for (int64_t r = n - 1; r >= 0; --r) {
            for (int64_t k = r + 1; k < n; ++k) x[r] -= M[r * n + k] * x[k];
            x[r] /= M[r * n + r];
        }
        for (int64_t r = 0; r < n; ++r) inv[r * n + c] = x[r];
    }
    return true;
}

}  // namespace

int amg_build(AmgCsr&& A, double theta, int max_levels, int64_t coarse_max, double omega, AmgHierarchy& H,
              std::string& err) {
    if (!(theta >= 0.0 && theta <= 1.0) || max_levels < 1 || max_levels > kAmgMaxLevels || coarse_max < 1 ||
        coarse_max > 4096 || !(omega > 0.0 && omega < 2.0)) {
        err = "bad multigrid options";
        return E_ARG;
    }
    if (A.n < 1) {
        err = "empty matrix";
        return E_ARG;
    }
    H = AmgHierarchy{};
    H.theta = theta;
    H.omega = omega;
    H.max_levels = max_levels;
    H.coarse_max = coarse_max;
    H.lv.emplace_back();
    H.lv[0].A = std::move(A);
    for (;;) {
        AmgLevel& L = H.lv.back();
        if (L.A.n <= coarse_max) break;
        if ((int)H.lv.size() == max_levels) {
            err = "coarsest level above coarse_max: raise max_levels";
            return E_ARG;
        }
        std::vector<int64_t> sptr;
        std::vector<int32_t> sidx;
        std::vector<double> sval;
        strength(L.A, theta, sptr, sidx, sval);
        const int64_t na = aggregate(L.A, sptr, sidx, sval, L.agg);
        if (na * 10 > L.A.n * 9) {
            err = "aggregation stalled (coarse level above 90% of the fine one)";
            return E_ARG;
        }
        L.ncoarse = na;
        AmgLevel next;
        galerkin(L.A, L.agg, na, next.A);
        H.lv.push_back(std::move(next));
    }
    if (!dense_inverse(H.lv.back().A, H.cinv)) {
        err = "singular coarsest matrix";
        return E_ARG;
    }
    return 0;
}

void amg_pack(const AmgHierarchy& h, std::vector<AmgPacked>& out) {
    const int nl = int(h.lv.size());
    out.assign(nl, AmgPacked());
    std::vector<int32_t> inv;                             // the coarser level's rows, old -> new
    for (int l = nl - 1; l >= 0; --l) {
        const AmgLevel& L = h.lv[l];
        AmgPacked& P = out[l];
        const int64_t n = L.A.n;
        std::vector<int32_t> order(n);                    // new -> old
        if (l == nl - 1) {
            for (int64_t i = 0; i < n; ++i) order[i] = int32_t(i);
        } else {
            P.mptr.assign(L.ncoarse + 1, 0);
            for (int64_t i = 0; i < n; ++i) P.mptr[inv[L.agg[i]] + 1]++;
            for (int64_t k = 0; k < L.ncoarse; ++k) P.mptr[k + 1] += P.mptr[k];
            std::vector<int32_t> pos(P.mptr.begin(), P.mptr.end() - 1);
            for (int64_t i = 0; i < n; ++i) order[pos[inv[L.agg[i]]]++] = int32_t(i);
        }
        if (l == 0) {                                     // the state's cells keep their order
            P.midx = nl > 1 ? order : std::vector<int32_t>();
            break;
        }
        std::vector<int32_t> here(n);
        for (int64_t i = 0; i < n; ++i) here[order[i]] = int32_t(i);
        P.diag.assign(n, 0.0);
        std::vector<int32_t> len(n, 0);
        for (int64_t r = 0; r < n; ++r) {
            const int64_t i = order[r];
            for (int64_t e = L.A.ptr[i]; e < L.A.ptr[i + 1]; ++e) {
                if (L.A.col[e] == i) P.diag[r] += L.A.val[e];
                else len[r]++;
            }
        }
        if (l < nl - 1) {
            // blocks of whole aggregates with at most 64 rows (one slice), or
            // one larger aggregate over several slices
            P.bslice.push_back(0);
            P.bagg.push_back(0);
            for (int64_t a = 0; a < L.ncoarse;) {
                const int32_t r0 = P.mptr[a];
                int64_t to = a + 1;
                while (to < L.ncoarse && P.mptr[to + 1] - r0 <= 64) ++to;
                for (int32_t r = r0; r < P.mptr[to]; r += 64) P.srow.push_back(r);
                P.bslice.push_back(int32_t(P.srow.size()));
                P.bagg.push_back(int32_t(to));
                a = to;
            }
            P.srow.push_back(int32_t(n));
            const int64_t ns = int64_t(P.srow.size()) - 1;
            P.off.assign(ns + 1, 0);
            P.width.assign(ns, 0);
            for (int64_t q = 0; q < ns; ++q) {
                for (int32_t r = P.srow[q]; r < P.srow[q + 1]; ++r) P.width[q] = std::max(P.width[q], len[r]);
                P.off[q + 1] = P.off[q] + int64_t(P.width[q]) * 64;
            }
            P.idx.assign(P.off[ns], 0);
            P.val.assign(P.off[ns], 0.0);
            for_chunks(ns, setup_threads(n), [&](int, int64_t lo, int64_t hi) {
                for (int64_t q = lo; q < hi; ++q)
                    for (int64_t lane = 0; lane < 64; ++lane) {
                        const int64_t r = P.srow[q] + lane;
                        int64_t at = P.off[q] + lane, k = 0;
                        if (r < P.srow[q + 1]) {
                            const int64_t i = order[r];
                            for (int64_t e = L.A.ptr[i]; e < L.A.ptr[i + 1]; ++e) {
                                if (L.A.col[e] == i) continue;
                                P.idx[at] = here[L.A.col[e]];
                                P.val[at] = L.A.val[e];
                                at += 64;
                                ++k;
                            }
                        }
                        for (; k < P.width[q]; ++k, at += 64) P.idx[at] = P.srow[q];   // value 0
                    }
            });
        }
        inv.swap(here);
    }
}

}  // namespace mifvm
