// ks_stedc.hip -- divide-and-conquer eigensolver of the real symmetric
// tridiagonal T = tridiag(e, d, e) (Cuppen's method with Gu-Eisenstat
// eigenvectors), the second half of the "diagonalize H'" step that the paper
// (Sec. 6) describes as dominated by matrix products.
//
// Tree: T is torn at the midpoints down to leaves of at most DC_LEAF rows; the
// tear at m uses T = diag(T1', T2') + |b| w w^T with b = e[m-1],
// w = e_{m-1} + sign(b) e_m and d[m-1], d[m] reduced by |b|.
// Leaves: implicit QL of their halves and a merge in LDS (one workgroup each).
// Merge of (D1, Q1), (D2, Q2) into D + rho z z^T, z = [Q1 row m-1;
// sign(b) Q2 row m] / sqrt(2), rho = 2|b|:
//   deflate  sort (D, z); drop |rho z_i| <= tol; rotate away z of nearly equal
//            pairs (tol = 8 eps max(|D|, rho |z|), so that it scales with T);
//   secular  one wavefront per root of 1 + rho sum z_i^2/(d_i - x) = 0, origin
//            at the nearer pole, safeguarded two-pole rational iteration with
//            bisection fallback;
//   vectors  z_hat from the computed roots (Gu-Eisenstat), u_j ~ z_hat/(d - x_j);
//   product  Q_new = Q_perm U on the matrix cores (grouped GEMM);
//   order    rank sort of the merged eigenvalues, columns permuted to match.
// Every size that depends on deflation stays on the device: kernels are
// launched for the undeflated size and idle workgroups exit, so the whole
// solve is enqueued without a host synchronisation.
// A batch of tridiagonals of one order shares the tree and every launch: the
// matrix index b is folded into the merge (group) index, G = b * nm + g, and
// selects the matrix's slices of the vectors (stride n) and matrices (n^2).
#include "ks_internal.hpp"
#include "ks_lanes.hpp"

namespace ks {

constexpr double DEPS = 1.1102230246251565e-16;  // unit roundoff 2^-53

// The slices of the merge work arrays that belong to matrix b of a batch
// (kk, nrot and rho are indexed by the folded group index instead).
__device__ inline DcWork dc_slice(DcWork w, int b, int n) {
    long o = (long)b * n;
    w.ds += o;
    w.zs += o;
    w.perm += o;
    w.ndl += o;
    w.dfl += o;
    w.dfval += o;
    w.dnd += o;
    w.znd += o;
    w.rot_idx += 2 * o;
    w.rot_cs += 2 * o;
    w.orig += o;
    w.tau += o;
    w.zhat += o;
    w.cinv += o;
    w.fval += o;
    w.fsrc += o;
    w.gpos += o;
    return w;
}

// ---------------------------------------------------------------- small merges
// The deflation test of two consecutive kept entries (d_p, z_p), (d_j, z_j):
// the Givens rotation (c, s) with c = z_j / tau, s = -z_p / tau, tau =
// hypot(z_p, z_j), zeroes z_p; the pair deflates if the off-diagonal it
// leaves, (d_j - d_p) c s, is at most tol in magnitude.
__device__ inline bool deflate_pair(double dp, double zp, double dj, double zj, double tol, double* c = nullptr,
                                    double* s = nullptr, double* t = nullptr) {
    const double tau = hypot(zj, zp);
    const double cs = zj / tau, sn = -zp / tau;
    if (c) {
        *c = cs;
        *s = sn;
        *t = tau;
    }
    return fabs((dj - dp) * cs * sn) <= tol;
}

// 1/sqrt(x) and 1/x for normal x > 0 and x != 0: the hardware's estimate (23
// bits) and one step of the cubic iteration.
__device__ __forceinline__ double rsqrt_step(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

__device__ __forceinline__ double rcp_step(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

// The next iterate of a secular root from tau: the two-pole rational model with
// the poles next to the root (D1, D2 from the iterate; the last root has one),
// kept inside the bracket (blo, bhi), which is halved where the model fails or
// is taken to (bisect).
__device__ __forceinline__ double secular_step(double tau, double f, double rho, double dpsi, double dphi, double D1,
                                               double D2, bool last, double blo, double bhi, bool bisect) {
    double tn;
    if (!last) {
        const double S1 = D1 * D1 * dpsi, S2 = D2 * D2 * dphi;
        const double c = f - rho * (S1 / D1 + S2 / D2);
        const double a2 = c, a1 = -(c * (D1 + D2) + rho * (S1 + S2)), a0 = D1 * D2 * f;
        double eta;
        if (a2 == 0.0) {
            eta = -a0 / a1;
        } else {
            const double disc = fmax(0.0, a1 * a1 - 4.0 * a2 * a0);
            const double q = -0.5 * (a1 + copysign(sqrt(disc), a1));
            const double e1 = q / a2, e2 = (q != 0.0) ? a0 / q : e1;
            const bool in1 = (tau + e1 > blo) && (tau + e1 < bhi);
            const bool in2 = (tau + e2 > blo) && (tau + e2 < bhi);
            if (in1 && in2) eta = (fabs(e1) < fabs(e2)) ? e1 : e2;
            else if (in2) eta = e2;
            else eta = e1;
        }
        tn = tau + eta;
    } else {
        const double S1 = D1 * D1 * dpsi;
        const double c = f - rho * S1 / D1;
        tn = (c > 0.0) ? tau + D1 + rho * S1 / c : 0.5 * (blo + bhi);
    }
    if (!(tn > blo && tn < bhi) || bisect) tn = 0.5 * (blo + bhi);
    return tn;
}

// The power of two that brings the largest entry of a merge to at most 1.
__device__ __forceinline__ int merge_scale(double big) {
    int ex = 0;
    if (big > 0.0 && big <= 1.7976931348623157e308) (void)frexp(big, &ex);
    return max(ex, -1000);
}

// A merge of at most KM rows in LDS, by 8 KM threads.
template <int KM>
struct MergeLds {
    double Q[2][KM][KM + 1];  // the block, and U / the merged block
    double lam[KM], ds[KM], zs[KM], dnd[KM], znd[KM], dfval[KM], dor[KM], tau[KM], zhat[KM], val[KM];
    double rot_c[KM], rot_s[KM];
    int perm[KM], ndl[KM], dfl[KM], rk[KM], rot_p[KM], rot_j[KM];
    unsigned long long mask[2];
    double red[2][KM / 8];
    int any, K, nrot;
};

// Sum over groups of eight lanes.
__device__ __forceinline__ double sum_oct(double v) { return sum21(sum4(v)); }

// The ascending rank of entry i, value v, among x[0 .. n-1] (ties by index),
// by the eight lanes (sub) of a group.
template <int KM>
__device__ __forceinline__ int rank_oct(const double* x, int n, double v, int i, int sub) {
    int r = 0;
#pragma unroll
    for (int q0 = 0; q0 < KM; q0 += 8) {
        const int q = q0 + sub;
        const double u = x[q];
        r += q < n && (u < v || (u == v && q < i));
    }
    r += __builtin_amdgcn_update_dpp(0, r, DPP_HALF_MIRROR, 0xf, 0xf, true);
    r += __builtin_amdgcn_update_dpp(0, r, DPP_XOR2, 0xf, 0xf, true);
    return r + __builtin_amdgcn_update_dpp(0, r, DPP_XOR1, 0xf, 0xf, true);
}

// Merge the children [0, n1) and [n1, K0) (eigenvalues M.lam in any order,
// vectors in the diagonal blocks of M.Q[cur]) across the tear of strength b, by
// the steps of the kernels below: deflation, secular equation (eight lanes per
// root), Gu-Eisenstat vectors, product, ascending order.  The result is in
// M.lam and M.Q[cur ^ 1].  Ends with a barrier; the whole workgroup calls it.
template <int KM>
__device__ inline void merge_lds(MergeLds<KM>& M, int cur, int K0, int n1, double b, int* info, int max_iter) {
    constexpr int NT = 8 * KM;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    double(*Q)[KM + 1] = M.Q[cur];
    double(*U)[KM + 1] = M.Q[cur ^ 1];
    const double sg = b >= 0.0 ? 1.0 : -1.0;
    double rho = 2.0 * fabs(b);
    if (t < K0) M.perm[t] = t;
    if (t == 0) M.any = 0;
    __syncthreads();
    // eight lanes per entry: (D, z) in ascending order of D
    const int jr = t >> 3, sub = t & 7;
    {
        double D = 0.0, z = 0.0;
        if (jr < K0) {
            D = M.lam[jr];
            z = 0.70710678118654752440 * (jr < n1 ? Q[n1 - 1][jr] : sg * Q[n1][jr]);
        }
        const int r = rank_oct<KM>(M.lam, K0, D, jr, sub);
        if (jr < K0 && sub == 0) {
            M.ds[r] = D;
            M.zs[r] = z;
            M.perm[r] = jr;
        }
        const double mxd = wave_max(fabs(D)), mxz = wave_max(fabs(z));
        if (lane == 0) {
            M.red[0][wave] = mxd;
            M.red[1][wave] = mxz;
        }
    }
    __syncthreads();
    double tol = 0.0, mz = 0.0;
#pragma unroll
    for (int q = 0; q < NT / 64; ++q) {
        tol = fmax(tol, M.red[0][q]);
        mz = fmax(mz, M.red[1][q]);
    }
    const int ex = merge_scale(fmax(tol, rho));
    const double sc = ldexp(1.0, -ex);
    rho *= sc;
    tol = 8.0 * DEPS * fmax(sc * tol, rho * mz);
    bool keep = false;
    double dj = 0.0, zj = 0.0;
    if (t < K0) {
        dj = sc * M.ds[t];
        M.ds[t] = dj;
        zj = M.zs[t];
        keep = !(rho * fabs(zj) <= tol);
    }
    if (t < 128) {
        const unsigned long long mk = __ballot(keep);
        if (lane == 0) M.mask[wave] = mk;
    }
    __syncthreads();
    const unsigned long long m0 = M.mask[0], m1 = K0 > 64 ? M.mask[1] : 0;
    const unsigned long long below = (1ULL << lane) - 1;
    const unsigned long long b0 = wave == 0 ? m0 & below : m0, b1 = wave == 0 ? 0 : m1 & below;
    if (keep) {
        const int prev = b1 ? 127 - __clzll(b1) : b0 ? 63 - __clzll(b0) : -1;
        if (prev >= 0 && deflate_pair(M.ds[prev], M.zs[prev], dj, zj, tol)) M.any = 1;
    }
    __syncthreads();
    if (!M.any) {
        const int nk = __popcll(b0) + __popcll(b1);
        if (t < K0) {
            if (keep) {
                M.ndl[nk] = M.perm[t];
                M.dnd[nk] = dj;
                M.znd[nk] = zj;
            } else {
                M.dfl[t - nk] = M.perm[t];
                M.dfval[t - nk] = dj;
            }
        }
        if (t == 0) {
            M.K = __popcll(m0) + __popcll(m1);
            M.nrot = 0;
        }
    } else if (t == 0) {  // the sequential scan of dc_deflate_kernel
        int K = 0, nd = 0, nrot = 0, pj = -1;
        double dp = 0.0, zp = 0.0;
        for (int q = 0; q < K0; ++q) {
            double dq = M.ds[q], zq = M.zs[q];
            const int c = M.perm[q];
            if (rho * fabs(zq) <= tol) {
                M.dfl[nd] = c;
                M.dfval[nd++] = dq;
                continue;
            }
            if (pj >= 0) {
                double cs, sn, tt;
                if (deflate_pair(dp, zp, dq, zq, tol, &cs, &sn, &tt)) {
                    M.rot_p[nrot] = pj;
                    M.rot_j[nrot] = c;
                    M.rot_c[nrot] = cs;
                    M.rot_s[nrot++] = sn;
                    M.dfl[nd] = pj;
                    M.dfval[nd++] = dp * cs * cs + dq * sn * sn;
                    dq = dp * sn * sn + dq * cs * cs;
                    zq = tt;
                } else {
                    M.ndl[K] = pj;
                    M.dnd[K] = dp;
                    M.znd[K++] = zp;
                }
            }
            pj = c;
            dp = dq;
            zp = zq;
        }
        if (pj >= 0) {
            M.ndl[K] = pj;
            M.dnd[K] = dp;
            M.znd[K++] = zp;
        }
        M.K = K;
        M.nrot = nrot;
    }
    __syncthreads();
    const int K = M.K, nrot = M.nrot;
    if (nrot > 0) {
        if (t < K0)
            for (int q = 0; q < nrot; ++q) {
                const int cp = M.rot_p[q], cj = M.rot_j[q];
                const double x = Q[t][cp], y = Q[t][cj];
                Q[t][cp] = M.rot_c[q] * x + M.rot_s[q] * y;
                Q[t][cj] = M.rot_c[q] * y - M.rot_s[q] * x;
            }
        __syncthreads();
    }
    // eight lanes per root; each keeps its entries i = sub + 8 q of the poles and
    // weights in registers
    constexpr int NI = KM / 8;
    const double* d = M.dnd;
    double dr[NI], zr[NI];
#pragma unroll
    for (int q = 0; q < NI; ++q) {
        const int i = sub + 8 * q;
        const double zi = i < K ? M.znd[i] : 0.0;
        dr[q] = i < K ? d[i] : 1e300;
        zr[q] = zi * zi;
    }
    if (jr < K) {  // root jr, as in dc_secular_kernel
        int o = 0;
        double tau = 0.0, dor = d[0];
        bool conv = K == 1;
        if (K == 1) {
            tau = rho * M.znd[0] * M.znd[0];
        } else {
            double blo, bhi, s = 0.0;
            const bool last = jr == K - 1;
            const double dj0 = d[jr], dj1 = d[last ? jr : jr + 1], gap = dj1 - dj0;
#pragma unroll
            for (int q = 0; q < NI; ++q) {
                if (8 * q >= K) break;
                s += last ? zr[q] : zr[q] * rcp_step((dr[q] - dj0) - 0.5 * gap);
            }
            s = sum_oct(s);
            if (last) {
                o = K - 1;
                blo = 0.0;
                bhi = rho * s;
            } else if (1.0 + rho * s >= 0.0) {
                o = jr;
                blo = 0.0;
                bhi = 0.5 * gap;
            } else {
                o = jr + 1;
                blo = -0.5 * gap;
                bhi = 0.0;
            }
            dor = o == jr ? dj0 : dj1;
            tau = 0.5 * (blo + bhi);
            if (!last) {  // from the middle of the gap, with the two poles' own weights
                const double h = 0.5 * gap, ih = 1.0 / (h * h), z0 = M.znd[jr], z1 = M.znd[jr + 1];
                tau = secular_step(o == jr ? h : -h, 1.0 + rho * s, rho, z0 * z0 * ih, z1 * z1 * ih, -h, h, false, blo,
                                   bhi, false);
            }
            for (int it = 0; it < max_iter; ++it) {
                double psi = 0.0, phi = 0.0, dpsi = 0.0, dphi = 0.0;
#pragma unroll
                for (int q = 0; q < NI; ++q) {
                    if (8 * q >= K) break;
                    const double rd = rcp_step((dr[q] - dor) - tau), tm = zr[q] * rd;
                    const bool lower = sub + 8 * q <= jr;
                    psi += lower ? tm : 0.0;
                    phi += lower ? 0.0 : tm;
                    const double dt = tm * rd;
                    dpsi += lower ? dt : 0.0;
                    dphi += lower ? 0.0 : dt;
                }
                psi = sum_oct(psi);
                phi = sum_oct(phi);
                dpsi = sum_oct(dpsi);
                dphi = sum_oct(dphi);
                const double f = 1.0 + rho * (psi + phi);
                // (every term of psi has one sign, every term of phi the other)
                const double err = 16.0 * DEPS * (1.0 + rho * (fabs(psi) + fabs(phi)) + fabs(tau) * rho * (dpsi + dphi));
                if (fabs(f) <= err) {
                    conv = true;
                    break;
                }
                if (f < 0.0) blo = tau;
                else bhi = tau;
                if (bhi - blo <= 2.0 * DEPS * fmax(fabs(blo), fabs(bhi))) {
                    conv = true;
                    break;
                }
                tau = secular_step(tau, f, rho, dpsi, dphi, (dj0 - dor) - tau, last ? 0.0 : (dj1 - dor) - tau, last, blo,
                                   bhi, it >= max_iter / 2);
            }
        }
        if (sub == 0) {
            if (!conv) set_info(info, KS_ERR_NO_CONVERGENCE, 2);
            M.dor[jr] = dor;
            M.tau[jr] = tau;
        }
    }
    __syncthreads();
    if (jr < K) {  // z_hat
        const double di = d[jr];
        double p = 1.0;
#pragma unroll
        for (int q = 0; q < NI; ++q) {
            if (8 * q >= K) break;
            const int j = sub + 8 * q, jc = min(j, K - 1);
            const double xj = (M.dor[jc] - di) + M.tau[jc];
            const double dk = d[min(j < jr ? j : j + 1, K - 1)] - di;
            const double fac = j < K - 1 || j < jr ? xj * rcp_step(dk) : xj;
            p *= j < K ? fac : 1.0;
        }
        p *= dpp_<DPP_HALF_MIRROR>(p);
        p *= dpp_<DPP_XOR2>(p);
        p *= dpp_<DPP_XOR1>(p);
        if (sub == 0) M.zhat[jr] = copysign(sqrt(fabs(p / rho)), M.znd[jr]);
    }
    __syncthreads();
    if (jr < K) {  // column jr of U
        const double dor = M.dor[jr], tj = M.tau[jr];
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < NI; ++q) {
            const int i = sub + 8 * q;
            zr[q] = i < K ? M.zhat[i] * rcp_step((dr[q] - dor) - tj) : 0.0;
            s = fma(zr[q], zr[q], s);
        }
        s = 1.0 / sqrt(sum_oct(s));
#pragma unroll
        for (int q = 0; q < NI; ++q) U[sub + 8 * q][jr] = zr[q] * s;
    }
    if (t < K0) M.val[t] = ldexp(t < K ? M.dor[t] + M.tau[t] : M.dfval[t - K], ex);
    // the product below takes inner entries up to the next multiple of four
    // (rows of U beyond K are zero)
    if (t < KM && t >= K) M.ndl[t] = 0;
    __syncthreads();
    // Q_new = Q[:, ndl] U on the matrix cores, TPW tiles of one row of 16 x 16
    // tiles per wavefront (as a register-tiled product of FMAs it was bound by
    // its LDS reads, 22000 clocks for 64 rows)
    constexpr int NTILE = KM / 16, TPW = NTILE * NTILE / (NT / 64);
    static_assert(NTILE % TPW == 0, "a wavefront's tiles are in one row");
    typedef double d4 __attribute__((ext_vector_type(4)));
    const int rt = wave * TPW / NTILE, ct = wave * TPW % NTILE;
    d4 acc[TPW];
#pragma unroll
    for (int x = 0; x < TPW; ++x) acc[x] = d4{0.0, 0.0, 0.0, 0.0};
    if (rt * 16 < K0 && ct * 16 < K) {
        const double* qr = Q[rt * 16 + (lane & 15)];
        for (int k = 0; k < K; k += 4) {
            const int kk = k + (lane >> 4);
            const double a = qr[M.ndl[kk]];
#pragma unroll
            for (int x = 0; x < TPW; ++x)
                acc[x] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, U[kk][(ct + x) * 16 + (lane & 15)], acc[x], 0, 0, 0);
        }
    }
    {  // ascending order
        const int r = rank_oct<KM>(M.val, K0, jr < K0 ? M.val[jr] : 0.0, jr, sub);
        if (jr < K0 && sub == 0) M.rk[jr] = r;
    }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < TPW; ++x) {
        const int j = (ct + x) * 16 + (lane & 15);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = rt * 16 + (lane >> 4) + 4 * r;
            if (i < K0 && j < K) U[i][M.rk[j]] = acc[x][r];
        }
    }
    for (int q = t; q < (K0 - K) * K0; q += NT) {
        const int c = q / K0, r = q % K0;
        U[r][M.rk[K + c]] = Q[r][M.dfl[c]];
    }
    if (t < K0) M.lam[M.rk[t]] = M.val[t];
    __syncthreads();
}

// ---------------------------------------------------------------- leaves
// Eigenvalues (lane i keeps the i-th, in no order) and vectors (columns off ..
// off + s - 1 of the same rows of Q, the identity on entry) of a symmetric
// tridiagonal of s <= 64 rows by one wavefront: implicit QL with Wilkinson's
// shift, the method of EISPACK's imtql2 (Dubrulle, Martin, Wilkinson, Numer.
// Math. 12, 1968).  Lane i holds d_i, e_i and row i of the vectors.
template <int LD>
__device__ inline double ql_wave(double d, double e, int s, double (*Q)[LD], int off, int* info, int max_sweeps) {
    const int lane = threadIdx.x & 63;
    const double big = wave_max(fmax(fabs(d), fabs(e)));
    const int ex = merge_scale(big);  // entries of at most 1: their squares stay in range
    d = ldexp(d, -ex);
    e = ldexp(e, -ex);
    double* row = &Q[off + min(lane, s - 1)][off];
    int l = 0, iter = 0;
    for (;;) {
        // the next block l .. m that is not yet split
        const double dn = __shfl(d, lane + 1, 64);
        const bool cut = lane >= s - 1 || fabs(e) <= DEPS * (fabs(d) + fabs(dn)) || fabs(e) <= 1e-18;
        const unsigned long long cuts = __ballot(cut);
        int m = l;
        while (l < s - 1) {
            m = __ffsll(cuts >> l) - 1 + l;
            if (m > l) break;
            ++l;
            iter = 0;
        }
        if (l >= s - 1) break;
        if (++iter > max_sweeps) {
            if (lane == 0) set_info(info, KS_ERR_NO_CONVERGENCE, 1);
            break;
        }
        const double dl = lane_get(d, l), el = lane_get(e, l), dm = lane_get(d, m);
        double g = (lane_get(d, l + 1) - dl) / (2.0 * el);
        g = dm - dl + el / (g + copysign(sqrt(fma(g, g, 1.0)), g));
        double si = 1.0, co = 1.0, p = 0.0, dnext = dm;
        double z1 = row[m];
        for (int i = m - 1; i >= l; --i) {
            const double di = lane_get(d, i), ei = lane_get(e, i), z0 = row[i];
            const double f = si * ei, b = co * ei;
            const double r2 = fma(g, g, f * f);
            const bool ok = r2 > 1e-290;  // else both vanish beside the block: any rotation will do
            const double ri = rsqrt_step(ok ? r2 : 1.0);
            co = ok ? g * ri : 1.0;
            si = ok ? f * ri : 0.0;
            const double h = dnext - p;
            const double r = fma(di - h, si, 2.0 * co * b);
            p = si * r;
            g = fma(co, r, -b);
            dnext = di;
            const bool me = lane == i + 1;
            d = me ? h + p : d;
            e = me ? (ok ? r2 * ri : 0.0) : e;
            row[i + 1] = fma(si, z0, co * z1);
            z1 = fma(co, z0, -si * z1);
        }
        row[l] = z1;
        d = lane == l ? dl - p : d;
        e = lane == l ? g : lane == m ? 0.0 : e;
    }
    return ldexp(d, ex);
}

// The leaves (size <= DC_LEAF), one workgroup each: the two halves by QL, one
// wavefront each, and their merge in LDS.  QL's cost is a chain of about
// 17 dependent operations per rotation and 27 s^2 / 32 rotations, so halving
// the leaf before it takes three quarters off.  Parallel Jacobi took 0.28 to
// 0.77 ms for the leaves of any order (four barriers a round), QL of whole
// leaves 0.11 to 0.23.  The tears are taken off the leaf's end entries here, and the
// leaf's rows of Z are cleared.
constexpr int QL_ROWS = DC_LEAF / 2;
__global__ __launch_bounds__(8 * DC_LEAF) void dc_leaf_kernel(int n, const int* leaf_lo, const int* leaf_hi,
                                                              const double* d, const double* e, double* lam, double* Z,
                                                              int* info, int max_sweeps, int max_iter) {
    constexpr int L = DC_LEAF, NT = 8 * L;
    __shared__ MergeLds<L> M;
    {
        const long o = (long)blockIdx.y * n;
        d += o;
        e += o;
        lam += o;
        Z += o * n;
    }
    const int lo = leaf_lo[blockIdx.x], hi = leaf_hi[blockIdx.x], s = hi - lo, t = threadIdx.x;
    const int n1 = s > QL_ROWS ? s / 2 : s;  // rows of the first half
    for (int q = t; q < L * L; q += NT) M.Q[0][q / L][q % L] = q / L == q % L ? 1.0 : 0.0;
    for (long q = t; q < (long)s * n; q += NT) Z[(long)lo * n + q] = 0.0;
    __syncthreads();
    const int h = t >> 6, i = t & 63, off = h == 0 ? 0 : n1, sh = h == 0 ? n1 : s - n1;
    if (h < 2 && sh > 0) {
        const int k = lo + off + i;
        double di = 0.0, ei = 0.0;
        if (i < sh) {
            di = d[k];
            if (i == 0 && k > 0) di -= fabs(e[k - 1]);
            if (i == sh - 1 && k + 1 < n) di -= fabs(e[k]);
            if (i < sh - 1) ei = e[k];
        }
        const double v = ql_wave<L + 1>(di, ei, sh, M.Q[0], off, info, max_sweeps);
        if (i < sh) M.lam[off + i] = v;
    }
    __syncthreads();
    int cur = 0;
    if (n1 < s) {
        merge_lds<L>(M, 0, s, n1, e[lo + n1 - 1], info, max_iter);
        cur = 1;
        if (t < s) M.rk[t] = t;
    } else {  // stable ascending rank
        const int j = t >> 3, r = rank_oct<L>(M.lam, s, j < s ? M.lam[j] : 0.0, j, t & 7);
        if (j < s && (t & 7) == 0) M.rk[j] = r;
    }
    __syncthreads();
    if (t < s) lam[lo + M.rk[t]] = M.lam[t];
    for (int q = t; q < s * s; q += NT) {
        const int r = q / s, c = q % s;
        Z[(long)(lo + r) * n + lo + M.rk[c]] = M.Q[cur][r][c];
    }
}

// One level of merges of at most SMALL_MERGE rows, one workgroup each, in place
// in Z and lam: one launch in the place of the ten below, which take 80 to
// 95 us for any such level (launches and round trips through memory).
constexpr int SMALL_MERGE = 96;  // two blocks fill the LDS
__global__ __launch_bounds__(8 * SMALL_MERGE) void dc_small_merge_kernel(int n, int nm, const int* mlo, const int* mmid,
                                                                         const int* mhi, const double* e, double* lam,
                                                                         double* Z, int* info, int max_iter) {
    constexpr int KM = SMALL_MERGE, NT = 8 * KM;
    __shared__ MergeLds<KM> M;
    const int G = blockIdx.x, g = G % nm, bm = G / nm, t = threadIdx.x;
    const int lo = mlo[g], K0 = mhi[g] - lo, n1 = mmid[g] - lo;
    e += (long)bm * n;
    lam += (long)bm * n + lo;
    Z += (long)bm * n * n + (long)lo * n + lo;
    for (int q = t; q < K0 * K0; q += NT) M.Q[0][q / K0][q % K0] = Z[(long)(q / K0) * n + q % K0];
    if (t < K0) M.lam[t] = lam[t];
    const double b = e[lo + n1 - 1];
    __syncthreads();
    merge_lds<KM>(M, 0, K0, n1, b, info, max_iter);
    if (t < K0) lam[t] = M.lam[t];
    for (int q = t; q < K0 * K0; q += NT) Z[(long)(q / K0) * n + q % K0] = M.Q[1][q / K0][q % K0];
}

// ---------------------------------------------------------------- merges
// One workgroup per merge: form (D, z), merge-sort, deflate.  With use_lds the
// launch provides K0 doubles of dynamic LDS and the two sorted lists are
// staged there for the merge's binary searches.
constexpr int DEFLATE_LDS_MAX = 8192;  // 64 KB of dynamic LDS
__global__ __launch_bounds__(256) void dc_deflate_kernel(int n, int nm, const int* mlo, const int* mmid,
                                                         const int* mhi, const double* e,
                                                         const double* lam, const double* Z,
                                                         DcWork w, int use_lds) {
    __shared__ double sd[64], sz[64];
    extern __shared__ double slam[];
    const int G = blockIdx.x, g = G % nm, bm = G / nm;
    w = dc_slice(w, bm, n);
    e += (long)bm * n;
    lam += (long)bm * n;
    Z += (long)bm * n * n;
    int lo = mlo[g], mid = mmid[g], hi = mhi[g];
    int K0 = hi - lo, n1 = mid - lo;
    int t = threadIdx.x;
    double b = e[mid - 1];
    double rho = 2.0 * fabs(b);
    double sg = (b >= 0.0) ? 1.0 : -1.0;
    const double rs2 = 0.70710678118654752440;
    double dmax = 0.0, zmax = 0.0;
    if (use_lds) {
        for (int c = t; c < K0; c += blockDim.x) slam[c] = lam[lo + c];
        __syncthreads();
    }
    const double* L = use_lds ? (const double*)slam : lam + lo;  // L[q] = lam[lo + q]
    for (int c = t; c < K0; c += blockDim.x) {
        double D = L[c];
        double z = (c < n1) ? Z[(long)(mid - 1) * n + lo + c] : sg * Z[(long)mid * n + lo + c];
        z *= rs2;
        // rank in the merged order (ties: first list first)
        int rank;
        if (c < n1) {
            int a = 0, bb = K0 - n1;  // count of second-list entries < D
            while (a < bb) {
                int h = (a + bb) >> 1;
                if (L[n1 + h] < D) a = h + 1;
                else bb = h;
            }
            rank = c + a;
        } else {
            int a = 0, bb = n1;  // count of first-list entries <= D
            while (a < bb) {
                int h = (a + bb) >> 1;
                if (L[h] <= D) a = h + 1;
                else bb = h;
            }
            rank = (c - n1) + a;
        }
        w.perm[lo + rank] = c;
        w.ds[lo + rank] = D;
        w.zs[lo + rank] = z;
        dmax = fmax(dmax, fabs(D));
        zmax = fmax(zmax, fabs(z));
    }
    // block max (fixed order)
    dmax = wave_max(dmax);
    zmax = wave_max(zmax);
    __shared__ double mx[2][4];
    if ((t & 63) == 0) {
        mx[0][t >> 6] = dmax;
        mx[1][t >> 6] = zmax;
    }
    __threadfence_block();
    __syncthreads();
    double tol = rho;
    for (int i = 0; i < 4; ++i) tol = fmax(tol, mx[0][i]);
    // the merge works on 2^-ex (D, rho), at most 1: its products stay in range
    // whatever the scale of T (dc_rank_kernel scales the values back)
    const int ex = merge_scale(tol);
    const double sc = ldexp(1.0, -ex);
    rho *= sc;
    tol = 0.0;
    for (int i = 0; i < 4; ++i) tol = fmax(tol, fmax(sc * mx[0][i], rho * mx[1][i]));
    tol *= 8.0 * DEPS;
    // Deflation in merged order: entry j deflates if rho |z_j| <= tol, and two
    // consecutive kept entries are rotated together (the rotated one carrying
    // on) if the Givens rotation that zeroes the first one's z leaves an
    // off-diagonal |(d_j - d_p) c s| <= tol.  Without such a pair the outcome
    // is a stable partition into deflated and kept entries, which all threads
    // form at once from contiguous chunks; a merge with a pair takes the
    // sequential scan below (same tests, same arithmetic).
    {
        __shared__ int cnt_d[256], cnt_k[256], cnt_k1[256], last_k[256];
        __shared__ int any_pair;
        const int per = (K0 + (int)blockDim.x - 1) / (int)blockDim.x;
        const int c0 = min(K0, t * per), c1 = min(K0, c0 + per);
        int nd = 0, nk = 0, nk1 = 0, firstk = -1, lastk = -1;
        bool pair = false;
        double dp = 0.0, zp = 0.0;
        for (int j = c0; j < c1; ++j) {
            const double dj = sc * w.ds[lo + j], zj = w.zs[lo + j];
            if (rho * fabs(zj) <= tol) {
                ++nd;
                continue;
            }
            if (lastk >= 0 && deflate_pair(dp, zp, dj, zj, tol)) pair = true;
            if (firstk < 0) firstk = j;
            lastk = j;
            dp = dj;
            zp = zj;
            ++nk;
            nk1 += w.perm[lo + j] < n1;
        }
        cnt_d[t] = nd;
        cnt_k[t] = nk;
        cnt_k1[t] = nk1;
        last_k[t] = lastk;
        if (t == 0) any_pair = 0;
        __syncthreads();
        if (firstk >= 0) {
            // the pair across the chunk boundary: the last kept entry before
            int pk = -1;
            for (int q = t - 1; q >= 0 && pk < 0; --q) pk = last_k[q];
            if (pk >= 0 && deflate_pair(sc * w.ds[lo + pk], w.zs[lo + pk], sc * w.ds[lo + firstk], w.zs[lo + firstk],
                                        tol))
                pair = true;
        }
        if (pair) any_pair = 1;
        __syncthreads();
        if (!any_pair) {
            // without rotations every kept column belongs to one child: the
            // merge product takes them grouped by child (first child's first,
            // each group in secular order), which halves its flops
            int od = 0, ok = 0, ok1 = 0, K1 = 0;
            for (int q = 0; q < (int)blockDim.x; ++q) {
                if (q < t) {
                    od += cnt_d[q];
                    ok += cnt_k[q];
                    ok1 += cnt_k1[q];
                }
                K1 += cnt_k1[q];
            }
            for (int j = c0; j < c1; ++j) {
                const double dj = sc * w.ds[lo + j], zj = w.zs[lo + j];
                if (rho * fabs(zj) <= tol) {
                    w.dfl[lo + od] = j;
                    w.dfval[lo + od] = dj;
                    ++od;
                } else {
                    const bool first = w.perm[lo + j] < n1;
                    w.ndl[lo + ok] = j;
                    w.dnd[lo + ok] = dj;
                    w.znd[lo + ok] = zj;
                    w.gpos[lo + ok] = first ? ok1 : K1 + (ok - ok1);
                    ok1 += first;
                    ++ok;
                }
            }
            if (t == (int)blockDim.x - 1) {
                w.kk[G] = ok;
                w.kk1[G] = K1;
                w.nrot[G] = 0;
                w.rho[G] = rho;
                w.ex[G] = ex;
            }
            return;
        }
    }
    // sequential deflation scan, streamed through LDS in chunks of 64
    if (t < 64) {
        int K = 0, nd = 0, nrot = 0, pj = -1;
        double dpj = 0.0, zpj = 0.0;
        for (int base = 0; base < K0; base += 64) {
            int cnt = min(64, K0 - base);
            if (t < cnt) {
                sd[t] = sc * w.ds[lo + base + t];
                sz[t] = w.zs[lo + base + t];
            }
            __threadfence_block();
            if (t == 0) {
                for (int q = 0; q < cnt; ++q) {
                    int jj = base + q;
                    double dj = sd[q], zj = sz[q];
                    if (rho * fabs(zj) <= tol) {
                        w.dfl[lo + nd] = jj;
                        w.dfval[lo + nd] = dj;
                        ++nd;
                        continue;
                    }
                    if (pj < 0) {
                        pj = jj;
                        dpj = dj;
                        zpj = zj;
                        continue;
                    }
                    double cs, sn, tau;
                    if (deflate_pair(dpj, zpj, dj, zj, tol, &cs, &sn, &tau)) {
                        w.rot_idx[2 * (lo + nrot)] = pj;
                        w.rot_idx[2 * (lo + nrot) + 1] = jj;
                        w.rot_cs[2 * (lo + nrot)] = cs;
                        w.rot_cs[2 * (lo + nrot) + 1] = sn;
                        ++nrot;
                        double tp = dpj * cs * cs + dj * sn * sn;
                        dj = dpj * sn * sn + dj * cs * cs;
                        w.dfl[lo + nd] = pj;
                        w.dfval[lo + nd] = tp;
                        ++nd;
                        pj = jj;
                        dpj = dj;
                        zpj = tau;
                    } else {
                        w.ndl[lo + K] = pj;
                        w.dnd[lo + K] = dpj;
                        w.znd[lo + K] = zpj;
                        ++K;
                        pj = jj;
                        dpj = dj;
                        zpj = zj;
                    }
                }
            }
            __threadfence_block();
        }
        if (t == 0) {
            if (pj >= 0) {
                w.ndl[lo + K] = pj;
                w.dnd[lo + K] = dpj;
                w.znd[lo + K] = zpj;
                ++K;
            }
            w.kk[G] = K;
            w.kk1[G] = -1;  // rotations may mix the children's columns
            w.nrot[G] = nrot;
            w.rho[G] = rho;
            w.ex[G] = ex;
        }
    }
}

// Apply the deflation rotations to the merge's columns of Z, one thread per row.
__global__ __launch_bounds__(256) void dc_rotate_kernel(int n, int nm, const int* mlo, const int* mhi,
                                                        DcWork w, double* Z) {
    const int G = blockIdx.y, g = G % nm, bm = G / nm;
    w = dc_slice(w, bm, n);
    Z += (long)bm * n * n;
    int lo = mlo[g], hi = mhi[g];
    int r = lo + blockIdx.x * blockDim.x + threadIdx.x;
    int nr = w.nrot[G];
    if (r >= hi || nr == 0) return;
    double* zr = Z + (long)r * n + lo;
    for (int q = 0; q < nr; ++q) {
        int pj = w.rot_idx[2 * (lo + q)], jj = w.rot_idx[2 * (lo + q) + 1];
        double c = w.rot_cs[2 * (lo + q)], s = w.rot_cs[2 * (lo + q) + 1];
        int cp = w.perm[lo + pj], cj = w.perm[lo + jj];
        double x = zr[cp], y = zr[cj];
        zr[cp] = c * x + s * y;
        zr[cj] = c * y - s * x;
    }
}

// Secular equation: one wavefront per root.
__global__ __launch_bounds__(256) void dc_secular_kernel(int n, int nm, const int* mlo, DcWork w, int* info,
                                                         int max_iter) {
    const int G = blockIdx.y, g = G % nm;
    w = dc_slice(w, G / nm, n);
    int lo = mlo[g];
    int K = w.kk[G];
    int jr = blockIdx.x * 4 + (threadIdx.x >> 6);
    int lane = threadIdx.x & 63;
    if (jr >= K) return;
    const double* d = w.dnd + lo;
    const double* z = w.znd + lo;
    double rho = w.rho[G];
    if (K == 1) {
        if (lane == 0) {
            w.orig[lo] = 0;
            w.tau[lo] = rho * z[0] * z[0];
        }
        return;
    }
    int o;
    double blo, bhi;
    if (jr < K - 1) {
        double D = d[jr + 1] - d[jr];
        double f = 0.0;
        for (int i = lane; i < K; i += 64) f += z[i] * z[i] / ((d[i] - d[jr]) - 0.5 * D);
        f = 1.0 + rho * wave_sum(f);
        if (f >= 0.0) {
            o = jr;
            blo = 0.0;
            bhi = 0.5 * D;
        } else {
            o = jr + 1;
            blo = -0.5 * D;
            bhi = 0.0;
        }
    } else {
        double zz = 0.0;
        for (int i = lane; i < K; i += 64) zz += z[i] * z[i];
        zz = wave_sum(zz);
        o = K - 1;
        blo = 0.0;
        bhi = rho * zz;
    }
    double dor = d[o];
    double tau = 0.5 * (blo + bhi);
    bool conv = false;
    for (int it = 0; it < max_iter; ++it) {
        double psi = 0.0, phi = 0.0, dpsi = 0.0, dphi = 0.0, eabs = 0.0;
        for (int i = lane; i < K; i += 64) {
            double del = (d[i] - dor) - tau;
            double tm = z[i] * z[i] / del;
            if (i <= jr) {
                psi += tm;
                dpsi += tm / del;
            } else {
                phi += tm;
                dphi += tm / del;
            }
            eabs += fabs(tm);
        }
        psi = wave_sum(psi);
        phi = wave_sum(phi);
        dpsi = wave_sum(dpsi);
        dphi = wave_sum(dphi);
        eabs = wave_sum(eabs);
        double f = 1.0 + rho * (psi + phi);
        double err = 16.0 * DEPS * (1.0 + rho * eabs + fabs(tau) * rho * (dpsi + dphi));
        if (fabs(f) <= err) {
            conv = true;
            break;
        }
        if (f < 0.0) blo = tau;
        else bhi = tau;
        if (bhi - blo <= 2.0 * DEPS * fmax(fabs(blo), fabs(bhi))) {
            conv = true;
            break;
        }
        // (the last root's one pole is d[K-1] = dor)
        const bool last = jr == K - 1;
        tau = secular_step(tau, f, rho, dpsi, dphi, last ? -tau : (d[jr] - dor) - tau,
                           last ? 0.0 : (d[jr + 1] - dor) - tau, last, blo, bhi, it >= max_iter / 2);
    }
    if (lane == 0) {
        if (!conv) set_info(info, KS_ERR_NO_CONVERGENCE, 2);
        w.orig[lo + jr] = o;
        w.tau[lo + jr] = tau;
    }
}

// Gu-Eisenstat: z_hat_i^2 = prod_j (x_j - d_i) / (rho prod_{j != i} (d_j - d_i)),
// paired so that every factor lies in (0, 1].
__global__ __launch_bounds__(256) void dc_zhat_kernel(int n, int nm, const int* mlo, DcWork w) {
    const int G = blockIdx.y, g = G % nm;
    w = dc_slice(w, G / nm, n);
    int lo = mlo[g];
    int K = w.kk[G];
    int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    int lane = threadIdx.x & 63;
    if (i >= K) return;
    const double* d = w.dnd + lo;
    double di = d[i];
    double p = 1.0;
    for (int j = lane; j < K; j += 64) {
        double xj = (d[w.orig[lo + j]] - di) + w.tau[lo + j];  // x_j - d_i
        if (j < i) p *= xj / (d[j] - di);
        else if (j < K - 1) p *= xj / (d[j + 1] - di);
        else p *= xj;
    }
    p = wave_prod(p);
    if (lane == 0) {
        double zh = sqrt(fabs(p / w.rho[G]));
        w.zhat[lo + i] = copysign(zh, w.znd[lo + i]);
    }
}

// 1/||u_j|| with u_ij = z_hat_i / (d_i - x_j).
__global__ __launch_bounds__(256) void dc_colnorm_kernel(int n, int nm, const int* mlo, DcWork w) {
    const int G = blockIdx.y, g = G % nm;
    w = dc_slice(w, G / nm, n);
    int lo = mlo[g];
    int K = w.kk[G];
    int jr = blockIdx.x * 4 + (threadIdx.x >> 6);
    int lane = threadIdx.x & 63;
    if (jr >= K) return;
    const double* d = w.dnd + lo;
    double dor = d[w.orig[lo + jr]], tj = w.tau[lo + jr];
    double s = 0.0;
    for (int i = lane; i < K; i += 64) {
        double u = w.zhat[lo + i] / ((d[i] - dor) - tj);
        s += u * u;
    }
    s = wave_sum(s);
    if (lane == 0) w.cinv[lo + jr] = 1.0 / sqrt(s);
}

// U block (K x K at (lo, lo), row stride n): U_ij = z_hat_i / (d_i - x_j) / ||u_j||.
__global__ __launch_bounds__(256) void dc_ugen_kernel(int n, int nm, const int* mlo, DcWork w, double* U) {
    const int G = blockIdx.z, g = G % nm, bm = G / nm;
    w = dc_slice(w, bm, n);
    U += (long)bm * n * n;
    int lo = mlo[g];
    int K = w.kk[G];
    int i = blockIdx.y;
    int jr = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= K || jr >= K) return;
    const double* d = w.dnd + lo;
    double u = w.zhat[lo + i] / ((d[i] - d[w.orig[lo + jr]]) - w.tau[lo + jr]);
    // row i of U pairs with column i of the gathered eigenvectors: both in the
    // child-grouped order when the merge has one
    const int gi = w.kk1[G] >= 0 ? w.gpos[lo + i] : i;
    U[(long)(lo + gi) * n + lo + jr] = u * w.cinv[lo + jr];
}

// Gather: Qp columns [0, K) = undeflated columns of Z in secular order, or in
// the child-grouped order gpos when the merge has one (kk1 >= 0); Z2 columns
// [K, K0) = deflated columns (both at the merge's block).
__global__ __launch_bounds__(256) void dc_gather_kernel(int n, int nm, const int* mlo, const int* mhi,
                                                        DcWork w, const double* Z, double* Qp, double* Z2) {
    const int G = blockIdx.z, g = G % nm, bm = G / nm;
    w = dc_slice(w, bm, n);
    const long o = (long)bm * n * n;
    Z += o;
    Qp += o;
    Z2 += o;
    int lo = mlo[g], hi = mhi[g];
    int K0 = hi - lo, K = w.kk[G];
    int r = lo + blockIdx.y;
    int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= hi || c >= K0) return;
    if (c < K) {
        int src = w.perm[lo + w.ndl[lo + c]];
        const int gc = w.kk1[G] >= 0 ? w.gpos[lo + c] : c;
        Qp[(long)r * n + lo + gc] = Z[(long)r * n + lo + src];
    } else {
        int src = w.perm[lo + w.dfl[lo + (c - K)]];
        Z2[(long)r * n + lo + c] = Z[(long)r * n + lo + src];
    }
}

// Final order: value of merged column c is x_c (c < K) or the deflated value;
// stable rank sort; lam[lo + rank] = value, src[lo + rank] = c.  The values
// every thread compares against pass through LDS in chunks, formed once per
// workgroup instead of gathered from memory by every thread.
constexpr int RANK_CHUNK = 2048;
__global__ __launch_bounds__(256) void dc_rank_kernel(int n, int nm, const int* mlo, const int* mhi, DcWork w) {
    __shared__ double sv[RANK_CHUNK];
    const int G = blockIdx.y, g = G % nm;
    w = dc_slice(w, G / nm, n);
    const int lo = mlo[g], hi = mhi[g];
    const int K0 = hi - lo, K = w.kk[G];
    if ((int)(blockIdx.x * blockDim.x) >= K0) return;  // the whole workgroup: no barrier is skipped
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    const bool act = c < K0;
    const double* d = w.dnd + lo;
    const int ex = w.ex[G];
    auto val = [&](int q) -> double {
        return ldexp((q < K) ? d[w.orig[lo + q]] + w.tau[lo + q] : w.dfval[lo + q - K], ex);
    };
    const double v = act ? val(c) : 0.0;
    int rk = 0;
    for (int q0 = 0; q0 < K0; q0 += RANK_CHUNK) {
        const int cnt = min(RANK_CHUNK, K0 - q0);
        __syncthreads();  // the previous chunk has been read
        for (int e = threadIdx.x; e < cnt; e += blockDim.x) sv[e] = val(q0 + e);
        __syncthreads();
        if (act)
            for (int e = 0; e < cnt; ++e) {
                const double u = sv[e];
                rk += (u < v) || (u == v && q0 + e < c);
            }
    }
    if (act) {
        w.fval[lo + rk] = v;
        w.fsrc[lo + rk] = c;
    }
}

__global__ __launch_bounds__(256) void dc_permute_kernel(int n, int nm, const int* mlo, const int* mhi,
                                                         DcWork w, const double* Z2, double* Z, double* lam) {
    const int G = blockIdx.z, g = G % nm, bm = G / nm;
    w = dc_slice(w, bm, n);
    const long o = (long)bm * n * n;
    Z2 += o;
    Z += o;
    lam += (long)bm * n;
    int lo = mlo[g], hi = mhi[g];
    int K0 = hi - lo;
    int r = lo + blockIdx.y;
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= hi || p >= K0) return;
    Z[(long)r * n + lo + p] = Z2[(long)r * n + lo + w.fsrc[lo + p]];
    if (r == lo) lam[lo + p] = w.fval[lo + p];
}

// Iteration caps of the leaf's QL sweeps (per eigenvalue) and of the secular-equation
// iterations.  A step that reaches its cap records KS_ERR_NO_CONVERGENCE and
// still finishes normally.  The defaults are far above what any input needs
// (quadratic convergence); a test hook lowers them to exercise that path.
namespace {
int g_leaf_sweeps = 40;
int g_secular_iters = 120;
}  // namespace

void stedc_set_caps(int leaf_sweeps, int secular_iters) {
    g_leaf_sweeps = leaf_sweeps > 0 ? leaf_sweeps : 40;
    g_secular_iters = secular_iters > 0 ? secular_iters : 120;
}

void stedc(hipStream_t s, const DcTree& tr, int batch, const double* d, const double* e, double* lam,
           double* Z, double* Z2, double* U, double* Qp, DcWork& w, int* info) {
    const int n = tr.n, B = batch;
    hipLaunchKernelGGL(dc_leaf_kernel, dim3(tr.nleaf, B), dim3(8 * DC_LEAF), 0, s, n, tr.d_leaf_lo, tr.d_leaf_hi, d,
                       e, lam, Z, info, g_leaf_sweeps, g_secular_iters);
    for (int l = tr.depth - 1; l >= 0; --l) {
        const int nm = 1 << l, NG = nm * B;
        const int off = nm - 1;
        const int* mlo = tr.d_mlo + off;
        const int* mmid = tr.d_mmid + off;
        const int* mhi = tr.d_mhi + off;
        const int mk = tr.max_k0[l];
        if (mk <= SMALL_MERGE) {
            hipLaunchKernelGGL(dc_small_merge_kernel, dim3(NG), dim3(8 * SMALL_MERGE), 0, s, n, nm, mlo, mmid, mhi, e,
                               lam, Z, info, g_secular_iters);
            continue;
        }
        const int dl = mk <= DEFLATE_LDS_MAX ? 1 : 0;
        hipLaunchKernelGGL(dc_deflate_kernel, dim3(NG), dim3(256), dl ? (size_t)mk * sizeof(double) : 0, s, n, nm,
                           mlo, mmid, mhi, e, lam, Z, w, dl);
        hipLaunchKernelGGL(dc_rotate_kernel, dim3(cdiv(mk, 256), NG), dim3(256), 0, s, n, nm, mlo, mhi, w, Z);
        hipLaunchKernelGGL(dc_secular_kernel, dim3(cdiv(mk, 4), NG), dim3(256), 0, s, n, nm, mlo, w, info,
                           g_secular_iters);
        hipLaunchKernelGGL(dc_zhat_kernel, dim3(cdiv(mk, 4), NG), dim3(256), 0, s, n, nm, mlo, w);
        hipLaunchKernelGGL(dc_colnorm_kernel, dim3(cdiv(mk, 4), NG), dim3(256), 0, s, n, nm, mlo, w);
        hipLaunchKernelGGL(dc_ugen_kernel, dim3(cdiv(mk, 256), mk, NG), dim3(256), 0, s, n, nm, mlo, w, U);
        hipLaunchKernelGGL(dc_gather_kernel, dim3(cdiv(mk, 256), mk, NG), dim3(256), 0, s, n, nm, mlo, mhi, w,
                           (const double*)Z, Qp, Z2);
        gemm_grouped_dc(s, nm, B, mk, mlo, mmid, mhi, w.kk, w.kk1, Qp, U, Z2, n);
        hipLaunchKernelGGL(dc_rank_kernel, dim3(cdiv(mk, 256), NG), dim3(256), 0, s, n, nm, mlo, mhi, w);
        hipLaunchKernelGGL(dc_permute_kernel, dim3(cdiv(mk, 256), mk, NG), dim3(256), 0, s, n, nm, mlo, mhi, w,
                           (const double*)Z2, Z, lam);
    }
}

// Host: the tear tree for order n (depth = smallest with ceil(n / 2^depth) <= leaf,
// leaf <= DC_LEAF).
void dc_tree_host(int n, int leaf, std::vector<int>& mlo, std::vector<int>& mmid, std::vector<int>& mhi,
                  std::vector<int>& leaf_lo, std::vector<int>& leaf_hi, int& depth,
                  std::vector<int>& max_k0) {
    leaf = std::max(2, std::min(leaf, DC_LEAF));
    depth = 0;
    while ((n + (1 << depth) - 1) / (1 << depth) > leaf) ++depth;
    // nodes level by level: level l has 2^l nodes, stored at offset 2^l - 1
    std::vector<int> lo{0}, hi{n};
    mlo.clear();
    mmid.clear();
    mhi.clear();
    max_k0.assign(depth > 0 ? depth : 1, 0);
    for (int l = 0; l < depth; ++l) {
        std::vector<int> nlo, nhi;
        for (size_t q = 0; q < lo.size(); ++q) {
            int a = lo[q], b = hi[q], m = a + (b - a) / 2;
            mlo.push_back(a);
            mmid.push_back(m);
            mhi.push_back(b);
            max_k0[l] = std::max(max_k0[l], b - a);
            nlo.push_back(a);
            nhi.push_back(m);
            nlo.push_back(m);
            nhi.push_back(b);
        }
        lo.swap(nlo);
        hi.swap(nhi);
    }
    leaf_lo = lo;
    leaf_hi = hi;
}

}  // namespace ks
