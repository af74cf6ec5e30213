// ks_backtr.hip -- back-transform of the tridiagonal eigenvectors,
// C = (I (x) L)^-H Q Z (Part 2-5 / Part 3-6 of the paper's flows, with the
// Cholesky factor in place of the Loewdin V), and the density build with
// Fermi-Dirac occupations (Parts 3-4 of Sec. 3.1, Parts 4-5 of Sec. 3.2).
//
// Q = H_0 H_1 ... H_{n-2} is applied in blocks of BT reflectors in compact-WY
// form, H_b ... H_{b+BT-1} = I - V T V^H (T upper triangular, built once per
// set of reflectors from G = V^H V and tau), so each block is three MFMA GEMMs:
// W1 = V^H X, W2 = T W1 (T^H W1 for Q^H), X -= V W2.  A batch of matrices of one
// order shares every launch (GEMM batch index, or blockIdx.y / z selecting the
// matrix).
#include "ks_internal.hpp"
#include "ks_lanes.hpp"

namespace ks {

// X (n x ncols, ld ldx, type T) = Z[:, c0 : c0 + ncols] (real).
template <typename T>
__global__ void load_z_kernel(int n, int ncols, const double* Z, int c0, T* X, int ldx, long sX) {
    Z += (long)blockIdx.y * n * n;
    X += blockIdx.y * sX;
    long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (long)n * ncols) return;
    int r = (int)(e / ncols), c = (int)(e % ncols);
    X[(long)r * ldx + c] = from_re<T>(Z[(long)r * n + c0 + c]);
}

// The triangular factors of the BACKTR_SUB-reflector sub-blocks ("quarters"
// of a 256-reflector block) of every block at once (blockIdx.x = block x
// sub-blocks per block + sub-block, blockIdx.y = matrix): T_q solves
// (diag(1/tau) + striu(G_qq)) T_q = I for the quarter's reflectors.  Blocks of
// 16 reflectors by back substitution on the identity (column c by lane c, the
// unknowns in registers, each new one taken off the rows above at once), then
// neighbours joined by T_12 = -T_1 G_12 T_2, 16 to 32 to 64, in LDS.  (One lane per
// column of the whole quarter was a chain of 2016 multiply-adds: 50 us real, 130
// complex at orders 64 and 520, now 18 and 26.)  G_b (= V_b^H V_b) and T_b share storage (leading dimension BT): each quarter reads its
// diagonal block of G into LDS before writing T_q over it, and zeroes the blocks to its
// left (T_b is upper triangular); the blocks above the diagonal still hold
// V_p^H V_q for the coupling terms.
constexpr int TF_Q = BACKTR_SUB;
constexpr int TF_S = 16;  // reflectors per back substitution
template <typename T>
__global__ __launch_bounds__(256) void t_factors_kernel(int n, int B, const T* tau, T* Tall, long sT) {
    constexpr int H = TF_Q, S = TF_S, NT = 256;
    const int nq = B / H;
    const int b = blockIdx.x / nq, qd = blockIdx.x % nq, z = blockIdx.y, t = threadIdx.x;
    const int b0 = b * B, jb = min(B, n - 1 - b0), o = qd * H, jh = min(H, jb - o);
    if (jh <= 0) return;
    T* Tb = Tall + z * sT + (long)b * B * B;
    T* Th = Tb + (long)o * B + o;
    tau += (long)z * n + b0 + o;
    __shared__ T sg[H][H + 1];  // G above the diagonal, T on and above it as it is formed
    __shared__ T sy[H / 2][H / 2 + 1];
    __shared__ T st[H];
    // (entries beyond a ragged quarter: zero G and tau, so T's there are zero)
    for (int e = t; e < H * H; e += NT) {
        const int i = e / H, j = e % H;
        sg[i][j] = i < j && j < jh ? Th[(long)i * B + j] : zero_<T>();
    }
    if (t < H) st[t] = t < jh ? tau[t] : zero_<T>();
    for (int e = t; e < jh * o; e += NT) Tb[(long)(o + e / o) * B + e % o] = zero_<T>();  // left of the quarter
    __syncthreads();
    if (t < H) {
        const int s0 = t / S * S, c = t % S;
        T w[S];
#pragma unroll
        for (int i = 0; i < S; ++i) w[i] = i == c ? from_re<T>(1.0) : zero_<T>();
#pragma unroll
        for (int i = S - 1; i >= 0; --i) {
            w[i] = st[s0 + i] * w[i];
#pragma unroll
            for (int l = 0; l < i; ++l) w[l] -= sg[s0 + l][s0 + i] * w[i];
        }
#pragma unroll
        for (int i = 0; i < S; ++i)
            if (i <= c) sg[s0 + i][s0 + c] = w[i];
    }
    __syncthreads();
    for (int hb = S; hb < H; hb *= 2) {
        const int np = H / (2 * hb), tot = np * hb * hb;  // pairs, entries of their couplings
        // Y = G_12 T_2 (upper triangular T_2: inner entries up to the column), then -T_1 Y
        for (int e = t; e < tot; e += NT) {
            const int pr = e / (hb * hb), i = e / hb % hb, j = e % hb, r0 = pr * 2 * hb, c0 = r0 + hb;
            T y = zero_<T>();
            for (int l = 0; l <= j; ++l) y += sg[r0 + i][c0 + l] * sg[c0 + l][c0 + j];
            sy[pr * hb + i][j] = y;
        }
        __syncthreads();
        for (int e = t; e < tot; e += NT) {
            const int pr = e / (hb * hb), i = e / hb % hb, j = e % hb, r0 = pr * 2 * hb, c0 = r0 + hb;
            T y = zero_<T>();
            for (int l = i; l < hb; ++l) y -= sg[r0 + i][r0 + l] * sy[pr * hb + l][j];
            sg[r0 + i][c0 + j] = y;
        }
        __syncthreads();
    }
    for (int e = t; e < jh * jh; e += NT) Th[(long)(e / jh) * B + e % jh] = sg[e / jh][e % jh];
}

// The compact-WY factors T_b (jb x jb, row-major with leading dimension BT, at
// Tall + b BT^2 per matrix) of every block of BT reflectors.  The reflector
// matrix is zero above each block, so G_b = V_b^H V_b can run over all n rows:
// one split-K GEMM batched over the full blocks (a ragged last block takes its
// own).  One launch forms the triangular factors of the quarters of every
// block; then pairs of neighbouring factors are joined, quarters into halves
// and halves into the block, by the coupling T_12 = -T_1 (V_1^H V_2) T_2 (the
// product of two compact-WY forms), two batched GEMMs per pair position.
template <typename T>
void backtransform_prepare(hipStream_t s, int n, int batch, const T* Vall, const T* tau, BacktrWork<T>& w) {
    const int bt = w.bt;
    const int nref = n - 1;
    if (nref <= 0) return;
    const int nblk = cdiv(nref, bt), nfull = nref / bt;
    const long sV = (long)n * n, bb = (long)bt * bt;
    const int jl = nref - nfull * bt;  // order of a ragged last block (0 if none)
    // the launches take the full blocks of one matrix or one block of every
    // matrix, whichever are more
    const bool by_matrix = batch > nfull;
    const int nout = by_matrix ? nfull : batch, nin = by_matrix ? batch : nfull;
    const long so = by_matrix ? bb : w.sTall, si = by_matrix ? w.sTall : bb;
    // G_b is staged where T_b goes
    for (int q = 0; q < nout && nfull > 0; ++q) {
        const T* V = Vall + (by_matrix ? q * (long)bt : q * sV);
        const long sv = by_matrix ? sV : bt;
        gemm_splitk<T>(s, OP_C, OP_N, bt, bt, n, 1.0, V, n, V, n, 0.0, w.Tall + q * so, bt, w.P, w.pelems, nin, sv, sv,
                       si);
    }
    if (jl > 0) {
        const T* V = Vall + (long)nfull * bt;
        gemm_splitk<T>(s, OP_C, OP_N, jl, jl, n, 1.0, V, n, V, n, 0.0, w.Tall + nfull * bb, bt, w.P, w.pelems, batch, sV,
                       sV, w.sTall);
    }
    hipLaunchKernelGGL((t_factors_kernel<T>), dim3((bt / TF_Q) * nblk, batch), dim3(256), 0, s, n, bt, tau, w.Tall,
                       w.sTall);
    // join pairs: Y = G_12 T_2 (in W1), then T_12 = -T_1 Y over G_12
    for (int hb = TF_Q; hb < bt; hb *= 2) {
        for (int po = 0; po < bt; po += 2 * hb) {
            const long o1 = (long)po * bt + po, o12 = o1 + hb, o2 = o1 + (long)hb * bt + hb;
            for (int q = 0; q < nout && nfull > 0; ++q) {
                T* Tq = w.Tall + q * so;
                gemm<T>(s, OP_N, OP_N, hb, hb, hb, 1.0, Tq + o12, bt, si, Tq + o2, bt, si, 0.0, w.W1, hb,
                        (long)hb * hb, nin);
                gemm<T>(s, OP_N, OP_N, hb, hb, hb, -1.0, Tq + o1, bt, si, w.W1, hb, (long)hb * hb, 0.0, Tq + o12, bt,
                        si, nin);
            }
            const int h2 = std::min(hb, jl - po - hb);  // the ragged block's second factor of this pair
            if (h2 > 0) {
                T* Tq = w.Tall + nfull * bb;
                gemm<T>(s, OP_N, OP_N, hb, h2, h2, 1.0, Tq + o12, bt, w.sTall, Tq + o2, bt, w.sTall, 0.0, w.W1, h2,
                        (long)hb * h2, batch);
                gemm<T>(s, OP_N, OP_N, hb, h2, hb, -1.0, Tq + o1, bt, w.sTall, w.W1, h2, (long)hb * h2, 0.0, Tq + o12,
                        bt, w.sTall, batch);
            }
        }
    }
}

template <typename T>
void backtransform_q(hipStream_t s, int n, int batch, const T* Vall, int ncols, T* X, int ldx, long sX,
                     BacktrWork<T>& w, bool adjoint) {
    const int bt = w.bt;
    const int B = batch;
    const long sV = (long)n * n;
    int nref = n - 1;
    if (nref <= 0 || ncols <= 0) return;
    int nblk = cdiv(nref, bt);
    // complex rank updates by 128 reflectors gain from the large tiles where there are
    // enough of them (16 x 1300: 3.1 -> 2.6 ms): the threshold without tuning means 128
    // for them, any other is the caller's
    const int big = gemm_big_min_k();
    GemmPolicy pol(std::is_same<T, cplx>::value && big == GEMM_BIG_MIN_K ? 128 : big);
    // Q X applies the blocks last to first; Q^H X = (H_{n-2}^H ... H_0^H) X applies them first to last
    for (int q = 0; q < nblk; ++q) {
        const int b = adjoint ? q : nblk - 1 - q;
        int b0 = b * bt;
        int jb = min(bt, nref - b0);
        int m = n - b0 - 1;
        const T* Vb = Vall + (long)(b0 + 1) * n + b0;
        const T* Tb = w.Tall + (long)b * bt * bt;
        T* Xb = X + (long)(b0 + 1) * ldx;
        gemm_splitk<T>(s, OP_C, OP_N, jb, ncols, m, 1.0, Vb, n, Xb, ldx, 0.0, w.W1, ncols, w.P, w.pelems, B, sV,
                       sX, (long)jb * ncols);
        gemm<T>(s, adjoint ? OP_C : OP_N, OP_N, jb, ncols, jb, 1.0, Tb, bt, w.sTall, w.W1, ncols, (long)jb * ncols,
                0.0, w.W2, ncols, (long)jb * ncols, B);
        gemm<T>(s, OP_N, OP_N, m, ncols, jb, -1.0, Vb, n, sV, w.W2, ncols, (long)jb * ncols, 1.0, Xb, ldx, sX, B);
    }
}

template <typename T>
void load_z(hipStream_t s, int n, int batch, int ncols, const double* Z, int c0, T* X, int ldx, long sX) {
    long tot = (long)n * ncols;
    hipLaunchKernelGGL((load_z_kernel<T>), dim3(cdiv(tot, 256), batch), dim3(256), 0, s, n, ncols, Z, c0, X, ldx,
                       sX);
}

// ---------------------------------------------------------------- Fermi level
// 1 / (1 + e^x); 1 to half a unit in the last place below -40, and 0 beyond the
// smallest number, without an exponential.
__device__ inline double fermi_F(double x) {
    if (x < -40.0) return 1.0;
    if (x > 800.0) return 0.0;
    const double e = exp(-fabs(x));
    return (x > 0.0 ? e : 1.0) / (1.0 + e);
}
// The same for the electron count, where a state beyond `none` is nothing.
__device__ inline double fermi_count(double x, double none) {
    if (x > none) return 0.0;
    if (x < -40.0) return 1.0;
    const double e = exp(-fabs(x)), r = 1.0 / (1.0 + e);
    return x > 0.0 ? e * r : r;
}

// One workgroup: mu by bisection on sum_k w_k sum_i g F((eps_ik - mu)/kT) = ne over
// [min eps - 50 kT, max eps + 50 kT] until hi - lo <= 1e-14 max(1, |mu|) (at most
// 200 halvings), mu = midpoint; then occ, E_band and the window check.
// A halving is a chain of exponentials, a sum over the workgroup and a barrier,
// 1.5 us however few the eigenvalues.  The eigenvalues are therefore taken in
// chunks of 64, of which only those near the point are looked at: a chunk 40 kT below
// it is full, and one beyond `none` = 44 + ln(states / electrons) is empty (all
// such states together hold less than 1e-19 of the electrons asked for, however few
// these are).  A lane keeps what a wavefront has to know of one of its chunks.
// Few chunks: every wavefront has them all, and the sixteen count at the 15 inner points
// of four halvings at once; beyond, the wavefronts share the chunks of one count.
// (Against all eigenvalues at every halving: order 64 76 -> 21 us, 8 x 208
// 230 -> 97, 1300 106 -> 50, 16 x 1300 800 -> 158.  The line, whole density builds in us, all chunks in
// every wavefront against shared: orders 448 and 512 60.0, 61.5 and 62.7, 62.5; of a
// batch, whose k-points each have a chunk near the level, 3 and 5 of order 64 51.8, 57.4
// and 68.0, 64.2.)
constexpr int FERMI_CHUNKS = 64;                   // chunks in LDS
constexpr int FERMI_FEW = 7, FERMI_FEW_BATCH = 4;  // chunks in every wavefront
__global__ __launch_bounds__(1024) void fermi_kernel(int batch, int order, const double* eps,
                                                     KWeights kw, double g, double ne, double kT,
                                                     int il, int iu, double* occ, double* mu_out,
                                                     double* eband_out, int* kwin, int* info) {
    __shared__ double red[2][16];
    __shared__ double se[FERMI_CHUNKS * 64];
    __shared__ int lastw[16];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int per = (order + 63) / 64;  // chunks of a k-point
    const long nchunk = (long)batch * per;
    const bool few = nchunk <= (batch == 1 ? FERMI_FEW : FERMI_FEW_BATCH), lds = nchunk <= FERMI_CHUNKS, held = nchunk <= 16 * 64;
    // chunk c of the wavefront: c itself, or c * 16 + wave
    auto chunk_id = [&](long c) { return few ? c : c * 16 + wave; };
    double mn = INFINITY, mx = -INFINITY;
    double cmin = INFINITY, cmax = INFINITY, cw = 0.0;  // of chunk `lane`: an absent one is empty
    long cbase = 0;
    int cnum = 0;
    for (long c = 0; chunk_id(c) < nchunk; ++c) {
        const long id = chunk_id(c), bq = id / per, base = bq * order + (id % per) * 64;
        const int num = min(64, (int)((bq + 1) * order - base));
        const bool in = lane < num;
        const double e = in ? eps[base + lane] : 0.0;
        if (few ? wave == (int)(c & 15) : lds) se[id * 64 + lane] = in ? e : INFINITY;
        const double a = wave_min(in ? e : INFINITY), z = wave_max(in ? e : -INFINITY);
        const bool nan = __any(e != e);  // such a chunk is neither full nor empty
        mn = fmin(mn, a);
        mx = fmax(mx, z);
        if (lane == c) {
            cmin = nan ? -INFINITY : a;
            cmax = nan ? INFINITY : z;
            cw = g * kw.w[bq];
            cbase = lds ? id * 64 : base;
            cnum = num;
        }
    }
    if (lane == 0) {
        red[0][wave] = mn;
        red[1][wave] = mx;
    }
    __syncthreads();
    double lo = INFINITY, hi = -INFINITY;
    for (int i = 0; i < 16; ++i) {
        lo = fmin(lo, red[0][i]);
        hi = fmax(hi, red[1][i]);
    }
    lo -= 50.0 * kT;
    hi += 50.0 * kT;
    __syncthreads();
    const double ikT = 1.0 / fmax(kT, 0x1p-1022);
    double states = 0.0;
    for (int b = 0; b < batch; ++b) states += g * kw.w[b] * order;
    const double none = 44.0 + log(fmax(1.0, states / ne));
    const double* src = lds ? se : eps;
    // the wavefront's chunks' electrons at x, in every lane
    auto count = [&](double x) {
        double cnt = 0.0;
        if (held) {
            bool act = false;
            if ((cmax - x) * ikT < -40.0) cnt = cw * cnum;
            else act = !((cmin - x) * ikT > none);
            unsigned long long mask = __ballot(act && cnum > 0);
            while (mask) {
                const int l = __builtin_amdgcn_readfirstlane(__ffsll(mask) - 1);
                mask &= mask - 1;
                const long base = __builtin_amdgcn_readlane((int)cbase, l);
                const int num = __builtin_amdgcn_readlane(cnum, l);
                if (lane < num) cnt += lane_get(cw, l) * fermi_count((src[base + lane] - x) * ikT, none);
            }
        } else {
            for (int b = 0; b < batch; ++b) {
                double sb = 0.0;
                for (int i = t; i < order; i += 1024) sb += fermi_count((eps[(long)b * order + i] - x) * ikT, none);
                cnt += g * kw.w[b] * sb;
            }
        }
        return lane_sum(cnt);
    };
    for (int it = 0; it < (few ? 50 : 200); ++it) {
        const double mid = 0.5 * (lo + hi);
        if (hi - lo <= 1e-14 * fmax(1.0, fabs(mid))) break;
        double* rd = red[it & 1];
        // wavefront w of few chunks counts at lo + (w + 1) / 16 (hi - lo)
        const double cnt = count(few ? lo + 0.0625 * (wave + 1) * (hi - lo) : mid);
        if (lane == 0) rd[wave] = cnt;
        __syncthreads();
        if (few) {
            int p = 0;  // the path of four halvings among the points
#pragma unroll
            for (int s = 8; s > 0; s >>= 1)
                if (rd[p + s - 1] < ne) p += s;
            const double w = hi - lo, l0 = lo;
            lo = l0 + 0.0625 * p * w;
            hi = p < 15 ? l0 + 0.0625 * (p + 1) * w : hi;
        } else {
            double sum = 0.0;
#pragma unroll
            for (int i = 0; i < 16; ++i) sum += rd[i];
            if (sum < ne) lo = mid;
            else hi = mid;
        }
    }
    double mu = 0.5 * (lo + hi);
    double eb = 0.0;
    int last = -1;  // last window column (0-based within [il-1, iu-1]) with f > g 1e-15
    for (int b = 0; b < batch; ++b) {
        double sb = 0.0;
        for (int i = t; i < order; i += blockDim.x) {
            double ei = eps[(long)b * order + i];
            double f = g * fermi_F((ei - mu) / kT);
            occ[(long)b * order + i] = f;
            sb += f * ei;
            bool occd = f > g * 1e-15;
            if ((i < il - 1 || i > iu - 1) && occd) set_info(info, KS_ERR_WINDOW, i + 1);
            if (occd && i >= il - 1 && i <= iu - 1) last = max(last, i - (il - 1));
        }
        eb += kw.w[b] * sb;
    }
    __syncthreads();
    eb = block_sum(eb, red[0]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) last = max(last, __shfl_xor(last, o, 64));
    if ((t & 63) == 0) lastw[t >> 6] = last;
    __syncthreads();
    if (t == 0) {
        int lw = -1;
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) lw = max(lw, lastw[i]);
        *kwin = lw + 1;
        *mu_out = mu;
        *eband_out = eb;
    }
}

void fermi(hipStream_t s, int batch, int order, const double* eps, const KWeights& kw, double g,
           double ne, double kT, int il, int iu, double* occ, double* mu, double* eband, int* kwin,
           int* info) {
    hipLaunchKernelGGL(fermi_kernel, dim3(1), dim3(1024), 0, s, batch, order, eps, kw, g, ne, kT, il, iu,
                       occ, mu, eband, kwin, info);
}

#define KS_INST(T)                                                                                 \
    template void backtransform_q<T>(hipStream_t, int, int, const T*, int, T*, int, long,            \
                                     BacktrWork<T>&, bool);                                       \
    template void backtransform_prepare<T>(hipStream_t, int, int, const T*, const T*, BacktrWork<T>&); \
    template void load_z<T>(hipStream_t, int, int, int, const double*, int, T*, int, long);
KS_INST(double)
KS_INST(cplx)
KS_INST(float)
KS_INST(cplx32)
#undef KS_INST

}  // namespace ks
