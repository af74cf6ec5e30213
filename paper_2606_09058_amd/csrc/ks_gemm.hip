// ks_gemm.hip -- matrix-core (MFMA) GEMM for gfx950, real and complex, FP64
// and (for the mixed-precision path) FP32 with FP32 accumulation.
//
// Every dense contraction of the eigensolver goes through this kernel: the
// Cholesky trailing update, the triangular-solve updates of the reduction
// L^-1 H L^-H, the two-sided rank-2k trailing update of the Householder
// tridiagonalisation, the divide-and-conquer merge products, the compact-WY
// back-transform and the density C f C^H.
//
// Tile: 64 x 64 outputs per 256-thread workgroup, K step 16, staged through
// LDS with a register prefetch of the next K step.  Each of the 4 waves owns
// a 32 x 32 quadrant = 2 x 2 blocks of v_mfma_f64_16x16x4_f64.  Lane l of an
// MFMA supplies A[l%16][l/16] and B[l/16][l%16] of the 16x4 / 4x16 operands
// and receives D[l/16 + 4r][l%16] in accumulator register r.  The FP32 tile
// uses v_mfma_f32_16x16x4_f32 with the same operand layout; its lane l receives
// D[4 (l/16) + r][l%16].  A complex product uses four real MFMAs
// (re*re - im*im, re*im + im*re) into separate real and imaginary accumulators.
#include <algorithm>
#include <type_traits>

#include "ks_internal.hpp"

namespace ks {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int BM = 64, BN = 64, BK = 16, LPAD = 2;

__device__ inline d4 mfma(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ inline f4 mfma(float a, float b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Row (within a 16 x 16 block) of accumulator register r of a lane.
template <typename T>
__device__ inline int out_row(int lane, int r) {
    if constexpr (sizeof(T) == 8 && !is_cplx<T>::value) return (lane >> 4) + 4 * r;  // f64 MFMA
    else if constexpr (is_cplx<T>::value && sizeof(T) == 16) return (lane >> 4) + 4 * r;
    else return 4 * (lane >> 4) + r;  // f32 MFMA
}

template <typename T, int OP>
__device__ inline T ld_op(const T* p) {
    T v = *p;
    if constexpr (OP == OP_C) v = conj_(v);
    return v;
}

// Load the BM x BK tile of op(A) starting at (m0, k0) into registers.
// Mapping A: element (m, k) of op(A) is A[m*lda + k] for OP_N, A[k*lda + m]
// otherwise.  The four elements a thread loads are contiguous in memory.
template <typename T, int OPA>
__device__ inline void load_a(T (&r)[4], const T* A, int lda, int m, int K, int m0, int k0,
                              const double* ks) {
    int t = threadIdx.x;
    if constexpr (OPA == OP_N) {
        int mm = m0 + (t >> 2), kk = k0 + (t & 3) * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            bool ok = mm < m && kk + i < K;
            r[i] = ok ? ld_op<T, OPA>(A + (long)mm * lda + kk + i) : zero_<T>();
            if (ks && ok) r[i] = r[i] * ks[kk + i];  // (a narrowing multiply for FP32 types)
        }
    } else {
        int kk = k0 + (t >> 4), mm = m0 + (t & 15) * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            bool ok = mm + i < m && kk < K;
            r[i] = ok ? ld_op<T, OPA>(A + (long)kk * lda + mm + i) : zero_<T>();
            if (ks && ok) r[i] = r[i] * ks[kk];
        }
    }
}

template <typename T, int OPA>
__device__ inline void store_a(const T (&r)[4], T (*sA)[BM + LPAD]) {
    int t = threadIdx.x;
    if constexpr (OPA == OP_N) {
        int mm = t >> 2, kk = (t & 3) * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) sA[kk + i][mm] = r[i];
    } else {
        int kk = t >> 4, mm = (t & 15) * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) sA[kk][mm + i] = r[i];
    }
}

// op(B) is K x N: element (k, n) is B[k*ldb + n] for OP_N, B[n*ldb + k] otherwise.
template <typename T, int OPB>
__device__ inline void load_b(T (&r)[4], const T* B, int ldb, int n, int K, int n0, int k0) {
    int t = threadIdx.x;
    if constexpr (OPB == OP_N) {
        int kk = k0 + (t >> 4), nn = n0 + (t & 15) * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            bool ok = nn + i < n && kk < K;
            r[i] = ok ? B[(long)kk * ldb + nn + i] : zero_<T>();
        }
    } else {
        int nn = n0 + (t >> 2), kk = k0 + (t & 3) * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            bool ok = nn < n && kk + i < K;
            r[i] = ok ? ld_op<T, OPB>(B + (long)nn * ldb + kk + i) : zero_<T>();
        }
    }
}

template <typename T, int OPB>
__device__ inline void store_b(const T (&r)[4], T (*sB)[BN + LPAD]) {
    int t = threadIdx.x;
    if constexpr (OPB == OP_N) {
        int kk = t >> 4, nn = (t & 15) * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) sB[kk][nn + i] = r[i];
    } else {
        int nn = t >> 2, kk = (t & 3) * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) sB[kk + i][nn] = r[i];
    }
}

template <typename T>
struct Acc;
template <>
struct Acc<double> {
    d4 c[2][2];
};
// FP64 complex tiles take three real products per complex one (p1 = Re a Re b,
// p2 = Im a Im b, p3 = (Re a + Im a)(Re b + Im b); Re = p1 - p2,
// Im = p3 - p1 - p2), a quarter fewer MFMAs than the four-product form with
// the same normwise error bound.
template <>
struct Acc<cplx> {
    d4 p1[2][2], p2[2][2], p3[2][2];
};
template <>
struct Acc<float> {
    f4 c[2][2];
};
template <>
struct Acc<cplx32> {
    f4 re[2][2], im[2][2];
};

__device__ inline void acc_zero(Acc<double>& a) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) a.c[i][j] = d4{0.0, 0.0, 0.0, 0.0};
}
__device__ inline void acc_zero(Acc<cplx>& a) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            a.p1[i][j] = d4{0.0, 0.0, 0.0, 0.0};
            a.p2[i][j] = d4{0.0, 0.0, 0.0, 0.0};
            a.p3[i][j] = d4{0.0, 0.0, 0.0, 0.0};
        }
}

__device__ inline void acc_zero(Acc<float>& a) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) a.c[i][j] = f4{0.f, 0.f, 0.f, 0.f};
}
__device__ inline void acc_zero(Acc<cplx32>& a) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            a.re[i][j] = f4{0.f, 0.f, 0.f, 0.f};
            a.im[i][j] = f4{0.f, 0.f, 0.f, 0.f};
        }
}

// Real tile product (FP64 or FP32 MFMA, the same operand layout).
template <typename R, typename V>
__device__ inline void tile_mma_real(V (&c)[2][2], R (*sA)[BM + LPAD], R (*sB)[BN + LPAD]) {
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6, wm = w >> 1, wn = w & 1;
    int li = lane & 15, lk = lane >> 4;
#pragma unroll
    for (int ks = 0; ks < BK / 4; ++ks) {
        int kr = ks * 4 + lk;
        R a0 = sA[kr][wm * 32 + li], a1 = sA[kr][wm * 32 + 16 + li];
        R b0 = sB[kr][wn * 32 + li], b1 = sB[kr][wn * 32 + 16 + li];
        c[0][0] = mfma(a0, b0, c[0][0]);
        c[0][1] = mfma(a0, b1, c[0][1]);
        c[1][0] = mfma(a1, b0, c[1][0]);
        c[1][1] = mfma(a1, b1, c[1][1]);
    }
}

// Complex tile product: four real MFMAs per block.
template <typename C, typename V>
__device__ inline void tile_mma_cplx(V (&re)[2][2], V (&im)[2][2], C (*sA)[BM + LPAD], C (*sB)[BN + LPAD]) {
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6, wm = w >> 1, wn = w & 1;
    int li = lane & 15, lk = lane >> 4;
#pragma unroll
    for (int ks = 0; ks < BK / 4; ++ks) {
        int kr = ks * 4 + lk;
        C a[2] = {sA[kr][wm * 32 + li], sA[kr][wm * 32 + 16 + li]};
        C b[2] = {sB[kr][wn * 32 + li], sB[kr][wn * 32 + 16 + li]};
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                re[i][j] = mfma(a[i].x, b[j].x, re[i][j]);
                re[i][j] = mfma(-a[i].y, b[j].y, re[i][j]);
                im[i][j] = mfma(a[i].x, b[j].y, im[i][j]);
                im[i][j] = mfma(a[i].y, b[j].x, im[i][j]);
            }
    }
}

__device__ inline void tile_mma(Acc<float>& acc, float (*sA)[BM + LPAD], float (*sB)[BN + LPAD]) {
    tile_mma_real<float, f4>(acc.c, sA, sB);
}
__device__ inline void tile_mma(Acc<cplx32>& acc, cplx32 (*sA)[BM + LPAD], cplx32 (*sB)[BN + LPAD]) {
    tile_mma_cplx<cplx32, f4>(acc.re, acc.im, sA, sB);
}
__device__ inline float acc_get(const Acc<float>& a, int i, int j, int r) { return a.c[i][j][r]; }
__device__ inline cplx32 acc_get(const Acc<cplx32>& a, int i, int j, int r) {
    return mk32(a.re[i][j][r], a.im[i][j][r]);
}

__device__ inline void tile_mma(Acc<double>& acc, double (*sA)[BM + LPAD], double (*sB)[BN + LPAD]) {
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6, wm = w >> 1, wn = w & 1;
    int li = lane & 15, lk = lane >> 4;
#pragma unroll
    for (int ks = 0; ks < BK / 4; ++ks) {
        int kr = ks * 4 + lk;
        double a0 = sA[kr][wm * 32 + li], a1 = sA[kr][wm * 32 + 16 + li];
        double b0 = sB[kr][wn * 32 + li], b1 = sB[kr][wn * 32 + 16 + li];
        acc.c[0][0] = mfma(a0, b0, acc.c[0][0]);
        acc.c[0][1] = mfma(a0, b1, acc.c[0][1]);
        acc.c[1][0] = mfma(a1, b0, acc.c[1][0]);
        acc.c[1][1] = mfma(a1, b1, acc.c[1][1]);
    }
}

__device__ inline void tile_mma(Acc<cplx>& acc, cplx (*sA)[BM + LPAD], cplx (*sB)[BN + LPAD]) {
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6, wm = w >> 1, wn = w & 1;
    int li = lane & 15, lk = lane >> 4;
#pragma unroll 2
    for (int ks = 0; ks < BK / 4; ++ks) {
        int kr = ks * 4 + lk;
        cplx a[2] = {sA[kr][wm * 32 + li], sA[kr][wm * 32 + 16 + li]};
        cplx b[2] = {sB[kr][wn * 32 + li], sB[kr][wn * 32 + 16 + li]};
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                acc.p1[i][j] = mfma(a[i].x, b[j].x, acc.p1[i][j]);
                acc.p2[i][j] = mfma(a[i].y, b[j].y, acc.p2[i][j]);
                acc.p3[i][j] = mfma(a[i].x + a[i].y, b[j].x + b[j].y, acc.p3[i][j]);
            }
    }
}

__device__ inline double acc_get(const Acc<double>& a, int i, int j, int r) { return a.c[i][j][r]; }
__device__ inline cplx acc_get(const Acc<cplx>& a, int i, int j, int r) {
    const double p1 = a.p1[i][j][r], p2 = a.p2[i][j][r];
    return mk(p1 - p2, a.p3[i][j][r] - p1 - p2);
}

// One 64 x 64 output tile at (m0, n0).
template <typename T, int OPA, int OPB>
__device__ inline void gemm_tile(int m, int n, int K, double alpha, const T* A, int lda, const T* B,
                                 int ldb, double beta, T* C, int ldc, const double* kscale, int uplo,
                                 int m0, int n0, int klo = 0) {
    __shared__ T sA[BK][BM + LPAD];
    __shared__ T sB[BK][BN + LPAD];
    Acc<T> acc;
    acc_zero(acc);
    T ra[4], rb[4];
    if (K > klo) {
        load_a<T, OPA>(ra, A, lda, m, K, m0, klo, kscale);
        load_b<T, OPB>(rb, B, ldb, n, K, n0, klo);
    }
    for (int k0 = klo; k0 < K; k0 += BK) {
        __syncthreads();
        store_a<T, OPA>(ra, sA);
        store_b<T, OPB>(rb, sB);
        __syncthreads();
        if (k0 + BK < K) {
            load_a<T, OPA>(ra, A, lda, m, K, m0, k0 + BK, kscale);
            load_b<T, OPB>(rb, B, ldb, n, K, n0, k0 + BK);
        }
        tile_mma(acc, sA, sB);
    }
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6, wm = w >> 1, wn = w & 1;
    // with beta != 0 a row of blocks' C values are all requested before any is
    // written back (see the large-tile kernel); complex tiles read C in place,
    // which keeps their register budget
    const bool acc_c = beta != 0.0;
    constexpr bool pre = !is_cplx<T>::value;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        T cv[2][4];
        if (pre && acc_c) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = m0 + wm * 32 + i * 16 + out_row<T>(lane, r);
                    const int col = n0 + wn * 32 + j * 16 + (lane & 15);
                    const bool ok = row < m && col < n && in_uplo(uplo, row, col);
                    cv[j][r] = ok ? C[(long)row * ldc + col] : zero_<T>();
                }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                int row = m0 + wm * 32 + i * 16 + out_row<T>(lane, r);
                int col = n0 + wn * 32 + j * 16 + (lane & 15);
                if (row < m && col < n && in_uplo(uplo, row, col)) {
                    T v = alpha * acc_get(acc, i, j, r);
                    T* pc = C + (long)row * ldc + col;
                    if (acc_c) v += beta * (pre ? cv[j][r] : *pc);
                    *pc = v;
                }
            }
    }
}

template <typename T, int OPA, int OPB>
__global__ __launch_bounds__(256) void gemm_kernel(int m, int n, int K, double alpha, const T* A,
                                                   int lda, long sa, const T* B, int ldb, long sb,
                                                   double beta, T* C, int ldc, long sc,
                                                   const double* kscale, long sk, int uplo,
                                                   const int* kdev, int tri) {
    int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    if (!in_uplo(uplo, m0 + BM - 1, n0)) return;  // tile strictly above the diagonal
    long b = blockIdx.z;
    if (kdev) K = min(K, *kdev);  // inner size decided on the device (occupied window)
    // triangular operands: skip the K range where the operand is known to be zero
    int klo = 0;
    if (tri == TRI_A_LOWER) K = min(K, m0 + BM);
    if (tri == TRI_B_UPPER) K = min(K, n0 + BN);
    if (tri == TRI_A_UPPER) klo = (m0 / BK) * BK;
    if (tri == TRI_B_LOWER) klo = (n0 / BK) * BK;
    gemm_tile<T, OPA, OPB>(m, n, K, alpha, A + b * sa, lda, B + b * sb, ldb, beta, C + b * sc, ldc,
                           kscale ? kscale + b * sk : nullptr, uplo, m0, n0, klo);
}


// ---------------------------------------------------------------- large tiles
// Large tiles only where they pay: enough k steps to amortise the tile's
// prologue and epilogue, and enough tiles to keep two workgroups on every CU
// (measured: rank-64 updates and 6656 x 1414 x 6656 FP64 products run faster
// on 64 x 64 tiles).
constexpr long BIG_MIN_TILES = 512;
constexpr int BIG_MIN_K = 256;
// The smallest k for the large tiles, set per plan call (the autotuner's
// knob) on the calling thread: launches are enqueued by the thread that calls
// the entry point, so a plan's setting holds for exactly its own launches.
static thread_local int g_big_min_k = BIG_MIN_K;
void gemm_set_big_min_k(int k) { g_big_min_k = k; }
int gemm_big_min_k() { return g_big_min_k; }
static thread_local long g_big_launches = 0;
long gemm_big_launches() { return g_big_launches; }
// Output tiles of BM x BN (128 x 128; 64 x 64 for FP64 complex) with one
// wave tile of BM/2 x BN/2 per wavefront (2 x 2 wavefronts), so that each k
// step feeds (BM/32)(BN/32) MFMA blocks per wavefront per operand fragment
// pair: half the L2 traffic per flop of the 64 x 64 tile.  The LDS stages are
// double-buffered (one barrier per k step) and each thread prefetches its
// share of the next stage into registers while the current one is used.
template <typename T>
struct Big;
// accumulator vector of one 16 x 16 MFMA block, and a complex value from its parts
template <typename T>
struct AccVec {
    using type = d4;
};
template <>
struct AccVec<float> {
    using type = f4;
};
template <>
struct AccVec<cplx32> {
    using type = f4;
};
__device__ inline cplx from_parts(double re, double im, const cplx*) { return mk(re, im); }
__device__ inline cplx32 from_parts(float re, float im, const cplx32*) { return mk32(re, im); }
template <>
struct Big<double> {
    static constexpr int BM = 128, BN = 128, BK = 16;
};
template <>
struct Big<float> {
    static constexpr int BM = 128, BN = 128, BK = 32;
};
template <>
struct Big<cplx> {
    static constexpr int BM = 64, BN = 64, BK = 16;  // (two workgroups per CU fit in LDS)
};
template <>
struct Big<cplx32> {
    static constexpr int BM = 128, BN = 128, BK = 16;
};

// Which element of a block with rows of C a thread takes as its i-th of E, counted
// along the rows: FP64 element t + 256 i, so that neighbours load and, in the
// layout of the LDS tiles, write neighbours (with a run of elements per thread
// bank conflicts took 23 % of the time of a complex product: 71 -> 77 TFLOP/s at
// order 4992); FP32 a run (its larger tiles have no registers for E addresses).
template <typename T>
constexpr bool BIG_RUN = sizeof(T) == 4 || std::is_same<T, cplx32>::value;
template <typename T, int E>
__device__ inline int big_elem(int t, int i) {
    return BIG_RUN<T> ? t * E + i : t + 256 * i;
}
// Load an R x C block of memory (row stride ld, C contiguous) starting at
// (r0, c0), zero outside rows < nr and columns < nc.
template <typename T, int R, int C, int OP>
__device__ inline void big_load(T (&v)[R * C / 256], const T* P, int ld, int nr, int nc, int r0, int c0,
                                int t) {
    constexpr int E = R * C / 256;
    static_assert(E * 256 == R * C && C % E == 0 && (256 % C == 0 || C % 256 == 0), "block shape");
#pragma unroll
    for (int i = 0; i < E; ++i) {
        const int e = big_elem<T, E>(t, i);
        const int rr = r0 + (BIG_RUN<T> ? t / (C / E) : e / C), cc = c0 + (BIG_RUN<T> ? t % (C / E) * E + i : e % C);
        const bool ok = rr < nr && cc < nc;
        v[i] = ok ? ld_op<T, OP>(P + (long)rr * ld + cc) : zero_<T>();
    }
}

template <typename T, int OPA, int OPB>
__global__ __launch_bounds__(256, 2) void gemm_big_kernel(int m, int n, int K, double alpha, const T* A, int lda,
                                                       long sa, const T* B, int ldb, long sb, double beta, T* C,
                                                       int ldc, long sc, int uplo, const int* kdev, int tri) {
    constexpr int BM = Big<T>::BM, BN = Big<T>::BN, BKb = Big<T>::BK;
    constexpr int WM = BM / 2, WN = BN / 2, MI = WM / 16, NI = WN / 16;
    constexpr int EA = BM * BKb / 256, EB = BN * BKb / 256;
    constexpr int PAD = std::is_same<T, cplx>::value ? 1 : LPAD;  // 16 rows of a column in different banks
    __shared__ T sA[2][BKb][BM + PAD];
    __shared__ T sB[2][BKb][BN + PAD];
    int bx = blockIdx.x, by = blockIdx.y;
    if (uplo == UPLO_FULL && tri == TRI_NONE) {
        // Consecutive workgroups go to the eight dies in turn: each die gets a run of
        // tiles of its own, in bands of eight tile rows, so that its L2 serves the
        // rows and columns its tiles share.
        const int gx = gridDim.x, gy = gridDim.y, tot = gx * gy, per = tot / 8;
        int l = by * gx + bx;
        if (l < 8 * per) l = (l % 8) * per + l / 8;
        const int band = l / (8 * gx), r = min(8, gy - 8 * band), w = l - band * 8 * gx;
        by = 8 * band + w % r;
        bx = w / r;
    }
    const int m0 = by * BM, n0 = bx * BN;
    if (!in_uplo(uplo, m0 + BM - 1, n0)) return;  // tile strictly above the diagonal
    const long b = blockIdx.z;
    A += b * sa;
    B += b * sb;
    C += b * sc;
    if (kdev) K = min(K, *kdev);
    int klo = 0;
    if (tri == TRI_A_LOWER) K = min(K, m0 + BM);
    if (tri == TRI_B_UPPER) K = min(K, n0 + BN);
    if (tri == TRI_A_UPPER) klo = (m0 / BKb) * BKb;
    if (tri == TRI_B_LOWER) klo = (n0 / BKb) * BKb;
    const int t = threadIdx.x;
    T ra[EA], rb[EB];
    // op(A) tile BM x BK: A is m x K (OP_N) or K x m; op(B) tile BK x BN: B is K x n (OP_N) or n x K
    auto load = [&](int k0) {
        if constexpr (OPA == OP_N) big_load<T, BM, BKb, OPA>(ra, A, lda, m, K, m0, k0, t);
        else big_load<T, BKb, BM, OPA>(ra, A, lda, K, m, k0, m0, t);
        if constexpr (OPB == OP_N) big_load<T, BKb, BN, OPB>(rb, B, ldb, K, n, k0, n0, t);
        else big_load<T, BN, BKb, OPB>(rb, B, ldb, n, K, n0, k0, t);
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int i = 0; i < EA; ++i) {
            const int e = big_elem<T, EA>(t, i);
            if constexpr (OPA == OP_N) sA[buf][e % BKb][e / BKb] = ra[i];
            else sA[buf][e / BM][e % BM] = ra[i];
        }
#pragma unroll
        for (int i = 0; i < EB; ++i) {
            const int e = big_elem<T, EB>(t, i);
            if constexpr (OPB == OP_N) sB[buf][e / BN][e % BN] = rb[i];
            else sB[buf][e % BKb][e / BKb] = rb[i];
        }
    };
    const int lane = t & 63, w = t >> 6, wm = w >> 1, wn = w & 1;
    const int li = lane & 15, lk = lane >> 4;
    using V = typename AccVec<T>::type;
    // complex: cre, cim and c3 hold the three real products of Acc<cplx>
    constexpr int CX = is_cplx<T>::value ? 1 : 0;
    V cre[MI][NI], cim[CX ? MI : 1][CX ? NI : 1], c3[CX ? MI : 1][CX ? NI : 1];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            cre[i][j] = V{};
            if constexpr (CX) {
                cim[i][j] = V{};
                c3[i][j] = V{};
            }
        }
    if (K > klo) {
        load(klo);
        store(0);
    }
    __syncthreads();
    int cur = 0;
    for (int k0 = klo; k0 < K; k0 += BKb) {
        const bool more = k0 + BKb < K;
        if (more) load(k0 + BKb);
#pragma unroll
        for (int ks = 0; ks < BKb / 4; ++ks) {
            const int kr = ks * 4 + lk;
            T a[MI], bb[NI];
#pragma unroll
            for (int i = 0; i < MI; ++i) a[i] = sA[cur][kr][wm * WM + 16 * i + li];
#pragma unroll
            for (int j = 0; j < NI; ++j) bb[j] = sB[cur][kr][wn * WN + 16 * j + li];
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    if constexpr (CX) {
                        cre[i][j] = mfma(a[i].x, bb[j].x, cre[i][j]);
                        cim[i][j] = mfma(a[i].y, bb[j].y, cim[i][j]);
                        c3[i][j] = mfma(a[i].x + a[i].y, bb[j].x + bb[j].y, c3[i][j]);
                    } else {
                        cre[i][j] = mfma(a[i], bb[j], cre[i][j]);
                    }
                }
        }
        if (more) store(cur ^ 1);
        __syncthreads();
        cur ^= 1;
    }
    // With beta != 0, one row of blocks at a time: its C values are all
    // requested before any of them is written back (a read of C placed after a
    // write to C would wait for the memory once per element, since the
    // compiler cannot tell that the addresses differ).
    const bool acc_c = beta != 0.0;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        T cv[NI][4];
        if (acc_c) {
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = m0 + wm * WM + i * 16 + out_row<T>(lane, r);
                    const int col = n0 + wn * WN + j * 16 + li;
                    const bool ok = row < m && col < n && in_uplo(uplo, row, col);
                    cv[j][r] = ok ? C[(long)row * ldc + col] : zero_<T>();
                }
        }
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = m0 + wm * WM + i * 16 + out_row<T>(lane, r);
                const int col = n0 + wn * WN + j * 16 + li;
                if (row < m && col < n && in_uplo(uplo, row, col)) {
                    T v;
                    if constexpr (CX) {
                        const auto p1 = cre[i][j][r], p2 = cim[i][j][r];
                        v = from_parts(p1 - p2, c3[i][j][r] - p1 - p2, (const T*)nullptr);
                    } else {
                        v = cre[i][j][r];
                    }
                    v = alpha * v;
                    if (acc_c) v += beta * cv[j][r];
                    C[(long)row * ldc + col] = v;
                }
            }
    }
}

// ---------------------------------------------------------------- thin products
// Products with fewer 64 x 64 tiles than compute units (FP64).  There the tile
// kernel above leaves most of the chip idle and pays a round trip through
// memory and LDS per 16 inner steps.  Here a workgroup takes a 32 x 32 tile, its
// four wavefronts a quarter of the inner dimension each, with the operands
// loaded straight into the MFMA layout (32 inner steps of loads in flight ahead
// of their use, 16 for complex data) and the four partial tiles added in LDS in
// order.  Lane (li, lk) takes inner index k + 2 lk + s in step s of eight, the
// same for both operands, so that it reads two neighbours of a row.
// (Averages over the products of one solve: order 333 real 10.5 -> 6.4 us, order
// 520 complex 18.5 -> 9.2 us per N N launch, 28.8 -> 10.7 us per N C launch.)
template <typename T, int OPA, int OPB>
__global__ __launch_bounds__(256) void gemm_thin_kernel(int m, int n, int K, double alpha, const T* A, int lda, long sa,
                                                        const T* B, int ldb, long sb, double beta, T* C, int ldc,
                                                        long sc, const double* kscale, long sk, int uplo,
                                                        const int* kdev, int tri) {
    constexpr int TS = 32, SETS = is_cplx<T>::value ? 2 : 4;
    __shared__ T part[4][TS][TS + 1];
    const int m0 = blockIdx.y * TS, n0 = blockIdx.x * TS;
    if (!in_uplo(uplo, m0 + TS - 1, n0)) return;  // tile strictly above the diagonal
    const long b = blockIdx.z;
    A += b * sa;
    B += b * sb;
    C += b * sc;
    if (kscale) kscale += b * sk;
    if (kdev) K = min(K, *kdev);
    int klo = 0;
    if (tri == TRI_A_LOWER) K = min(K, m0 + TS);
    if (tri == TRI_B_UPPER) K = min(K, n0 + TS);
    if (tri == TRI_A_UPPER) klo = m0;
    if (tri == TRI_B_LOWER) klo = n0;
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int li = lane & 15, lk = lane >> 4;
    const int kq = max(0, K - klo + 31) / 32 * 8;  // a wavefront's share, a multiple of eight
    const int kb = klo + w * kq, ke = min(K, kb + kq);
    const int ra[2] = {min(m0 + li, m - 1), min(m0 + 16 + li, m - 1)};
    const int cb[2] = {min(n0 + li, n - 1), min(n0 + 16 + li, n - 1)};
    constexpr int CX = is_cplx<T>::value ? 1 : 0;
    d4 c1[2][2], c2[CX ? 2 : 1][CX ? 2 : 1], c3[CX ? 2 : 1][CX ? 2 : 1];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            c1[i][j] = d4{0.0, 0.0, 0.0, 0.0};
            if constexpr (CX) c2[i][j] = c3[i][j] = d4{0.0, 0.0, 0.0, 0.0};
        }
    T av[2][SETS][2][2], bv[2][SETS][2][2];
    auto load = [&](int buf, int k0) {
#pragma unroll
        for (int q = 0; q < SETS; ++q)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int kk = k0 + 8 * q + 2 * lk + s, kc = min(kk, ke - 1);
                const bool ok = kk < ke;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    T x = OPA == OP_N ? A[(long)ra[i] * lda + kc] : ld_op<T, OPA>(A + (long)kc * lda + ra[i]);
                    if (kscale) x = x * kscale[kc];
                    av[buf][q][s][i] = pick(ok, x, zero_<T>());
                    const T y = OPB == OP_N ? B[(long)kc * ldb + cb[i]] : ld_op<T, OPB>(B + (long)cb[i] * ldb + kc);
                    bv[buf][q][s][i] = pick(ok, y, zero_<T>());
                }
            }
    };
    auto use = [&](int buf) {
#pragma unroll
        for (int q = 0; q < SETS; ++q)
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const T x = av[buf][q][s][i], y = bv[buf][q][s][j];
                        if constexpr (CX) {
                            c1[i][j] = mfma(x.x, y.x, c1[i][j]);
                            c2[i][j] = mfma(x.y, y.y, c2[i][j]);
                            c3[i][j] = mfma(x.x + x.y, y.x + y.y, c3[i][j]);
                        } else {
                            c1[i][j] = mfma(x, y, c1[i][j]);
                        }
                    }
    };
    constexpr int KS = 8 * SETS;
    if (kb < ke) {
        load(0, kb);
        for (int k = kb; k < ke; k += 2 * KS) {
            if (k + KS < ke) load(1, k + KS);
            use(0);
            if (k + KS < ke) {
                if (k + 2 * KS < ke) load(0, k + 2 * KS);
                use(1);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                T v;
                if constexpr (CX) {
                    const double p1 = c1[i][j][r], p2 = c2[i][j][r];
                    v = mk(p1 - p2, c3[i][j][r] - p1 - p2);
                } else {
                    v = c1[i][j][r];
                }
                part[w][16 * i + out_row<T>(lane, r)][16 * j + li] = v;
            }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < TS * TS / 256; ++q) {
        const int e = t + 256 * q, r = e / TS, cc = e % TS, row = m0 + r, col = n0 + cc;
        if (row < m && col < n && in_uplo(uplo, row, col)) {
            T v = alpha * ((part[0][r][cc] + part[1][r][cc]) + (part[2][r][cc] + part[3][r][cc]));
            T* pc = C + (long)row * ldc + col;
            if (beta != 0.0) v += beta * (*pc);
            *pc = v;
        }
    }
}

// FP64 products that take the thin kernel: fewer 64 x 64 tiles than THIN_TILES, one
// per compute unit (beyond, the larger tiles' reuse is worth more than the split),
// and with an inner dimension above THIN_K no more 32 x 32 tiles than THIN_WGS: there
// the four wavefronts have work enough, and twice the operand bytes per product decide.
// (Triangular operands cut the inner dimension differently for every tile, which the
// small ones even out: order 1000 reduction real 146 -> 103 us, complex 331 -> 233.)
// Whole calls (us, 64 x 64 tiles against thin) on both sides of the lines: the lower
// triangle of C w C^H (energy density) real 900 97, 73, 1000 105, 131, complex 900 194, 180,
// 1000 204, 278; six full products (backward) real 700 322, 243, 800 367, 403, complex 800 826,
// 738, 900 945, 1080; the lower triangle of V^H (H V) (Loewdin reduction) complex 800 271,
// 252, 900 311, 345, real ones up to the tiles' line (1300 277, 233).
constexpr long THIN_TILES = 256;
constexpr int THIN_K = 256;
template <typename T, int OPA>
constexpr long thin_wgs(bool lower) {
    if (std::is_same<T, cplx>::value) return !lower ? 640 : OPA == OP_N ? 450 : 350;
    return !lower ? 512 : OPA == OP_N ? 450 : 4 * THIN_TILES;
}
template <typename T, int OPA>
static bool thin(int m, int n, int k, int batch, Uplo uplo, Tri tri) {
    if (!std::is_same<T, double>::value && !std::is_same<T, cplx>::value) return false;
    const int half = uplo != UPLO_FULL ? 2 : 1;
    if ((long)cdiv(m, BM) * cdiv(n, BN) * batch / half >= THIN_TILES) return false;
    return k <= THIN_K || tri != TRI_NONE ||
           (long)cdiv(m, 32) * cdiv(n, 32) * batch / half <= thin_wgs<T, OPA>(half == 2);
}

// They replace a split-K product of the back-transform up to these inner dimensions,
// for complex data only with few tiles: whole back-transforms by blocks of 128 (us, split-K
// against thin) 760 real 274, 257, 900 real 362 both, 1100 494, 501; 600 complex 453
// both, 680 508, 522; four complex matrices of 400 (56 tiles) 493, 444, of 520 (72 tiles) 735, 820.
template <typename T>
constexpr int THIN_SPLITK = std::is_same<T, cplx>::value ? 640 : 800;
constexpr long THIN_SPLITK_TILES = 64;
template <typename T>
static bool thin_splitk(int k, long tiles) {
    return k <= THIN_SPLITK<T> && (!std::is_same<T, cplx>::value || tiles <= THIN_SPLITK_TILES);
}
template <typename T, int OPA, int OPB>
static void launch(hipStream_t s, int m, int n, int k, double alpha, const T* A, int lda, long sa,
                   const T* B, int ldb, long sb, double beta, T* C, int ldc, long sc, int batch,
                   const double* kscale, long sk, Uplo uplo, const int* kdev, Tri tri) {
    constexpr int BBM = Big<T>::BM, BBN = Big<T>::BN;
    const long big_tiles = (long)cdiv(m, BBM) * cdiv(n, BBN) * batch / (uplo != UPLO_FULL ? 2 : 1);
    // FP32 gains from large tiles at one round of workgroups, FP64 from two
    const long min_tiles = (sizeof(T) == 4 || std::is_same<T, cplx32>::value) ? BIG_MIN_TILES : 2 * BIG_MIN_TILES;
    if (!kscale && k >= g_big_min_k && big_tiles >= min_tiles) {
        ++g_big_launches;
        dim3 grid(cdiv(n, BBN), cdiv(m, BBM), batch);
        hipLaunchKernelGGL((gemm_big_kernel<T, OPA, OPB>), grid, dim3(256), 0, s, m, n, k, alpha, A, lda, sa, B,
                           ldb, sb, beta, C, ldc, sc, (int)uplo, kdev, (int)tri);
        return;
    }
    if constexpr (std::is_same<T, double>::value || std::is_same<T, cplx>::value) {
        if (thin<T, OPA>(m, n, k, batch, uplo, tri)) {
            dim3 grid(cdiv(n, 32), cdiv(m, 32), batch);
            hipLaunchKernelGGL((gemm_thin_kernel<T, OPA, OPB>), grid, dim3(256), 0, s, m, n, k, alpha, A, lda, sa, B,
                               ldb, sb, beta, C, ldc, sc, kscale, sk, (int)uplo, kdev, (int)tri);
            return;
        }
    }
    dim3 grid(cdiv(n, BN), cdiv(m, BM), batch);
    hipLaunchKernelGGL((gemm_kernel<T, OPA, OPB>), grid, dim3(256), 0, s, m, n, k, alpha, A, lda, sa,
                       B, ldb, sb, beta, C, ldc, sc, kscale, sk, (int)uplo, kdev, (int)tri);
}

template <typename T>
void gemm(hipStream_t s, Op opa, Op opb, int m, int n, int k, double alpha, const T* A, int lda,
          long sa, const T* B, int ldb, long sb, double beta, T* C, int ldc, long sc, int batch,
          const double* kscale, long sk, Uplo uplo, const int* kdev, Tri tri) {
    if (m <= 0 || n <= 0 || batch <= 0) return;
#define KS_GEMM_CASE(OA, OB)                                                                      \
    if (opa == OA && opb == OB)                                                                   \
        return launch<T, OA, OB>(s, m, n, k, alpha, A, lda, sa, B, ldb, sb, beta, C, ldc, sc, batch, \
                                 kscale, sk, uplo, kdev, tri);
    KS_GEMM_CASE(OP_N, OP_N)
    KS_GEMM_CASE(OP_N, OP_T)
    KS_GEMM_CASE(OP_N, OP_C)
    KS_GEMM_CASE(OP_T, OP_N)
    KS_GEMM_CASE(OP_C, OP_N)
#undef KS_GEMM_CASE
}

template void gemm<double>(hipStream_t, Op, Op, int, int, int, double, const double*, int, long,
                           const double*, int, long, double, double*, int, long, int, const double*,
                           long, Uplo, const int*, Tri);
template void gemm<cplx>(hipStream_t, Op, Op, int, int, int, double, const cplx*, int, long,
                         const cplx*, int, long, double, cplx*, int, long, int, const double*, long,
                         Uplo, const int*, Tri);
template void gemm<float>(hipStream_t, Op, Op, int, int, int, double, const float*, int, long,
                          const float*, int, long, double, float*, int, long, int, const double*, long,
                          Uplo, const int*, Tri);
template void gemm<cplx32>(hipStream_t, Op, Op, int, int, int, double, const cplx32*, int, long,
                           const cplx32*, int, long, double, cplx32*, int, long, int, const double*, long,
                           Uplo, const int*, Tri);

// ---------------------------------------------------------------- split K
// Partial products over K chunks: P[b][z] = op(A_b)[:, Kz] op(B_b)[Kz, :] for
// chunk z of matrix b of the batch (blockIdx.z = b * nz + z).
template <typename T, int OPA, int OPB>
__global__ __launch_bounds__(256) void gemm_splitk_kernel(int m, int n, int K, int kc, int nz, const T* A,
                                                          int lda, long sa, const T* B, int ldb, long sb, T* P) {
    int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    int z = blockIdx.z % nz, b = blockIdx.z / nz;
    int k0 = z * kc;
    int kz = min(kc, K - k0);
    A += b * sa;
    B += b * sb;
    const T* Az = (OPA == OP_N) ? A + k0 : A + (long)k0 * lda;
    const T* Bz = (OPB == OP_N) ? B + (long)k0 * ldb : B + k0;
    gemm_tile<T, OPA, OPB>(m, n, kz, 1.0, Az, lda, Bz, ldb, 0.0, P + (long)blockIdx.z * m * n, n, nullptr,
                           UPLO_FULL, m0, n0);
}

// C_b = alpha sum_z P[b][z] + beta C_b, summed in chunk order (deterministic).
template <typename T>
__global__ void splitk_reduce_kernel(int m, int n, int nz, const T* P, double alpha, double beta, T* C,
                                     int ldc, long sc) {
    long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (long)m * n) return;
    const int b = blockIdx.y;
    P += (long)b * nz * m * n;
    int i = (int)(e / n), j = (int)(e % n);
    T s = zero_<T>();
    for (int z = 0; z < nz; ++z) s += P[(long)z * m * n + e];
    T v = alpha * s;
    T* pc = C + b * sc + (long)i * ldc + j;
    if (beta != 0.0) v += beta * (*pc);
    *pc = v;
}

template <typename T>
void gemm_splitk(hipStream_t s, Op opa, Op opb, int m, int n, int k, double alpha, const T* A, int lda,
                 const T* B, int ldb, double beta, T* C, int ldc, T* work, long work_elems, int batch, long sa,
                 long sb, long sc) {
    if (m <= 0 || n <= 0 || batch <= 0) return;
    // the chunking depends on one matrix's shape only, so a batched product rounds
    // like the same product on its own (as long as both are thin or neither is)
    long tiles = (long)cdiv(m, BM) * cdiv(n, BN);
    int nz = (int)std::max<long>(1, std::min<long>(cdiv(1024, tiles), cdiv(k, 256)));
    while (nz > 1 && (long)nz * m * n * batch > work_elems) --nz;
    int kc = ((cdiv(k, nz) + BK - 1) / BK) * BK;
    nz = cdiv(k, kc);
    // (short inner dimensions fit the thin kernel's four wavefronts)
    if (nz <= 1 || k <= 0 || (thin_splitk<T>(k, tiles * batch) && thin<T, OP_C>(m, n, k, batch, UPLO_FULL, TRI_NONE))) {
        gemm<T>(s, opa, opb, m, n, k, alpha, A, lda, sa, B, ldb, sb, beta, C, ldc, sc, batch);
        return;
    }
    dim3 grid(cdiv(n, BN), cdiv(m, BM), nz * batch);
#define KS_SK_CASE(OA, OB)                                                                            \
    if (opa == OA && opb == OB)                                                                      \
        hipLaunchKernelGGL((gemm_splitk_kernel<T, OA, OB>), grid, dim3(256), 0, s, m, n, k, kc, nz, A, lda, sa, \
                           B, ldb, sb, work);
    KS_SK_CASE(OP_N, OP_N)
    KS_SK_CASE(OP_C, OP_N)
    KS_SK_CASE(OP_T, OP_N)
#undef KS_SK_CASE
    long tot = (long)m * n;
    hipLaunchKernelGGL((splitk_reduce_kernel<T>), dim3(cdiv(tot, 256), batch), dim3(256), 0, s, m, n, nz, work,
                       alpha, beta, C, ldc, sc);
}

template void gemm_splitk<double>(hipStream_t, Op, Op, int, int, int, double, const double*, int, const double*,
                                  int, double, double*, int, double*, long, int, long, long, long);
template void gemm_splitk<cplx>(hipStream_t, Op, Op, int, int, int, double, const cplx*, int, const cplx*, int,
                                double, cplx*, int, cplx*, long, int, long, long, long);
template void gemm_splitk<float>(hipStream_t, Op, Op, int, int, int, double, const float*, int, const float*,
                                 int, double, float*, int, float*, long, int, long, long, long);
template void gemm_splitk<cplx32>(hipStream_t, Op, Op, int, int, int, double, const cplx32*, int,
                                  const cplx32*, int, double, cplx32*, int, cplx32*, long, int, long, long, long);

// ---------------------------------------------------------------- grouped
__global__ __launch_bounds__(256) void gemm_grouped_dc_kernel(int nm, int part, const int* lo, const int* mid,
                                                              const int* hi, const int* kk, const int* kk1,
                                                              const double* A, const double* B, double* C,
                                                              int ld) {
    const int G = blockIdx.z, g = G % nm;  // merge g of matrix G / nm of a batch
    const int l = lo[g], md = mid[g], K = kk[G], K1 = kk1[G];
    // part 0: rows l .. md-1; part 1: rows md .. hi-1; inner range [k0, k1)
    const int r0 = part == 0 ? l : md, rows = part == 0 ? md - l : hi[g] - md;
    const int k0 = (K1 >= 0 && part == 1) ? K1 : 0, k1 = (K1 >= 0 && part == 0) ? K1 : K;
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    if (m0 >= rows || n0 >= K) return;
    const long base = (long)(G / nm) * ld * ld;
    gemm_tile<double, OP_N, OP_N>(rows, K, k1 - k0, 1.0, A + base + (long)r0 * ld + l + k0, ld,
                                  B + base + (long)(l + k0) * ld + l, ld, 0.0, C + base + (long)r0 * ld + l, ld,
                                  nullptr, UPLO_FULL, m0, n0);
}

void gemm_grouped_dc(hipStream_t s, int ngroups, int batch, int max_rows, const int* d_lo, const int* d_mid,
                     const int* d_hi, const int* d_kk, const int* d_kk1, const double* A, const double* B,
                     double* C, int ld) {
    if (ngroups <= 0 || max_rows <= 0 || batch <= 0) return;
    // each part covers at most max_rows - max_rows / 2 rows (the tear splits a merge in halves)
    const int half = max_rows - max_rows / 2;
    dim3 grid(cdiv(max_rows, BN), cdiv(half, BM), ngroups * batch);
    for (int part = 0; part < 2; ++part)
        hipLaunchKernelGGL(gemm_grouped_dc_kernel, grid, dim3(256), 0, s, ngroups, part, d_lo, d_mid, d_hi, d_kk,
                           d_kk1, A, B, C, ld);
}

}  // namespace ks
