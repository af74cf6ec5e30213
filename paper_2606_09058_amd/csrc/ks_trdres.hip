// ks_trdres.hip -- the last columns of the Householder tridiagonalisation with
// the trailing matrix held in registers (the whole reduction of a matrix that
// fits).  The two-launch column of ks_hetrd.hip costs 11 to 14 us (real) or 13
// to 20 us (complex) however small the trailing matrix is: two kernel
// boundaries and two dependent rounds of loads.  Here a column is one pass over
// registers and one exchange between workgroups, bound by the latency of the
// exchange (0.75 us from the store to the last reader) and of two barriers.
// Measured, whole tridiagonalisation: order 64 real 0.70 -> 0.07 ms, 333 real
// 4.0 -> 0.68, 520 complex 9.1 -> 1.6, 1024 real 13.1 -> 2.4, 1300 complex
// 24.4 -> 5.0, 2048 complex 40.5 -> 11.0, 2600 real 36.7 -> 7.7, 16 x 1300
// complex 41.7 -> 24.6 ms.
//
// A gang of workgroups owns the full rows of the trailing matrix cyclically
// (local row i on workgroup i mod P, slot i / P), a thread C columns of them.
// Every workgroup keeps the column vector x (one entry per owned column in each
// thread) and forms the same reflector from it, so that a column needs one
// exchange only: the products z_i = (A x)_i of the owned rows with the raw
// column x, which wait for no reduction, and the raw row k+1 (by symmetry
// column k+1) of its owner.  While they are on their way every workgroup forms
// the reflector (v = s x + c e_{k+1}); from them p = A v = s z + c a_{k+1},
// v^H p, w and the next column x' = a_{k+1} - v conj(w_{k+1}) - w.  The rank-2
// update A -= v w^H + w v^H of column k and the product of column k+1 are one
// pass over the registers, with w_i = tau p_i + alw v_i of the own rows taken
// apart so that the pass needs only v_i and p_i.
//
// Gangs whose rows fit one workgroup (trd_wave_kernel) exchange through LDS,
// with a wavefront in the place of a workgroup.
//
// The exchange: the data are the flags.  The buffers hold a NaN pattern that
// no arithmetic result has (a result with those bits is changed); a reader
// polls its entries until none has the pattern left.  Entries are stored
// through to memory and read past the caches (agent-scope relaxed atomics), so
// no fence is needed.  Three slots, column k in slot k mod 3: once a workgroup
// has read all of column k's entries, every workgroup has published column k
// and so has read all of column k-1's; each entry of column k-1 is then reset by its
// writer, and the reset is in memory (s_waitcnt) before that workgroup
// publishes column k+1, after which alone the slot's next writer, in column
// k+2, can write.
//
// A gang waits for its own workgroups, so all of them have to be resident.
// They first count in; if they do not all arrive in time (other kernels hold
// compute units), the gang leaves without having touched the matrix, and
// a kernel launched behind it does the columns instead: the same gang with its
// rows in memory (on half the chip, or a quarter where that is not free either)
// behind one that takes the whole chip, one workgroup (trd_single_kernel) behind
// the others.  Waits inside a gang that is complete are bounded as well
// (KS_ERR_NO_CONVERGENCE, detail -4).

// Sums as they are written: the forms of a gang would give other bits if the compiler
// chose for each which products it fuses.
#pragma clang fp contract(off)
#include "ks_gang.hpp"
#include "ks_lanes.hpp"

namespace ks {

namespace {

// Entry (i, j) of the trailing matrix from its lower triangle.
template <typename T, typename S>
__device__ __forceinline__ T herm_entry(const S* A, long lda, int i, int j) {
    if (i > j) return widen(A[i * lda + j]);
    if (i < j) return conj_(widen(A[j * lda + i]));
    return from_re<T>(re_(widen(A[i * lda + j])));
}

__device__ __forceinline__ void put(double* p, double v) { *p = v; }
__device__ __forceinline__ void put(cplx* p, cplx v) { *p = v; }
__device__ __forceinline__ void put(float* p, double v) { *p = narrow(v); }
__device__ __forceinline__ void put(cplx32* p, cplx v) { *p = narrow(v); }

// Zero the entries of the reflector columns k0 .. k0+kend-1 on and above the
// diagonal, rows i = first, first + step, ...
template <typename T>
__device__ __forceinline__ void zero_above(int n, int k0, int kend, T* Vall, int first, int step, int t, int nt) {
    for (int i = first; i < n; i += step) {
        const int c0 = max(0, i - k0);
        for (int c = c0 + t; c < kend; c += nt) Vall[(long)i * n + k0 + c] = zero_<T>();
    }
}

}  // namespace

// ---------------------------------------------------------------- one workgroup
// NW wavefronts; wavefront g owns local rows g, g + NW, ... (R of them), a lane
// the columns lane + 64 c; every wavefront keeps the vectors of all columns.
// Per column one barrier: it publishes z and the raw row k+1 (LDS, two buffers
// by column parity).
template <typename T, typename S, int NW, int C, int R>
__global__ __launch_bounds__(64 * NW) void trd_wave_kernel(int n, int k0, const S* A, int lda, long sA, T* Vall,
                                                           double* d, double* e, T* taua) {
    constexpr int RC = R <= 4 ? 4 : R <= 8 || is_cplx<T>::value ? 8 : 16;  // rows summed at a time
    __shared__ T zbuf[2][NW * R], rbuf[2][64 * C];
    __shared__ T vp[NW][2][R];  // v and p on the wavefront's own rows
    const int z = blockIdx.x, lane = threadIdx.x & 63, g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = n - k0;
    A += z * sA + (long)k0 * lda + k0;
    Vall += (long)z * n * n;
    d += (long)z * n + k0;
    e += (long)z * n + k0;
    taua += (long)z * n + k0;
    zero_above<T>(n, k0, m - 1, Vall, g, NW, lane, 64);
    T* V = Vall + (long)k0 * n + k0;
    T a[R][C], x[C], ua[C], ta[C];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int i = g + NW * r, j = lane + 64 * c;
            a[r][c] = i < m && j < m ? herm_entry<T, S>(A, lda, i, j) : zero_<T>();
        }
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int j = lane + 64 * c;
        x[c] = j >= 1 && j < m ? widen(A[(long)j * lda]) : zero_<T>();
        ua[c] = ta[c] = zero_<T>();
        if (j % NW == g) vp[g][0][j / NW] = vp[g][1][j / NW] = zero_<T>();
    }
    if (threadIdx.x == 0) d[0] = re_(widen(A[0]));
    for (int k = 0; k < m - 1; ++k) {
        const int k1 = k + 1;
        double nx = 0.0;
        T xk = zero_<T>();
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int j = lane + 64 * c;
            add_abs2(nx, pick(j > k1, x[c], zero_<T>()));
            xk = pick(c == (k1 >> 6), x[c], xk);
        }
        const double xn2 = lane_sum(nx);
        const T alpha = lane_get(xk, k1 & 63);
        T sc, tv;
        double beta;
        form_reflector<T>(alpha, xn2, sc, tv, beta);
        T c1 = from_re<T>(1.0);
        fma_(c1, -sc, alpha);
        T* zb = zbuf[k & 1];
        T* rb = rbuf[k & 1];
        const int r1 = k1 / NW;  // slot of the raw row, on wavefront k1 % NW
#pragma unroll
        for (int r0 = 0; r0 < R; r0 += RC) {
            if (NW * (r0 + RC) <= k1) continue;  // every row of these slots is done (uniform)
            T acc[RC];
#pragma unroll
            for (int q = 0; q < RC; ++q) {
                acc[q] = zero_<T>();
                const int r = r0 + q;
                if (r >= R) continue;
                if (q % (is_cplx<T>::value ? 2 : 4) == 0) asm volatile("" ::: "memory");
                const T vr = vp[g][0][r], pr = vp[g][1][r];
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    rank2_(a[r][c], vr, ua[c], pr, ta[c]);
                    fma_(acc[q], a[r][c], x[c]);
                }
            }
            if (g == k1 % NW && r1 >= r0 && r1 < r0 + RC) {
#pragma unroll
                for (int q = 0; q < RC; ++q) {
                    if (r0 + q >= R || r1 != r0 + q) continue;
#pragma unroll
                    for (int c = 0; c < C; ++c) rb[lane + 64 * c] = a[r0 + q < R ? r0 + q : 0][c];
                }
            }
            const T s = lane_sums(acc, lane);
            constexpr int LPR = 64 / RC;
            const int r = r0 + lane / LPR;
            if (lane % LPR == 0 && r < R) zb[g * R + r] = s;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            e[k] = beta;
            taua[k] = tv;
        }
        T v[C], p[C], row[C];
        double gs = 0.0;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int j = lane + 64 * c;
            const bool in = j > k && j < m;
            v[c] = pick(j == k1, from_re<T>(1.0), mul_(sc, x[c]));
            const T zj = zb[(j % NW) * R + j / NW];
            row[c] = in ? conj_(rb[j]) : zero_<T>();
            p[c] = mul_(c1, row[c]);
            fma_(p[c], sc, zj);
            p[c] = pick(in, p[c], zero_<T>());
            add_dot(gs, v[c], p[c]);
            if (j % NW == g) {  // own rows: for the update, and the reflector's entries
                vp[g][0][j / NW] = v[c];
                vp[g][1][j / NW] = p[c];
                if (in) V[(long)j * n + k] = v[c];
            }
        }
        T p1 = mul_(c1, conj_(rb[k1]));
        fma_(p1, sc, zb[(k1 % NW) * R + k1 / NW]);
        const double alw = -0.5 * abs2_(tv) * lane_sum(gs);
        T w1 = from_re<T>(alw);
        fma_(w1, tv, p1);
        w1 = conj_(w1);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int j = lane + 64 * c;
            T w = mul_(tv, p[c]);
            add_scaled(w, alw, v[c]);
            ta[c] = -mul_(tv, conj_(v[c]));
            ua[c] = -conj_(w);
            add_scaled(ua[c], -alw, conj_(v[c]));
            T y = w;
            fma_(y, v[c], w1);
            x[c] = pick(j > k1, row[c] - y, zero_<T>());
            if (j == k1 && g == 0) d[k1] = re_(row[c]) - 2.0 * re_(w1);
        }
    }
}

// ---------------------------------------------------------------- a gang
// NT threads, C columns per thread, R rows per workgroup; P = 1 << lp
// workgroups per matrix (blockIdx.y the matrix), P R = NT C.  Columns 0 ..
// kend-1 (kend >= 1) of the trailing matrix; with kend < m-1 the rest is
// written back for the next kernel.  Every workgroup has a row beyond the last
// column (m - kend >= P): a workgroup that is read from no more would not be
// waited for.
//
// WPE: wavefronts per SIMD that the registers leave room for (the share of a
// compute unit that a workgroup takes).  MEM: the rows live in memory instead
// of registers, each thread's own entries where only it reaches them: the
// form behind a gang that takes the whole chip, when that could not gather.
// Its workgroups take half a compute unit each and all fit half the chip; where
// even that is taken, half of them do the rows of two each.  Either way every
// sum is formed as in registers, so the results are the same.
template <typename T, typename S, int NT, int C, int R, int WPE, bool MEM>
__global__ __launch_bounds__(NT, WPE) void trd_gang_kernel(int n, int k0, int kend, int lp, S* A, int lda, long sA,
                                                           T* Vall, double* d, double* e, T* taua, GangWork<T> gw,
                                                           long long gate, int half, int* info) {
    constexpr int NW = NT / 64, QM = MEM ? 2 : 1;
    static_assert(R <= NT, "one thread per row");
    // rows summed at a time
    constexpr int RC = MEM || R % 8 == 4 || (is_cplx<T>::value && R * C >= 32) ? 4 : R <= 8 || is_cplx<T>::value ? 8 : 16;
    __shared__ double red1[NW], red2[NW];
    __shared__ T salpha, sp1;
    __shared__ T sv[QM][R], sp[QM][R];  // v and p on the workgroup's own rows
    __shared__ T rowred[QM][NW][R];
    __shared__ int sstate, sfail, snum;
    const int t = threadIdx.x, lane = t & 63, g = t >> 6;
    const int P = 1 << lp, z = blockIdx.y;
    const int m = n - k0;
    int b = blockIdx.x, np = P;  // the workgroup's number, and how many there are
    // the thread's columns jc[c]: entry t + NT c of the exchange buffers, in
    // the order (workgroup, slot) of the rows, so that a workgroup writes and a
    // wavefront reads whole cache lines (entries in the order of the columns,
    // eight workgroups to a line, were 10 % slower per column)
    int jc[C];
#pragma unroll
    for (int c = 0; c < C; ++c) jc[c] = (((t + NT * c) % R) << lp) + (t + NT * c) / R;
    int* state = gw.state + GANG_STATE * z + (MEM ? GS_MEM : 0);
    if (MEM && state[GS_STATE - GS_MEM] != GANG_LEFT) return;
    if (t == 0) {
        sfail = 0;
        if constexpr (MEM) {
            snum = gather_in_memory(state, state[GS_CHIP - GS_MEM] ? half : P / 2, P / 2, gate, np);
            sstate = np;
        } else {
            sstate = gather(state, P, gate, gw.chip);
        }
    }
    if (t < R)
        for (int q = 0; q < QM; ++q) sv[q][t] = sp[q][t] = zero_<T>();
    __syncthreads();
    if constexpr (MEM) {
        b = snum;
        np = sstate;
        if (b >= np) return;
    } else {
        if (sstate != GANG_GO) return;
    }
    // f(q, o) for the owners o of rows o, o + P, ... whose rows are this workgroup's
    auto each = [&](auto&& f) {
        if constexpr (MEM) {
            for (int q = 0; b + q * np < P; ++q) f(q, b + q * np);
        } else {
            f(0, b);
        }
    };
    A += z * sA + (long)k0 * lda + k0;
    Vall += (long)z * n * n;
    d += (long)z * n + k0;
    e += (long)z * n + k0;
    taua += (long)z * n + k0;
    each([&](int, int o) { zero_above<T>(n, k0, kend, Vall, (o + k0) & (P - 1), P, t, NT); });
    T* V = Vall + (long)k0 * n + k0;
    T* xp = gw.xp + z * gw.sxp;
    T* xr = gw.xr + z * gw.sxr;
    const int slotn = NT * C;
    T a[MEM ? 1 : R][MEM ? 1 : C], x[C], ua[C], ta[C];
    auto rows = [&](int o) { return gw.mem + z * gw.smem + (long)o * R * C * NT + t; };
    each([&](int, int o) {
        T* am = MEM ? rows(o) : nullptr;
#pragma unroll(MEM ? 1 : R)
        for (int r = 0; r < R; ++r) {
            if (r % 4 == 0) asm volatile("" ::: "memory");  // four rows' addresses and loads at a time
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int i = o + P * r, j = jc[c];
                const T q = i < m && j < m ? herm_entry<T, S>(A, lda, i, j) : zero_<T>();
                if constexpr (MEM) am[(long)(r * C + c) * NT] = q;
                else a[r][c] = q;
            }
        }
    });
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int j = jc[c];
        x[c] = j >= 1 && j < m ? widen(A[(long)j * lda]) : zero_<T>();
        ua[c] = ta[c] = zero_<T>();
    }
    if (b == 0 && t == 0) d[0] = re_(widen(A[0]));
    // the one of the thread's columns that is a row of owner o (entries o R ..
    // o R + R - 1), its row's slot, and where its reflector entries go
    auto mine = [&](int o, int& co, int& ro, int& jo) {
        co = -1;
#pragma unroll
        for (int c = 0; c < C; ++c)
            if ((t + NT * c) / R == o) co = c;
        ro = (t + NT * max(co, 0)) % R;
        jo = co < 0 ? m : o + (ro << lp);
    };
    int co = -1, ro = 0, jo = m;
    if (!MEM) mine(b, co, ro, jo);
    T* Vo = V + (long)min(jo, m - 1) * n;
    const T* xpt = xp + t;
    const T* xrt = xr + t;
    int slot = 0, prev = 2;  // column k's slot and column k-1's
    int k = 0;  // kend >= 1 (a loop that may not run at all took 100 registers more)
    do {
        const int k1 = k + 1, b1 = k1 & (P - 1), r1 = k1 >> lp;  // row k1: workgroup and slot,
        const int e1 = b1 * R + r1, c1e = e1 / NT, t1 = e1 % NT;   // column k1: entry, the thread's column, thread
        const bool is1 = t == t1;
        double nx = 0.0;
        T x1 = x[0];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            add_abs2(nx, pick(jc[c] > k1, x[c], zero_<T>()));
            x1 = pick(c == c1e, x[c], x1);
        }
        if (is1) salpha = x1;
        each([&](int qo, int o) {
            T* am = MEM ? rows(o) : nullptr;
#pragma unroll(MEM ? 1 : R)
            for (int r0 = 0; r0 < R; r0 += RC) {
                if (((r0 + RC) << lp) <= k1) continue;  // every row of these slots is done (uniform)
                T acc[RC];
#pragma unroll
                for (int q = 0; q < RC; ++q) {
                    const int r = r0 + q;
                    acc[q] = zero_<T>();
                    if (r >= R) continue;
                    // (keeps the LDS reads of later rows behind: all at once they
                    // would take the registers of the matrix)
                    if (q % (is_cplx<T>::value ? 2 : 4) == 0) asm volatile("" ::: "memory");
                    const T vr = sv[qo][r], pr = sp[qo][r];
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        T y;
                        if constexpr (MEM) y = am[(long)(r * C + c) * NT];
                        else y = a[r][c];
                        rank2_(y, vr, ua[c], pr, ta[c]);
                        fma_(acc[q], y, x[c]);
                        if constexpr (MEM) am[(long)(r * C + c) * NT] = y;
                        else a[r][c] = y;
                    }
                }
                if (b1 == o && r1 >= r0 && r1 < r0 + RC) {
#pragma unroll
                    for (int q = 0; q < RC; ++q) {
                        if (r0 + q >= R || r1 != r0 + q) continue;
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            const int j = jc[c];
                            if (j > k && j < m) {
                                if constexpr (MEM) publish(&xr[slot * slotn + t + NT * c], am[(long)((r0 + q) * C + c) * NT]);
                                else publish(&xr[slot * slotn + t + NT * c], a[r0 + q < R ? r0 + q : 0][c]);
                            }
                        }
                    }
                }
                const T s = lane_sums(acc, lane);
                constexpr int LPR = 64 / RC;
                if (lane % LPR == 0 && r0 + lane / LPR < R) rowred[qo][g][r0 + lane / LPR] = s;
            }
        });
        nx = lane_sum(nx);
        if (lane == 0) red1[g] = nx;
        // this workgroup's resets of the slot of column k+1 are in memory
        // before it publishes column k (they were issued a column ago)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (t < R)
            each([&](int qo, int o) {
                T s = zero_<T>();
#pragma unroll
                for (int q = 0; q < NW; ++q) s += rowred[qo][q][t];
                publish(&xp[slot * slotn + o * R + t], s);
            });
        // the reflector, while the products are on their way
        double xn2 = 0.0;
#pragma unroll
        for (int q = 0; q < NW; ++q) xn2 += red1[q];
        const T alpha = salpha;
        T sc, tv;
        double beta;
        form_reflector<T>(alpha, xn2, sc, tv, beta);
        T c1 = from_re<T>(1.0);
        fma_(c1, -sc, alpha);
        T v[C], p[C], row[C], vo = zero_<T>(), po = vo;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int j = jc[c];
            v[c] = pick(j == k1, from_re<T>(1.0), mul_(sc, x[c]));
            vo = pick(c == co, v[c], vo);
            p[c] = row[c] = j > k && j < m ? empty_<T>() : zero_<T>();
        }
        if constexpr (MEM)
            each([&](int, int o) {
                mine(o, co, ro, jo);
                T x = zero_<T>();
#pragma unroll
                for (int c = 0; c < C; ++c) x = pick(c == co, v[c], x);
                if (jo > k && jo < m) V[(long)jo * n + k] = x;
            });
        else if (jo > k && jo < m) Vo[k] = vo;
        if (b == 0 && t == 0) {
            e[k] = beta;
            taua[k] = tv;
        }
        // every z_j and the raw row, straight into the threads of their columns
        {
            const T* pp = xpt + slot * slotn;
            const T* pr = xrt + slot * slotn;
            long long t0 = 0;
            for (int spin = 0;; ++spin) {
                bool wait = false;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    if (is_empty(p[c])) p[c] = peek(pp + c * NT);
                    if (is_empty(row[c])) row[c] = peek(pr + c * NT);
                }
#pragma unroll
                for (int c = 0; c < C; ++c) wait |= is_empty(p[c]) || is_empty(row[c]);
                if (!wait) break;
                if ((spin & 1023) == 1023) {
                    const long long now = wall_clock64();
                    if (t0 == 0) t0 = now;
                    if (now - t0 > WAIT_MS * TICKS) atomicExch(&state[0], GANG_FAILED);
                    if (__hip_atomic_load(&state[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == GANG_FAILED) {
                        sfail = 1;
                        break;
                    }
                }
            }
        }
        double gs = 0.0;
        T p1 = zero_<T>(), row1 = p1;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            row[c] = conj_(row[c]);
            const T z = p[c];  // A v = s A x + c a_{k+1}
            p[c] = mul_(c1, row[c]);
            fma_(p[c], sc, z);
            add_dot(gs, v[c], p[c]);
            p1 = pick(c == c1e, p[c], p1);
            row1 = pick(c == c1e, row[c], row1);
            po = pick(c == co, p[c], po);
        }
        if (is1) sp1 = p1;
        if constexpr (MEM) {
            each([&](int qo, int o) {
                mine(o, co, ro, jo);
                T x = zero_<T>(), y = x;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    x = pick(c == co, v[c], x);
                    y = pick(c == co, p[c], y);
                }
                if (co >= 0) {
                    sv[qo][ro] = x;
                    sp[qo][ro] = y;
                }
            });
        } else if (co >= 0) {
            sv[0][ro] = vo;
            sp[0][ro] = po;
        }
        gs = lane_sum(gs);
        if (lane == 0) red2[g] = gs;
        __syncthreads();
        if (sfail) {
            if (t == 0) set_info(info, KS_ERR_NO_CONVERGENCE, -4);
            return;
        }
        // column k's entries have all been read here, so column k-1's are free
        if (k > 0)
            each([&](int, int o) {
                if (t < R) empty_out(&xp[prev * slotn + o * R + t]);
                if ((k & (P - 1)) == o) {
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        const int j = jc[c];
                        if (j > k - 1 && j < m) empty_out(&xr[prev * slotn + t + NT * c]);
                    }
                }
            });
        prev = slot;
        slot = slot == 2 ? 0 : slot + 1;
        double gr = 0.0;
#pragma unroll
        for (int q = 0; q < NW; ++q) gr += red2[q];
        const double alw = -0.5 * abs2_(tv) * gr;
        T w1 = from_re<T>(alw);
        fma_(w1, tv, sp1);
        w1 = conj_(w1);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int j = jc[c];
            T w = mul_(tv, p[c]);
            add_scaled(w, alw, v[c]);
            // A -= v w^H + w v^H with w_i = tau p_i + alw v_i on the own rows:
            // v_i (conj(w_j) + alw conj(v_j)) + p_i tau conj(v_j)
            ta[c] = -mul_(tv, conj_(v[c]));
            ua[c] = -conj_(w);
            add_scaled(ua[c], -alw, conj_(v[c]));
            T y = w;
            fma_(y, v[c], w1);
            x[c] = pick(j > k1, row[c] - y, zero_<T>());
        }
        if (b == 0 && is1) d[k1] = re_(row1) - 2.0 * re_(w1);
    } while (++k < kend);
    if (kend >= m - 1) return;
    each([&](int qo, int o) {
        T* am = MEM ? rows(o) : nullptr;
#pragma unroll(MEM ? 1 : R)
        for (int r = 0; r < R; ++r) {
            const int i = o + (r << lp);
            asm volatile("" ::: "memory");
            const T vr = sv[qo][r], pr = sp[qo][r];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int j = jc[c];
                T y;
                if constexpr (MEM) y = am[(long)(r * C + c) * NT];
                else y = a[r][c];
                rank2_(y, vr, ua[c], pr, ta[c]);
                if (i >= kend && i < m && j >= kend && j <= i) put(&A[(long)i * lda + j], y);
            }
        }
    });
}

// The whole-chip gangs of a device take turns: 0 = free, 1 = taken, 2 = by a gang whose
// workgroups have gathered.  Before a gang its init kernel waits for its turn, bounded by
// TURN_MS, but only TURN_US while the chip is taken and not gathered: the gang that
// took it may need the compute unit that the wait itself is on.  Who has to go without
// takes a quarter of the chip.  (Two solves of order 6656 on two streams: 319 ms when a gang
// that found the chip taken left at once, 251 with the wait; 290 with two launches per column.)
__device__ int g_chip = 0;
constexpr long long TURN_US = 200, TURN_MS = 20;
// After a panel that could not gather its workgroups, so many panels leave at once
// before one waits for them again, doubled up to the most: what holds a compute
// unit for longer than a gang waits (CHIP_GATE_MS) holds it for many panels.  (The gangs of
// the last columns are few and long, and always wait.)
constexpr int SKIP_FIRST = 4, SKIP_MOST = 32;

// Before a gang: its buffers empty (those of a panel: words entries at p), its
// state cleared, the chip taken if it needs that.
template <typename T>
__global__ void gang_init_kernel(GangWork<T> gw, int slotn, int chip, T* p, long words) {
    const int z = blockIdx.y;
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    for (long e = i; e < words; e += (long)gridDim.x * blockDim.x) empty_out(&p[e]);
    if (i < 3 * slotn) {
        empty_out(&gw.xp[z * gw.sxp + i]);
        empty_out(&gw.xr[z * gw.sxr + i]);
    }
    if (i == 0) {
        int* state = gw.state + GANG_STATE * z;
        int skip = 0, next = 0;
        if (!gw.fresh) {
            skip = state[GS_SKIP];
            next = state[GS_SKIP_NEXT];
            if (state[GS_TRIED]) {
                next = state[GS_STATE] != GANG_LEFT ? 0 : next ? min(2 * next, SKIP_MOST) : SKIP_FIRST;
                skip = next;
            }
        }
        bool got = false;
        if (chip) {
            const long long t0 = wall_clock64();
            long long t1 = t0;  // since when the chip has been taken and not gathered
            for (;;) {
                const int was = atomicCAS(gw.chip, 0, 1);
                const long long now = wall_clock64();
                got = was == 0;
                if (was == 2) t1 = now;
                if (got || now - t1 >= TURN_US * TICKS / 1000 || now - t0 >= TURN_MS * TICKS) break;
                __builtin_amdgcn_s_sleep(8);
            }
        }
        const bool panel = words > 0, tries = got && !(panel && skip > 0);
        if (panel && skip > 0) --skip;
        state[GS_STATE] = chip && !tries ? GANG_LEFT : GANG_NONE;
        state[GS_ARRIVED] = 0;
        state[GS_MEM + GS_STATE] = GANG_NONE;
        state[GS_MEM + GS_ARRIVED] = 0;
        state[GS_CHIP] = got;
        state[GS_SKIP] = skip;
        state[GS_SKIP_NEXT] = next;
        state[GS_TRIED] = tries;
    }
}

// Behind a gang (and, with mem, behind its form in memory): gives the chip
// back, and where the gang could not gather its workgroups does columns 0 ..
// kend-1 of the trailing matrix with one workgroup, in place in global memory.
// The vectors v, w live at vb, the gang's exchange buffer.  For a panel (VW not
// null; kend = HETRD_NB) the reflectors go to the panel's buffer too, and WV becomes
// zero: the trailing update has been done.
template <typename T, typename S>
__global__ __launch_bounds__(1024) void trd_single_kernel(int n, int k0, int kend, S* A, int lda, long sA, T* Vall,
                                                          double* d, double* e, T* taua, GangWork<T> gw, int mem,
                                                          T* vb, long svb, T* VW, T* WV) {
    __shared__ double red[16];
    const int t = threadIdx.x, NT = blockDim.x, z = blockIdx.x, m = n - k0;
    const int* state = gw.state + GANG_STATE * z;
    if (t == 0 && state[GS_CHIP]) atomicExch(gw.chip, 0);
    if (state[GS_STATE] != GANG_LEFT || (mem && state[GS_MEM + GS_STATE] != GANG_LEFT)) return;
    A += z * sA + (long)k0 * lda + k0;
    Vall += (long)z * n * n;
    d += (long)z * n + k0;
    e += (long)z * n + k0;
    taua += (long)z * n + k0;
    T* v = vb + z * svb;
    T* w = v + m;
    zero_above<T>(n, k0, kend, Vall, 0, 1, t, NT);
    T* V = Vall + (long)k0 * n + k0;
    for (int k = 0; k < kend; ++k) {
        double nx = 0.0;
        for (int i = k + 2 + t; i < m; i += NT) nx += abs2_(widen(A[(long)i * lda + k]));
        const double xn2 = block_sum(nx, red);
        T sc, tv;
        double beta;
        form_reflector<T>(widen(A[(long)(k + 1) * lda + k]), xn2, sc, tv, beta);
        if (t == 0) {
            d[k] = re_(widen(A[(long)k * lda + k]));
            e[k] = beta;
            taua[k] = tv;
        }
        for (int i = k + 1 + t; i < m; i += NT) {
            const T vi = i == k + 1 ? from_re<T>(1.0) : sc * widen(A[(long)i * lda + k]);
            v[i] = vi;
            V[(long)i * n + k] = vi;
        }
        __syncthreads();
        double gl = 0.0;
        for (int i = k + 1 + t; i < m; i += NT) {
            T p = zero_<T>();
            for (int j = k + 1; j < m; ++j) p += herm_entry<T, S>(A, lda, i, j) * v[j];
            w[i] = p;
            gl += re_(conj_(v[i]) * p);
        }
        const double alw = -0.5 * abs2_(tv) * block_sum(gl, red);
        for (int i = k + 1 + t; i < m; i += NT) w[i] = tv * w[i] + alw * v[i];
        __syncthreads();
        for (int i = k + 1 + t; i < m; i += NT) {
            const T vi = v[i], wi = w[i];
            for (int j = k + 1; j <= i; ++j)
                put(&A[(long)i * lda + j],
                    widen(A[(long)i * lda + j]) - (vi * conj_(w[j]) + wi * conj_(v[j])));
        }
        __syncthreads();
    }
    if (t == 0 && kend >= m - 1) d[m - 1] = re_(widen(A[(long)(m - 1) * lda + m - 1]));
    if (!VW) return;
    for (int c = 0; c < HETRD_NB; ++c)
        for (int i = c + 1 + t; i < m; i += NT) {
            VW[(long)c * n + k0 + i] = V[(long)i * n + c];
            VW[(long)(HETRD_NB + c) * n + k0 + i] = zero_<T>();
            WV[(long)c * n + k0 + i] = zero_<T>();
            WV[(long)(HETRD_NB + c) * n + k0 + i] = zero_<T>();
        }
}

// ---------------------------------------------------------------- host side
namespace {

thread_local int g_leave = 0;  // test hook, see trd_set_leave

template <typename T, typename S, int NT, int C, int R, int LP, int WPE, bool CHIP>
void gang_run(hipStream_t s, int n, int k0, int kend, int B, S* A, int lda, long sA, T* Vall, double* d, double* e,
              T* tau, GangWork<T>& gw, int* info) {
    static_assert(NT * C == R << LP && NT * C <= GANG_ORDER, "columns");
    const long long gate = CHIP ? gang_gate(1) : gang_gate(2);
    hipLaunchKernelGGL((gang_init_kernel<T>), dim3(cdiv(3 * NT * C, 256), B), dim3(256), 0, s, gw, NT * C, (int)CHIP,
                       (T*)nullptr, 0L);
    hipLaunchKernelGGL((trd_gang_kernel<T, S, NT, C, R, WPE, false>), dim3(1 << LP, B), dim3(NT), 0, s, n, k0, kend,
                       LP, A, lda, sA, Vall, d, e, tau, gw, gate, 0, info);
    if constexpr (CHIP)
        hipLaunchKernelGGL((trd_gang_kernel<T, S, NT, C, R, 4, true>), dim3(1 << LP, B), dim3(NT), 0, s, n, k0, kend,
                           LP, A, lda, sA, Vall, d, e, tau, gw, gang_gate(2), gang_half(1 << LP, 1 << (LP - 1)), info);
    hipLaunchKernelGGL((trd_single_kernel<T, S>), dim3(B), dim3(1024), 0, s, n, k0, kend, A, lda, sA, Vall, d, e, tau,
                       gw, (int)CHIP, gw.xr, gw.sxr, (T*)nullptr, (T*)nullptr);
}

// A shape of the gang: the largest order it takes, its workgroups per matrix
// (1 << lp), the compute units they fill together, its time per column (us) on
// one matrix of that order, and whether it takes more than a quarter of the
// chip.  HIP runs at most four kernels of a process at once (its hardware
// queues), so gangs of a quarter always find room beside each other; a larger
// one takes turns (GangWork::chip) and has its form in memory for when it cannot.
struct GangShape {
    int order, lp, cus;
    double us;
};
constexpr int CHIP_CUS = 256;
// us per column measured on an MI355X (the largest shape of each type keeps some
// of its registers in scratch memory; the one below it takes over as soon as it can:
// 2600 real 13.8 -> 11.5 ms, 2048 complex with its backward pass 26.8 -> 26.1); the
// two-launch column costs 12 to 15 (real) and 16 to 23 (complex) at these orders
constexpr GangShape SHAPES_R[] = {{256, 5, 8, 2.0}, {512, 6, 16, 2.1}, {1024, 7, 64, 2.45}, {2048, 8, CHIP_CUS, 2.85},
                                  {2560, 8, CHIP_CUS, 3.7}, {3072, 8, CHIP_CUS, 8.3}};
constexpr GangShape SHAPES_C[] = {{256, 5, 8, 2.5},   {512, 6, 32, 2.9},          {512, 4, 16, 4.8},
                                  {1024, 6, 64, 4.35}, {1536, 8, CHIP_CUS, 4.45}, {1792, 8, CHIP_CUS, 8.5},
                                  {2048, 8, CHIP_CUS, 12.0}};
constexpr int NSHAPE_R = sizeof(SHAPES_R) / sizeof(GangShape), NSHAPE_C = sizeof(SHAPES_C) / sizeof(GangShape);
template <typename T>
const GangShape* shapes(int& n) {
    n = is_cplx<T>::value ? NSHAPE_C : NSHAPE_R;
    return is_cplx<T>::value ? SHAPES_C : SHAPES_R;
}

// Time per column of a batch in one shape: gangs that do not fit the chip
// together follow each other.
double gang_us(const GangShape& g, int batch, int ncu) { return g.us * cdiv((long)batch * g.cus, ncu); }

// The shape with the least time per column among those that take order m
// (-1: none); ncu: compute units that the stream may use, chip: whether gangs
// that take all of them are allowed.
template <typename T>
int pick_shape(int m, int batch, int ncu, bool chip) {
    int n, best = -1;
    const GangShape* g = shapes<T>(n);
    for (int i = 0; i < n; ++i) {
        if (g[i].order < m || g[i].cus > ncu || (g[i].cus == CHIP_CUS && !chip)) continue;
        if (best < 0 || gang_us(g[i], batch, ncu) < gang_us(g[best], batch, ncu)) best = i;
    }
    return best;
}

constexpr int WAVE_ORDER = 128;  // largest order of trd_wave_kernel
// Order from which on one workgroup takes over: complex columns of order 65 to
// 128 take 3.3 us there and 2.4 in a gang (real ones 1.8 and 2.0), as long as
// the gangs of the batch fit the chip together.
template <typename T>
int wave_order(int batch, int ncu) {
    return is_cplx<T>::value && batch * SHAPES_C[0].cus <= ncu ? WAVE_ORDER / 2 : WAVE_ORDER;
}

template <typename T, typename S>
void gang_columns(int shape, hipStream_t s, int n, int k0, int kend, int B, S* A, int lda, long sA, T* Vall, double* d,
                  double* e, T* tau, GangWork<T> gw, int* info) {
    if constexpr (is_cplx<T>::value) {
        switch (shape) {
            case 0: return gang_run<T, S, 256, 1, 8, 5, 4, false>(s, n, k0, kend, B, A, lda, sA, Vall, d, e, tau, gw, info);
            case 1: return gang_run<T, S, 256, 2, 8, 6, 2, false>(s, n, k0, kend, B, A, lda, sA, Vall, d, e, tau, gw, info);
            case 2: return gang_run<T, S, 512, 1, 32, 4, 2, false>(s, n, k0, kend, B, A, lda, sA, Vall, d, e, tau, gw, info);
            case 3: return gang_run<T, S, 512, 2, 16, 6, 2, false>(s, n, k0, kend, B, A, lda, sA, Vall, d, e, tau, gw, info);
            case 4: return gang_run<T, S, 512, 3, 6, 8, 2, true>(s, n, k0, kend, B, A, lda, sA, Vall, d, e, tau, gw, info);
            case 5: return gang_run<T, S, 448, 4, 7, 8, 2, true>(s, n, k0, kend, B, A, lda, sA, Vall, d, e, tau, gw, info);
            case 6: return gang_run<T, S, 512, 4, 8, 8, 2, true>(s, n, k0, kend, B, A, lda, sA, Vall, d, e, tau, gw, info);
        }
    } else {
        switch (shape) {
            case 0: return gang_run<T, S, 256, 1, 8, 5, 4, false>(s, n, k0, kend, B, A, lda, sA, Vall, d, e, tau, gw, info);
            case 1: return gang_run<T, S, 256, 2, 8, 6, 4, false>(s, n, k0, kend, B, A, lda, sA, Vall, d, e, tau, gw, info);
            case 2: return gang_run<T, S, 256, 4, 8, 7, 2, false>(s, n, k0, kend, B, A, lda, sA, Vall, d, e, tau, gw, info);
            case 3: return gang_run<T, S, 512, 4, 8, 8, 2, true>(s, n, k0, kend, B, A, lda, sA, Vall, d, e, tau, gw, info);
            case 4: return gang_run<T, S, 512, 5, 10, 8, 2, true>(s, n, k0, kend, B, A, lda, sA, Vall, d, e, tau, gw, info);
            case 5: return gang_run<T, S, 512, 6, 12, 8, 2, true>(s, n, k0, kend, B, A, lda, sA, Vall, d, e, tau, gw, info);
        }
    }
}

}  // namespace

void trd_set_leave(int level) { g_leave = level; }

int* gang_chip() {
    void* p = nullptr;
    return hipGetSymbolAddress(&p, HIP_SYMBOL(g_chip)) == hipSuccess ? (int*)p : nullptr;
}

long long gang_gate(int form) {
    if (form == 1) return g_leave ? 0 : CHIP_GATE_MS * TICKS;
    return g_leave == 2 ? 0 : GATE_MS * TICKS;
}
int gang_half(int half, int few) { return g_leave == 3 ? few : half; }

template <typename T>
void gang_open(hipStream_t s, GangWork<T> gw, T* p, long words) {
    hipLaunchKernelGGL((gang_init_kernel<T>), dim3(1024), dim3(256), 0, s, gw, 0, 1, p, words);
}

template <typename T, typename S>
void trd_single_panel(hipStream_t s, int n, int k0, int kend, S* A, int lda, T* Vall, double* d, double* e, T* tau,
                      T* VW, T* WV, GangWork<T> gw) {
    hipLaunchKernelGGL((trd_single_kernel<T, S>), dim3(1), dim3(1024), 0, s, n, k0, kend, A, lda, 0L, Vall, d, e, tau,
                       gw, 1, gw.mem, 0L, VW, WV);
}

// Gangs up to the largest order where one is faster than the two launches of a
// column (which overlap for the two halves of a batch: bound by the bytes of
// the product there).
template <typename T>
int resident_order(int batch, int ncu) {
    int n, best = wave_order<T>(batch, ncu);
    const GangShape* g = shapes<T>(n);
    for (int i = 0; i < n; ++i) {
        const double bytes = (double)batch * g[i].order * g[i].order / 2 * sizeof(T);
        const double two = is_cplx<T>::value ? std::max(16.0, 8.0 + bytes / 5e6) : std::max(12.0, 6.0 + bytes / 5e6);
        const int p = pick_shape<T>(g[i].order, batch, ncu, batch <= GANG_CHIP_BATCH);
        if (p >= 0 && gang_us(g[p], batch, ncu) < two) best = std::max(best, g[i].order);
    }
    return best;
}

template <typename T>
long gang_mem(int order, int batch) {
    if (batch > GANG_CHIP_BATCH) return 0;
    int n;
    long need = 0;
    const GangShape* g = shapes<T>(n);
    for (int i = 0; i < n; ++i) {
        if (g[i].cus != CHIP_CUS) {
            if (g[i].order >= order) return 0;  // never larger than a quarter of the chip
            continue;
        }
        need = (long)g[i].order * g[i].order;
        if (g[i].order >= order) break;
    }
    return need;
}

// Columns k0 .. n-1: a gang hands over to a smaller shape where that takes at
// least a tenth less per column (a hand-over costs three launches and two
// passes over the rest), and the last columns to one workgroup.  (Whole tridiagonalisations, us,
// with the line at 0.7, 0.8, 0.9 and 1: 520 real 1224, 1223, 1143, 1114; 2600 real 8299,
// 7662, 7484, 7496; 1300 complex 4921, 4902, 4802, 5002; 2048 complex 12021, 11160, 11057, 11520.)
template <typename T, typename S>
void hetrd_resident(hipStream_t s, int n, int k0, S* A, int lda, long sA, int B, double* d, double* e, T* tau, T* Vall,
                    GangWork<T> gw, int* info) {
    int ns;
    const GangShape* g = shapes<T>(ns);
    const int last = wave_order<T>(B, gw.ncu);
    while (n - k0 > last) {
        const int m = n - k0, p = pick_shape<T>(m, B, gw.ncu, gw.mem != nullptr);
        int next = std::max(last, 1 << g[p].lp);
        for (int i = 0; i < ns; ++i) {
            const int q = g[i].order < m ? pick_shape<T>(g[i].order, B, gw.ncu, gw.mem != nullptr) : -1;
            if (q >= 0 && gang_us(g[q], B, gw.ncu) <= 0.9 * gang_us(g[p], B, gw.ncu)) next = std::max(next, g[i].order);
        }
        const int kend = m - std::min(next, m - 1);
        // gangs that take the whole chip: one matrix's launches behind the other's, so
        // that each finds it free.  (In one launch one of them got it and the others'
        // columns were done in memory: 2 x 3072 real 66.6 -> 21.3 ms, 47.1 with two
        // launches per column; 4 x 2048 real 33.8 -> 15.0, 31.2.)
        const int step = g[p].cus == CHIP_CUS ? 1 : B;
        for (int z = 0; z < B; z += step)
            gang_columns<T, S>(p, s, n, k0, kend, step, A + z * sA, lda, sA, Vall + (long)z * n * n, d + (long)z * n,
                               e + (long)z * n, tau + (long)z * n, gw.at(z), info);
        gw.fresh = false;
        k0 += kend;
    }
    const int m = n - k0;
    if (m <= 64)
        hipLaunchKernelGGL((trd_wave_kernel<T, S, 8, 1, 8>), dim3(B), dim3(512), 0, s, n, k0, A, lda, sA, Vall, d, e,
                           tau);
    else
        hipLaunchKernelGGL((trd_wave_kernel<T, S, 8, 2, 16>), dim3(B), dim3(512), 0, s, n, k0, A, lda, sA, Vall, d, e,
                           tau);
}

#define KS_INST(T, S)                                                                                          \
    template void hetrd_resident<T, S>(hipStream_t, int, int, S*, int, long, int, double*, double*, T*, T*,     \
                                       GangWork<T>, int*);                                                      \
    template void trd_single_panel<T, S>(hipStream_t, int, int, int, S*, int, T*, double*, double*, T*, T*, T*,  \
                                         GangWork<T>);
KS_INST(double, double)
KS_INST(cplx, cplx)
KS_INST(double, float)
KS_INST(cplx, cplx32)
#undef KS_INST
template void gang_open<double>(hipStream_t, GangWork<double>, double*, long);
template void gang_open<cplx>(hipStream_t, GangWork<cplx>, cplx*, long);
template int resident_order<double>(int, int);
template int resident_order<cplx>(int, int);
template long gang_mem<double>(int, int);
template long gang_mem<cplx>(int, int);

}  // namespace ks
