// ks_trdpanel.hip -- a panel of the Householder tridiagonalisation in one launch,
// for one matrix too large for the registers of the chip (ks_trdres.hip).
// The two-launch column of ks_hetrd.hip is bound by the bytes of the lower
// triangle per column, plus 10 us of its column kernel, kernel boundaries and
// launch ramps.  Here one workgroup per compute unit stays for the panel's
// columns and keeps what fits of the matrix, which the panel does not change, in
// registers; the rest is read each column.
//
// The lower triangle of the trailing matrix is cut into PQ block rows and columns
// of h: block (I, J), J <= I, on workgroup I (I + 1) / 2 + J.  A wavefront holds
// rows g, g + 8, ... of its block, a lane the columns lane + 64 c.  With the raw
// column x (as in the other gangs) the block gives the partial products
// A_IJ x_J of block row I and A_IJ^H x_I of block row J.  Rows belong to
// owners, PO of ro = h / PR rows each, which keep their rows of the panel's V and
// W in LDS.  A column is two exchanges (the data are the flags, ks_gang.hpp):
//   A  blocks read x, publish their partial products and their share of x^H A x;
//      meanwhile the three workgroups without a block add the owners' shares of
//      |x|^2, W^H x and V^H x;
//   B  every workgroup forms the reflector from those sums; the owners add the
//      partial products of their rows, take the panel's part off and publish
//      the next column and their shares of its products with the panel.
// Slots: column j's entries in slot j mod 3 (x: mod 4).  Who has read the sums of
// column j knows that every workgroup has finished column j - 1, so it resets
// its own entries of column j - 1 (and its shares of column j's sums) at the end
// of column j, and these resets are in memory before it publishes its shares of
// column j + 2.
//
// A column of trailing order 3100 to 4100 (real, all of it kept) takes 8.8 us:
// four round trips past the caches of about 1 us (x, the sums, the partial products,
// and those overlapped with work), 1.7 us of products, and sums over LDS.
// Larger ones add what is not kept at 5 to 6.5 TB/s.  Against two launches per column,
// whole solves: 6656 real 170 -> 127 ms, 4160 complex in FP32 storage 104 -> 74,
// 9984 complex 944 -> 773.
//
// Residency, the gate and what happens when the workgroups do not gather are
// as in ks_trdres.hip: a form of 128 workgroups that does two blocks each (64 and four
// where these are not free) and keeps nothing, but forms the same sums, then one
// workgroup.  Whole tridiagonalisations with their panels in that form (two launches per
// column): 6656 real 114 ms (144), 4160 complex 99 (109), 9984 complex 765 (727), 10000
// real 442 (359); on 64 workgroups 179, 165, 1295 and 802.

// Sums as they are written: the forms of a gang would give other bits if the compiler
// chose for each which products it fuses.
#pragma clang fp contract(off)
#include "ks_gang.hpp"
#include "ks_lanes.hpp"

namespace ks {

namespace {

constexpr int PQ = 22, PB = PQ * (PQ + 1) / 2;  // block rows; blocks
constexpr int PR = 11, PO = PQ * PR;            // owners per block row, owners
constexpr int PV = 256;                         // workgroups (virtual ones of the small form)
constexpr int PNW = 8, PNT = 64 * PNW;
constexpr int NB = HETRD_NB;
// shares of W^H x and V^H x, and at the place that column 31 of W would have of |x|^2
constexpr int ND = 2 * NB, DN = NB - 1;
static_assert(ND == 64, "one lane per share");
constexpr int PS = PV - PB;                     // workgroups that add the shares

template <typename T, typename S>
struct Panel {
    int n, k0, jb;           // order, first column, columns
    int m, ro, rop, h, q;    // trailing order, rows of an owner (padded), of a block, block rows in use
    int lda;
    const S* A;              // at (k0, k0)
    T *VW, *WV;              // panel buffers, at row k0
    double *d, *e;
    T* tau;
    T *xb, *pb, *db, *sb, *vb, *hb;  // exchange: column, partial products, shares, sums, x^H A x, head rows
    int *state, *chip;
    int* info;
};

__device__ __forceinline__ void block_of(int v, int& I, int& J) {
    I = (int)((sqrtf(8.f * v + 1.f) - 1.f) * 0.5f);
    while (I * (I + 1) / 2 > v) --I;
    while ((I + 1) * (I + 2) / 2 <= v) ++I;
    I = __builtin_amdgcn_readfirstlane(I);
    J = v - I * (I + 1) / 2;
}

// widen(), not ahead of the loop over the columns (the results would take twice
// the registers).
__device__ __forceinline__ double widen_here(double v) { return v; }
__device__ __forceinline__ cplx widen_here(cplx v) { return v; }
__device__ __forceinline__ double widen_here(float v) {
    double r;
    asm volatile("v_cvt_f64_f32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}
__device__ __forceinline__ cplx widen_here(cplx32 v) { return mk(widen_here(v.x), widen_here(v.y)); }

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float read(__amdgpu_buffer_rsrc_t r, float, int v, int s) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, v, s, 0));
}
__device__ __forceinline__ double read(__amdgpu_buffer_rsrc_t r, double, int v, int s) {
    const u32x2 x = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, v, s, 0));
    return __hiloint2double(x.y, x.x);
}
__device__ __forceinline__ cplx32 read(__amdgpu_buffer_rsrc_t r, cplx32, int v, int s) {
    const u32x2 x = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, v, s, 0));
    return mk32(__uint_as_float(x.x), __uint_as_float(x.y));
}
__device__ __forceinline__ cplx read(__amdgpu_buffer_rsrc_t r, cplx, int v, int s) {
    const u32x4 x = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, v, s, 0));
    return mk(__hiloint2double(x.y, x.x), __hiloint2double(x.w, x.z));
}

// Formed before any later load is issued (the scheduler would hold several rows).
__device__ __forceinline__ void here(double& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void here(cplx& v) { asm volatile("" : "+v"(v.x), "+v"(v.y)); }

// Polls N entries until none is empty (v[i] is empty where it is wanted).
template <int N, typename T>
__device__ __forceinline__ void poll(T (&v)[N], const T* const (&p)[N], int* state, int* sfail) {
    long long t0 = 0;
    for (int spin = 0;; ++spin) {
        bool wait = false;
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (is_empty(v[i])) v[i] = peek(p[i]);
#pragma unroll
        for (int i = 0; i < N; ++i) wait |= is_empty(v[i]);
        if (!wait) break;
        if ((spin & 1023) == 1023) {
            const long long now = wall_clock64();
            if (t0 == 0) t0 = now;
            if (now - t0 > WAIT_MS * TICKS) atomicExch(&state[0], GANG_FAILED);
            if (__hip_atomic_load(&state[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == GANG_FAILED) {
                *sfail = 1;
                break;
            }
        }
    }
}

}  // namespace

// RT: row slots of a wavefront that the form in registers keeps; from there on the
// rows are read in turn (MEM reads them all, in the same order).
template <typename T, typename S, int C, int RR, int RL, int RT, bool MEM>
__global__ __launch_bounds__(PNT, 2) void trd_panel_kernel(Panel<T, S> a, long long gate, int half) {
    constexpr int H = 64 * C;                      // largest block
    constexpr int RK = RR + RL;                    // row slots of a wavefront that are kept (RL of them in LDS)
    constexpr bool ALL = PNW * RK >= H;            // every row
    constexpr int RC = ALL && !is_cplx<T>::value ? 8 : 4;  // rows summed at a time
    constexpr int ROM = H / PR + 1;                // most rows of an owner
    constexpr int SG = C * sizeof(S) <= 64 ? 2 : 1;  // rows on their way beside those in use, of those that are not kept
    // rows so long that the time goes to reading them: a diagonal block's only up
    // to the diagonal, the wavefronts in step (at shorter rows either cost more
    // than it gave: 6656 real 57 against 52 ms of its panels)
    constexpr bool LONG = C * sizeof(S) >= 64;
    constexpr int NS = 2 * PNW * 64 > PNW * H ? 2 * PNW * 64 : PNW * H;
    __shared__ T sxr[H + 64], sxc[H], szr[H + 64], szc[NS];
    __shared__ T sV[MEM ? 1 : NB][MEM ? 1 : ROM], sW[MEM ? 1 : NB][MEM ? 1 : ROM];
    __shared__ S kept[RL > 0 ? RL * C : 1][PNT];
    __shared__ T svj[64], swj[64], sxe[64], sS[64], sH[64], sal, sz1;
    __shared__ double red[PNW];
    __shared__ int sstate, sfail, scount, snum;
    int t = threadIdx.x, lane = t & 63;
    const int g = __builtin_amdgcn_readfirstlane(t >> 6);
    // what is derived from the lane is derived again in each phase: kept, it
    // would take the registers of the matrix
    auto fresh = [&] {
        t = threadIdx.x;
        asm volatile("" : "+v"(t));
        lane = t & 63;
    };
    const int m = a.m, ro = a.ro, h = a.h, lda = a.lda;
    int b = blockIdx.x, P = PV;  // the workgroup's number, and how many there are
    int* state = a.state + (MEM ? GS_MEM : 0);
    if (MEM && state[GS_STATE - GS_MEM] != GANG_LEFT) return;
    if (t == 0) {
        sfail = scount = 0;
        if constexpr (MEM) {
            snum = gather_in_memory(state, state[GS_CHIP - GS_MEM] ? half : PV / 4, PV / 4, gate, P);
            sstate = P;
        } else {
            sstate = gather(state, PV, gate, a.chip);
        }
    }
    for (int i = t; i < H + 64; i += PNT) sxr[i] = zero_<T>();
    if constexpr (!MEM)
        for (int i = t; i < NB * ROM; i += PNT) sV[i / ROM][i % ROM] = sW[i / ROM][i % ROM] = zero_<T>();
    __syncthreads();
    if constexpr (MEM) {
        b = __builtin_amdgcn_readfirstlane(snum);
        P = __builtin_amdgcn_readfirstlane(sstate);
        if (b >= P) return;
    } else {
        if (sstate != GANG_GO) return;
    }
    T* party = szc;  // [PNW][64] each, in phase B
    T* partc = szc + PNW * 64;
    // partial products of an owner's row: block row s at offset s rop
    const int ps = PO * PQ * a.rop;
    auto row_at = [&](int i) { return (i / ro) * (PQ * a.rop) + i % ro; };
    int atI = 0, atJ = 0;  // of the thread's row t in block rows I and J

    // ---- the block's rows that stay in registers
    S res[RR > 0 ? RR : 1][C];
    int bI = 0, bJ = 0;
    const S* Ab = a.A;
    int hI = 1, hJ = 1;
    auto set_block = [&](int v) {
        block_of(v, bI, bJ);
        hI = min(h, m - bI * h);
        Ab = a.A + (long)bI * h * lda + bJ * h;
        hJ = min(h, m - bJ * h);
        atI = row_at(bI * h + t);
        atJ = row_at(bJ * h + t);
    };
    // (the matrix through a descriptor: a lane offset and a scalar one for the row,
    // where pointers would take two registers for each load)
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)a.A, 0, (int)((((unsigned)m - 1) * lda + m) * (unsigned)sizeof(S)), 0x00027000);
    auto entry = [&](int r, int c) {  // row slot r of this wavefront
        const int i = min(PNW * r + g, hI - 1);
        return read(rsrc, S{}, min(lane + 64 * c, LONG && bI == bJ ? min(i, hJ - 1) : hJ - 1) * (int)sizeof(S),
                    (int)(((unsigned)(bI * h + i) * lda + bJ * h) * (unsigned)sizeof(S)));
    };
    // on or above the diagonal of a diagonal block, whose lower triangle counts
    auto upper = [&](int r, int c) { return min(lane + 64 * c, hJ - 1) >= min(PNW * r + g, hI - 1); };
    auto kept_entry = [&](int r, int c) {
        const S x = entry(r, c);
        return bI == bJ && upper(r, c) ? S{} : x;
    };
    if constexpr (!MEM) {
        if (b < PB) {
            set_block(b);
            if (bI < a.q) {
#pragma unroll
                for (int r = 0; r < RR; ++r) {
                    if (r % 4 == 0) asm volatile("" ::: "memory");
#pragma unroll
                    for (int c = 0; c < C; ++c) res[r][c] = kept_entry(r, c);
                }
#pragma unroll 1
                for (int r = 0; r < RL; ++r)
#pragma unroll
                    for (int c = 0; c < C; ++c) kept[r * C + c][t] = kept_entry(RR + r, c);
            }
        }
    }
    const int rall = (h + PNW - 1) / PNW;  // row slots of a wavefront

    // ---- column k0
    for (int v = b; v < PV; v += P) {
        if (g != 0) continue;
        const int i = v * ro + lane;
        const bool in = v < PO && lane < ro && i < m;
        T x = in ? widen(a.A[(long)i * lda]) : zero_<T>();
        if (in && i == 0) a.d[0] = re_(x);
        if (in && i >= 1) publish(&a.xb[i], x);
        const double s = lane_sum(in && i >= 2 ? abs2_(x) : 0.0);
        if (lane == 0) publish(&a.db[v * ND + DN], from_re<T>(s));
        if (!MEM) sxe[lane] = x;
    }

    // column k + 1 of the matrix at the owner's rows (first wavefront), and its diagonal entry
    T ar = zero_<T>();
    double a11 = 0.0;
    auto raw_column = [&](int v, int i1) {
        if (g != 0) return;
        const int i = v * ro + lane;
        if (v < PO && lane < ro && i < m && i >= i1) ar = widen(a.A[(long)i * lda + i1]);
        a11 = re_(widen(a.A[(long)i1 * lda + i1]));
    };
    // Loads of entries that are due soon are issued ahead of the work before them
    // (a load past the caches takes 1 us).
    T xa[2] = {zero_<T>(), zero_<T>()}, sa[PS];  // x at the thread's row and column of the block, the sums
    // how: 0 = pointers only, 1 = and mark what is wanted, 2 = and load it
    auto ask_x = [&](int j, const T* X, const T* (&p)[2], int how) {
        const int i[2] = {bI * h + t, bJ * h + t};
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            p[u] = X + min(i[u], m - 1);
            if (how) xa[u] = t < h && i[u] > j && i[u] < m ? (how == 2 ? peek(p[u]) : empty_<T>()) : zero_<T>();
        }
    };
    auto ask_sums = [&](int j, const T* X, const T* Sm, const T* (&p)[PS], int how) {
        const int l = lane & (NB - 1);
#pragma unroll
        for (int u = 0; u < PS; ++u) {
            bool want = false;
            p[u] = Sm + u * ND + lane;
            if (g == 0) want = l < j || lane == DN;
            if (u == 0 && g == 1) {
                want = lane == 0;
                p[0] = X + j + 1;
            } else if (u == 0 && g == 2) {
                want = l < j;
                p[0] = a.hb + lane * NB + j;
            }
            if (how) sa[u] = want ? (how == 2 ? peek(p[u]) : empty_<T>()) : zero_<T>();
        }
    };
    int slot = 0, prev = 2, xslot = 0;
    for (int j = 0; j < a.jb; ++j) {
        const int i1 = j + 1, nslot = slot == 2 ? 0 : slot + 1;
        const bool next = j + 1 < a.jb;
        const int at1 = row_at(i1);
        bool asked = false;
        const T* X = a.xb + (long)xslot * m;
        T* Pj = a.pb + slot * ps;
        T* Pp = a.pb + prev * ps;
        T* D = a.db + slot * ND * PV;
        T* Sm = a.sb + slot * PS * ND;
        T* Vx = a.vb + slot * PV;
        T* Vp = a.vb + prev * PV;

        // ---------------- A
        fresh();
        if (!MEM) raw_column(b, i1);
        for (int v = b; v < PV; v += P) {
            if (v >= PB) {  // sums of the owners' shares
                constexpr int NU = (PV + PS * PNW - 1) / (PS * PNW), NC = is_cplx<T>::value ? (NU + 1) / 2 : NU;
                const bool share = lane == DN || (lane & (NB - 1)) < j;
                T r = zero_<T>();
#pragma unroll 1
                for (int i0 = 0; i0 < NU; i0 += NC) {
                    T x[NC];
                    const T* p[NC];
#pragma unroll
                    for (int i = 0; i < NC; ++i) {
                        const int o = (v - PB) * PNW + g + (i0 + i) * PS * PNW;
                        x[i] = share && o < PV ? empty_<T>() : zero_<T>();
                        p[i] = D + min(o, PV - 1) * ND + lane;
                    }
                    poll<NC, T>(x, p, state, &sfail);
#pragma unroll
                    for (int i = 0; i < NC; ++i) r += x[i];
                }
                szc[g * 64 + lane] = r;
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
                if (g == 0 && share) {
                    r = zero_<T>();
#pragma unroll 2
                    for (int q = 0; q < PNW; ++q) r += szc[q * 64 + lane];
                    publish(&Sm[(v - PB) * ND + lane], r);
                    if (j > 0) empty_out(&a.sb[(prev * PS + v - PB) * ND + lane]);
                }
                continue;
            }
            if constexpr (MEM) set_block(v);
            if (bI >= a.q) continue;
            // the rows that are not kept, from the last one in every other column:
            // what the column before read last is still in the memory-side cache
            auto turn = [&](int r) { return (j & 1) && r >= RT && r < rall ? RT + rall - 1 - r : r; };
            S buf[2][SG][C];
            auto load = [&](int r, int p) {
#pragma unroll
                for (int q = 0; q < SG; ++q)
#pragma unroll
                    for (int c = 0; c < C; ++c) buf[p][q][c] = entry(turn(r + q), c);
            };
            {
                const T* p[2];
                ask_x(j, X, p, MEM || j == 0 ? 1 : 0);
                poll<2, T>(xa, p, state, &sfail);
                if (t < H) {
                    sxr[t] = xa[0];
                    sxc[t] = xa[1];
                }
            }
            T dx = zero_<T>();  // diagonal part of a diagonal block
            if (bI == bJ && t < hI) dx = from_re<T>(re_(widen(Ab[(long)t * lda + t])));
            if (!ALL) load(RK, 0);
            __syncthreads();
            if (sfail) {
                if (t == 0) set_info(a.info, KS_ERR_NO_CONVERGENCE, -4);
                return;
            }
            T xc[C], zc[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                xc[c] = sxc[lane + 64 * c];
                zc[c] = zero_<T>();
            }
            auto rowsum = [&](int r, const T (&acc)[RC], int cnt, bool streamed) {  // row slots r .. r + RC - 1
                const T s = lane_sums(acc, lane);
                constexpr int LPR = 64 / RC;
                const int i = PNW * (streamed ? turn(r + lane / LPR) : r + lane / LPR) + g;
                if (lane % LPR == 0 && lane / LPR < cnt && i < h) szr[i] = s;
            };
#pragma unroll
            for (int r0 = 0; r0 < RR; r0 += RC) {
                T acc[RC];
#pragma unroll
                for (int q = 0; q < RC; ++q) {
                    acc[q] = zero_<T>();
                    if (r0 + q >= RR) continue;
                    if (q % 2 == 0) asm volatile("" ::: "memory");
                    const T xi = sxr[PNW * (r0 + q) + g];
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        const T e = widen_here(res[r0 + q < RR ? r0 + q : 0][c]);
                        fma_(acc[q], e, xc[c]);
                        fma_(zc[c], conj_(e), xi);
                        here(zc[c]);
                    }
                    here(acc[q]);
                }
                rowsum(r0, acc, min(RC, RR - r0), false);
            }
#pragma unroll 1
            for (int r0 = 0; r0 < RL; r0 += RC) {
                T acc[RC];
#pragma unroll
                for (int q = 0; q < RC; ++q) {
                    acc[q] = zero_<T>();
                    if (RL % RC && r0 + q >= RL) continue;
                    const T xi = sxr[PNW * (RR + r0 + q) + g];
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        const T e = widen(kept[(r0 + q) * C + c][t]);
                        fma_(acc[q], e, xc[c]);
                        fma_(zc[c], conj_(e), xi);
                        here(zc[c]);
                    }
                    here(acc[q]);
                }
                rowsum(RR + r0, acc, min(RC, RL - r0), false);
            }
            if constexpr (!ALL) {
                // (a diagonal block: columns below the row's)
                const int dlim = bI == bJ ? 0 : 64 * C + PNW * 64 * C;
#pragma unroll 1
                for (int r0 = RK; r0 < rall; r0 += RC) {
                    T acc[RC];
#pragma unroll
                    for (int u = 0; u < RC / SG; ++u) {
                        load(r0 + (u + 1) * SG, (u + 1) & 1);
#pragma unroll
                        for (int w = 0; w < SG; ++w) {
                            const int q = u * SG + w;
                            acc[q] = zero_<T>();
                            // (rows beyond the block: x is zero there)
                            const int rq = turn(r0 + q);
                            const T xi = sxr[min(PNW * rq + g, H + 63)];
#pragma unroll
                            for (int c = 0; c < C; ++c) {
                                T e = widen(buf[u & 1][w][c]);
                                e = pick(min(lane + 64 * c, hJ - 1) >= min(PNW * rq + g, hI - 1) + dlim, zero_<T>(), e);
                                fma_(acc[q], e, xc[c]);
                                fma_(zc[c], conj_(e), xi);
                                here(zc[c]);
                            }
                            here(acc[q]);
                        }
                        asm volatile("" ::: "memory");
                    }
                    rowsum(r0, acc, RC, true);
                    // the wavefronts stay together: left alone, the first ones were through a
                    // third before the last, which could not keep the memory busy
                    if (LONG) __builtin_amdgcn_s_barrier();
                }
            }
            if (!MEM) {
                const T* p[PS];
                ask_sums(j, X, Sm, p, 2);
                asked = true;
            }
#pragma unroll
            for (int c = 0; c < C; ++c) szc[g * H + lane + 64 * c] = zc[c];
            __syncthreads();
            double va = 0.0;
            if (t < h) {
                T zs = zero_<T>();
#pragma unroll
                for (int q = 0; q < PNW; ++q) zs += szc[q * H + t];
                const T zr = szr[t], x = sxr[t];
                const int i = bI * h + t, jj = bJ * h + t;
                if (bI == bJ) {
                    const T z = (zr + zs) + dx * x;
                    if (i >= i1 && i < m) {
                        publish(Pj + atI + bI * a.rop, z);
                        va = re_(conj_(x) * z);
                    }
                } else {
                    if (i >= i1 && i < m) {
                        publish(Pj + atI + bJ * a.rop, zr);
                        va = 2.0 * re_(conj_(x) * zr);
                    }
                    if (jj >= i1) publish(Pj + atJ + bI * a.rop, zs);
                }
            }
            va = lane_sum(va);
            if (lane == 0) {  // the last wavefront adds them up
                red[g] = va;
                __threadfence_block();
                if (atomicAdd(&scount, 1) == PNW - 1) {
                    __threadfence_block();
                    scount = 0;
                    double s = 0.0;
#pragma unroll
                    for (int q = 0; q < PNW; ++q) s += ((volatile double*)red)[q];
                    publish(&Vx[v], from_re<T>(s));
                }
            }
            if (MEM) __syncthreads();
        }

        // ---------------- B: the sums, x_{k+1}, row k+1 of V and W
        fresh();
        {
            const T* p[PS];
            ask_sums(j, X, Sm, p, asked ? 0 : 1);
            poll<PS, T>(sa, p, state, &sfail);
            if (g == 0) sS[lane] = (sa[0] + sa[1]) + sa[2];
            if (g == 1 && lane == 0) sal = sa[0];
            if (g == 2) sH[lane] = sa[0];
        }
        __syncthreads();
        if (sfail) {
            if (t == 0) set_info(a.info, KS_ERR_NO_CONVERGENCE, -4);
            return;
        }
        const T alpha = sal;
        T sc, tv;
        double beta;
        form_reflector<T>(alpha, re_(sS[DN]), sc, tv, beta);
        const T c1 = from_re<T>(1.0) - sc * alpha;
        T cs = zero_<T>();
        double cr = 0.0;
        if (g == 0) {
            const int l = lane;
            if (l < j) {
                const T vk = sH[l], wk = sH[NB + l];
                const T pl = conj_(wk) + sc * sS[l], ql = conj_(vk) + sc * sS[NB + l];
                cs = vk * pl + wk * ql;
                cr = re_(conj_(ql) * pl);
            }
            cs = lane_sum(cs);
            cr = lane_sum(cr);
        }
        for (int v = b; v < PV; v += P) {
            fresh();
            const int i = v * ro + lane, r = min(i, m - 1);
            const bool in = v < PO && lane < ro && i < m && i >= i1;
            if (MEM) raw_column(v, i1);
            // the partial products; x^H A x; z_{k+1}
            T x[4];
            const T* p[4];
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                const int s = g + PNW * u;
                p[u] = Pj + (min(v, PO - 1) * PQ + min(s, PQ - 1)) * a.rop + min(lane, ro - 1);
                x[u] = in && s < a.q ? peek(p[u]) : zero_<T>();
            }
            bool want = false;
            p[3] = Pj;
            if (g >= 1 && g <= 4) {
                const int f = (g - 1) * 64 + lane;
                want = f < a.q * (a.q + 1) / 2;
                p[3] = Vx + f;
            } else if (g == 5) {
                want = lane < a.q;
                p[3] = Pj + at1 + min(lane, PQ - 1) * a.rop;
            }
            x[3] = want ? peek(p[3]) : zero_<T>();
            // what the panel takes off A v and off the next column
            T cy = zero_<T>(), cx = zero_<T>();
#pragma unroll(is_cplx<T>::value ? 1 : 4)
            for (int u = 0; u < NB / PNW; ++u) {
                const int l = g + PNW * u;
                if (l < j) {
                    const T vk = sH[l], wk = sH[NB + l];
                    const T pl = conj_(wk) + sc * sS[l], ql = conj_(vk) + sc * sS[NB + l];
                    T vl, wl;
                    if constexpr (MEM) {
                        vl = in ? a.VW[(long)l * a.n + r] : zero_<T>();
                        wl = in ? a.VW[(long)(NB + l) * a.n + r] : zero_<T>();
                    } else {
                        vl = sV[l][min(lane, ROM - 1)];
                        wl = sW[l][min(lane, ROM - 1)];
                    }
                    fma_(cy, vl, pl);
                    fma_(cy, wl, ql);
                    fma_(cx, vl, conj_(wk));
                    fma_(cx, wl, conj_(vk));
                }
            }
            {
                poll<4, T>(x, p, state, &sfail);
                party[g * 64 + lane] = sc * ((x[0] + x[1]) + x[2]) - cy;
                partc[g * 64 + lane] = cx;
                const T s = lane_sum(x[3]);
                if (lane == 0) {
                    red[g] = re_(s);
                    if (g == 5) sz1 = s;
                }
            }
            __syncthreads();
            if (sfail) {
                if (t == 0) set_info(a.info, KS_ERR_NO_CONVERGENCE, -4);
                return;
            }
            if (g == 0) {
                T y = zero_<T>(), cc = zero_<T>();
#pragma unroll(is_cplx<T>::value ? 4 : PNW)
                for (int q = 0; q < PNW; ++q) {
                    y += party[q * 64 + lane];
                    cc += partc[q * 64 + lane];
                }
                const double xAx = (red[1] + red[2]) + (red[3] + red[4]);
                const T z1 = sz1;
                const double vAv = abs2_(sc) * xAx + 2.0 * re_(conj_(sc) * c1 * conj_(z1)) + abs2_(c1) * a11;
                const double alw = -0.5 * abs2_(tv) * (vAv - 2.0 * cr);
                const T w1 = tv * (sc * z1 + c1 * from_re<T>(a11) - cs) + from_re<T>(alw);
                T vv = zero_<T>(), ww = zero_<T>(), xn = zero_<T>();
                if (in) {
                    if (i == i1) ar = from_re<T>(a11);
                    const T xr = MEM ? peek(X + i) : sxe[lane];
                    vv = i == i1 ? from_re<T>(1.0) : sc * xr;
                    ww = i == i1 ? w1 : tv * (y + c1 * ar) + alw * vv;
                    xn = ar - cc - (vv * conj_(w1) + ww);
                    if (i == i1) a.d[i1] = re_(xn);
                    if (next && i > i1) {
                        publish(&a.xb[(long)((xslot + 1) & 3) * m + i], xn);
                        if (i <= NB) {
                            publish(&a.hb[j * NB + i - 1], vv);
                            publish(&a.hb[(NB + j) * NB + i - 1], ww);
                        }
                    }
                    a.VW[(long)j * a.n + i] = vv;
                    a.VW[(long)(NB + j) * a.n + i] = ww;
                    a.WV[(long)j * a.n + i] = conj_(ww);
                    a.WV[(long)(NB + j) * a.n + i] = conj_(vv);
                }
                svj[lane] = vv;
                swj[lane] = ww;
                sxe[lane] = i > i1 ? xn : zero_<T>();
                if constexpr (!MEM)
                    if (lane < ROM) {
                        sV[j][lane] = vv;
                        sW[j][lane] = ww;
                    }
                if (v == 0 && lane == 0) {
                    a.e[j] = beta;
                    a.tau[j] = tv;
                }
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            // shares of the next column's products with the panel
            if (next) {
                const T xe = i > i1 + 1 ? sxe[lane] : zero_<T>();
                T* Dn = a.db + ((long)nslot * PV + v) * ND;
                T prod[2 * NB / PNW];
#pragma unroll
                for (int u = 0; u < NB / PNW; ++u) {
                    const int l = g + PNW * u;
                    T vl = zero_<T>(), wl = zero_<T>();
                    if (l == j) {
                        vl = svj[lane];
                        wl = swj[lane];
                    } else if (l < j) {
                        if constexpr (MEM) {
                            vl = in ? a.VW[(long)l * a.n + r] : zero_<T>();
                            wl = in ? a.VW[(long)(NB + l) * a.n + r] : zero_<T>();
                        } else {
                            vl = sV[l][min(lane, ROM - 1)];
                            wl = sW[l][min(lane, ROM - 1)];
                        }
                    }
                    prod[2 * u] = conj_(wl) * xe;
                    prod[2 * u + 1] = conj_(vl) * xe;
                    here(prod[2 * u]);
                    here(prod[2 * u + 1]);
                }
                const T s = lane_sums(prod, lane);
                constexpr int LPQ = 64 * PNW / (2 * NB);
                const int q = lane / LPQ, l = g + PNW * (q >> 1);
                if (lane % LPQ == 0 && l <= j) publish(&Dn[((q & 1) ? NB : 0) + l], s);
                if (g == 0) {
                    const double nn = lane_sum(abs2_(xe));
                    if (lane == 0) publish(&Dn[DN], from_re<T>(nn));
                }
            }
            if (!MEM && next && b < PB && bI < a.q) {
                const T* p[2];
                ask_x(j + 1, a.xb + (long)((xslot + 1) & 3) * m, p, 2);
            }
            // entries that everybody has read
            if (j > 0) {
                if (v < PB) {
                    if constexpr (MEM) set_block(v);
                    if (bI < a.q && t < h) {
                        const int ii = bI * h + t, jj = bJ * h + t;
                        if (ii >= j && ii < m) empty_out(Pp + atI + bJ * a.rop);
                        if (bI != bJ && jj >= j) empty_out(Pp + atJ + bI * a.rop);
                        if (t == 0) empty_out(&Vp[v]);
                    }
                }
                if (g == 0 && v < PO && lane < ro && i >= j && i < m) empty_out(&a.xb[(long)((xslot + 3) & 3) * m + i]);
            }
            if (g == 1 && (lane == DN || (lane & (NB - 1)) < j)) empty_out(&D[v * ND + lane]);
            if (MEM) __syncthreads();
        }
        prev = slot;
        slot = nslot;
        xslot = (xslot + 1) & 3;
    }
}

// ---------------------------------------------------------------- host side
namespace {

template <typename T>
long panel_words(int m, int rop) {
    return 4L * m + 3L * PO * PQ * rop + 3L * ND * PV + 3 * PS * ND + 3 * PV + 2 * NB * NB;
}

template <typename T, typename S, int C, int RR, int RL>
void panel_run(hipStream_t s, const Panel<T, S>& a) {
    hipLaunchKernelGGL((trd_panel_kernel<T, S, C, RR, RL, RR + RL, false>), dim3(PV), dim3(PNT), 0, s, a, gang_gate(1), 0);
    hipLaunchKernelGGL((trd_panel_kernel<T, S, C, 0, 0, RR + RL, true>), dim3(PV / 2), dim3(PNT), 0, s, a, gang_gate(2),
                       gang_half(PV / 2, PV / 4));
}

}  // namespace

// Largest trailing order: blocks of 64 x 8.
template <typename T>
int panel_order() {
    return (64 * 8 / PR) * PO;
}

// Columns k0 .. k0 + HETRD_NB - 1 of one matrix (more than HETRD_NB + 2 left).
template <typename T, typename S>
void hetrd_panel(hipStream_t s, int n, int k0, S* A, int lda, double* d, double* e, T* tau, T* Vall, T* VW, T* WV,
                 GangWork<T> gw, int* info) {
    Panel<T, S> a;
    a.n = n;
    a.k0 = k0;
    a.jb = NB;
    a.m = n - k0;
    a.ro = cdiv(a.m, PO);
    a.rop = cdiv(a.ro, 8) * 8;
    a.h = PR * a.ro;
    a.q = cdiv(a.m, a.h);
    a.lda = lda;
    a.A = A + (long)k0 * lda + k0;
    a.VW = VW + k0;
    a.WV = WV + k0;
    a.d = d + k0;
    a.e = e + k0;
    a.tau = tau + k0;
    a.state = gw.state;
    a.chip = gw.chip;
    a.info = info;
    const long words = panel_words<T>(a.m, a.rop);
    T* p = gw.mem;
    a.xb = p;
    a.pb = a.xb + 4L * a.m;
    a.db = a.pb + 3L * PO * PQ * a.rop;
    a.sb = a.db + 3L * ND * PV;
    a.vb = a.sb + 3 * PS * ND;
    a.hb = a.vb + 3 * PV;
    gang_open<T>(s, gw, p, words);
    const int c = cdiv(a.h, 64);
    constexpr bool cx = is_cplx<T>::value, lo = !std::is_same<T, S>::value;
#define KS_PANEL(CC, RR_, RL_) panel_run<T, S, CC, RR_, RL_>(s, a)
    // rows in registers (what 256 hold beside x, the column sums and the rows on
    // their way) and in LDS
    if constexpr (!cx && !lo) {
        if (c <= 3) KS_PANEL(3, 16, 8);
        else if (c == 4) KS_PANEL(4, 12, 7);
        else if (c == 5) KS_PANEL(5, 8, 5);
        else if (c == 6) KS_PANEL(6, 5, 4);
        else KS_PANEL(8, 2, 2);
    } else if constexpr (cx && !lo) {
        if (c <= 2) KS_PANEL(2, 10, 6);
        else if (c == 3) KS_PANEL(3, 4, 4);
        else if (c == 4) KS_PANEL(4, 1, 2);
        else if (c == 5) KS_PANEL(5, 1, 1);
        else if (c == 6) KS_PANEL(6, 0, 1);
        else KS_PANEL(8, 0, 0);
    } else if constexpr (cx) {
        if (c <= 2) KS_PANEL(2, 16, 0);
        else if (c == 3) KS_PANEL(3, 16, 8);
        else if (c == 4) KS_PANEL(4, 5, 5);
        else if (c == 5) KS_PANEL(5, 2, 3);
        else if (c == 6) KS_PANEL(6, 0, 2);
        else KS_PANEL(8, 0, 0);
    } else {
        if (c <= 3) KS_PANEL(3, 24, 0);
        else if (c == 4) KS_PANEL(4, 24, 8);
        else if (c == 5) KS_PANEL(5, 18, 10);
        else if (c == 6) KS_PANEL(6, 14, 8);
        else KS_PANEL(8, 8, 5);
    }
#undef KS_PANEL
    trd_single_panel<T, S>(s, n, k0, NB, A, lda, Vall, d, e, tau, VW, WV, gw);
}

#define KS_INST(T, S)                                                                                       \
    template void hetrd_panel<T, S>(hipStream_t, int, int, S*, int, double*, double*, T*, T*, T*, T*,        \
                                    GangWork<T>, int*);
KS_INST(double, double)
KS_INST(cplx, cplx)
KS_INST(double, float)
KS_INST(cplx, cplx32)
#undef KS_INST
template int panel_order<double>();
template int panel_order<cplx>();

}  // namespace ks
