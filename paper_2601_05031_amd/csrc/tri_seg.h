// Segmented tridiagonal solves in y of the Poisson problems (main text eq. (5b), (5c)) in
// registers: the device code, the row-count dispatch and the segment layouts, shared by the single
// solves (k_tri.hip) and the vorticity + stream-vector pair solves (k_tri_pair.hip).
#pragma once

#include "spectral.h"

namespace vs {

// Segment layout for M interior rows: S lanes per mode, at most LMAX rows per lane; 0 = the
// two-lane solve (M < 4 or M > 256).
int seg_shape(int M);

namespace {

// ---------------------------------------------------------------- segmented tridiagonal solve
// Partition solve of T x = f for one mode, T = tridiag(1, beta, 1) of size M with zero ends
// (the walls are folded into f). The column is cut into S consecutive segments, one lane each;
// a segment of L rows lives in registers. A 256-lane block owns 256/S consecutive modes, and
// its lanes are ordered mode-fastest, so each wave holds consecutive modes (consecutive q of
// one spectral row) of one or more segments and every row load or store covers whole runs.
// With G = T_L^{-1}, segment k obeys x_k = G (f_k - E_{k-1} e_1 - F_{k+1} e_L), where F_k, E_k
// are the first and last unknowns of segment k (E_{-1} = F_S = 0). Its ends give the coupled
// relations  F_k = p_k - g11 E_{k-1} - g1L F_{k+1},  E_k = q_k - g1L E_{k-1} - g11 F_{k+1}
// (p, q: ends of G f_k; g11 = G_11 = G_LL, g1L = G_1L = G_L1 since T_L is symmetric and
// persymmetric). A forward sweep over the segments, E_k = a_k - b_k F_{k+1},
// F_k = phi_k - chi_k F_{k+1}, and the back sweep both run redundantly in every lane of the
// mode, after the segment ends are exchanged through LDS. The segment is then finished from
// its forward-eliminated rows d'_j:
// the corrections of f enter d' as -E_{k-1} pi_j (pi = forward elimination of e_1) and
// -F_{k+1} c'_L at the last row. Pivots c'_j = 1/(beta - c'_{j-1}) come from the class table,
// so no lane divides in the row loops; beta itself is the table's last row.
//
// Segments have Lm rows (the first nlong of them) or Lm - 1 rows. Every lane walks Lm rows so
// that the row loops depend on wave-uniform values only; a short segment's extra last row is a
// phantom whose value is forced to zero by selects on the last two rows.
// Buffer-instruction access for the segmented solve (see seg_load).
typedef __amdgpu_buffer_rsrc_t BufRes;
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ BufRes buf_res(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ double buf_ld(BufRes r, unsigned voff, unsigned soff, const double*) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
__device__ __forceinline__ double buf_ld(BufRes r, unsigned voff, unsigned soff, const float*) {
    return (double)__builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
__device__ __forceinline__ void buf_st(BufRes r, unsigned voff, unsigned soff, double v, double*) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, voff, soff, 0);
}
__device__ __forceinline__ void buf_st(BufRes r, unsigned voff, unsigned soff, double v, float*) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, (float)v), r, voff, soff, 0);
}

// T: the arithmetic type of the solve (that of the spectral storage: FP64, or FP32 in the
// refined mode); the pivots come from the FP64 table, rounded to T.
template <int LMAX, class T>
struct SegCoef {
    T c[LMAX];
    T beta, g11l, g11s, g1ll, g1ls;   // G_11 and G_1L for Lm and Lm - 1 rows
};

template <int LMAX, class T>
__device__ __forceinline__ void seg_coef(SegCoef<LMAX, T>& cf, const double* __restrict__ tri,
                                         unsigned cls, unsigned ncls, int M, int Lm) {
    const BufRes r = buf_res(tri, (unsigned)(M + 1) * ncls * 8u);
#pragma unroll
    for (int u = 0; u < LMAX; ++u) cf.c[u] = (u < Lm) ? (T)buf_ld(r, cls * 8u, u * ncls * 8u, tri) : (T)0;
    cf.beta = (T)buf_ld(r, cls * 8u, (unsigned)M * ncls * 8u, tri);
    // G_11(L) = c'_L; G_1L(L) = (-1)^(L-1) c'_1 ... c'_L
    T prod = 1;
    cf.g11l = cf.g11s = cf.g1ll = cf.g1ls = 0;
#pragma unroll
    for (int u = 0; u < LMAX; ++u) {
        if (u < Lm) {
            prod *= -cf.c[u];
            if (u == Lm - 2) {
                cf.g1ls = -prod;
                cf.g11s = cf.c[u];
            }
            if (u == Lm - 1) {
                cf.g1ll = -prod;
                cf.g11l = cf.c[u];
            }
        }
    }
}

// xch: 512 values of LDS for the exchange of the segment ends; every thread of the 256-thread
// block calls this (it holds two barriers).
template <int S, int LMAX, class T>
__device__ __forceinline__ void seg_solve(T (&x)[LMAX], const SegCoef<LMAX, T>& cf, int k,
                                          bool shortl, int Lm, int nlong, T* xch) {
    const T* c = cf.c;
    // forward elimination in place; q = last d', piL = pi at the last row (phantom row zeroed)
    T acc = 0, pi = 0, q = 0, piL = 0;
#pragma unroll
    for (int u = 0; u < LMAX; ++u) {
        if (u < Lm) {
            acc = c[u] * (x[u] - acc);
            pi = (u == 0) ? c[0] : -c[u] * pi;
            if (u == Lm - 2) {
                q = acc;
                piL = pi;
            }
            if (u == Lm - 1) {
                q = shortl ? q : acc;
                piL = shortl ? piL : pi;
                x[u] = shortl ? (T)0 : acc;
            } else {
                x[u] = acc;
            }
        }
    }
    // p = first unknown of the zero-end segment solve (back substitution, nothing stored)
    T p = 0;
#pragma unroll
    for (int u = LMAX - 1; u >= 0; --u)
        if (u < Lm) p = x[u] - c[u] * p;
    // reduced system. Every segment's p and q are gathered first (through LDS: the S lanes of
    // a mode sit 256/S lanes apart); every lane then runs the forward sweep and the back
    // substitution of the whole reduced system itself, keeping phi and chi of every segment,
    // so no value has to travel between lanes after the gather.
    constexpr int NM = 256 / S;
    const int m = (int)threadIdx.x % NM;
    xch[threadIdx.x] = p;
    xch[256 + threadIdx.x] = q;
    __syncthreads();
    T P[S], Q[S];
#pragma unroll
    for (int kk = 0; kk < S; ++kk) {
        P[kk] = xch[kk * NM + m];
        Q[kk] = xch[256 + kk * NM + m];
    }
    __syncthreads();   // xch is free again
    T a = 0, b = 0, alp = 0, bep = 0;
    T PH[S], CH[S];
#pragma unroll
    for (int kk = 0; kk < S; ++kk) {
        const bool lng = nlong == 0 || kk < nlong;   // nlong = 0: all segments have Lm rows
        const T g11 = lng ? cf.g11l : cf.g11s;
        const T g1l = lng ? cf.g1ll : cf.g1ls;
        const T rden = (T)1 / ((T)1 - g11 * b);
        const T ph = (P[kk] - g11 * a) * rden;
        const T ch = g1l * rden;
        const T an = Q[kk] - g1l * a + g1l * b * ph;
        const T bn = g11 + g1l * b * ch;
        PH[kk] = ph;
        CH[kk] = ch;
        if (kk == k - 1) {   // alpha, beta of the segment before this lane's
            alp = an;
            bep = bn;
        }
        a = an;
        b = bn;
    }
    // back substitution F_kk = phi_kk - chi_kk F_{kk+1} (F_S = 0); this lane keeps F_k, F_{k+1}
    T F = 0, Fk = 0, Fnext = 0;
#pragma unroll
    for (int kk = S - 1; kk >= 0; --kk) {
        if (kk == k) Fnext = F;
        F = PH[kk] - CH[kk] * F;
        if (kk == k) Fk = F;
    }
    // E_{k-1} = alpha_{k-1} - beta_{k-1} F_k
    const T Eprev = k > 0 ? alp - bep * Fk : (T)0;
    // finish the segment bottom up
    T xn = 0, pc = 0;
#pragma unroll
    for (int u = LMAX - 1; u >= 0; --u) {
        if (u < Lm) {
            T f;
            if (u == Lm - 1) {
                pc = shortl ? (T)0 : piL;
                f = shortl ? (T)0 : Fnext * c[u];
            } else if (u == Lm - 2) {
                pc = shortl ? piL : -pc * (cf.beta - c[u]);
                f = shortl ? Fnext * c[u] : (T)0;
            } else {
                pc = -pc * (cf.beta - c[u]);
                f = 0;
            }
            xn = (x[u] - Eprev * pc - f) - c[u] * xn;
            x[u] = xn;
        }
    }
}

template <int S>
struct SegLane {
    int p, q, k, Lm, nlong;
    int a;          // first interior row (0-based) of the lane's segment
    bool act, shortl;
    unsigned cls, ncls;
    unsigned off;   // offset of (p, first row of the segment, q); grids stay below 2^31 nodes
};

template <int S>
__device__ __forceinline__ SegLane<S> seg_lane(const Dims& d) {
    SegLane<S> sl;
    // a block owns 256/S consecutive modes; lane t of the block takes mode t % (256/S) and
    // segment t / (256/S), so the lanes of a wave hold consecutive modes (consecutive q) of
    // one or two segments, and a row's loads and stores cover whole runs of a spectral row
    constexpr int NM = 256 / S;
    const int mode = (int)blockIdx.x * NM + (int)threadIdx.x % NM;   // blockIdx.x: mode block
    sl.k = (int)threadIdx.x / NM;
    sl.act = mode < d.nx * d.nz;
    const int mm = sl.act ? mode : 0;
    sl.p = mm / d.nz;
    sl.q = mm - sl.p * d.nz;
    const int base = d.M / S;
    sl.nlong = d.M - base * S;
    sl.Lm = base + (sl.nlong > 0);
    sl.shortl = sl.nlong > 0 && sl.k >= sl.nlong;
    const int a = sl.k * base + min(sl.k, sl.nlong);
    sl.a = a;
    const int pc = min(sl.p, d.nx - sl.p);
    const int qc = min(sl.q, d.nz - sl.q);
    sl.ncls = (unsigned)((d.nx / 2 + 1) * (d.nz / 2 + 1));
    sl.cls = (unsigned)(pc * (d.nz / 2 + 1) + qc);
    sl.off = (unsigned)(sl.p * d.ny * d.nz + (1 + a) * d.nz + sl.q);
    return sl;
}

// Segment rows go through buffer instructions: one buffer resource per array (wave-uniform),
// the lane's 32-bit byte offset in a VGPR and the row offset u * sj in an SGPR, so no lane
// keeps an address per row. Accesses beyond the array's extent read zero and drop stores.
// A short segment's phantom row reads the next segment's first row, or the wall row
// j = ny-1: in bounds, and zeroed by the solve.
template <int S, int LMAX, class ST>
__device__ __forceinline__ void seg_load(ST (&x)[LMAX], const ST* base, unsigned nelem,
                                         unsigned off, unsigned sj, int Lm, ST scale) {
    const BufRes r = buf_res(base, nelem * (unsigned)sizeof(ST));
    const unsigned vo = off * (unsigned)sizeof(ST);
#pragma unroll
    for (int u = 0; u < LMAX; ++u)
        x[u] = (u < Lm) ? scale * (ST)buf_ld(r, vo, u * sj * (unsigned)sizeof(ST), base) : (ST)0;
}

template <int S, int LMAX, class ST>
__device__ __forceinline__ void seg_store(const ST (&x)[LMAX], ST* base, unsigned nelem,
                                          unsigned sj, const SegLane<S>& sl) {
    const BufRes r = buf_res(base, nelem * (unsigned)sizeof(ST));
    const unsigned vo = sl.off * (unsigned)sizeof(ST);
    if (!sl.act) return;
#pragma unroll
    for (int u = 0; u < LMAX; ++u) {
        const unsigned so = u * sj * (unsigned)sizeof(ST);
        if (u < sl.Lm - 1) buf_st(r, vo, so, x[u], base);
        if (u == sl.Lm - 1 && !sl.shortl) buf_st(r, vo, so, x[u], base);
    }
}

// Segmented solves. Grids with ny = n in {32, 48, 64, 96, 128, 256} (M = n - 2) get their
// segment lengths and long-segment counts as compile-time constants, other M in [17, 256] in FP64
// the length alone: with a run-time length every row of the unrolled loops sits behind a branch,
// which keeps the loads from being in flight together (pair solves at
// 72 x 51 x 108 17.9 -> 9.2 us, 96 x 112 x 96 32 -> 17, 128 x 120 x 128 66 -> 26). M below 17 and FP32
// with another M than those of the six grids take a run-time length (compile-time ones were not
// measured there).
#define VS_SEG_L(X, C, S_, L_) case C + L_: X(S_, L_, L_, -1); return true;
#define VS_SEG_L8(X, C, S_)                                                                    \
    VS_SEG_L(X, C, S_, 9) VS_SEG_L(X, C, S_, 10) VS_SEG_L(X, C, S_, 11) VS_SEG_L(X, C, S_, 12) \
    VS_SEG_L(X, C, S_, 13) VS_SEG_L(X, C, S_, 14) VS_SEG_L(X, C, S_, 15) VS_SEG_L(X, C, S_, 16)
#define VS_SEG_SHAPES(X)                                                                       \
    switch (d.M) {                                                                             \
    case 30: X(4, 8, 8, 2); return true;                                                       \
    case 46: X(4, 16, 12, 2); return true;                                                     \
    case 62: X(4, 16, 16, 2); return true;                                                     \
    case 94: X(8, 16, 12, 6); return true;                                                     \
    case 126: X(8, 16, 16, 6); return true;                                                    \
    case 254: X(16, 16, 16, 14); return true;                                                  \
    default: break;                                                                            \
    }                                                                                          \
    if constexpr (sizeof(ST) == 8) {                                                           \
        const int sc = d.M <= 64 ? 0 : d.M <= 128 ? 100 : 200;                                 \
        const int sg = sc == 0 ? 4 : sc == 100 ? 8 : 16;                                       \
        if (d.M >= 17 && d.M <= 256) switch (sc + (d.M + sg - 1) / sg) {                       \
            VS_SEG_L(X, 0, 4, 5) VS_SEG_L(X, 0, 4, 6) VS_SEG_L(X, 0, 4, 7)                     \
            VS_SEG_L(X, 0, 4, 8) VS_SEG_L8(X, 0, 4) VS_SEG_L8(X, 100, 8)                       \
            VS_SEG_L8(X, 200, 16)                                                              \
            default: break;                                                                    \
        }                                                                                      \
    }                                                                                          \
    switch (seg_shape(d.M)) {                                                                  \
    case 8: X(4, 8, 0, 0); return true;                                                        \
    case 16: X(4, 16, 0, 0); return true;                                                      \
    case 32: X(4, 32, 0, 0); return true;                                                      \
    case 832: X(8, 32, 0, 0); return true;                                                     \
    default: return false;                                                                     \
    }

}  // namespace
}  // namespace vs
