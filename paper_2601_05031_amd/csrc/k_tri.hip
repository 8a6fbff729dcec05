// Tridiagonal solves in y of one Poisson problem per component (main text eq. (5b) or (5c)) per
// Hartley mode: the segmented register solve (tri_seg.h), and the two-lane solves of very short or
// tall columns.
#include <type_traits>

#include "tri_seg.h"

namespace vs {

namespace {

// Twisted tridiagonal solve of
//   U_{j-1} + beta U_j + U_{j+1} = f_j,  j = 1..M,  U_0 = U_{M+1} = 0,
// beta = 2 cos(2 pi p/nx) + 2 cos(2 pi q/nz) - 6, shared by a lane pair: the even lane
// eliminates rows 1..m downwards (pivots c'_s = 1/(beta - c'_{s-1}), rows read as
// U_j + c'_j U_{j+1} = d'_j), the odd lane rows M..m+1 upwards with the same pivots counted
// from the bottom (the matrix is symmetric Toeplitz), the two meet in a 2x2 system at rows
// m, m+1 (values exchanged by a lane shuffle), then each back-substitutes away from the
// middle. f_j = rhs(j, v) with v the value read at row j of rd; d' and then U are written to
// wr (which may alias rd). Pivots come from cp[s * ncls]; loads run one chunk ahead. All lanes
// of the wave call this together; inactive lanes pass act = false.
// INPLACE: rd == wr (one pointer is used for both); otherwise rd and wr are distinct buffers.
template <bool INPLACE, class ST, class Rhs>
__device__ __forceinline__ void twisted_half(const ST* __restrict__ rd, ST* __restrict__ wr,
                                             long sj, int M, int half, bool act,
                                             const double* __restrict__ cp, size_t ncls, Rhs rhs) {
    const int m = (M + 1) / 2;
    const int nr = act ? (half ? M - m : m) : 0;      // rows eliminated by this lane
    const int j0 = half ? M : 1;                       // row of step 0 (the wall end)
    const int jd = half ? -1 : 1;
    const long dj = jd * sj;
    ST* wb = wr + (long)j0 * sj;
    const ST* rb = INPLACE ? wb : rd + (long)j0 * sj;
    constexpr int CH = 8;
    double fv[CH], cv[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u) {
        fv[u] = (u < nr) ? rhs(j0 + u * jd, ld(rb + u * dj)) : 0.0;
        cv[u] = (u < nr) ? cp[(size_t)u * ncls] : 0.0;
    }
    double acc = 0.0, clast = 0.0;
    for (int s0 = 0; s0 < nr; s0 += CH) {
        double nf[CH], nc[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int sn = s0 + CH + u;
            nf[u] = (sn < nr) ? rhs(j0 + sn * jd, ld(rb + sn * dj)) : 0.0;
            nc[u] = (sn < nr) ? cp[(size_t)sn * ncls] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            if (s0 + u < nr) {
                acc = cv[u] * (fv[u] - acc);
                clast = cv[u];
                st(wb + (s0 + u) * dj, acc);
            }
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            fv[u] = nf[u];
            cv[u] = nc[u];
        }
    }
    // interface: top lane holds (d'_m, c'_m), bottom lane (g'_{m+1}, e'_{m+1}); a lane with no
    // rows contributes (0, 0), i.e. the wall value U = 0.
    const double oacc = __shfl_xor(acc, 1, 64);
    const double oc = __shfl_xor(clast, 1, 64);
    if (nr == 0) return;
    const double dm = half ? oacc : acc, cm = half ? oc : clast;
    const double gm = half ? acc : oacc, em = half ? clast : oc;
    const double Um = (dm - cm * gm) / (1.0 - cm * em);
    double unext = half ? (gm - em * Um) : Um;        // U at this lane's last row
    st(wb + (nr - 1) * dj, unext);
    // back substitution from step nr-2 towards the wall: U = d' - c' U_next
#pragma unroll
    for (int u = 0; u < CH; ++u) {
        const int sn = nr - 2 - u;
        fv[u] = (sn >= 0) ? ld(wb + sn * dj) : 0.0;
        cv[u] = (sn >= 0) ? cp[(size_t)(sn >= 0 ? sn : 0) * ncls] : 0.0;
    }
    for (int s0 = nr - 2; s0 >= 0; s0 -= CH) {
        double nf[CH], nc[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int sn = s0 - CH - u;
            nf[u] = (sn >= 0) ? ld(wb + sn * dj) : 0.0;
            nc[u] = (sn >= 0) ? cp[(size_t)(sn >= 0 ? sn : 0) * ncls] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            if (s0 - u >= 0) {
                unext = fv[u] - cv[u] * unext;
                st(wb + (s0 - u) * dj, unext);
            }
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            fv[u] = nf[u];
            cv[u] = nc[u];
        }
    }
}

struct ModeLane {
    int p, q, half;
    bool act;
    const double* cp;
    size_t ncls;
    long off;   // offset of the (p, row 0, q) element
};

__device__ __forceinline__ ModeLane mode_lane(const Dims& d, const double* __restrict__ tri) {
    ModeLane ml;
    const int t = blockIdx.x * 64 + threadIdx.x;
    const int pair = t >> 1;
    ml.half = t & 1;
    ml.act = pair < d.nx * d.nz;
    const int pp = ml.act ? pair : 0;
    ml.p = pp / d.nz;
    ml.q = pp - ml.p * d.nz;
    const int pc = min(ml.p, d.nx - ml.p);
    const int qc = min(ml.q, d.nz - ml.q);
    ml.ncls = (size_t)(d.nx / 2 + 1) * (d.nz / 2 + 1);
    ml.cp = tri + (size_t)(pc * (d.nz / 2 + 1) + qc);
    ml.off = (long)ml.p * d.ny * d.nz + ml.q;
    return ml;
}

// tridiag_y: one Poisson problem per component blockIdx.y: f_j = scale * B_j (B = the 2D
// Hartley spectrum of the right-hand side, scale = h^2/(nx nz)), in place.
// wlo, whi: wall terms folded into mode (0, 0) (zero when the right-hand side holds them).
template <class ST>
__global__ __launch_bounds__(64) void k_tridiag_y(Dims d, const double* __restrict__ tri,
                                                 SPtr3<ST> spec, const int* gate, double scale,
                                                 double3 wlo, double3 whi) {
    if (gate && *gate) return;
    const ModeLane ml = mode_lane(d, tri);
    const int c = blockIdx.y;
    ST* col = spec.p[c] + ml.off;
    const bool m00 = (ml.p == 0 && ml.q == 0);
    const double a = c == 0 ? wlo.x : (c == 1 ? wlo.y : wlo.z);
    const double b = c == 0 ? whi.x : (c == 1 ? whi.y : whi.z);
    const int M = d.M;
    twisted_half<true, ST>(nullptr, col, d.nz, d.M, ml.half, ml.act, ml.cp, ml.ncls,
                           [&](int j, double v) {
                               double f = scale * v;
                               if (m00) {
                                   if (j == 1) f -= a;
                                   if (j == M) f -= b;
                               }
                               return f;
                           });
}

// tridiag_psi: the stream-vector problem lap psi = -w from the vorticity modes U_w = T w/(nx nz)
// left in spec by tridiag_y (T the 2D Hartley transform): its transformed right-hand side is
// -(nx nz) U_w minus the wall terms, whose transform for wall values constant over each wall
// plane lives only in mode (0, 0):
//   f_j = -h^2 U_w(j) - [p = q = 0] ([j = 1] psi_lo + [j = M] psi_hi);
// solved into spec2, leaving spec unchanged.
template <class ST>
__global__ __launch_bounds__(64) void k_tridiag_psi(Dims d, const double* __restrict__ tri,
                                                   SPtr3<ST> spec, SPtr3<ST> spec2, double3 plo,
                                                   double3 phi_, const int* gate) {
    if (gate && *gate) return;
    const ModeLane ml = mode_lane(d, tri);
    const int c = blockIdx.y;
    const ST* col = spec.p[c] + ml.off;
    ST* col2 = spec2.p[c] + ml.off;
    const bool m00 = (ml.p == 0 && ml.q == 0);
    const double wlo = c == 0 ? plo.x : (c == 1 ? plo.y : plo.z);
    const double whi = c == 0 ? phi_.x : (c == 1 ? phi_.y : phi_.z);
    const double h2 = d.h * d.h;
    const int M = d.M;
    twisted_half<false, ST>(col, col2, d.nz, d.M, ml.half, ml.act, ml.cp, ml.ncls, [&](int j, double v) {
        double f = -h2 * v;
        if (m00) {
            if (j == 1) f -= wlo;
            if (j == M) f -= whi;
        }
        return f;
    });
}

// Segmented tridiag_y: f_j = scale * B_j per component blockIdx.y, solved in place.
// LMF, NLF: the segment length Lm and long-segment count nlong fixed at compile time (LMF = 0: both
// taken from M at run time; NLF = -1: the count alone).
template <int S, int LMAX, class ST, int LMF, int NLF>
__global__ __launch_bounds__(256) void k_tridiag_seg(Dims d, const double* __restrict__ tri,
                                                    SPtr3<ST> spec, const int* gate, double scale) {
    if (gate && *gate) return;
    SegLane<S> sl = seg_lane<S>(d);
    if (LMF) sl.Lm = LMF;
    if (LMF && NLF >= 0) {
        sl.nlong = NLF;
        sl.shortl = NLF > 0 && sl.k >= NLF;
    }
    __shared__ ST xch[512];
    SegCoef<LMAX, ST> cf;
    seg_coef<LMAX, ST>(cf, tri, sl.cls, sl.ncls, d.M, sl.Lm);
    ST* col = spec.p[blockIdx.y];
    const unsigned N = (unsigned)(d.nx * d.ny * d.nz);
    ST x[LMAX];
    seg_load<S, LMAX, ST>(x, col, N, sl.off, d.nz, sl.Lm, (ST)scale);
    seg_solve<S, LMAX, ST>(x, cf, sl.k, sl.shortl, sl.Lm, sl.nlong, xch);
    seg_store<S, LMAX, ST>(x, col, N, d.nz, sl);
}

}  // namespace

// Segment layout for M interior rows: S lanes per mode, at most LMAX rows per lane.
// 0 = the twisted two-lane solve (M < 4 or M > 256).
int seg_shape(int M) {
    if (M < 4 || M > 256) return 0;
    if (M <= 32) return 8;
    if (M <= 64) return 16;
    if (M <= 128) return 32;
    return 832;   // S = 8, LMAX = 32
}

template <int S, int LMAX, class ST, int LMF, int NLF>
void seg_launch_single(hipStream_t s, const Dims& d, const double* tri, void* const spec[3],
                       int ncomp, const int* gate) {
    const double scale = d.h * d.h / ((double)d.nx * d.nz);
    const dim3 grid((unsigned)(((long)d.nx * d.nz * S + 255) / 256), ncomp);
    launch_kernel((k_tridiag_seg<S, LMAX, ST, LMF, NLF>), grid, dim3(256), 0, s, d, tri,
                  sptr<ST>(spec, ncomp), gate, scale);
}

template <class ST>
bool seg_single(hipStream_t s, const Dims& d, const double* tri, void* const spec[3], int ncomp,
                const int* gate) {
#define VS_X(S_, L_, F_, N_) seg_launch_single<S_, L_, ST, F_, N_>(s, d, tri, spec, ncomp, gate)
    VS_SEG_SHAPES(VS_X)
#undef VS_X
}

template <class ST>
void tridiag_y_t(hipStream_t s, const Dims& d, const double* tri, void* const spec[3], int ncomp,
                 const int* gate) {
    const double3 z = make_double3(0.0, 0.0, 0.0);
    if (seg_single<ST>(s, d, tri, spec, ncomp, gate)) return;
    const double scale = d.h * d.h / ((double)d.nx * d.nz);
    const dim3 grid((2 * d.nx * d.nz + 63) / 64, ncomp);
    launch_kernel(k_tridiag_y<ST>, grid, dim3(64), 0, s, d, tri, sptr<ST>(spec, ncomp), gate,
                  scale, z, z);
}

void launch_tridiag_y(hipStream_t s, const Dims& d, const double* tri, void* const spec[3],
                      int ncomp, bool f32, const int* gate) {
    if (f32)
        tridiag_y_t<float>(s, d, tri, spec, ncomp, gate);
    else
        tridiag_y_t<double>(s, d, tri, spec, ncomp, gate);
}

void launch_tri_pair(hipStream_t s, const Dims& d, bool f32, bool corr, const Over<TriArgs>& a) {
    if (seg_tri_pair(s, d, f32, corr, a)) return;
    // M < 4 or M > 256: the two-lane solves, one instance (no correction form)
    const TriArgs& t = a.one;
    const double scale = d.h * d.h / ((double)d.nx * d.nz);
    const dim3 grid((2 * d.nx * d.nz + 63) / 64, 3);
    const double3 olo = make_double3(t.olo[0], t.olo[1], t.olo[2]);
    const double3 ohi = make_double3(t.ohi[0], t.ohi[1], t.ohi[2]);
    const double3 lo = make_double3(t.plo[0], t.plo[1], t.plo[2]);
    const double3 hi = make_double3(t.phi[0], t.phi[1], t.phi[2]);
    void* const sp[3] = {t.spec[0], t.spec[1], t.spec[2]};
    void* const sp2[3] = {t.spec2[0], t.spec2[1], t.spec2[2]};
    if (f32) {
        launch_kernel(k_tridiag_y<float>, grid, dim3(64), 0, s, d, t.triw, sptr<float>(sp, 3),
                      t.gate, scale, olo, ohi);
        launch_kernel(k_tridiag_psi<float>, grid, dim3(64), 0, s, d, t.tri, sptr<float>(sp, 3),
                      sptr<float>(sp2, 3), lo, hi, t.gate);
    } else {
        launch_kernel(k_tridiag_y<double>, grid, dim3(64), 0, s, d, t.triw, sptr<double>(sp, 3),
                      t.gate, scale, olo, ohi);
        launch_kernel(k_tridiag_psi<double>, grid, dim3(64), 0, s, d, t.tri, sptr<double>(sp, 3),
                      sptr<double>(sp2, 3), lo, hi, t.gate);
    }
}

void launch_tridiag_pair(hipStream_t s, const Dims& d, const double* tri, const double* triw,
                         void* const spec[3], void* const spec2[3], const double om_lo[3],
                         const double om_hi[3], const double psi_lo[3], const double psi_hi[3],
                         bool f32) {
    TriArgs t{};
    t.tri = tri;
    t.triw = triw ? triw : tri;
    for (int c = 0; c < 3; ++c) {
        t.spec[c] = spec[c];
        t.spec2[c] = spec2[c];
        t.olo[c] = om_lo[c];
        t.ohi[c] = om_hi[c];
        t.plo[c] = psi_lo[c];
        t.phi[c] = psi_hi[c];
    }
    t.gate = nullptr;
    launch_tri_pair(s, d, f32, false, over_one(t));
}

}  // namespace vs
