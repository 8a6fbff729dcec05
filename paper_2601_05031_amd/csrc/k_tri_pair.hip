// Segmented vorticity + stream-vector tridiagonal solves of a step's flow pass (main text eq. (5b),
// then (5c)); the device code is in tri_seg.h.
#include <type_traits>

#include "tri_seg.h"

namespace vs {

namespace {

// Segmented vorticity + stream-vector pair: the vorticity modes U_w (f = scale * B) are solved
// and stored in spec, then the stream-vector problem lap psi = -w is solved from them in
// registers, f_j = -h^2 U_w(j) - [p = q = 0]([j = 1] psi_lo + [j = M] psi_hi), into spec2.
// triw holds the vorticity's pivots: tri itself, or those of the shifted operator L_h - a of
// the inertial variant (SM eq. (36)).
// CORR (the corrections of a defect-correction cycle, homogeneous walls): spec holds the
// transformed vorticity residual R_w and spec2 the stream-vector residual R_psi; the
// corrections are U_ew = T^{-1}(scale R_w) and U_epsi = T^{-1}(scale R_psi - h^2 U_ew), since the
// stream-vector correction solves L e_psi = r_psi - e_w.
// Grid: x = mode blocks, y = component (3) [x instances].
template <int S, int LMAX, class ST, int LMF, int NLF, bool CORR, bool BATCH>
__global__ __launch_bounds__(256) void k_tridiag_pair_seg(Dims d, TriArgs one,
                                                         const TriArgs* __restrict__ tab) {
    const int inst = BATCH ? (int)blockIdx.y / 3 : 0;
    const int c3 = (int)blockIdx.y - inst * 3;
    const TriArgs& ta = inst_args<BATCH>(one, tab, inst);
    if (ta.gate && *ta.gate) return;
    SegLane<S> sl = seg_lane<S>(d);
    if (LMF) sl.Lm = LMF;
    if (LMF && NLF >= 0) {
        sl.nlong = NLF;
        sl.shortl = NLF > 0 && sl.k >= NLF;
    }
    __shared__ ST xch[512];
    SegCoef<LMAX, ST> cf;
    seg_coef<LMAX, ST>(cf, ta.triw, sl.cls, sl.ncls, d.M, sl.Lm);
    ST* col = (ST*)pick(ta.spec, c3);
    ST* col2 = (ST*)pick(ta.spec2, c3);
    const unsigned N = (unsigned)(d.nx * d.ny * d.nz);
    const ST scale = (ST)(d.h * d.h / ((double)d.nx * d.nz));
    ST x[LMAX];
    seg_load<S, LMAX, ST>(x, col, N, sl.off, d.nz, sl.Lm, scale);
    ST y[LMAX];
    if (CORR) seg_load<S, LMAX, ST>(y, col2, N, sl.off, d.nz, sl.Lm, scale);
    const bool m00 = sl.p == 0 && sl.q == 0;
    // the row j = M is the last real row of segment S - 1 (short if nlong > 0)
    const int ulast = sl.nlong > 0 ? sl.Lm - 2 : sl.Lm - 1;
    if (!CORR) {
        // vorticity wall terms, constant over each wall plane: mode (0, 0) only
        const ST a = (ST)pick(ta.olo, c3);
        const ST b = (ST)pick(ta.ohi, c3);
#pragma unroll
        for (int u = 0; u < LMAX; ++u) {
            if (m00 && sl.k == 0 && u == 0) x[u] -= a;
            if (m00 && sl.k == S - 1 && u == ulast) x[u] -= b;
        }
    }
    seg_solve<S, LMAX, ST>(x, cf, sl.k, sl.shortl, sl.Lm, sl.nlong, xch);
    seg_store<S, LMAX, ST>(x, col, N, d.nz, sl);
    // the stream-vector problem has no shift: its own pivots when the vorticity's differ
    if (ta.triw != ta.tri) seg_coef<LMAX, ST>(cf, ta.tri, sl.cls, sl.ncls, d.M, sl.Lm);
    const ST h2 = (ST)(d.h * d.h);
    const ST wlo = CORR ? (ST)0 : (ST)pick(ta.plo, c3);
    const ST whi = CORR ? (ST)0 : (ST)pick(ta.phi, c3);
#pragma unroll
    for (int u = 0; u < LMAX; ++u) {
        ST f = CORR ? y[u] - h2 * x[u] : -h2 * x[u];
        if (m00 && sl.k == 0 && u == 0) f -= wlo;
        if (m00 && sl.k == S - 1 && u == ulast) f -= whi;
        x[u] = f;
    }
    seg_solve<S, LMAX, ST>(x, cf, sl.k, sl.shortl, sl.Lm, sl.nlong, xch);
    seg_store<S, LMAX, ST>(x, col2, N, d.nz, sl);
}

template <int S, int LMAX, class ST, int LMF, int NLF>
void seg_launch_pair(hipStream_t s, const Dims& d, bool corr, const Over<TriArgs>& a) {
    const unsigned ni = a.tab ? (unsigned)a.n : 1u;
    const dim3 grid((unsigned)(((long)d.nx * d.nz * S + 255) / 256), 3 * ni);
    if constexpr (sizeof(ST) == 4) {   // the correction form serves the refined mode only
        if (corr) {
            if (a.tab) launch_kernel((k_tridiag_pair_seg<S, LMAX, ST, LMF, NLF, true, true>), grid, dim3(256), 0, s, d, a.one, a.tab);
            else launch_kernel((k_tridiag_pair_seg<S, LMAX, ST, LMF, NLF, true, false>), grid, dim3(256), 0, s, d, a.one, a.tab);
            return;
        }
    }
    {
        if (a.tab) launch_kernel((k_tridiag_pair_seg<S, LMAX, ST, LMF, NLF, false, true>), grid, dim3(256), 0, s, d, a.one, a.tab);
        else launch_kernel((k_tridiag_pair_seg<S, LMAX, ST, LMF, NLF, false, false>), grid, dim3(256), 0, s, d, a.one, a.tab);
    }
}

// The pair solves have a second layout for each compile-time row count, twice (or half) the
// lanes per mode, which the autotuner may pick (seg_alt).
template <class ST>
bool seg_pair(hipStream_t s, const Dims& d, bool corr, const Over<TriArgs>& a) {
#define VS_X(S_, L_, F_, N_) seg_launch_pair<S_, L_, ST, F_, N_>(s, d, corr, a)
    if (tuning_for(d).seg_alt) {
        switch (d.M) {
        case 30: VS_X(8, 4, 4, 6); return true;
        case 46: VS_X(8, 8, 6, 6); return true;
        case 62: VS_X(8, 8, 8, 6); return true;
        case 94: VS_X(16, 8, 6, 14); return true;
        case 126: VS_X(16, 8, 8, 14); return true;
        case 254: VS_X(8, 32, 32, 6); return true;
        default: break;
        }
    }
    VS_SEG_SHAPES(VS_X)
#undef VS_X
}

}  // namespace

bool seg_has_alt(int M) {
    return M == 30 || M == 46 || M == 62 || M == 94 || M == 126 || M == 254;
}

bool seg_tri_pair(hipStream_t s, const Dims& d, bool f32, bool corr, const Over<TriArgs>& a) {
    return f32 ? seg_pair<float>(s, d, corr, a) : seg_pair<double>(s, d, corr, a);
}

}  // namespace vs
