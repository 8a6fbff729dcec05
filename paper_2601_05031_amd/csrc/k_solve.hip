// Residual norms and convergence checks that verify every Poisson solve (main text eq. (5b), (5c))
// on the device, and the residuals of the refined mode's correction cycles.
#include <type_traits>

#include "spectral.h"

namespace vs {

namespace {

// resid_norm: block partials of sum (b - L_h u)_c^2 and sum b~_c^2 over the interior. A block
// owns one component c and a slab of ci consecutive x-planes; each thread owns one interior
// (j, k) and walks the slab with u_c at x-1 and x kept in registers, so one new centre value
// is read per plane. Blocks are ordered per XCD. Streaming a single component (u_c and b_c)
// per block keeps two arrays in flight per wave instead of six, which runs close to the copy
// rate where reading every component at each node does not.
__global__ __launch_bounds__(kBlock) void k_resid_norm(Dims d, RhsArgs rhs, CPtr3 u, int ncomp,
                                                      SlabGrid sg, double* __restrict__ partials,
                                                      const int* gate, int slot0) {
    if (gate && *gate) return;
    __shared__ double sh[2 * 4];
    const int nb = sg.gx * sg.gi;
    const int lb0 = xcd_block(blockIdx.x, ncomp * nb);
    const int c = lb0 / nb;
    const int lb = lb0 - c * nb;
    const int bi = lb / sg.gx;
    const int t = (lb - bi * sg.gx) * kBlock + threadIdx.x;
    // block-uniform selects keep the pointer choice in scalar registers
    const double* uc = c == 0 ? u.p[0] : c == 1 ? u.p[1] : u.p[2];
    const double* fc = c == 0 ? rhs.f[0] : c == 1 ? rhs.f[1] : rhs.f[2];
    const double sgn = (rhs.mode == RHS_NEGW) ? -1.0 : 1.0;
    double rr = 0.0, bb = 0.0;
    if (t < d.M * d.nz) {
        const int jj = t / d.nz;
        const int k = t - jj * d.nz;
        const int j = jj + 1;
        const int plane = d.ny * d.nz;
        const int off = j * d.nz + k;
        const int kp = (k + 1 == d.nz) ? 0 : k + 1;
        const int km = (k == 0) ? d.nz - 1 : k - 1;
        const int i0 = bi * sg.ci;
        const int i1 = min(d.nx, i0 + sg.ci);
        const int im0 = (i0 == 0) ? d.nx - 1 : i0 - 1;
        double um = uc[im0 * plane + off];
        double ux = uc[i0 * plane + off];
#pragma unroll 2
        for (int i = i0; i < i1; ++i) {
            const int ip = (i + 1 == d.nx) ? 0 : i + 1;
            const int rb = i * plane + j * d.nz;
            const int c0 = rb + k;
            const double up = uc[ip * plane + off];
            const double b = sgn * fc[c0];
            const double ylo = uc[c0 - d.nz], yhi = uc[c0 + d.nz];
            const double w = (j == 1 ? ylo : 0.0) + (j == d.M ? yhi : 0.0);
            const double lap = (up + um + ylo + yhi + uc[rb + kp] + uc[rb + km] - 6.0 * ux) *
                               d.inv_h2;
            const double r = b - lap;
            const double bt = b - w * d.inv_h2;
            rr += r * r;
            bb += bt * bt;
            um = ux;
            ux = up;
        }
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    rr = wave_sum(rr);
    bb = wave_sum(bb);
    if (lane == 0) {
        sh[w] = rr;
        sh[4 + w] = bb;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const int q = threadIdx.x;
        partials[(slot0 + 3 * q + c) * kMaxPartialBlocks + lb] =
            sh[4 * q + 0] + sh[4 * q + 1] + sh[4 * q + 2] + sh[4 * q + 3];
    } else if (c == 0 && threadIdx.x < 8) {
        // the check sums three components: the blocks of component 0 clear the absent ones
        const int q = (threadIdx.x - 2) / 3, cc = (threadIdx.x - 2) - 3 * q;
        if (cc >= ncomp) partials[(slot0 + 3 * q + cc) * kMaxPartialBlocks + lb] = 0.0;
    }
}

// resid_flow: both residual norms of the flow solve in one pass, in the layout of resid_norm
// (vorticity in slots 0-5, stream vector in slots 6-11). A block owns one component c and
// streams omega_c, S_c and psi_c: omega_c is read once for both problems (its stencil for
// eq. (5b), its centre as the right-hand side -omega_c of eq. (5c)). Sums are those of
// resid_norm, term for term.
// This one-z form serves n_z not a multiple of 32 (k_resid_flow2 below takes the others).
// The source S is stored as SS (double, or float in the refined mode); sums are FP64.
template <bool BATCH, class SS>
__global__ __launch_bounds__(kBlock) void k_resid_flow(Dims d, SlabGrid sg, ResArgs one,
                                                      const ResArgs* __restrict__ tab) {
    __shared__ double sh[4 * 4];
    const int nb = sg.gx * sg.gi;
    const int lbi = xcd_block(blockIdx.x, gridDim.x);
    const int inst = BATCH ? lbi / (3 * nb) : 0;
    const ResArgs& ra = inst_args<BATCH>(one, tab, inst);
    if (ra.gate && *ra.gate) return;
    const double ashift = ra.ashift;
    Gl<double>* __restrict__ partials = (Gl<double>*)ra.part;
    const int lb0 = lbi - inst * 3 * nb;
    const int c = lb0 / nb;
    const int lb = lb0 - c * nb;
    const int bi = lb / sg.gx;
    const int t = (lb - bi * sg.gx) * kBlock + threadIdx.x;
    const Gl<double>* wc = (const Gl<double>*)(c == 0 ? ra.om[0] : c == 1 ? ra.om[1] : ra.om[2]);
    const Gl<SS>* sc = (const Gl<SS>*)(c == 0 ? ra.src[0] : c == 1 ? ra.src[1] : ra.src[2]);
    const Gl<double>* pc = (const Gl<double>*)(c == 0 ? ra.ps[0] : c == 1 ? ra.ps[1] : ra.ps[2]);
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    if (t < d.M * d.nz) {
        const int jj = t / d.nz;
        const int k = t - jj * d.nz;
        const int j = jj + 1;
        const int plane = d.ny * d.nz;
        const int off = j * d.nz + k;
        const int kp = (k + 1 == d.nz) ? 0 : k + 1;
        const int km = (k == 0) ? d.nz - 1 : k - 1;
        // z neighbours of u at plane row rb
        auto zpair = [&](const Gl<double>* u, int rb, double, double& zp, double& zm) {
            zp = u[rb + kp];
            zm = u[rb + km];
        };
        const int i0 = bi * sg.ci;
        const int i1 = min(d.nx, i0 + sg.ci);
        const int im0 = (i0 == 0) ? d.nx - 1 : i0 - 1;
        double wm = wc[im0 * plane + off], wx = wc[i0 * plane + off];
        double pm = pc[im0 * plane + off], px = pc[i0 * plane + off];
#pragma unroll 2
        for (int i = i0; i < i1; ++i) {
            const int ip = (i + 1 == d.nx) ? 0 : i + 1;
            const int rb = i * plane + j * d.nz;
            const int c0 = rb + k;
            const double wp = wc[ip * plane + off];
            const double pp = pc[ip * plane + off];
            {
                const double b = (double)sc[c0];
                const double ylo = wc[c0 - d.nz], yhi = wc[c0 + d.nz];
                const double w = (j == 1 ? ylo : 0.0) + (j == d.M ? yhi : 0.0);
                double zp, zm;
                zpair(wc, rb, wx, zp, zm);
                const double lap = (wp + wm + ylo + yhi + zp + zm - 6.0 * wx) * d.inv_h2;
                // the inertial variant solves (L_h - a) omega = b
                const double r = b - (ashift != 0.0 ? lap - ashift * wx : lap);
                const double bt = b - w * d.inv_h2;
                a[0] += r * r;
                a[1] += bt * bt;
            }
            {
                const double b = -wx;
                const double ylo = pc[c0 - d.nz], yhi = pc[c0 + d.nz];
                const double w = (j == 1 ? ylo : 0.0) + (j == d.M ? yhi : 0.0);
                double zp, zm;
                zpair(pc, rb, px, zp, zm);
                const double lap = (pp + pm + ylo + yhi + zp + zm - 6.0 * px) * d.inv_h2;
                const double r = b - lap;
                const double bt = b - w * d.inv_h2;
                a[2] += r * r;
                a[3] += bt * bt;
            }
            wm = wx;
            wx = wp;
            pm = px;
            px = pp;
        }
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const double v = wave_sum(a[q]);
        if (lane == 0) sh[4 * q + w] = v;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int q = threadIdx.x;   // 0: omega r, 1: omega b~, 2: psi r, 3: psi b~
        partials[(3 * q + c) * kMaxPartialBlocks + lb] =
            sh[4 * q + 0] + sh[4 * q + 1] + sh[4 * q + 2] + sh[4 * q + 3];
    }
}


// resid_flow with two consecutive z per lane: W lanes (64, 32 or 16) cover 2W consecutive z of
// one row, n_z a multiple of 2W. Every load moves 16 bytes, half the load instructions of the
// one-z form; the z neighbours inside the pair come from the pair itself, across lanes by
// width-W shuffles, and the segment's two edge values by one load each. The next plane's
// centres are loaded last (a scheduling barrier keeps them there), so they stay in flight
// while the current plane is summed. Same sums per node as k_resid_flow; a lane adds its two
// nodes' squares together.
template <int W, bool BATCH, class SS>
__global__ __launch_bounds__(kBlock) void k_resid_flow2(Dims d, SlabGrid sg, ResArgs one,
                                                       const ResArgs* __restrict__ tab) {
    __shared__ double sh[4 * 4];
    const int nb = sg.gx * sg.gi;
    const int lbi = xcd_block(blockIdx.x, gridDim.x);
    const int inst = BATCH ? lbi / (3 * nb) : 0;
    const ResArgs& ra = inst_args<BATCH>(one, tab, inst);
    if (ra.gate && *ra.gate) return;
    const double ashift = ra.ashift;
    Gl<double>* __restrict__ partials = (Gl<double>*)ra.part;
    const int lb0 = lbi - inst * 3 * nb;
    const int c = lb0 / nb;
    const int lb = lb0 - c * nb;
    const int bi = lb / sg.gx;
    const int t = (lb - bi * sg.gx) * kBlock + threadIdx.x;
    const Gl<double>* wc = (const Gl<double>*)(c == 0 ? ra.om[0] : c == 1 ? ra.om[1] : ra.om[2]);
    const Gl<SS>* sc = (const Gl<SS>*)(c == 0 ? ra.src[0] : c == 1 ? ra.src[1] : ra.src[2]);
    const Gl<double>* pc = (const Gl<double>*)(c == 0 ? ra.ps[0] : c == 1 ? ra.ps[1] : ra.ps[2]);
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    const int hz = d.nz >> 1;
    if (t < d.M * hz) {
        const int jj = t / hz;
        const int k = 2 * (t - jj * hz);
        const int j = jj + 1;
        const int plane = d.ny * d.nz;
        const int off = j * d.nz + k;
        const int ln = threadIdx.x & (W - 1);
        const int k0 = k - 2 * ln;
        const int kpe = (k0 + 2 * W == d.nz) ? 0 : k0 + 2 * W;
        const int kme = (k0 == 0) ? d.nz - 1 : k0 - 1;
        auto ld2v = [](const Gl<double>* q) { return ldg2(q); };
        auto zn = [&](double2 v, double em, double ep, double& zm0, double& zp1) {
            const double prev = __shfl_up(v.y, 1, W), next = __shfl_down(v.x, 1, W);
            zm0 = ln == 0 ? em : prev;
            zp1 = ln == W - 1 ? ep : next;
        };
        const int i0 = bi * sg.ci;
        const int i1 = min(d.nx, i0 + sg.ci);
        const int im0 = (i0 == 0) ? d.nx - 1 : i0 - 1;
        double2 wm = ld2v(wc + im0 * plane + off), wx = ld2v(wc + i0 * plane + off);
        double2 pm = ld2v(pc + im0 * plane + off), px = ld2v(pc + i0 * plane + off);
        const bool lo = j == 1, hi = j == d.M;
#pragma unroll 2
        for (int i = i0; i < i1; ++i) {
            const int ip = (i + 1 == d.nx) ? 0 : i + 1;
            const int rb = i * plane + j * d.nz;
            const int c0 = rb + k;
            const double2 b = ldg2(sc + c0);
            const double2 ylo = ld2v(wc + c0 - d.nz), yhi = ld2v(wc + c0 + d.nz);
            const double2 qlo = ld2v(pc + c0 - d.nz), qhi = ld2v(pc + c0 + d.nz);
            const int ome = rb + kme, ope = rb + kpe;
            const double wem = wc[ome], wep = wc[ope], pem = pc[ome], pep = pc[ope];
            // the next plane's centres last: they stay in flight while this plane is summed
            const double2 wp = ld2v(wc + ip * plane + off);
            const double2 pp = ld2v(pc + ip * plane + off);
            __builtin_amdgcn_sched_barrier(0);
            {
                double zm0, zp1;
                zn(wx, wem, wep, zm0, zp1);
                const double l0 = (wp.x + wm.x + ylo.x + yhi.x + wx.y + zm0 - 6.0 * wx.x) * d.inv_h2;
                const double l1 = (wp.y + wm.y + ylo.y + yhi.y + zp1 + wx.x - 6.0 * wx.y) * d.inv_h2;
                const double r0 = b.x - (ashift != 0.0 ? l0 - ashift * wx.x : l0);
                const double r1 = b.y - (ashift != 0.0 ? l1 - ashift * wx.y : l1);
                const double t0 = b.x - ((lo ? ylo.x : 0.0) + (hi ? yhi.x : 0.0)) * d.inv_h2;
                const double t1 = b.y - ((lo ? ylo.y : 0.0) + (hi ? yhi.y : 0.0)) * d.inv_h2;
                a[0] += r0 * r0 + r1 * r1;
                a[1] += t0 * t0 + t1 * t1;
            }
            {
                const double2 ylo = qlo, yhi = qhi;
                double zm0, zp1;
                zn(px, pem, pep, zm0, zp1);
                const double l0 = (pp.x + pm.x + ylo.x + yhi.x + px.y + zm0 - 6.0 * px.x) * d.inv_h2;
                const double l1 = (pp.y + pm.y + ylo.y + yhi.y + zp1 + px.x - 6.0 * px.y) * d.inv_h2;
                const double r0 = -wx.x - l0, r1 = -wx.y - l1;
                const double t0 = -wx.x - ((lo ? ylo.x : 0.0) + (hi ? yhi.x : 0.0)) * d.inv_h2;
                const double t1 = -wx.y - ((lo ? ylo.y : 0.0) + (hi ? yhi.y : 0.0)) * d.inv_h2;
                a[2] += r0 * r0 + r1 * r1;
                a[3] += t0 * t0 + t1 * t1;
            }
            wm = wx;
            wx = wp;
            pm = px;
            px = pp;
        }
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const double v = wave_sum(a[q]);
        if (lane == 0) sh[4 * q + w] = v;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int q = threadIdx.x;
        partials[(3 * q + c) * kMaxPartialBlocks + lb] =
            sh[4 * q + 0] + sh[4 * q + 1] + sh[4 * q + 2] + sh[4 * q + 3];
    }
}

// The first step of the refined mode's first correction cycle: both flow residuals at the
// predicted fields u* = u + p (p of order H: 0, the last increment i1, or 2 i1 - i2; the same
// arithmetic as the update of k_hz_out), r_w = S - L_h omega* (eq. (5b)) and
// r_psi = -omega* - L_h psi* (eq. (5c)), formed in FP64 and stored in FP32 at the node offsets of
// spec (vorticity) and spec2 (stream vector) for the z transform that follows. The walk of
// k_resid_flow2: a block owns one component, W lanes cover 2W consecutive z of one interior
// row, the slab marches along x with the x-neighbours in registers. Wall rows enter as stored
// (their increments are zero).
template <int W, bool BATCH>
__global__ __launch_bounds__(kBlock) void k_rhs_pred(Dims d, SlabGrid sg, RhsFlowArgs one,
                                                    const RhsFlowArgs* __restrict__ tab) {
    const int nb = sg.gx * sg.gi;
    const int lbi = xcd_block(blockIdx.x, gridDim.x);
    const int inst = BATCH ? lbi / (3 * nb) : 0;
    const RhsFlowArgs& a = inst_args<BATCH>(one, tab, inst);
    if (a.gate && *a.gate) return;
    const int lb0 = lbi - inst * 3 * nb;
    const int c = lb0 / nb;
    const int lb = lb0 - c * nb;
    const int bi = lb / sg.gx;
    const int t = (lb - bi * sg.gx) * kBlock + threadIdx.x;
    const int hz = d.nz >> 1;
    if (t >= d.M * hz) return;
    const Gl<double>* wc = (const Gl<double>*)pick(a.om, c);
    const Gl<double>* pc = (const Gl<double>*)pick(a.ps, c);
    const Gl<double>* sc = (const Gl<double>*)pick(a.src, c);
    const Gl<float>* w1 = (const Gl<float>*)pick(a.i1, c);
    const Gl<float>* w2 = (const Gl<float>*)pick(a.i2, c);
    const Gl<float>* p1 = (const Gl<float>*)pick(a.i1, 3 + c);
    const Gl<float>* p2 = (const Gl<float>*)pick(a.i2, 3 + c);
    Gl<float>* ow = (Gl<float>*)pick(a.spec, c);
    Gl<float>* op = (Gl<float>*)pick(a.spec2, c);
    const int h = a.hist ? *a.hist : 0;
    const int jj = t / hz;
    const int k = 2 * (t - jj * hz);
    const int j = jj + 1;
    const int plane = d.ny * d.nz;
    const int off = j * d.nz + k;
    const int ln = threadIdx.x & (W - 1);
    const int k0 = k - 2 * ln;
    const int kpe = (k0 + 2 * W == d.nz) ? 0 : k0 + 2 * W;
    const int kme = (k0 == 0) ? d.nz - 1 : k0 - 1;
    const int i0 = bi * sg.ci;
    const int i1 = min(d.nx, i0 + sg.ci);
    const int im0 = (i0 == 0) ? d.nx - 1 : i0 - 1;
    auto walk = [&](auto hc) {
        constexpr int H = decltype(hc)::value;
        // u* at a pair of nodes or at one node: the values as loaded, and their combination. Kept apart
        // so that the scheduling barrier below holds loads only: combined at the load, every plane
        // waited for its last load, the next plane's centres: 176 us at 128 x 128 x 256, now 157
        // (4.5 TB/s of the 704 MB it must move).
        struct Raw2 {
            double2 u;
            gf2v a, b;
        };
        struct Raw1 {
            double u;
            float a, b;
        };
        auto ld2 = [&](const Gl<double>* u, const Gl<float>* f1, const Gl<float>* f2, int o) -> Raw2 {
            Raw2 r;
            r.u = ldg2(u + o);
            if constexpr (H >= 1) r.a = *reinterpret_cast<const Gl<gf2v>*>(f1 + o);
            if constexpr (H == 2) r.b = *reinterpret_cast<const Gl<gf2v>*>(f2 + o);
            return r;
        };
        auto ld1 = [&](const Gl<double>* u, const Gl<float>* f1, const Gl<float>* f2, int o) -> Raw1 {
            Raw1 r;
            r.u = u[o];
            if constexpr (H >= 1) r.a = f1[o];
            if constexpr (H == 2) r.b = f2[o];
            return r;
        };
        auto at2 = [](const Raw2& r) -> double2 {
            double2 v = r.u;
            if constexpr (H == 1) {
                v.x = v.x + (double)r.a.x;
                v.y = v.y + (double)r.a.y;
            } else if constexpr (H == 2) {
                v.x = v.x + (2.0 * (double)r.a.x - (double)r.b.x);
                v.y = v.y + (2.0 * (double)r.a.y - (double)r.b.y);
            }
            return v;
        };
        auto at1 = [](const Raw1& r) -> double {
            if constexpr (H == 0) return r.u;
            else if constexpr (H == 1) return r.u + (double)r.a;
            else return r.u + (2.0 * (double)r.a - (double)r.b);
        };
        auto zn = [&](double2 v, double em, double ep, double& zm0, double& zp1) {
            const double prev = __shfl_up(v.y, 1, W), next = __shfl_down(v.x, 1, W);
            zm0 = ln == 0 ? em : prev;
            zp1 = ln == W - 1 ? ep : next;
        };
        double2 wm = at2(ld2(wc, w1, w2, im0 * plane + off)), wx = at2(ld2(wc, w1, w2, i0 * plane + off));
        double2 pm = at2(ld2(pc, p1, p2, im0 * plane + off)), px = at2(ld2(pc, p1, p2, i0 * plane + off));
#pragma unroll 1
        for (int i = i0; i < i1; ++i) {
            const int ip = (i + 1 == d.nx) ? 0 : i + 1;
            const int rb = i * plane + j * d.nz;
            const int c0 = rb + k;
            const double2 b = ldg2(sc + c0);
            const Raw2 rylo = ld2(wc, w1, w2, c0 - d.nz), ryhi = ld2(wc, w1, w2, c0 + d.nz);
            const Raw2 rqlo = ld2(pc, p1, p2, c0 - d.nz), rqhi = ld2(pc, p1, p2, c0 + d.nz);
            const int ome = rb + kme, ope = rb + kpe;
            const Raw1 rwem = ld1(wc, w1, w2, ome), rwep = ld1(wc, w1, w2, ope);
            const Raw1 rpem = ld1(pc, p1, p2, ome), rpep = ld1(pc, p1, p2, ope);
            // the next plane's centres last: they stay in flight while this plane is formed
            const Raw2 rwp = ld2(wc, w1, w2, ip * plane + off);
            const Raw2 rpp = ld2(pc, p1, p2, ip * plane + off);
            __builtin_amdgcn_sched_barrier(0);
            const double2 ylo = at2(rylo), yhi = at2(ryhi), qlo = at2(rqlo), qhi = at2(rqhi);
            const double wem = at1(rwem), wep = at1(rwep), pem = at1(rpem), pep = at1(rpep);
            const double2 wp = at2(rwp), pp = at2(rpp);
            {
                double zm0, zp1;
                zn(wx, wem, wep, zm0, zp1);
                const double l0 = (wp.x + wm.x + ylo.x + yhi.x + wx.y + zm0 - 6.0 * wx.x) * d.inv_h2;
                const double l1 = (wp.y + wm.y + ylo.y + yhi.y + zp1 + wx.x - 6.0 * wx.y) * d.inv_h2;
                stc<float>(ow + c0, (float)(b.x - l0), (float)(b.y - l1));
            }
            {
                double zm0, zp1;
                zn(px, pem, pep, zm0, zp1);
                const double l0 = (pp.x + pm.x + qlo.x + qhi.x + px.y + zm0 - 6.0 * px.x) * d.inv_h2;
                const double l1 = (pp.y + pm.y + qlo.y + qhi.y + zp1 + px.x - 6.0 * px.y) * d.inv_h2;
                stc<float>(op + c0, (float)(-wx.x - l0), (float)(-wx.y - l1));
            }
            wm = wx;
            wx = wp;
            pm = px;
            px = pp;
        }
    };
    if (h == 0) walk(std::integral_constant<int, 0>{});
    else if (h == 1) walk(std::integral_constant<int, 1>{});
    else walk(std::integral_constant<int, 2>{});
}

// The final decision of k_check, from the wave sums of r^2 (sh) and b~^2 (sh + 16).
__device__ __forceinline__ void check_one(const double* sh, int nw, double rtol, int last_cycle,
                                          double* scal, int* istat, int role, double* log) {
    double rr = 0.0, bb = 0.0;
    for (int i = 0; i < nw; ++i) {
        rr += sh[i];
        bb += sh[16 + i];
    }
    double rel;
    if (bb > 0.0)
        rel = sqrt(rr / bb);
    else
        rel = (rr > 0.0) ? INFINITY : 0.0;
    if (rr != rr || bb != bb) rel = NAN;
    const int conv = (rel <= rtol) ? 1 : 0;
    istat[IS_CONV] = conv;
    istat[IS_CYCLES] += 1;
    scal[SC_RELRES_LAST] = rel;
    if (conv || last_cycle) {
        const double prev = scal[SC_RELRES_MAX];
        scal[SC_RELRES_MAX] = (rel != rel || rel > prev) ? rel : prev;
        if (role == 1) scal[SC_RELRES_W] = rel;
        if (role == 2 && log) {   // the step's record (the per-step log; see flow_check.h)
            const double rw = scal[SC_RELRES_W];
            const int n = istat[IS_LOGN];
            double* r = log + (size_t)(n % kLogCap) * kLogFields;
            r[0] = (double)n;
            r[1] = (double)istat[IS_CYCLES];
            r[2] = (rw != rw || rw > rel) ? rw : rel;
            r[3] = scal[SC_V];
            r[4] = scal[SC_A];
            r[5] = scal[SC_LAMV];
            r[6] = scal[SC_GAMMA];
            r[7] = (double)((conv && rw <= rtol) ? 1 : 0);
            istat[IS_LOGN] = n + 1;
        }
    }
    if (!conv && last_cycle) istat[IS_FLAGS] |= ST_NOCONV;
    if (!isfinite(rr) || !isfinite(bb)) istat[IS_FLAGS] |= ST_NONFINITE;
}

// check: relative residual sqrt(sum_c r^2 / sum_c b~^2) in a fixed summation order; sets the
// convergence flag that gates the following cycles, counts the cycle and raises ST_NOCONV
// on the last allowed cycle, ST_NONFINITE on NaN/Inf.
__global__ __launch_bounds__(1024) void k_check(const double* __restrict__ partials,
                                               int nblocks, double rtol, int last_cycle,
                                               double* scal, int* istat, const int* gate,
                                               int slot0, int role, double* log, char* host) {
    if (gate && *gate) return;
    __shared__ double sh[2 * 16];
    double rr = 0.0, bb = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += blockDim.x) {
        const double* pb = partials + (size_t)slot0 * kMaxPartialBlocks + b;
        rr += pb[0 * kMaxPartialBlocks] + pb[1 * kMaxPartialBlocks] + pb[2 * kMaxPartialBlocks];
        bb += pb[3 * kMaxPartialBlocks] + pb[4 * kMaxPartialBlocks] + pb[5 * kMaxPartialBlocks];
    }
    rr = wave_sum(rr);
    bb = wave_sum(bb);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if (lane == 0) {
        sh[w] = rr;
        sh[16 + w] = bb;
    }
    __syncthreads();
    if (threadIdx.x == 0) check_one(sh, nw, rtol, last_cycle, scal, istat, role, log);
    if (host) {
        __syncthreads();
        status_to_host(scal, istat, host);
    }
}

// Convergence checks of the two flow solves of a step in one launch (flow_check.h); one block
// per instance.
template <bool BATCH>
__global__ __launch_bounds__(1024) void k_check_flow(int nblocks, int mode, ChkArgs one,
                                                    const ChkArgs* __restrict__ tab) {
    const ChkArgs& a = inst_args<BATCH>(one, tab, (int)blockIdx.x);
    __shared__ double sh[4 * 16];
    if (!(a.gate && *a.gate)) flow_check_block(a.part, nblocks, a.rtol, a.scal, a.istat, sh, mode, a.log);
    if (a.host) status_to_host(a.scal, a.istat, a.host);
}

}  // namespace

int seg_shape(int M);   // k_tri.hip

bool fused_flow_ok(const Dims& d) {
    int B, A;
    two_pass_shape(d.nx, B, A);
    if (!B) return false;
    two_pass_shape(d.nz, B, A);
    if (!B) return false;
    return seg_shape(d.M) != 0;
}

bool refined_ok(const Dims& d) {
    auto len = [](int n) { return n == 32 || n == 48 || n == 64 || n == 96 || n == 128 || n == 192 || n == 256; };
    return len(d.nx) && len(d.nz) && seg_shape(d.M) != 0;
}

// Residual blocks per component: slabs of x-planes chosen so that about a thousand blocks
// cover one component (each component adds as many again).
static SlabGrid resid_grid(const Dims& d) { return slab_grid(d.M * d.nz, d.nx, 1024); }

int resid_blocks(const Dims& d) {
    const SlabGrid g = resid_grid(d);
    return g.gx * g.gi;
}

// The block cap per component (tuned; 1024 by default).
static SlabGrid resid_flow_grid(const Dims& d) {
    const int maxb = tuning_for(d).res_maxb;
    return slab_grid(d.nz % 32 == 0 ? d.M * d.nz / 2 : d.M * d.nz, d.nx, maxb);
}

int resid_flow_blocks(const Dims& d) {
    const SlabGrid g = resid_flow_grid(d);
    return g.gx * g.gi;
}

void launch_resid_norm(hipStream_t s, const Dims& d, const RhsArgs& rhs,
                       const double* const u[3], int ncomp, double* partials, const int* gate,
                       int slot0) {
    CPtr3 uu{{u[0], ncomp > 1 ? u[1] : nullptr, ncomp > 2 ? u[2] : nullptr}};
    const SlabGrid g = resid_grid(d);
    launch_kernel(k_resid_norm, dim3(ncomp * g.gx * g.gi), dim3(kBlock), 0, s, d, rhs, uu, ncomp,
                  g, partials, gate, slot0);
}

template <class SS>
static void resid_flow_t(hipStream_t s, const Dims& d, const Over<ResArgs>& a) {
    const SlabGrid g = resid_flow_grid(d);
    const unsigned ni = a.tab ? (unsigned)a.n : 1u;
    const dim3 gr(3 * g.gx * g.gi * ni);
    auto go = [&](auto kt, auto kf) {
        if (a.tab) launch_kernel(kt, gr, dim3(kBlock), 0, s, d, g, a.one, a.tab);
        else launch_kernel(kf, gr, dim3(kBlock), 0, s, d, g, a.one, a.tab);
    };
    if (d.nz % 128 == 0) go(k_resid_flow2<64, true, SS>, k_resid_flow2<64, false, SS>);
    else if (d.nz % 64 == 0) go(k_resid_flow2<32, true, SS>, k_resid_flow2<32, false, SS>);
    else if (d.nz % 32 == 0) go(k_resid_flow2<16, true, SS>, k_resid_flow2<16, false, SS>);
    else go(k_resid_flow<true, SS>, k_resid_flow<false, SS>);
}

void launch_resid_flow_over(hipStream_t s, const Dims& d, bool f32src, const Over<ResArgs>& a) {
    if (f32src)
        resid_flow_t<float>(s, d, a);
    else
        resid_flow_t<double>(s, d, a);
}

void launch_rhs_pred(hipStream_t s, const Dims& d, const Over<RhsFlowArgs>& a) {
    const SlabGrid g = slab_grid(d.M * (d.nz / 2), d.nx, tuning_for(d).res_maxb);
    const unsigned ni = a.tab ? (unsigned)a.n : 1u;
    const dim3 gr(3 * g.gx * g.gi * ni);
    auto go = [&](auto kt, auto kf) {
        if (a.tab) launch_kernel(kt, gr, dim3(kBlock), 0, s, d, g, a.one, a.tab);
        else launch_kernel(kf, gr, dim3(kBlock), 0, s, d, g, a.one, a.tab);
    };
    if (d.nz % 128 == 0) go(k_rhs_pred<64, true>, k_rhs_pred<64, false>);
    else if (d.nz % 64 == 0) go(k_rhs_pred<32, true>, k_rhs_pred<32, false>);
    else if (d.nz % 32 == 0) go(k_rhs_pred<16, true>, k_rhs_pred<16, false>);
    else go(k_rhs_pred<8, true>, k_rhs_pred<8, false>);
}

void launch_resid_flow(hipStream_t s, const Dims& d, const double* const om[3],
                       const double* const src[3], const double* const ps[3], double ashift,
                       double* partials) {
    ResArgs r{};
    for (int c = 0; c < 3; ++c) {
        r.om[c] = om[c];
        r.src[c] = src[c];
        r.ps[c] = ps[c];
    }
    r.part = partials;
    r.ashift = ashift;
    launch_resid_flow_over(s, d, false, over_one(r));
}

void launch_check_flow_over(hipStream_t s, const Dims& d, int mode, const Over<ChkArgs>& a) {
    const unsigned ni = a.tab ? (unsigned)a.n : 1u;
    const int nb = resid_flow_blocks(d);
    if (a.tab)
        launch_kernel(k_check_flow<true>, dim3(ni), dim3(1024), 0, s, nb, mode, a.one, a.tab);
    else
        launch_kernel(k_check_flow<false>, dim3(1), dim3(1024), 0, s, nb, mode, a.one, a.tab);
}

void launch_check_flow(hipStream_t s, const Dims& d, const double* partials, double rtol,
                       double* scal, int* istat) {
    ChkArgs c{};
    c.part = partials;
    c.scal = scal;
    c.istat = istat;
    c.rtol = rtol;
    launch_check_flow_over(s, d, CK_LAST, over_one(c));
}

void launch_check(hipStream_t s, const double* partials, int nblocks, double rtol, int cycle,
                  int last_cycle, double* scal, int* istat, const int* gate, int slot0, int role,
                  double* log, char* host) {
    (void)cycle;
    launch_kernel(k_check, dim3(1), dim3(1024), 0, s, partials, nblocks, rtol,
                       last_cycle, scal, istat, gate, slot0, role, log, host);
}

}  // namespace vs
