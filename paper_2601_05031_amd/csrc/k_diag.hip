// Diagnostics of a state and the wall-speed change, FP64, gfx950.
//   * in-plane shear stress (main text "In plane shear"): sigma_ij = eta (d_j v_i + d_i v_j),
//     sigma_t = sqrt(sigma_xy^2 + sigma_yz^2 + sigma_xz^2), central differences of v (curl psi
//     inside, the wall speed on the walls), on the interior rows; 0 on the wall rows;
//   * the flow observables of the results section: int |omega - omega_0|^2 and
//     int |psi - psi_0|^2 about the no-body channel fields, trapezoid weights in y;
//   * the free-energy density: g^2 (bending, SM eq. (30) without the area term) or
//     1/4 (phi^2 - 1)^2 + (sigma/2) |D phi|^2 (Cahn-Hilliard, eq. F_CH);
//   * the gauge defect (D . psi)^2 on the interior rows (the Coulomb gauge is assumed, not
//     imposed) and the largest speed |v|;
//   * time-dependent walls (SM "Time-dependency and inertial flow"): the Poisson problems
//     are linear in the wall data and the no-body fields (polynomials of degree <= 3 in y)
//     solve them exactly, so a change of wall speeds adds the difference of the no-body fields
//     to omega_x and psi_x.
#include "flow_check.h"
#include "stencil.h"

namespace vs {

namespace {

// Bound by the memory side: 7 fields read, 3 written and read again, sigma_t written (the scratch
// velocity mostly from the 256 MB cache). A call with sigma_t, 128^3: 98 us with one node per
// lane, every neighbour loaded and the observables apart from the velocity; 78 now (64 where the
// state is still in the cache).
// Both node kernels: two consecutive z per lane, one lane per pair of the (y, z) plane (every
// even n_z), walking the ci x-planes of its block with the x neighbours held in registers. A
// field's read of a pair moves 16 bytes; the z neighbours outside the pair are one 8-byte load
// each. All loads of a plane are issued before the first use (scheduling barrier), so that one
// latency is paid a plane.
__device__ __forceinline__ double block_max(double v, double* sh) {   // in thread 0, fixed order
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_down(v, off, 64));
    if (lane == 0) sh[wv] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        v = 0.0;
        for (int q = 0; q < (int)(blockDim.x >> 6); ++q) v = fmax(v, sh[q]);
    }
    return v;
}

// The velocity on every node into three scratch fields (curl psi inside, the wall velocity on
// the walls), so that the shear stress reads each neighbour's velocity once instead of
// evaluating the curl there again; and what needs omega and psi only: the flow
// observables, the gauge defect and the largest speed.
__global__ __launch_bounds__(kBlock) void k_diag_flow(const double* __restrict__ o0,
                                                     const double* __restrict__ o1,
                                                     const double* __restrict__ o2, Vel vel,
                                                     const double* __restrict__ prof, Dims d,
                                                     SlabGrid sg, double* __restrict__ v0,
                                                     double* __restrict__ v1,
                                                     double* __restrict__ v2,
                                                     double* __restrict__ partials) {
    __shared__ double sh[3 * 16];
    __shared__ double shm[16];
    double acc[3] = {0.0, 0.0, 0.0};
    double vmax = 0.0;
    const PairLane L = pair_lane(d, sg);
    if (L.ok) {
        const double *__restrict__ px = vel.px, *__restrict__ py = vel.py, *__restrict__ pz = vel.pz;
        const double w = wrow(d, L.j);
        const double pw = prof[L.j], ow = prof[d.ny + L.j];
        const bool in = interior(d, L.j);
        const double vwall = L.j == 0 ? vel.vz_lo : vel.vz_hi;
        size_t b = (size_t)wrap(L.i0 - 1, d.nx) * L.plane;
        double2 xm = ldp(px + b + L.o), ym = ldp(py + b + L.o), zm = ldp(pz + b + L.o);
        b = (size_t)L.i0 * L.plane;
        double2 xc = ldp(px + b + L.o), yc = ldp(py + b + L.o), zc = ldp(pz + b + L.o);
#pragma unroll 1
        for (int i = L.i0; i < L.i1; ++i) {
            const size_t c = (size_t)i * L.plane, bn = (size_t)wrap(i + 1, d.nx) * L.plane;
            const double2 a0 = ldp(o0 + c + L.o), a1 = ldp(o1 + c + L.o), a2 = ldp(o2 + c + L.o);
            const double2 xyp = ldp(px + c + L.oyp), xym = ldp(px + c + L.oym);
            const double2 yyp = ldp(py + c + L.oyp), yym = ldp(py + c + L.oym);
            const double2 zyp = ldp(pz + c + L.oyp), zym = ldp(pz + c + L.oym);
            const double xl = px[c + L.ol], xr = px[c + L.orr];
            const double yl = py[c + L.ol], yr = py[c + L.orr];
            const double zl = pz[c + L.ol], zr = pz[c + L.orr];
            const double2 xp = ldp(px + bn + L.o), yp = ldp(py + bn + L.o), zp = ldp(pz + bn + L.o);
            __builtin_amdgcn_sched_barrier(0);
            double2 vx, vy, vz;
            auto one = [&](double om0, double om1, double om2, double cx, double cy, double cz,
                           double x_xp, double x_xm, double x_yp, double x_ym, double x_zp, double x_zm,
                           double y_xp, double y_xm, double y_yp, double y_ym, double y_zp, double y_zm,
                           double z_xp, double z_xm, double z_yp, double z_ym, double z_zp, double z_zm,
                           double& u0, double& u1, double& u2) {
                const double e0 = om0 - ow, b0 = cx - pw;
                acc[0] += w * (e0 * e0 + om1 * om1 + om2 * om2);
                acc[1] += w * (b0 * b0 + cy * cy + cz * cz);
                u0 = 0.0;
                u1 = 0.0;
                u2 = vwall;
                if (in) {
                    u0 = ((z_yp - z_ym) - (y_zp - y_zm)) * d.inv_2h;
                    u1 = ((x_zp - x_zm) - (z_xp - z_xm)) * d.inv_2h;
                    u2 = ((y_xp - y_xm) - (x_yp - x_ym)) * d.inv_2h;
                    const double dv = (x_xp - x_xm) * d.inv_2h + (y_yp - y_ym) * d.inv_2h +
                                      (z_zp - z_zm) * d.inv_2h;
                    acc[2] += dv * dv;
                }
                vmax = fmax(vmax, sqrt(u0 * u0 + u1 * u1 + u2 * u2));
            };
            one(a0.x, a1.x, a2.x, xc.x, yc.x, zc.x, xp.x, xm.x, xyp.x, xym.x, xc.y, xl,
                yp.x, ym.x, yyp.x, yym.x, yc.y, yl, zp.x, zm.x, zyp.x, zym.x, zc.y, zl,
                vx.x, vy.x, vz.x);
            one(a0.y, a1.y, a2.y, xc.y, yc.y, zc.y, xp.y, xm.y, xyp.y, xym.y, xr, xc.x,
                yp.y, ym.y, yyp.y, yym.y, yr, yc.x, zp.y, zm.y, zyp.y, zym.y, zr, zc.x,
                vx.y, vy.y, vz.y);
            *reinterpret_cast<double2*>(v0 + c + L.o) = vx;
            *reinterpret_cast<double2*>(v1 + c + L.o) = vy;
            *reinterpret_cast<double2*>(v2 + c + L.o) = vz;
            xm = xc; xc = xp;
            ym = yc; yc = yp;
            zm = zc; zc = zp;
        }
    }
    block_sum<3>(acc, sh);
    vmax = block_max(vmax, shm);
    if (threadIdx.x == 0) {
        partials[0 * kMaxPartialBlocks + blockIdx.x] = acc[0];
        partials[1 * kMaxPartialBlocks + blockIdx.x] = acc[1];
        partials[3 * kMaxPartialBlocks + blockIdx.x] = acc[2];
        partials[5 * kMaxPartialBlocks + blockIdx.x] = vmax;
    }
}

// The shear stress from the velocity's scratch fields, its largest value, and the free energy.
// sigma_t is the caller's: `pairs` says that it is 16-byte aligned.
__global__ __launch_bounds__(kBlock) void k_diag_shear(const double* __restrict__ phi,
                                                      const double* __restrict__ v0,
                                                      const double* __restrict__ v1,
                                                      const double* __restrict__ v2, Dims d,
                                                      SlabGrid sg, double eta, int model, double eps,
                                                      double sigma, double* __restrict__ sigma_t,
                                                      int pairs, double* __restrict__ partials) {
    __shared__ double sh[16];
    __shared__ double shm[16];
    double acc[1] = {0.0};
    double smax = 0.0;
    const PairLane L = pair_lane(d, sg);
    if (L.ok) {
        const double w = wrow(d, L.j);
        const double eps2 = eps * eps;
        const bool in = interior(d, L.j);
        size_t b = (size_t)wrap(L.i0 - 1, d.nx) * L.plane;
        double2 fm = ldp(phi + b + L.o), ym = ldp(v1 + b + L.o), zm = ldp(v2 + b + L.o);
        b = (size_t)L.i0 * L.plane;
        double2 fc = ldp(phi + b + L.o), yc = ldp(v1 + b + L.o), zc = ldp(v2 + b + L.o);
#pragma unroll 1
        for (int i = L.i0; i < L.i1; ++i) {
            const size_t c = (size_t)i * L.plane, bn = (size_t)wrap(i + 1, d.nx) * L.plane;
            const double2 fyp = ldp(phi + c + L.oyp), fym = ldp(phi + c + L.oym);
            const double2 xc = ldp(v0 + c + L.o);
            const double2 xyp = ldp(v0 + c + L.oyp), xym = ldp(v0 + c + L.oym);
            const double2 zyp = ldp(v2 + c + L.oyp), zym = ldp(v2 + c + L.oym);
            const double fl = phi[c + L.ol], fr = phi[c + L.orr];
            const double xl = v0[c + L.ol], xr = v0[c + L.orr];
            const double yl = v1[c + L.ol], yr = v1[c + L.orr];
            const double2 fp = ldp(phi + bn + L.o), yp = ldp(v1 + bn + L.o), zp = ldp(v2 + bn + L.o);
            __builtin_amdgcn_sched_barrier(0);
            double2 st;
            auto one = [&](double p, double f_xp, double f_xm, double f_yp, double f_ym, double f_zp,
                           double f_zm, double x_yp, double x_ym, double x_zp, double x_zm,
                           double y_xp, double y_xm, double y_zp, double y_zm, double z_xp,
                           double z_xm, double z_yp, double z_ym) -> double {
                if (model == VS_CAHN_HILLIARD) {
                    const double dx = (f_xp - f_xm) * d.inv_2h;
                    const double dy = (f_yp - f_ym) * d.inv_2h;
                    const double dz = (f_zp - f_zm) * d.inv_2h;
                    const double q = p * p - 1.0;
                    acc[0] += w * (0.25 * q * q + 0.5 * sigma * (dx * dx + dy * dy + dz * dz));
                } else {
                    const double g = p * p * p - p -
                                     eps2 * ((f_xp + f_xm + f_yp + f_ym + f_zp + f_zm - 6.0 * p) * d.inv_h2);
                    acc[0] += w * g * g;
                }
                if (!in) return 0.0;
                const double sxy = (x_yp - x_ym) + (y_xp - y_xm);
                const double syz = (y_zp - y_zm) + (z_yp - z_ym);
                const double sxz = (x_zp - x_zm) + (z_xp - z_xm);
                return eta * d.inv_2h * sqrt(sxy * sxy + syz * syz + sxz * sxz);
            };
            st.x = one(fc.x, fp.x, fm.x, fyp.x, fym.x, fc.y, fl, xyp.x, xym.x, xc.y, xl,
                       yp.x, ym.x, yc.y, yl, zp.x, zm.x, zyp.x, zym.x);
            st.y = one(fc.y, fp.y, fm.y, fyp.y, fym.y, fr, fc.x, xyp.y, xym.y, xr, xc.x,
                       yp.y, ym.y, yr, yc.x, zp.y, zm.y, zyp.y, zym.y);
            if (sigma_t) {
                double* const so = sigma_t + c + L.o;
                if (pairs) {
                    *reinterpret_cast<double2*>(so) = st;
                } else {
                    so[0] = st.x;
                    so[1] = st.y;
                }
            }
            smax = fmax(smax, fmax(st.x, st.y));
            fm = fc; fc = fp;
            ym = yc; yc = yp;
            zm = zc; zc = zp;
        }
    }
    block_sum<1>(acc, sh);
    smax = block_max(smax, shm);
    if (threadIdx.x == 0) {
        partials[2 * kMaxPartialBlocks + blockIdx.x] = acc[0];
        partials[4 * kMaxPartialBlocks + blockIdx.x] = smax;
    }
}

__global__ __launch_bounds__(1024) void k_diag_finalize(const double* __restrict__ partials,
                                                       int nblocks, double* scal, const int* istat,
                                                       char* host) {
    __shared__ double sh[4 * 16];
    __shared__ double shm[2 * 16];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    double m = 0.0, mv = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += blockDim.x) {
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] += partials[q * kMaxPartialBlocks + b];
        m = fmax(m, partials[4 * kMaxPartialBlocks + b]);
        mv = fmax(mv, partials[5 * kMaxPartialBlocks + b]);
    }
    block_sum<4>(acc, sh);
    const double mm = block_max(m, shm), mmv = block_max(mv, shm + 16);
    if (threadIdx.x == 0) {
        scal[SC_DG_OMEGA] = acc[0];
        scal[SC_DG_PSI] = acc[1];
        scal[SC_DG_ENERGY] = acc[2];
        scal[SC_DG_GAUGE] = acc[3];
        scal[SC_DG_SMAX] = mm;
        scal[SC_DG_VMAX] = mmv;
    }
    __syncthreads();
    status_to_host(scal, istat, host);
}

__global__ __launch_bounds__(kBlock) void k_shift_profiles(double* __restrict__ om,
                                                          double* __restrict__ ps, Dims d,
                                                          const double* __restrict__ dprof) {
    int i, j, k;
    bool ok;
    plane_index(d, i, j, k, ok);
    if (!ok) return;
    const int c = node(d, i, j, k);
    ps[c] += dprof[j];
    om[c] += dprof[d.ny + j];
}

}  // namespace

void launch_diagnostics(hipStream_t s, const Dims& d, const double* phi, double* const omega[3],
                        double* const psi[3], const double* prof, double vz_lo, double vz_hi,
                        double eta, int model, double eps, double sigma, double* sigma_t,
                        double* part, double* scal, double* const vscratch[3], const int* istat,
                        char* host) {
    // two blocks a CU: the lanes' loads in flight suffice, and longer walks read less twice
    // (128^3: 78.4, 80.9, 80.4, 87.3 us at up to 512, 1024, 2048, 4096 blocks; 108 x 51 x 72: 36.3
    // to 38; 64^3: equal)
    const SlabGrid g = slab_grid(d.ny * (d.nz / 2), d.nx, 512);
    const Vel vel{psi[0], psi[1], psi[2], vz_lo, vz_hi};
    const int nb = g.gx * g.gi;
    const int pairs = ((uintptr_t)sigma_t & 15) == 0;
    launch_kernel(k_diag_flow, dim3(nb), dim3(kBlock), 0, s, (const double*)omega[0],
                  (const double*)omega[1], (const double*)omega[2], vel, prof, d, g, vscratch[0],
                  vscratch[1], vscratch[2], part);
    launch_kernel(k_diag_shear, dim3(nb), dim3(kBlock), 0, s, phi, (const double*)vscratch[0],
                  (const double*)vscratch[1], (const double*)vscratch[2], d, g, eta, model, eps,
                  sigma, sigma_t, pairs, part);
    launch_kernel(k_diag_finalize, dim3(1), dim3(1024), 0, s, (const double*)part, nb, scal, istat, host);
}

void launch_shift_profiles(hipStream_t s, const Dims& d, double* omega_x, double* psi_x,
                           const double* dprof) {
    launch_kernel(k_shift_profiles, plane_grid(d), dim3(kBlock), 0, s, omega_x, psi_x, d, dprof);
}

}  // namespace vs
