// Plane passes of the spectral Poisson solves (main text eq. (5b), (5c)) for the lengths without a
// kernel of their own in k_plane.hip: both Hartley transforms of a direction in one pass over each
// (x, z) plane held in LDS, FP64, n_x and n_z any two-pass length up to 108 whose plane fits in 79 KB.
// One kernel per LDS class takes every pair of lengths: the two 1D passes are chosen by a switch, the
// lines run in rounds of as many as the block has lanes for.
//
// Bound by the launch and load latency of such small planes, of which one pass needs half of what two
// line passes do (forward + inverse, plane against lines): 24^3 12.3 against 17.2 us, 36^3 14.6
// against 19.7, 54^3 21.9 against 30.2, 72^3 29.7 against 35.5, 72 x 51 x 108 41.6 against 44.5. Longer
// lines and larger planes gained nothing or lost (16 x 100 x 144 27.3 against 25.2, 108^3 82.6
// against 85.0, 192 x 96 x 64 82 against 66: few planes, each on one CU): they keep the line passes.
#include <algorithm>

#include "spectral.h"

namespace vs {

namespace {

struct PlaneAny {
    int rs;      // row stride of the plane in LDS (doubles)
    int rpw;     // rows a wave loads or stores at once (a row has at most 54 pairs)
};

// One 1D Hartley transform of the nlp line pairs (ROWS: x-rows, element m at P[row * RS + m]; else
// z-columns, element m at P[m * RS + col]), in place, as plane_hartley of k_plane.hip. Line pairs
// are independent, so each round of LPR of them runs on its own.
template <int B, int A, bool ROWS, int NT>
__device__ __forceinline__ void any_hartley(double* __restrict__ P, int RS, int nlp,
                                            const tw2v* __restrict__ tw) {
    using C = double2;
    constexpr int IT = A > B / 2 ? A : B / 2, LPR = NT / IT;
    constexpr int SW = ROWS && (A & (A - 1)) == 0 ? A - 1 : 0;   // LDS bank spread, see k_plane.hip
    static_assert(SW == 0 || 64 % A == 0, "the lanes of a swizzled line pair share a wave");
    auto ld = [&](int lp, int m) -> C {
        if constexpr (ROWS) return make_double2(P[(2 * lp) * RS + m], P[(2 * lp + 1) * RS + m]);
        else return *reinterpret_cast<const C*>(&P[m * RS + 2 * lp]);
    };
    auto st = [&](int lp, int m, double a, double b) {
        if constexpr (ROWS) {
            P[(2 * lp) * RS + m] = a;
            P[(2 * lp + 1) * RS + m] = b;
        } else {
            *reinterpret_cast<C*>(&P[m * RS + 2 * lp]) = make_double2(a, b);
        }
    };
#pragma unroll 1
    for (int l0 = 0; l0 < nlp; l0 += LPR) {
        const int cnt = min(LPR, nlp - l0);
        // through an empty asm statement: otherwise the LDS offsets of every pass of the switch are
        // held (and spilled) across the plane loop
        int it = threadIdx.x;
        asm volatile("" : "+v"(it));
        {
            const int q = ROWS ? it / A : it % LPR, k1 = ROWS ? it % A : it / LPR;
            if (q < cnt && k1 < A) {
                const int lp = l0 + q;
                C x[B];
#pragma unroll
                for (int k2 = 0; k2 < B; ++k2) x[k2] = ld(lp, k1 + A * k2);
                fftr::DFT<B>::run(x);
#pragma unroll
                for (int p2 = 1; p2 < B; ++p2) x[p2] = cmul_tw<double>(x[p2], tw[k1 * p2]);
                if constexpr (SW != 0) swizzle_order();
#pragma unroll
                for (int p2 = 0; p2 < B; ++p2) st(lp, (k1 ^ (p2 & SW)) + A * p2, x[p2].x, x[p2].y);
            }
        }
        __syncthreads();
        const int q = ROWS ? it / (B / 2) : it % LPR, s0 = ROWS ? it % (B / 2) : it / LPR;
        const bool act = q < cnt && s0 < B / 2;
        // every lane computes (an idle one on the round's first pair), so the arrays stay in registers
        const int lp = act ? l0 + q : l0, s = act ? s0 : 0;
        const int pa = s, pb = (s == 0) ? B / 2 : B - s;
        C xa[A], xb[A];
#pragma unroll
        for (int k1 = 0; k1 < A; ++k1) {
            xa[k1] = ld(lp, (k1 ^ (pa & SW)) + A * pa);
            xb[k1] = ld(lp, (k1 ^ (pb & SW)) + A * pb);
        }
        fftr::DFT<A>::run(xa);
        fftr::DFT<A>::run(xb);
        __syncthreads();
        if (act) {
            // exact blends, as in k_plane.hip
            const double f = (s == 0) ? 1.0 : 0.0, g = 1.0 - f;
            auto blend = [&](const C& u, const C& v) -> C {
                return make_double2(__builtin_fma(f, u.x, g * v.x), __builtin_fma(f, u.y, g * v.y));
            };
#pragma unroll
            for (int p1 = 0; p1 < A; ++p1) {
                const C za = xa[p1];
                const C ma = blend(xa[(A - p1) % A], xb[A - 1 - p1]);
                st(lp, pa + B * p1, 0.5 * (za.x + ma.x - za.y + ma.y), 0.5 * (za.x - ma.x + za.y + ma.y));
                const C zb = xb[p1];
                const C mb = blend(xb[A - 1 - p1], xa[A - 1 - p1]);
                st(lp, pb + B * p1, 0.5 * (zb.x + mb.x - zb.y + mb.y), 0.5 * (zb.x - mb.x + zb.y + mb.y));
            }
        }
    }
    __syncthreads();
}

template <bool ROWS, int NT>
__device__ __forceinline__ void any_pass(int n, double* __restrict__ P, int RS, int nlp,
                                         const tw2v* __restrict__ tw) {
    switch (n) {   // the shapes of two_pass_shape
    case 16: any_hartley<8, 2, ROWS, NT>(P, RS, nlp, tw); break;
    case 24: any_hartley<8, 3, ROWS, NT>(P, RS, nlp, tw); break;
    case 32: any_hartley<8, 4, ROWS, NT>(P, RS, nlp, tw); break;
    case 36: any_hartley<12, 3, ROWS, NT>(P, RS, nlp, tw); break;
    case 48: any_hartley<16, 3, ROWS, NT>(P, RS, nlp, tw); break;
    case 54: any_hartley<18, 3, ROWS, NT>(P, RS, nlp, tw); break;
    case 64: any_hartley<16, 4, ROWS, NT>(P, RS, nlp, tw); break;
    case 72: any_hartley<12, 6, ROWS, NT>(P, RS, nlp, tw); break;
    case 96: any_hartley<16, 6, ROWS, NT>(P, RS, nlp, tw); break;
    default: any_hartley<12, 9, ROWS, NT>(P, RS, nlp, tw); break;   // 108
    }
}

// As k_hxz_plane (ZFIRST: z then x from z.spec into x.spec, with z.wall the right-hand side of a
// direct solve; otherwise x then z from x.spec into z.u; gated per instance by z.gate). LDSD: doubles
// of LDS, WPE: waves per SIMD the registers are held to. Loads and stores need 8-byte alignment only.
template <int LDSD, int NT, int WPE, bool ZFIRST, bool BATCH>
__global__ __launch_bounds__(NT, WPE) void k_plane_any(Dims d, int nc, PlaneAny pa, ZArgs zone,
                                                       const ZArgs* __restrict__ ztab, HxArgs xone,
                                                       const HxArgs* __restrict__ xtab, int nplanes) {
    __shared__ double P[LDSD];
    const int nx = d.nx, nz = d.nz, RS = pa.rs;
    tw2v* TWX = reinterpret_cast<tw2v*>(P + nx * RS);
    tw2v* TWZ = TWX + nx;
    const size_t pstride = (size_t)d.ny * nz;
    {
        const ZArgs& z0 = inst_args<BATCH>(zone, ztab, 0);
        const HxArgs& x0 = inst_args<BATCH>(xone, xtab, 0);
        const Gl<tw2v>* gz = (const Gl<tw2v>*)z0.tw;
        const Gl<tw2v>* gx = (const Gl<tw2v>*)x0.tw;
        for (int t = threadIdx.x; t < nx; t += NT) TWX[t] = gx[t];
        for (int t = threadIdx.x; t < nz; t += NT) TWZ[t] = gz[t];
    }
    if (ZFIRST && !BATCH && zone.reset && blockIdx.x + threadIdx.x == 0) clear_status(zone.scal, zone.reset);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, h = nz >> 1;
    const int r = lane / h, kc = 2 * (lane - r * h);    // the lane's row of the wave's rpw, its first z
    const bool ok = r < pa.rpw;
    const int stride = (NT / 64) * pa.rpw;
    constexpr int U = 8;
    for (int p = blockIdx.x; p < nplanes; p += (int)gridDim.x) {
        const int cg = p / d.M, j = 1 + (p - cg * d.M);
        const int inst = BATCH ? cg / nc : 0, c = cg - inst * nc;
        const ZArgs& za = inst_args<BATCH>(zone, ztab, inst);
        const HxArgs& xa = inst_args<BATCH>(xone, xtab, inst);
        if (za.gate && *(const Gl<int>*)za.gate) continue;   // block-uniform
        const Gl<double>* in = (const Gl<double>*)(ZFIRST ? pick(za.spec, c) : pick(xa.spec, c)) + (size_t)j * nz;
        Gl<double>* out = (Gl<double>*)(ZFIRST ? pick(xa.spec, c) : pick(za.u, c)) + (size_t)j * nz;
        for (int i0 = wv * pa.rpw; i0 < nx; i0 += U * stride) {
            double2 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = ldg2u(in + min(i0 + r + u * stride, nx - 1) * pstride + kc);
            if (ZFIRST && !BATCH && za.wall[0]) {
                const Gl<double>* w = (const Gl<double>*)pick(za.wall, c) + kc;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const Gl<double>* wi = w + min(i0 + r + u * stride, nx - 1) * pstride;
                    v[u].x *= za.sgn;
                    v[u].y *= za.sgn;
                    if (j == 1) {
                        const double2 q = ldg2u(wi);
                        v[u].x -= q.x * d.inv_h2;
                        v[u].y -= q.y * d.inv_h2;
                    }
                    if (j == d.M) {
                        const double2 q = ldg2u(wi + (size_t)(d.ny - 1) * nz);
                        v[u].x -= q.x * d.inv_h2;
                        v[u].y -= q.y * d.inv_h2;
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + r + u * stride;
                if (ok && i < nx) *reinterpret_cast<double2*>(&P[i * RS + kc]) = v[u];
            }
        }
        __syncthreads();
        if constexpr (ZFIRST) {
            any_pass<true, NT>(nz, P, RS, nx >> 1, TWZ);
            any_pass<false, NT>(nx, P, RS, h, TWX);
        } else {
            any_pass<false, NT>(nx, P, RS, h, TWX);
            any_pass<true, NT>(nz, P, RS, nx >> 1, TWZ);
        }
        for (int i0 = wv * pa.rpw; i0 < nx; i0 += U * stride) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + r + u * stride;
                if (ok && i < nx) {
                    const double2 q = *reinterpret_cast<const double2*>(&P[i * RS + kc]);
                    stg2u(out + i * pstride + kc, q.x, q.y);
                }
            }
        }
        __syncthreads();   // the plane's LDS is read out before the next one is written
    }
}

// Row stride: the two dwords of the A lanes of a line pair's pass 1 lie next to the following pair's,
// in other banks (a pair of rows is 4 RS dwords, of 64 banks).
int any_row(int nz) {
    int B, A;
    two_pass_shape(nz, B, A);
    const int want = (2 * A + 7) / 8 * 8;
    int rs = nz + 2;
    while ((4 * rs) % 64 != want) rs += 2;
    return rs;
}
size_t any_lds(const Dims& d) { return (size_t)d.nx * any_row(d.nz) * 8 + (size_t)(d.nx + d.nz) * 16; }

constexpr int kSmall = 40 * 1024 / 8, kMid = 79 * 1024 / 8;

template <int LDSD, int NT, int WPE, int PER_CU>
void any_go(hipStream_t s, const Dims& d, bool zfirst, int ncomp, const Over<ZArgs>& z, const Over<HxArgs>& x) {
    const int h = d.nz / 2;
    const PlaneAny pa{any_row(d.nz), 64 / h};
    const int nplanes = d.M * ncomp * (z.tab ? z.n : 1);
    const dim3 g((unsigned)std::min(nplanes, PER_CU * plane_blocks())), blk((unsigned)NT);
    auto go = [&](auto kf, auto kt) {
        if (z.tab) launch_kernel(kt, g, blk, 0, s, d, ncomp, pa, z.one, z.tab, x.one, x.tab, nplanes);
        else launch_kernel(kf, g, blk, 0, s, d, ncomp, pa, z.one, z.tab, x.one, x.tab, nplanes);
    };
    if (zfirst) go(k_plane_any<LDSD, NT, WPE, true, false>, k_plane_any<LDSD, NT, WPE, true, true>);
    else go(k_plane_any<LDSD, NT, WPE, false, false>, k_plane_any<LDSD, NT, WPE, false, true>);
}

}  // namespace

bool plane_any_fits(const Dims& d) {
    int bx, ax, bz, az;
    two_pass_shape(d.nx, bx, ax);
    two_pass_shape(d.nz, bz, az);
    return bx > 0 && bz > 0 && d.nx <= 108 && d.nz <= 108 && any_lds(d) <= (size_t)kMid * 8;
}

void launch_plane_any(hipStream_t s, const Dims& d, bool zfirst, int ncomp, const Over<ZArgs>& z,
                      const Over<HxArgs>& x) {
    const size_t lds = any_lds(d);
    if (lds <= (size_t)kSmall * 8) any_go<kSmall, 256, 3, 3>(s, d, zfirst, ncomp, z, x);
    else any_go<kMid, 256, 2, 2>(s, d, zfirst, ncomp, z, x);
}

}  // namespace vs
