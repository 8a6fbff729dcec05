// Plane passes of the spectral Poisson solves (main text eq. (5b), (5c)): both Hartley transforms
// of a direction in one pass over each (x, z) plane held in LDS. The pass structure and the 1D
// transforms are those of k_spectral.hip.
#include <algorithm>
#include <type_traits>

#include "spectral.h"

namespace vs {

namespace {

// ---------------------------------------------------------------------------------------
// Both transform directions of one interior row in one pass: the whole (x, z) plane of row j
// and one component sits in LDS (n_x rows of plane_row doubles, 132 KB at 128 x 128), so the spectral
// data crosses HBM once per direction instead of twice. Each 1D
// transform is the two-pass form above done in place in the plane: pass 1 overwrites the B
// inputs of its (line pair, k1), or with the swizzle below those of its line pair, with their twiddled
// B-point DFT, pass 2 reads the A values of rows pa, pb, and after a barrier writes the Hartley values. z lines are pairs of x-rows
// (i, i+1), x lines pairs of z-columns (q, q+1) as in k_hx.
// Padded row of the plane for z lines of shape (B, A): the 2 A (FP64) or A (FP32) dwords that A
// lanes of a line pair read land next to those of the following pairs, in other banks.
constexpr int plane_row(int nz, int A) { return nz + (A >= 16 ? 8 : A >= 6 ? 4 : 2); }
constexpr int kPlaneThreads = 512;

// One 1D Hartley transform of every line pair of the plane. ROWS: lines are x-rows (element m
// at P[row * RS + m]); otherwise z-columns (element m at P[m * RS + col]). T: the precision
// of the plane (FP64, or FP32 for the refined mode's corrections).
template <int B, int A, int NLP, int RS, bool ROWS, class T, int NT = kPlaneThreads>
__device__ __forceinline__ void plane_hartley(T* __restrict__ P, const tw2v* __restrict__ tw, int it) {
    using C = C2<T>;
    static_assert(NLP * A <= NT && NLP * (B / 2) <= NT, "one item per lane");
    auto ld = [&](int lp, int m) -> C {
        if constexpr (ROWS) return mkc<T>(P[(2 * lp) * RS + m], P[(2 * lp + 1) * RS + m]);
        else return *reinterpret_cast<const C*>(&P[m * RS + 2 * lp]);
    };
    auto st = [&](int lp, int m, T a, T b) {
        if constexpr (ROWS) {
            P[(2 * lp) * RS + m] = a;
            P[(2 * lp + 1) * RS + m] = b;
        } else {
            *reinterpret_cast<C*>(&P[m * RS + 2 * lp]) = mkc<T>(a, b);
        }
    };
    auto fma_t = [](T a, T b, T c) -> T {
        if constexpr (sizeof(T) == 8) return __builtin_fma(a, b, c);
        else return __builtin_fmaf(a, b, c);
    };
    // z lines with A a power of two hold their pass-1 result k1 of row p2 at A p2 + (k1 ^ p2 mod A):
    // in place of k1 + A p2, where the B/2 lanes of a line pair would read pass 2 in a stride of
    // A, on a few banks. A lane then overwrites inputs of the line pair's other lanes: all A of them
    // are in one wave, which issues its loads before its stores (swizzle_order)
    constexpr int SW = ROWS && (A & (A - 1)) == 0 ? A - 1 : 0;
    static_assert(SW == 0 || 64 % A == 0, "the lanes of a swizzled line pair share a wave");
    // pass 1: B-point DFTs over k2, twiddled, back to the same positions k1 + A p2
    if (it < NLP * A) {
        const int lp = ROWS ? it / A : it % NLP;
        const int k1 = ROWS ? it % A : it / NLP;
        C x[B];
#pragma unroll
        for (int k2 = 0; k2 < B; ++k2) x[k2] = ld(lp, k1 + A * k2);
        fftr::DFT<B>::run(x);
#pragma unroll
        for (int p2 = 1; p2 < B; ++p2) x[p2] = cmul_tw<T>(x[p2], tw[k1 * p2]);
        if constexpr (SW != 0) swizzle_order();
#pragma unroll
        for (int p2 = 0; p2 < B; ++p2) st(lp, (k1 ^ (p2 & SW)) + A * p2, x[p2].x, x[p2].y);
    }
    __syncthreads();
    // pass 2: A-point DFTs of rows pa and pb, then the Hartley values of both lines
    const bool act = it < NLP * (B / 2);
    const int lp = act ? (ROWS ? it / (B / 2) : it % NLP) : 0;
    const int s = act ? (ROWS ? it % (B / 2) : it / NLP) : 0;
    const int pa = s, pb = (s == 0) ? B / 2 : B - s;
    // every lane computes (an idle one on line pair 0), so the arrays stay in registers
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
        const T half = (T)0.5;
        // the partner Z_{n-p} comes from the lane's other row, except for s = 0 (rows 0 and
        // B/2, each its own partner); blended as f*u + (1-f)*v, exact for finite values (a
        // select here is turned into an indexed load from scratch memory)
        const T f = (s == 0) ? (T)1 : (T)0, g = (T)1 - f;
        auto blend = [&](const C& u, const C& v) -> C {
            return mkc<T>(fma_t(f, u.x, g * v.x), fma_t(f, u.y, g * v.y));
        };
#pragma unroll
        for (int p1 = 0; p1 < A; ++p1) {
            const C za = xa[p1];
            const C ma = blend(xa[(A - p1) % A], xb[A - 1 - p1]);
            st(lp, pa + B * p1, half * (za.x + ma.x - za.y + ma.y), half * (za.x - ma.x + za.y + ma.y));
            const C zb = xb[p1];
            const C mb = blend(xb[A - 1 - p1], xa[A - 1 - p1]);
            st(lp, pb + B * p1, half * (zb.x + mb.x - zb.y + mb.y), half * (zb.x - mb.x + zb.y + mb.y));
        }
    }
    __syncthreads();
}

// FP64 plane passes of n_x x n_z: a block per plane with as many lanes as the largest 1D pass has
// items, and as many blocks per CU as the LDS holds (at most 16 waves, so that a lane has 128
// registers): 64^2 planes 8.0 / 10.8 us forward / inverse at 64^3 against 11.0 / 16.0 us of line
// passes. Planes above 75 KB run alone on a CU with 512 lanes and keep the next plane's loads in
// flight while they transform (96^2: 21.4 / 31.7 us; two blocks per CU without the prefetch 23.7 /
// 35.6, with it 34.9 / 51.0, as its registers spill; 128^2: 29 / 44 us, 4.4 TB/s inverse). Below,
// the CU's other blocks give the overlap.
template <int BX, int AX, int BZ, int AZ>
struct PlaneShape {
    static constexpr int NX = BX * AX, NZ = BZ * AZ, RS = plane_row(NZ, AZ);
    static constexpr int imax(int a, int b) { return a > b ? a : b; }
    static constexpr int ITEMS = imax(imax(NX / 2 * AZ, NX / 2 * (BZ / 2)), imax(NZ / 2 * AX, NZ / 2 * (BX / 2)));
    static constexpr int LDS = NX * RS * 8 + (NX + NZ) * 16;
    static constexpr int FIT = LDS > 75 * 1024 ? 1 : 160 * 1024 / LDS;
    static constexpr int NT = FIT == 1 ? 512 : imax(128, (ITEMS + 63) / 64 * 64);
    static constexpr int WAVES = 16 / (NT / 64);
    static constexpr int PER_CU = FIT < WAVES ? FIT : WAVES;
    static constexpr int WPE = imax(1, PER_CU * (NT / 64) / 4);   // waves per SIMD
    static constexpr bool PF = PER_CU == 1;
};

// ZFIRST (the source's forward transform): z then x, from the field z.spec[c] (FP64, the
// interior rows) into the spectral buffer x.spec[c]. Otherwise (the inverse of the omega and
// psi modes): x then z, from x.spec[c] into the field z.u[c]. FP64 only, no accumulation; planes
// of an instance whose z.gate is set are skipped. Persistent: block b takes the planes b, b + G, ... (G = gridDim.x; plane
// p = (instance * nc + component) * M + j - 1) and, with PF, keeps the loads of its next plane in
// flight in registers while it works on the current one: the first half (NR1 values per lane)
// during the transforms, the rest during the stores (the whole plane beside a transform pass
// would not fit in the registers). The twiddles sit in LDS, so no global load inside the
// transforms waits behind the prefetch.
// RHS (with ZFIRST): the right-hand side of a direct solve, z.sgn times the field minus the wall
// terms, which the planes j = 1 and j = M take from the wall rows of z.wall. Its field and walls, and
// z.u, may be the caller's arrays: 8-byte aligned.
template <int BX, int AX, int BZ, int AZ, bool ZFIRST, bool BATCH, bool RHS = false>
__global__ __launch_bounds__((PlaneShape<BX, AX, BZ, AZ>::NT), (PlaneShape<BX, AX, BZ, AZ>::WPE)) void k_hxz_plane(
    Dims d, int nc, ZArgs zone, const ZArgs* __restrict__ ztab, HxArgs xone,
    const HxArgs* __restrict__ xtab, int nplanes) {
    using SH = PlaneShape<BX, AX, BZ, AZ>;
    constexpr int NX = SH::NX, NZ = SH::NZ, RS = SH::RS, NT = SH::NT;
    constexpr bool PF = SH::PF;
    constexpr int NV = NX * NZ / 2;                          // double2 values of the plane
    constexpr int NR = (NV + NT - 1) / NT;
    __shared__ double P[NX * RS];
    __shared__ tw2v TWX[NX], TWZ[NZ];
    const size_t pstride = (size_t)d.ny * NZ;
    // twiddles of the two lengths (the same table for every instance)
    {
        const ZArgs& z0 = inst_args<BATCH>(zone, ztab, 0);
        const HxArgs& x0 = inst_args<BATCH>(xone, xtab, 0);
        const Gl<tw2v>* gz = (const Gl<tw2v>*)z0.tw;
        const Gl<tw2v>* gx = (const Gl<tw2v>*)x0.tw;
        for (int t = threadIdx.x; t < NX; t += NT) TWX[t] = gx[t];
        for (int t = threadIdx.x; t < NZ; t += NT) TWZ[t] = gz[t];
    }
    // the source and destination of plane p
    auto src_of = [&](int p) -> const Gl<double>* {
        const int cg = p / d.M;
        const int j = 1 + (p - cg * d.M);
        const int inst = BATCH ? cg / nc : 0;
        const int c = cg - inst * nc;
        const ZArgs& za = inst_args<BATCH>(zone, ztab, inst);
        const HxArgs& xa = inst_args<BATCH>(xone, xtab, inst);
        return (const Gl<double>*)(ZFIRST ? pick(za.spec, c) : pick(xa.spec, c)) + (size_t)j * NZ;
    };
    auto dst_of = [&](int p) -> Gl<double>* {
        const int cg = p / d.M;
        const int j = 1 + (p - cg * d.M);
        const int inst = BATCH ? cg / nc : 0;
        const int c = cg - inst * nc;
        const ZArgs& za = inst_args<BATCH>(zone, ztab, inst);
        const HxArgs& xa = inst_args<BATCH>(xone, xtab, inst);
        return (Gl<double>*)(ZFIRST ? pick(xa.spec, c) : pick(za.u, c)) + (size_t)j * NZ;
    };
    // the next plane from q on (stride: the grid) whose instance is not gated off
    auto live = [&](int q) {
        while (q < nplanes) {
            const int inst = BATCH ? q / (d.M * nc) : 0;
            const ZArgs& za = inst_args<BATCH>(zone, ztab, inst);
            if (!(za.gate && *(const Gl<int>*)za.gate)) break;
            if (!BATCH) return nplanes;
            q += (int)gridDim.x;
        }
        return q;
    };
    // x-row i of a plane at P[i * RS]; 16-byte values, NZ / 2 per row
    constexpr int NR1 = (NR + 1) / 2;
    double2 v[NR];
    auto load = [&](int p, int r0, int r1) {
        const Gl<double>* in = src_of(p);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            if (r < r0 || r >= r1) continue;
            const int t = min((int)threadIdx.x + r * NT, NV - 1);
            const int i = t / (NZ / 2), k2 = t - i * (NZ / 2);
            v[r] = RHS ? ldg2u(in + i * pstride + 2 * k2) : ldg2(in + i * pstride + 2 * k2);
        }
        if constexpr (RHS) {
            const int cg = p / d.M, j = 1 + (p - cg * d.M);
            const double sg = zone.sgn;
            const bool wall = j == 1 || j == d.M;
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                if (r < r0 || r >= r1) continue;
                v[r].x *= sg;
                v[r].y *= sg;
                if (!wall) continue;
                const int t = min((int)threadIdx.x + r * NT, NV - 1);
                const int i = t / (NZ / 2), k2 = t - i * (NZ / 2);
                const Gl<double>* w = (const Gl<double>*)pick(zone.wall, cg) + i * pstride + 2 * k2;
                if (j == 1) {
                    const double2 u = ldg2u(w);
                    v[r].x -= u.x * d.inv_h2;
                    v[r].y -= u.y * d.inv_h2;
                }
                if (j == d.M) {
                    const double2 u = ldg2u(w + (size_t)(d.ny - 1) * NZ);
                    v[r].x -= u.x * d.inv_h2;
                    v[r].y -= u.y * d.inv_h2;
                }
            }
        }
    };
    int p = live(blockIdx.x);
    if constexpr (RHS) {
        if (zone.reset && blockIdx.x + threadIdx.x == 0) clear_status(zone.scal, zone.reset);
    }
    if (PF && p < nplanes) load(p, 0, NR);
    while (p < nplanes) {
        if (!PF) load(p, 0, NR);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int t = threadIdx.x + r * NT;
            if (t < NV) {
                const int i = t / (NZ / 2), k2 = t - i * (NZ / 2);
                *reinterpret_cast<double2*>(&P[i * RS + 2 * k2]) = v[r];
            }
        }
        __syncthreads();
        const int pn = BATCH ? live(p + (int)gridDim.x) : p + (int)gridDim.x;
        if (PF && pn < nplanes) load(pn, 0, NR1);   // in flight while this plane is transformed
        // the lane index through an empty asm statement: the transforms' LDS offsets are then
        // recomputed in every round instead of held (and spilled) across the loop
        int it = threadIdx.x;
        asm volatile("" : "+v"(it));
        if constexpr (ZFIRST) {
            plane_hartley<BZ, AZ, NX / 2, RS, true, double, NT>(P, TWZ, it);
            plane_hartley<BX, AX, NZ / 2, RS, false, double, NT>(P, TWX, it);
        } else {
            plane_hartley<BX, AX, NZ / 2, RS, false, double, NT>(P, TWX, it);
            plane_hartley<BZ, AZ, NX / 2, RS, true, double, NT>(P, TWZ, it);
        }
        if (PF && pn < nplanes) load(pn, NR1, NR);  // in flight while this plane is stored
        Gl<double>* out = dst_of(p);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int t = threadIdx.x + r * NT;
            if (t < NV) {
                const int i = t / (NZ / 2), k2 = t - i * (NZ / 2);
                const double2 w = *reinterpret_cast<const double2*>(&P[i * RS + 2 * k2]);
                stg2u(out + i * pstride + 2 * k2, w.x, w.y);
            }
        }
        __syncthreads();   // the plane's LDS is read out before the next one is written
        p = pn;
    }
}

// The refined mode's plane passes: FP32 spectral data, the (x, z) plane of one interior row
// and component in LDS as floats (n_x rows of plane_row floats: 66 KB at 128 x 128). ZFIRST: the forward
// transforms, z then x, of the FP32 residuals in place (z.spec[c], c < 6: vorticity then stream vector). Otherwise the inverse transforms, x then z,
// of the FP32 corrections (x.spec[c]) added to the FP64 fields (z.u[c]) as k_hz_out adds them:
// the time increments of the first cycle's update (z.inc, z.pinc, z.hist, z.hist_out) or of a
// later cycle (z.inc), or a plain add (z.add, the initial solve). Planes of an instance whose
// z.gate is set are skipped. Persistent, with the next plane's loads in flight, as k_hxz_plane.
template <int BX, int AX, int BZ, int AZ, bool ZFIRST, bool BATCH>
__global__ __launch_bounds__(kPlaneThreads) void k_plane32(Dims d, ZArgs zone,
                                                         const ZArgs* __restrict__ ztab,
                                                         HxArgs xone,
                                                         const HxArgs* __restrict__ xtab,
                                                         int nplanes) {
    constexpr int NC = 6;
    constexpr int NX = BX * AX, NZ = BZ * AZ, RS = plane_row(NZ, AZ);
    constexpr int NT = kPlaneThreads;
    constexpr int NV = NX * NZ / 2;                          // float pairs of the plane
    constexpr int NR = (NV + NT - 1) / NT;
    constexpr int NR1 = (NR + 1) / 2;
    // planes of more than 16 pairs per lane (128 x 256): transforms over halves of the lines
    // (one item per lane), and no prefetch (its registers would spill)
    constexpr bool PF = NR <= 16;
    constexpr int ZH = (NX / 2) * AZ > NT ? 2 : 1;
    constexpr int XH = (NZ / 2) * AX > NT ? 2 : 1;
    __shared__ float P[NX * RS];
    __shared__ tw2v TWX[NX], TWZ[NZ];
    const size_t pstride = (size_t)d.ny * NZ;
    {
        const ZArgs& z0 = inst_args<BATCH>(zone, ztab, 0);
        const HxArgs& x0 = inst_args<BATCH>(xone, xtab, 0);
        const Gl<tw2v>* gz = (const Gl<tw2v>*)z0.tw;
        const Gl<tw2v>* gx = (const Gl<tw2v>*)x0.tw;
        for (int t = threadIdx.x; t < NX; t += NT) TWX[t] = gx[t];
        for (int t = threadIdx.x; t < NZ; t += NT) TWZ[t] = gz[t];
    }
    struct Where {
        int inst, c, j;
    };
    auto where = [&](int p) -> Where {
        const int cg = p / d.M;
        const int inst = BATCH ? cg / NC : 0;
        return Where{inst, cg - inst * NC, 1 + (p - cg * d.M)};
    };
    auto live = [&](int q) {   // the next plane from q on (stride: the grid) not gated off
        while (q < nplanes) {
            const ZArgs& za = inst_args<BATCH>(zone, ztab, where(q).inst);
            if (!(za.gate && *(const Gl<int>*)za.gate)) break;
            q += (int)gridDim.x;
        }
        return q;
    };
    auto src_of = [&](int p) -> const Gl<float>* {
        const Where w = where(p);
        const ZArgs& za = inst_args<BATCH>(zone, ztab, w.inst);
        const HxArgs& xa = inst_args<BATCH>(xone, xtab, w.inst);
        return (const Gl<float>*)(ZFIRST ? pick(za.spec, w.c) : pick(xa.spec, w.c)) + (size_t)w.j * NZ;
    };
    float2 v[NR];
    auto load = [&](int p, int r0, int r1) {
        const Gl<float>* in = src_of(p);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            if (r < r0 || r >= r1) continue;
            const int t = min((int)threadIdx.x + r * NT, NV - 1);
            const int i = t / (NZ / 2), k2 = t - i * (NZ / 2);
            const gf2v q = *reinterpret_cast<const Gl<gf2v>*>(in + i * pstride + 2 * k2);
            v[r] = make_float2(q.x, q.y);
        }
    };
    int p = live(blockIdx.x);
    if (PF && p < nplanes) load(p, 0, NR);
    while (p < nplanes) {
        if constexpr (PF) {
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int t = threadIdx.x + r * NT;
                if (t < NV) {
                    const int i = t / (NZ / 2), k2 = t - i * (NZ / 2);
                    *reinterpret_cast<float2*>(&P[i * RS + 2 * k2]) = v[r];
                }
            }
        } else {
            const Gl<float>* in = src_of(p);
#pragma unroll 8
            for (int r = 0; r < NR; ++r) {
                const int t = threadIdx.x + r * NT;
                const int i = t / (NZ / 2), k2 = t - i * (NZ / 2);
                const gf2v q = *reinterpret_cast<const Gl<gf2v>*>(in + i * pstride + 2 * k2);
                *reinterpret_cast<float2*>(&P[i * RS + 2 * k2]) = make_float2(q.x, q.y);
            }
        }
        __syncthreads();
        const int pn = live(p + (int)gridDim.x);
        if (PF && pn < nplanes) load(pn, 0, NR1);
        int it = threadIdx.x;
        asm volatile("" : "+v"(it));
        auto zpass = [&] {
#pragma unroll
            for (int q = 0; q < ZH; ++q)
                plane_hartley<BZ, AZ, NX / 2 / ZH, RS, true>(P + q * (NX / ZH) * RS, TWZ, it);
        };
        auto xpass = [&] {
#pragma unroll
            for (int q = 0; q < XH; ++q)
                plane_hartley<BX, AX, NZ / 2 / XH, RS, false>(P + q * (NZ / XH), TWX, it);
        };
        if constexpr (ZFIRST) {
            zpass();
            xpass();
        } else {
            xpass();
            zpass();
        }
        if (PF && pn < nplanes) load(pn, NR1, NR);
        const Where w = where(p);
        const ZArgs& za = inst_args<BATCH>(zone, ztab, w.inst);
        if constexpr (ZFIRST) {
            Gl<float>* out = (Gl<float>*)pick(za.spec, w.c) + (size_t)w.j * NZ;
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int t = threadIdx.x + r * NT;
                if (t < NV) {
                    const int i = t / (NZ / 2), k2 = t - i * (NZ / 2);
                    const float2 e = *reinterpret_cast<const float2*>(&P[i * RS + 2 * k2]);
                    stc<float>(out + i * pstride + 2 * k2, e.x, e.y);
                }
            }
        } else {
            Gl<double>* uc = (Gl<double>*)pick(za.u, w.c) + (size_t)w.j * NZ;
            Gl<float>* __restrict__ ic = (Gl<float>*)pick(za.inc, w.c);
            const Gl<float>* __restrict__ pc = (const Gl<float>*)pick(za.pinc, w.c);
            if (ic) ic += (size_t)w.j * NZ;
            if (pc) pc += (size_t)w.j * NZ;
            const int h = za.hist ? *(const Gl<int>*)za.hist : -1;
            if (za.hist_out && w.c == 0 && w.j == 1 && threadIdx.x == 0)
                *(Gl<int>*)za.hist_out = h < 2 ? h + 1 : 2;
            const int add = za.add;
            // MODE as in k_hz_out: 0 plain store or add, 1 a later cycle, 2 + H the first cycle
            auto put = [&](auto mc) {
                constexpr int MODE = decltype(mc)::value;
#pragma unroll 4
                for (int r = 0; r < NR; ++r) {
                    const int t = threadIdx.x + r * NT;
                    if (t < NV) {
                        const int i = t / (NZ / 2), k2 = t - i * (NZ / 2);
                        const float2 ef = *reinterpret_cast<const float2*>(&P[i * RS + 2 * k2]);
                        const double e0 = (double)ef.x, e1 = (double)ef.y;
                        const size_t o = i * pstride + 2 * k2;
                        const double2 u = ldg2(uc + o);
                        if constexpr (MODE == 0) {
                            if (add) stc<double>(uc + o, u.x + e0, u.y + e1);
                            else stc<double>(uc + o, e0, e1);
                        } else if constexpr (MODE == 1) {
                            const double2 q = ldg2(ic + o);
                            stc<double>(uc + o, u.x + e0, u.y + e1);
                            stc<float>(ic + o, (float)(q.x + e0), (float)(q.y + e1));
                        } else {
                            double p0 = 0.0, p1 = 0.0;
                            if constexpr (MODE == 3) {
                                const double2 a = ldg2(pc + o);
                                p0 = a.x;
                                p1 = a.y;
                            } else if constexpr (MODE == 4) {
                                const double2 a = ldg2(pc + o), b = ldg2(ic + o);
                                p0 = 2.0 * a.x - b.x;
                                p1 = 2.0 * a.y - b.y;
                            }
                            stc<double>(uc + o, (u.x + p0) + e0, (u.y + p1) + e1);
                            stc<float>(ic + o, (float)(p0 + e0), (float)(p1 + e1));
                        }
                    }
                }
            };
            if (!add || !ic) put(std::integral_constant<int, 0>{});
            else if (h < 0) put(std::integral_constant<int, 1>{});
            else if (h == 0) put(std::integral_constant<int, 2>{});
            else if (h == 1) put(std::integral_constant<int, 3>{});
            else put(std::integral_constant<int, 4>{});
        }
        __syncthreads();   // the plane's LDS is read out before the next one is written
        p = pn;
    }
}

}  // namespace

// Blocks of a persistent plane launch: the compute units of the current device.
int plane_blocks() {
    static int n = 0;
    if (n == 0) {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0)
            n = cus;
        else
            n = 256;
    }
    return n;
}

// The grids with kernels of their own; the others take launch_plane_any where it fits.
static bool plane_own(const Dims& d) {
    auto len = [](int n) { return n == 32 || n == 48 || n == 64 || n == 96 || n == 128; };
    return len(d.nx) && len(d.nz);
}
bool plane_fits(const Dims& d) { return plane_own(d) || plane_any_fits(d); }

namespace {

template <int BX, int AX, int BZ, int AZ>
void plane_go(hipStream_t s, const Dims& d, bool zfirst, int ncomp, const Over<ZArgs>& z,
              const Over<HxArgs>& x) {
    using SH = PlaneShape<BX, AX, BZ, AZ>;
    const int nplanes = d.M * ncomp * (z.tab ? z.n : 1);
    // persistent: as many blocks as the CUs hold at once, up to the plane count
    const dim3 g((unsigned)std::min(nplanes, SH::PER_CU * plane_blocks())), blk((unsigned)SH::NT);
    auto go = [&](auto kf, auto kt) {
        if (z.tab) launch_kernel(kt, g, blk, 0, s, d, ncomp, z.one, z.tab, x.one, x.tab, nplanes);
        else launch_kernel(kf, g, blk, 0, s, d, ncomp, z.one, z.tab, x.one, x.tab, nplanes);
    };
    if (zfirst && z.one.wall[0] && !z.tab)
        launch_kernel((k_hxz_plane<BX, AX, BZ, AZ, true, false, true>), g, blk, 0, s, d, ncomp, z.one, z.tab,
                      x.one, x.tab, nplanes);
    else if (zfirst) go(k_hxz_plane<BX, AX, BZ, AZ, true, false>, k_hxz_plane<BX, AX, BZ, AZ, true, true>);
    else go(k_hxz_plane<BX, AX, BZ, AZ, false, false>, k_hxz_plane<BX, AX, BZ, AZ, false, true>);
}

template <int BX, int AX>
void plane_go_x(hipStream_t s, const Dims& d, bool zfirst, int ncomp, const Over<ZArgs>& z,
                const Over<HxArgs>& x) {
    switch (d.nz) {
    case 32: plane_go<BX, AX, 8, 4>(s, d, zfirst, ncomp, z, x); return;
    case 48: plane_go<BX, AX, 16, 3>(s, d, zfirst, ncomp, z, x); return;
    case 64: plane_go<BX, AX, 16, 4>(s, d, zfirst, ncomp, z, x); return;
    case 96: plane_go<BX, AX, 16, 6>(s, d, zfirst, ncomp, z, x); return;
    default: plane_go<BX, AX, 16, 8>(s, d, zfirst, ncomp, z, x); return;
    }
}

}  // namespace

bool launch_plane(hipStream_t s, const Dims& d, bool zfirst, int ncomp, const Over<ZArgs>& z,
                  const Over<HxArgs>& x) {
    if (!plane_fits(d) || ncomp < 1 || ncomp > 6 || z.one.add) return false;
    if ((z.tab != nullptr) != (x.tab != nullptr) || (z.tab && z.n != x.n)) return false;
    if (!plane_own(d)) {
        launch_plane_any(s, d, zfirst, ncomp, z, x);
        return true;
    }
    switch (d.nx) {
    case 32: plane_go_x<8, 4>(s, d, zfirst, ncomp, z, x); break;
    case 48: plane_go_x<16, 3>(s, d, zfirst, ncomp, z, x); break;
    case 64: plane_go_x<16, 4>(s, d, zfirst, ncomp, z, x); break;
    case 96: plane_go_x<16, 6>(s, d, zfirst, ncomp, z, x); break;
    default: plane_go_x<16, 8>(s, d, zfirst, ncomp, z, x); break;
    }
    return true;
}

// The refined mode's FP32 plane forms: square planes of n_x = n_z in {32, 48, 64, 96, 128}
// and the 128 x 256 plane (132 KB of floats).
bool plane32_fits(const Dims& d) {
    return (d.nx == d.nz && plane_own(d)) || (d.nx == 128 && d.nz == 256);
}

bool launch_plane32(hipStream_t s, const Dims& d, bool zfirst, const Over<ZArgs>& z,
                    const Over<HxArgs>& x) {
    if (!plane32_fits(d)) return false;
    const bool batch = z.tab != nullptr;
    if (batch != (x.tab != nullptr) || (batch && z.n != x.n)) return false;
    const int ni = batch ? z.n : 1;
    const int nplanes = d.M * 6 * ni;
    // persistent: as many blocks as fit on the CUs at once (two per CU for planes up to
    // 80 KB of LDS)
    const size_t lds = (size_t)d.nx * (d.nz + 8) * sizeof(float) + (size_t)(d.nx + d.nz) * sizeof(tw2v);
    const int per_cu = lds <= 80 * 1024 ? 2 : 1;
    const dim3 g((unsigned)std::min(nplanes, per_cu * plane_blocks()));
    const dim3 blk((unsigned)kPlaneThreads);   // the kernels' launch bound
    auto go = [&](auto kf, auto kt) {
        if (batch) launch_kernel(kt, g, blk, 0, s, d, z.one, z.tab, x.one, x.tab, nplanes);
        else launch_kernel(kf, g, blk, 0, s, d, z.one, z.tab, x.one, x.tab, nplanes);
    };
#define VS_PLANE32(nx_, nz_, bx, ax, bz, az)                                                     \
    if (d.nx == nx_ && d.nz == nz_) {                                                            \
        if (zfirst)                                                                              \
            go(k_plane32<bx, ax, bz, az, true, false>, k_plane32<bx, ax, bz, az, true, true>);    \
        else                                                                                     \
            go(k_plane32<bx, ax, bz, az, false, false>, k_plane32<bx, ax, bz, az, false, true>);  \
        return true;                                                                             \
    }
    VS_PLANE32(32, 32, 8, 4, 8, 4)
    VS_PLANE32(48, 48, 16, 3, 16, 3)
    VS_PLANE32(64, 64, 16, 4, 16, 4)
    VS_PLANE32(96, 96, 16, 6, 16, 6)
    VS_PLANE32(128, 128, 16, 8, 16, 8)
    VS_PLANE32(128, 256, 16, 8, 16, 16)
#undef VS_PLANE32
    return false;
}

}  // namespace vs
