// grmhd_sweep.hip -- one FP64 substep of a grid (or its right-hand side) in one
// launch (two for flux-CT), MC or PPM reconstruction.
//
// A wave owns 62 consecutive positions of a plane's rows laid end to end (each
// row with one ghost position at either end) and marches over a segment of
// planes; lanes 0 and 63 repeat the neighbouring waves' edge positions, so that
// a wave needs nothing from another one: no barriers, no shared staging.
//   x  every lane reconstructs its own cell and solves the face on its left; the
//      left state comes from the lane to the left, the flux through the right
//      face from the lane to the right (DPP wave shifts);
//   y  both faces of the cell, from the rows beside it (the caches serve a row
//      again to the waves of its neighbours);
//   z  the face above the cell; the flux below, the left state and the next cell
//      are carried from plane to plane in LDS (each lane its own words).
// Then sources, Runge-Kutta combination, recovery and the new primitives, which
// go to another cache with their ghost images.  Flux-CT leaves the cell to a
// second launch (k_ct_update).
//
// Bound by vector issue and by memory together: a curved 192^3 substep (0.90 ms)
// takes 2,900 vector instructions a cell (issue 58 % of the time, at two waves per
// SIMD) and moves 487 B a cell (336 by design), at 79 % of a copy's rate; with PPM
// (128^3) 5,000 instructions and 620 B.  185 to 222 registers for a substep, to 230
// for flux-CT, to 256 for the 1D instances (the curved one spills 2).  It replaced,
// for three RK3 steps or as stated: face kernels and an update on 2D grids (500 x
// 300, five steps: 551 to 342 us) and with PPM (128^3, two steps: 3.59 to 2.75 ms), a
// kernel that staged 32 x 8 tiles in LDS between two barriers a plane on 3D grids
// (192^3: 9.11 to 8.8 ms; 101 x 87 x 75, where tiles are ragged: 1.25 to 0.93 ms; kept
// where it takes a round less, substep_tiled), and nine launches of a right-hand
// side (24 x 20 x 16: 41 to 11.5 us).  Three waves per SIMD spilled 30 to 50 registers
// and took 13.3 ms for the 9.1 of two.
#include "grmhd_cell.h"
#include "grmhd_device.h"
#include "grmhd_internal.h"

namespace grmhd {

static constexpr int SWEEP_USED = 62;   // positions a wave updates

struct SweepKernelArgs {
    SweepArgs A;
    Dev d;
};

__device__ __forceinline__ SweepKernelArgs sweep_args()
{
    return kernel_args<SweepKernelArgs>();
}

// Lower and upper edge values of the middle cell of a line of cells at(-2 .. 2).
template <bool PPM, typename At>
__device__ __forceinline__ void cell_edges(At&& at, double& lo, double& hi)
{
    if constexpr (PPM) {
        ppm_edges(at(-2), at(-1), at(0), at(1), at(2), lo, hi);
    } else {
        const double c = at(0), h = mc_hslope(at(-1), c, at(1));
        lo = c - h;
        hi = c + h;
    }
}

// Index c of an axis of n cells mapped into the domain by the boundary rule.
__device__ __forceinline__ int map_cell(int c, int n, int bc)
{
    if (c >= 0 && c < n)
        return c;
    if (bc != 0)
        return c < 0 ? 0 : n - 1;
    return c < 0 ? c + n : c - n;
}

// Where the primitives come from: the ghosted cache, or, for a right-hand side
// that does not overlap them, the caller's dense array with indices mapped by the
// boundary rule.
template <bool DENSE, int G>
struct Source {
    static constexpr int X = G - 1;          // cells read beside one along x
    unsigned o;                              // the lane's own position
    unsigned ox[2 * X + 1], oy[2 * G + 1];   // dense: shifted along x, along y

    __device__ __forceinline__ Source(const Dev& d, int i, int j)
    {
        if constexpr (DENSE) {
            const int im = map_cell(i, d.n[0], d.bc[0]);
            o = (unsigned)(im + d.n[0] * j) * 8u;
#pragma unroll
            for (int m = -X; m <= X; ++m)
                ox[m + X] = d.act[0] ? (unsigned)(map_cell(i + m, d.n[0], d.bc[0]) + d.n[0] * j) * 8u : o;
#pragma unroll
            for (int m = -G; m <= G; ++m)
                oy[m + G] = d.act[1] ? (unsigned)(im + d.n[0] * map_cell(j + m, d.n[1], d.bc[1])) * 8u : o;
        } else {
            o = (unsigned)((j + d.g[1]) * d.px + i + d.g[0]) * 8u;
        }
    }

    // Variable v of the cell shifted by (x, y, z) (one of them at most not 0) in plane k.
    __device__ __forceinline__ double at(const SweepArgs& A, const Dev& d, int v, int k, int x, int y, int z) const
    {
        if constexpr (DENSE) {
            const int kk = d.act[2] ? map_cell(k + z, d.n[2], d.bc[2]) : 0;
            const double* p = A.P + v * d.N + (long long)kk * d.n[0] * d.n[1];
            return buf_load(p, x != 0 ? ox[x + X] : (y != 0 ? oy[y + G] : o));
        } else {
            // shifts count from the lowest cell read, which keeps the offsets positive
            const double* p = A.Pc + v * d.sv + (long long)(k + d.g[2] + z) * d.px * d.py - X;
            if (y != 0)
                return buf_load(p - G * d.px, o + 8u * X, (unsigned)((y + G) * d.px) * 8u);
            return buf_load(p, o + 8u * (x + X));
        }
    }
};

// Store the new primitives p of a cell (i, j, k) at cache position o of its plane
// and at the ghost positions whose boundary rule copies it (as store_prim).
__device__ __forceinline__ void sweep_store(double* Pn, const Dev& d, unsigned o, int i, int j, int k,
                                            const double* p)
{
    const long long st = (long long)d.px * d.py;
    auto put = [&](int plane, unsigned at) {
#pragma unroll
        for (int v = 0; v < 9; ++v)
            buf_store(Pn + v * d.sv + (plane + d.g[2]) * st, at, p[v]);
    };
    put(k, o);
    auto images = [&](int a, int idx, int n, int g, unsigned step) {
        if (!d.act[a])
            return;
        if (d.bc[a] == 0) {
            if (idx < g)
                put(k, o + (unsigned)n * step);
            if (idx >= n - g)
                put(k, o - (unsigned)n * step);
        } else if (idx == 0 || idx == n - 1) {
            for (int e = 1; e <= g; ++e)
                put(k, idx == 0 ? o - (unsigned)e * step : o + (unsigned)e * step);
        }
    };
    images(0, i, d.n[0], d.g[0], 8u);
    images(1, j, d.n[1], d.g[1], 8u * (unsigned)d.px);
    if (d.act[2]) {
        const int n = d.n[2], g = d.g[2];
        if (d.bc[2] == 0) {
            if (k < g)
                put(k + n, o);
            if (k >= n - g)
                put(k - n, o);
        } else if (k == 0 || k == n - 1) {
            for (int e = 1; e <= g; ++e)
                put(k == 0 ? -e : k + e, o);
        }
    }
}

// The face solver: on 1D grids (LINE) the plain order of operations, whichever axis
// they lie along.
template <int D, bool LINE>
__device__ __forceinline__ void sweep_face(double* qL, double* qR, const GeoT<double>& g, const Dev& d, double* F)
{
    if constexpr (LINE)
        face_solve<D>(qL, qR, g, d, F);
    else
        face_solve64<D>(qL, qR, g, d, F);
}

// What a sweep leaves: the new state; the right-hand side; or, for flux-CT, the
// flux differences and sources of mass, energy and momentum (and the flux
// differences of the field along an inactive axis, which no edge value corrects)
// and the transverse field fluxes of every face, which k_ct_update takes further.  DENSE: the
// primitives come from the caller's array.
enum { SWEEP_STEP = 0, SWEEP_RHS = 1, SWEEP_CT = 2 };

// The transverse field components of a face's flux along D into its records.
template <int D>
__device__ __forceinline__ void put_transverse(double* F, long long nf, long long f, const double* Fo)
{
    constexpr int B = D == 0 ? 1 : 0, C = D == 2 ? 1 : 2;
    F[(5 + B) * nf + f] = Fo[5 + B];
    F[(5 + C) * nf + f] = Fo[5 + C];
}

template <int KIND, bool PPM, int ROLE, bool DENSE, bool LINE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_sweep(SweepKernelArgs)
{
    constexpr int G = PPM ? 3 : 2, X = G - 1;
    // carried along z: the left state and the flux of the next face, the next cell
    // (and for PPM the cell below)
    __shared__ double sL[9 * 64], sF[9 * 64], sQ[9 * 64], sM[PPM ? 9 * 64 : 1];

    const SweepKernelArgs K0 = sweep_args();
    const SweepArgs& A0 = K0.A;
    // items (row group, segment), the row group fastest, in contiguous runs per XCD
    const unsigned run = gridDim.x / 8;
    const unsigned item = (blockIdx.x % 8) * run + blockIdx.x / 8;
    if (item >= (unsigned)A0.ngrp * (unsigned)A0.nseg)
        return;
    const int seg = (int)(item / (unsigned)A0.ngrp), grp = (int)(item - (unsigned)seg * (unsigned)A0.ngrp);
    const int lane = threadIdx.x;
    const int nx = K0.d.n[0], ny = K0.d.n[1];
    const bool ax = K0.d.act[0], ay = K0.d.act[1], az = K0.d.act[2];
    const int wx = ax ? nx + 2 : nx;
    const int s = grp * SWEEP_USED + lane - 1, total = ny * wx;
    const int sc = min(max(s, 0), total - 1);
    const int j = sc / wx, i = sc - j * wx - (ax ? 1 : 0);
    const bool used = s == sc && lane >= 1 && lane <= SWEEP_USED, own = used && i >= 0 && i < nx;
    const int k0 = seg * A0.seg, k1 = min(k0 + A0.seg, K0.d.n[2]);
    const int ic = min(max(i, 0), nx - 1);   // a cell of the row, also for the lanes at its ends
    const unsigned oc = (unsigned)(ic + nx * j) * 8u;
    const Source<DENSE, G> P(K0.d, i, j);

    double q0[9];
#pragma unroll
    for (int v = 0; v < 9; ++v)
        q0[v] = P.at(A0, K0.d, v, k0, 0, 0, 0);
    if (az) {
        const Dev& d = K0.d;
        double qL[9], qR[9], F[9];
#pragma unroll
        for (int v = 0; v < 9; ++v) {
            double q[2 * G + 1], e, hi;   // planes k0 - G .. k0 + G
#pragma unroll
            for (int m = -G; m < G; ++m)
                q[m + G] = m == 0 ? q0[v] : P.at(A0, d, v, k0, 0, 0, m);
            cell_edges<PPM>([&](int m) { return q[m - 1 + G]; }, e, qL[v]);
            cell_edges<PPM>([&](int m) { return q[m + G]; }, qR[v], hi);
            sL[v * 64 + lane] = hi;
            sQ[v * 64 + lane] = q[1 + G];
            if (PPM)
                sM[v * 64 + lane] = q[-1 + G];
        }
        const Geo g = face_geo<2, KIND, double>(d, d.lo[0] + (i + 0.5) * d.dx[0], d.lo[1] + (j + 0.5) * d.dx[1],
                                        d.lo[2] + k0 * d.dx[2], ic + (long long)nx * (j + (long long)ny * k0));
        sweep_face<2, LINE>(qL, qR, geo_cast<double>(g), d, F);
#pragma unroll
        for (int v = 0; v < 9; ++v)
            sF[v * 64 + lane] = F[v];
    }
    int nfail = 0, natm = 0, npf = 0, nfb = 0, itmax = 0;

    // The loads of a plane go out in groups (left to itself the compiler loads a
    // variable's stencil, waits and loads the next: 40 exposed latencies a plane,
    // and 1.6 ms instead of 1.0 ms for a 192^3 substep).
    for (int k = k0; k < k1; ++k) {
        double R[9];
#pragma unroll
        for (int v = 0; v < 9; ++v)
            R[v] = 0.0;
        if (ay) {
            const SweepKernelArgs K = sweep_args();
            const Dev& d = K.d;
            double lL[9], lR[9], hL[9], hR[9], Fl[9], Fh[9];
            // PPM: in three batches of variables, which bounds the registers
            constexpr int NB = PPM ? 3 : 9;
#pragma unroll
            for (int b = 0; b < 9; b += NB) {
                double r[NB][2 * G + 1];
#pragma unroll
                for (int v = 0; v < NB; ++v)
#pragma unroll
                    for (int m = -G; m <= G; ++m)
                        r[v][m + G] = m == 0 ? q0[b + v] : P.at(K.A, d, b + v, k, 0, m, 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int v = 0; v < NB; ++v) {
                    double e;
                    cell_edges<PPM>([&](int m) { return r[v][m - 1 + G]; }, e, lL[b + v]);
                    cell_edges<PPM>([&](int m) { return r[v][m + G]; }, lR[b + v], hL[b + v]);
                    cell_edges<PPM>([&](int m) { return r[v][m + 1 + G]; }, hR[b + v], e);
                }
            }
            const double x = d.lo[0] + (i + 0.5) * d.dx[0], z = d.lo[2] + (k + 0.5) * d.dx[2];
            const long long f = ic + (long long)nx * (j + (long long)(ny + 1) * k);
            sweep_face<1, LINE>(
                lL, lR, geo_cast<double>(face_geo<1, KIND, double>(d, x, d.lo[1] + j * d.dx[1], z, f)), d, Fl);
            sweep_face<1, LINE>(
                hL, hR, geo_cast<double>(face_geo<1, KIND, double>(d, x, d.lo[1] + (j + 1) * d.dx[1], z, f + nx)), d,
                Fh);
            if (ROLE == SWEEP_CT && own) {
                put_transverse<1>(K.A.F[1], d.nf[1], f, Fl);
                if (j == ny - 1)
                    put_transverse<1>(K.A.F[1], d.nf[1], f + nx, Fh);
            }
#pragma unroll
            for (int v = 0; v < 9; ++v)
                R[v] = -(Fh[v] - Fl[v]) * d.idx[1];
        }
        double q2[9], q3[9];
        if (ax) {
            const SweepKernelArgs K = sweep_args();
            const Dev& d = K.d;
            double r[9][2 * X + 1], qL[9], qR[9], F[9];
#pragma unroll
            for (int v = 0; v < 9; ++v)
#pragma unroll
                for (int m = -X; m <= X; ++m)
                    r[v][m + X] = m == 0 ? q0[v] : P.at(K.A, d, v, k, m, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int v = 0; v < 9; ++v) {
                double hi;
                cell_edges<PPM>([&](int m) { return r[v][m + X]; }, qR[v], hi);
                qL[v] = from_left(hi);
            }
            if (!PPM && az) {
#pragma unroll
                for (int v = 0; v < 9; ++v)
                    q2[v] = P.at(K.A, d, v, k, 0, 0, 2);
                __builtin_amdgcn_sched_barrier(0);
            }
            const long long f = max(i, 0) + (long long)(nx + 1) * (j + (long long)ny * k);
            const GeoT<double> g = geo_cast<double>(face_geo<0, KIND, double>(
                d, d.lo[0] + i * d.dx[0], d.lo[1] + (j + 0.5) * d.dx[1], d.lo[2] + (k + 0.5) * d.dx[2], f));
            sweep_face<0, LINE>(qL, qR, g, d, F);
            if (ROLE == SWEEP_CT && used && i >= 0)
                put_transverse<0>(K.A.F[0], d.nf[0], f, F);
#pragma unroll
            for (int v = 0; v < 9; ++v)
                R[v] -= (from_right(F[v]) - F[v]) * d.idx[0];
        }
        double q[9];
#pragma unroll
        for (int v = 0; v < 9; ++v)
            q[v] = q0[v];
        if (az) {
            const SweepKernelArgs K = sweep_args();
            const Dev& d = K.d;
            double qL[9], qR[9], F[9];
            if (PPM || !ax) {
#pragma unroll
                for (int v = 0; v < 9; ++v) {
                    q2[v] = P.at(K.A, d, v, k, 0, 0, 2);
                    q3[v] = PPM ? P.at(K.A, d, v, k, 0, 0, 3) : 0.0;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int v = 0; v < 9; ++v) {
                double hi;
                const double q1 = sQ[v * 64 + lane], qm = PPM ? sM[v * 64 + lane] : 0.0;
                cell_edges<PPM>(
                    [&](int m) {
                        return m == -2 ? qm : (m == -1 ? q[v] : (m == 0 ? q1 : (m == 1 ? q2[v] : q3[v])));
                    },
                    qR[v], hi);
                qL[v] = sL[v * 64 + lane];
                sL[v * 64 + lane] = hi;
                if (PPM)
                    sM[v * 64 + lane] = q[v];
                q0[v] = q1;
                sQ[v * 64 + lane] = q2[v];
            }
            const GeoT<double> g = geo_cast<double>(
                face_geo<2, KIND, double>(d, d.lo[0] + (i + 0.5) * d.dx[0], d.lo[1] + (j + 0.5) * d.dx[1],
                                  d.lo[2] + (k + 1) * d.dx[2], ic + (long long)nx * (j + (long long)ny * (k + 1))));
            sweep_face<2, LINE>(qL, qR, g, d, F);
            if (ROLE == SWEEP_CT && own) {
                double Fp[9];
#pragma unroll
                for (int v = 5; v < 7; ++v)
                    Fp[v] = sF[v * 64 + lane];
                const long long f = ic + (long long)nx * (j + (long long)ny * k);
                put_transverse<2>(K.A.F[2], d.nf[2], f, Fp);
                if (k == d.n[2] - 1)
                    put_transverse<2>(K.A.F[2], d.nf[2], f + (long long)nx * ny, F);
            }
#pragma unroll
            for (int v = 0; v < 9; ++v) {
                R[v] -= (F[v] - sF[v * 64 + lane]) * d.idx[2];
                sF[v * 64 + lane] = F[v];
            }
        }
        const SweepKernelArgs K = sweep_args();
        const Dev& d = K.d;
        const SweepArgs& A = K.A;
        const long long plane = (long long)nx * ny * k;   // uniform
        double un[9], us[9];
        // U^n, U^s and U^(s+1) are touched once per cell and substep: past the
        // last-level cache's size streaming accesses keep them from displacing the
        // primitives that neighbouring waves read again
        if constexpr (ROLE == SWEEP_STEP) {
            if (d.nt) {
#pragma unroll
                for (int v = 0; v < 9; ++v)
                    un[v] = buf_load<true>(A.Un + v * d.N + plane, oc);
                if (A.Us) {
#pragma unroll
                    for (int v = 0; v < 9; ++v)
                        us[v] = buf_load<true>(A.Us + v * d.N + plane, oc);
                }
            } else {
#pragma unroll
                for (int v = 0; v < 9; ++v)
                    un[v] = buf_load(A.Un + v * d.N + plane, oc);
                if (A.Us) {
#pragma unroll
                    for (int v = 0; v < 9; ++v)
                        us[v] = buf_load(A.Us + v * d.N + plane, oc);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        Geo g;
        add_sources<KIND>(d, d.lo[0] + (i + 0.5) * d.dx[0], d.lo[1] + (j + 0.5) * d.dx[1],
                          d.lo[2] + (k + 0.5) * d.dx[2], plane + oc / 8u, q, g, R);
        if constexpr (ROLE != SWEEP_STEP) {
            if (own) {
#pragma unroll
                for (int v = 0; v < (ROLE == SWEEP_CT ? 5 : 9); ++v)
                    buf_store(A.R + v * d.N + plane, oc, R[v]);
                if (ROLE == SWEEP_CT)
#pragma unroll
                    for (int a = 0; a < 3; ++a)
                        if (!d.act[a])
                            buf_store(A.Ri + plane, oc, R[5 + a]);
                if (DENSE && A.Pn)
                    sweep_store(A.Pn, d, (unsigned)((j + d.g[1]) * d.px + i + d.g[0]) * 8u, i, j, k, q);
            }
        } else {
            double u[9], p[9];
#pragma unroll
            for (int v = 0; v < 9; ++v) {
                const double ub = A.Us ? us[v] : un[v];
                u[v] = ub + A.a * (un[v] - ub) + A.b * (A.dt * R[v]);
            }
            int flags = 0, iters = 0;
            if (own) {
                flags = recover_cell<double>(d, g, u, q, p, iters);
                const SweepKernelArgs K2 = sweep_args();
                const SweepArgs& B = K2.A;
                const Dev& e = K2.d;
                if (e.nt) {
#pragma unroll
                    for (int v = 0; v < 9; ++v)
                        buf_store<true>(B.Uo + v * e.N + plane, oc, u[v]);
                } else {
#pragma unroll
                    for (int v = 0; v < 9; ++v)
                        buf_store(B.Uo + v * e.N + plane, oc, u[v]);
                }
                sweep_store(B.Pn, e, P.o, i, j, k, p);
                if (B.fout)
                    B.fout[plane + oc / 8u] = (unsigned char)flags;
            }
            if (__any(flags != 0)) {
                nfail += __popcll(__ballot(flags & FLAG_FAIL));
                natm += __popcll(__ballot(flags & FLAG_ATM));
                npf += __popcll(__ballot(flags & FLAG_PFLOOR));
                nfb += __popcll(__ballot(flags & FLAG_FALLBACK));
            }
            itmax = max(itmax, iters);
        }
    }
    if constexpr (ROLE == SWEEP_STEP) {
        for (int m = 32; m > 0; m >>= 1)
            itmax = max(itmax, __shfl_xor(itmax, m));
        if (lane == 0) {
            unsigned long long* cnt = A0.cnt + (size_t)(blockIdx.x % CNT_SLOTS) * CNT_WORDS;
            if (nfail)
                atomicAdd(&cnt[CNT_FAIL], (unsigned long long)nfail);
            if (natm)
                atomicAdd(&cnt[CNT_ATM], (unsigned long long)natm);
            if (npf)
                atomicAdd(&cnt[CNT_PFLOOR], (unsigned long long)npf);
            if (nfb)
                atomicAdd(&cnt[CNT_FALLBACK], (unsigned long long)nfb);
            atomicMax(&cnt[CNT_MAXIT], (unsigned long long)itmax);
        }
    }
}

// Planes per wave: a wave's planes and its first face and loads (half a plane)
// times the waves, and a tail of unevenly finished work worth 1280 waves (of the
// 2048 that are resident).  The line lies where measured: 64^3 (4416, 2208, 1518
// waves) 43.2, 46.8, 44.5 us a substep with 1, 2, 3 planes, 96 x 80 x 72 87, 86,
// 84, 98, 86, 93 us with 1 to 6, 192^3 0.917, 0.920, 0.933, 0.952 ms with 8, 12,
// 16, 32.
static int sweep_segment(long long ngrp, int nz)
{
    int best = 1;
    double cost = 0.0;
    for (int seg = 1; seg <= nz && seg <= 64; ++seg) {
        const double c = (double)(ngrp * ((nz + seg - 1) / seg) + 1280) * (seg + 0.5);
        if (seg == 1 || c < cost) {
            cost = c;
            best = seg;
        }
    }
    return best;
}

// Waves of a plane.
long long sweep_groups(const Dev& d)
{
    const long long wx = d.act[0] ? d.n[0] + 2 : d.n[0];
    return (wx * d.n[1] + SWEEP_USED - 1) / SWEEP_USED;
}

template <int ROLE, bool DENSE, bool LINE>
static hipError_t launch_sweep_l(int kind, const SweepArgs& A, const Dev& d, hipStream_t s)
{
    const long long wx = d.act[0] ? d.n[0] + 2 : d.n[0];
    const long long total = wx * d.n[1];
    // byte offsets within a plane are 32-bit (such grids take the face kernels)
    if ((long long)d.px * d.py * 8 >= (1LL << 32) || total >= (1LL << 31) - 64)
        return hipErrorInvalidValue;
    SweepKernelArgs K{A, d};
    const long long ngrp = sweep_groups(d);
    K.A.ngrp = (int)ngrp;
    K.A.seg = d.act[2] ? sweep_segment(ngrp, d.n[2]) : 1;
    K.A.nseg = (d.n[2] + K.A.seg - 1) / K.A.seg;
    const long long items = ngrp * K.A.nseg, blocks = (items + 7) / 8 * 8;
    if (blocks >= (1LL << 31))
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(64);
#define GRMHD_SWEEP(KIND)                                                                       \
    if (d.ppm)                                                                                  \
        hipLaunchKernelGGL((k_sweep<KIND, true, ROLE, DENSE, LINE>), grid, block, 0, s, K);     \
    else                                                                                        \
        hipLaunchKernelGGL((k_sweep<KIND, false, ROLE, DENSE, LINE>), grid, block, 0, s, K);
    if (kind == FLAT) {
        GRMHD_SWEEP(FLAT)
    } else if (kind == ISO) {
        GRMHD_SWEEP(ISO)
    } else {
        GRMHD_SWEEP(STORED)
    }
#undef GRMHD_SWEEP
    return hipGetLastError();
}

template <int ROLE, bool DENSE>
static hipError_t launch_sweep_r(int kind, const SweepArgs& A, const Dev& d, hipStream_t s)
{
    if constexpr (ROLE != SWEEP_CT) {   // (edge values need two active axes)
        if (d.act[0] + d.act[1] + d.act[2] <= 1)
            return launch_sweep_l<ROLE, DENSE, true>(kind, A, d, s);
    }
    return launch_sweep_l<ROLE, DENSE, false>(kind, A, d, s);
}

// The second half of a flux-CT substep or right-hand side: per cell the field's
// flux differences from the edge values around it (Toth 2000).  The edge value of
// the axes (a, b) at a-face fa and b-face fb is
//   W = 1/4 [F^b(Bd^a) at the two b-faces beside the edge
//            - F^a(Bd^b) at the two a-faces beside it],
// the corrected fluxes are F^a(Bd^b) = -1/2 and F^b(Bd^a) = +1/2 the sum of the
// edge values at a face's two edges.  Every cell forms its four edge values per
// pair itself, the lower neighbour's term first, so that the cells around an edge
// agree on its value to the last bit; the caches serve the repeated reads.  By
// design the two launches move 560 B a cell (measured 290 and 420 at 128^3); face
// records, edge values and corrected fluxes as arrays of their own took 1160 B in
// six launches (three RK2 steps of the 128^3 box 3310 us, 2465 now).
template <int KIND, bool RHS>
__global__ __launch_bounds__(256) void k_ct_update(SweepArgs A, Dev d)
{
    const long long c = (long long)blockIdx.x * 256 + threadIdx.x;
    int nfail = 0, natm = 0, npf = 0, nfb = 0, itmax = 0;
    if (c < d.N) {
        int ix[3];
        if (d.N <= 0x7fffffffLL) {
            const unsigned cu = (unsigned)c, t = cu / (unsigned)d.n[0];
            ix[2] = (int)(t / (unsigned)d.n[1]);
            ix[1] = (int)(t - (unsigned)ix[2] * (unsigned)d.n[1]);
            ix[0] = (int)(cu - t * (unsigned)d.n[0]);
        } else {
            ix[0] = (int)(c % d.n[0]);
            const long long t = c / d.n[0];
            ix[1] = (int)(t % d.n[1]);
            ix[2] = (int)(t / d.n[1]);
        }
        double R[9];
#pragma unroll
        for (int v = 0; v < 5; ++v)
            R[v] = A.R5[v * d.N + c];
#pragma unroll
        for (int v = 5; v < 9; ++v)
            R[v] = v < 8 && !d.act[v - 5] ? A.Ri[c] : 0.0;
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const int a = p == 2 ? 1 : 0, b = p == 0 ? 1 : 2;
            if (!d.act[a] || !d.act[b])
                continue;
            const int ca[3] = {map_cell(ix[a] - 1, d.n[a], d.bc[a]), ix[a], map_cell(ix[a] + 1, d.n[a], d.bc[a])};
            const int cb[3] = {map_cell(ix[b] - 1, d.n[b], d.bc[b]), ix[b], map_cell(ix[b] + 1, d.n[b], d.bc[b])};
            auto record = [&](int dir, int v, int ia, int ib) {
                int q[3] = {ix[0], ix[1], ix[2]};
                q[a] = ia;
                q[b] = ib;
                const long long m0 = d.n[0] + (dir == 0), m1 = d.n[1] + (dir == 1);
                return A.F[dir][v * d.nf[dir] + (q[2] * m1 + q[1]) * m0 + q[0]];
            };
            double gb[3][2], ga[2][3], W[2][2];
#pragma unroll
            for (int m = 0; m < 3; ++m)
#pragma unroll
                for (int f = 0; f < 2; ++f) {
                    gb[m][f] = record(b, 5 + a, ca[m], ix[b] + f);
                    ga[f][m] = record(a, 5 + b, ix[a] + f, cb[m]);
                }
#pragma unroll
            for (int fa = 0; fa < 2; ++fa)
#pragma unroll
                for (int fb = 0; fb < 2; ++fb)
                    W[fa][fb] = 0.25 * ((gb[fa][fb] + gb[fa + 1][fb]) - (ga[fa][fb] + ga[fa][fb + 1]));
            R[5 + a] -= 0.5 * ((W[0][1] + W[1][1]) - (W[0][0] + W[1][0])) * d.idx[b];
            R[5 + b] += 0.5 * ((W[1][0] + W[1][1]) - (W[0][0] + W[0][1])) * d.idx[a];
        }
        if (RHS) {
#pragma unroll
            for (int v = 0; v < 9; ++v)
                A.R[v * d.N + c] = R[v];
        } else {
            const long long pc = cache_index(d, ix[0], ix[1], ix[2]);
            double q[9], u[9], p[9];
#pragma unroll
            for (int v = 0; v < 9; ++v) {
                q[v] = A.Pc[v * d.sv + pc];
                const double un = A.Un[v * d.N + c];
                const double us = A.Us ? A.Us[v * d.N + c] : un;
                u[v] = us + A.a * (un - us) + A.b * (A.dt * R[v]);
            }
            const Geo g = cell_geo<KIND, double>(d, d.lo[0] + (ix[0] + 0.5) * d.dx[0], d.lo[1] + (ix[1] + 0.5) * d.dx[1],
                                         d.lo[2] + (ix[2] + 0.5) * d.dx[2], c);
            int iters = 0;
            const int flags = recover_cell<double>(d, g, u, q, p, iters);
#pragma unroll
            for (int v = 0; v < 9; ++v)
                A.Uo[v * d.N + c] = u[v];
            store_prim(d, A.Pn, pc, ix[0], ix[1], ix[2], p);
            tally(flags, iters, nfail, natm, npf, nfb, itmax);
        }
    }
    if (!RHS)
        count_sums(A.cnt, nfail, natm, npf, nfb, itmax);
}

hipError_t launch_ct_update(int kind, const SweepArgs& A, const Dev& d, hipStream_t s)
{
    const dim3 grid((unsigned)((d.N + 255) / 256)), block(256);
#define GRMHD_CT(KIND)                                                           \
    if (A.R)                                                                     \
        hipLaunchKernelGGL((k_ct_update<KIND, true>), grid, block, 0, s, A, d);  \
    else                                                                         \
        hipLaunchKernelGGL((k_ct_update<KIND, false>), grid, block, 0, s, A, d);
    if (kind == FLAT) {
        GRMHD_CT(FLAT)
    } else if (kind == ISO) {
        GRMHD_CT(ISO)
    } else {
        GRMHD_CT(STORED)
    }
#undef GRMHD_CT
    return hipGetLastError();
}

// One whole Runge-Kutta step of a 1D grid along x (flat metric, MC) in a wave's
// registers: its 64 cells take all stages, and the two cells at either end that
// each stage's stencil spoils repeat cells of the neighbouring waves (RK3: 52 of 64
// lanes are its own, RK2: 56).  A periodic image evolves as its cell does; beyond
// an outflow end the lanes take the end cell's primitives after every stage.
//   direct: one workgroup of up to 4 waves (one per SIMD) holds the whole grid, so
//   the new state may be stored in place once all of it has read the old one;
//   else it goes to Uo and Pn, and k_line_copy takes it over.
// Bound by the serial chain of the stages (roots, divisions and the Newton
// iteration of one wave per SIMD).  An RK3 step of 200 cells takes 12.7 us in one
// launch, of 400 to 2000 cells 14.6 us in two (8 waves in one workgroup: 17.3 us);
// a launch per stage took 21 us.
// The stages: Runge-Kutta coefficients, and for a recorded step the caches that
// keep their primitives (recovery flags in fout).
struct LineStages {
    double a[3], b[3];
    double* P[3];
};

template <bool RK3>
__global__ __launch_bounds__(256) void k_line(SweepArgs A, Dev d, LineStages rk, int direct)
{
    constexpr int NS = RK3 ? 3 : 2, H = 2 * NS, OWN = 64 - 2 * H;
    const int lane = threadIdx.x & 63, n = d.n[0];
    const int wave = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int c0 = wave * OWN - H, c = c0 + lane;
    int im = c;
    if (d.bc[0] == 0) {
        im = c % n;
        im += im < 0 ? n : 0;
    } else {
        im = min(max(c, 0), n - 1);
    }
    const bool own = lane >= H && lane < 64 - H && c < n;
    double q[9], un[9], ub[9];
#pragma unroll
    for (int v = 0; v < 9; ++v) {
        q[v] = A.Pc[v * d.sv + d.g[0] + im];
        un[v] = A.Un[v * d.N + im];
        ub[v] = un[v];
    }
    if (direct)
        __syncthreads();
    int nfail = 0, natm = 0, npf = 0, nfb = 0, itmax = 0;
    const Geo g = geo_at<FLAT, double>(d, 0.0, 0.0, 0.0);
#pragma nounroll
    for (int s = 0; s < NS; ++s) {
        const double a = rk.a[s], b = rk.b[s];
        double qL[9], qR[9], F[9], R[9];
#pragma unroll
        for (int v = 0; v < 9; ++v) {
            const double h = mc_hslope(from_left(q[v]), q[v], from_right(q[v]));
            qR[v] = q[v] - h;
            qL[v] = from_left(q[v] + h);
        }
        face_solve<0>(qL, qR, geo_cast<double>(g), d, F);
#pragma unroll
        for (int v = 0; v < 9; ++v)
            R[v] = -(from_right(F[v]) - F[v]) * d.idx[0];
        Geo gs;
        add_sources<FLAT>(d, 0.0, 0.0, 0.0, 0, q, gs, R);
        double u[9], p[9];
#pragma unroll
        for (int v = 0; v < 9; ++v)
            u[v] = ub[v] + a * (un[v] - ub[v]) + b * (A.dt * R[v]);
        // lanes whose stencil is still whole (the others' values are not used)
        if (lane >= 2 * (s + 1) && lane < 64 - 2 * (s + 1) && (d.bc[0] == 0 || (c >= 0 && c < n))) {
            int iters = 0;
            const int flags = recover_cell<double>(d, g, u, q, p, iters);
#pragma unroll
            for (int v = 0; v < 9; ++v) {
                q[v] = p[v];
                ub[v] = u[v];
            }
            if (own) {
                tally(flags, iters, nfail, natm, npf, nfb, itmax);
                if (rk.P[s]) {
                    store_prim(d, rk.P[s], cache_index(d, c, 0, 0), c, 0, 0, q);
                    A.fout[s * d.N + c] = (unsigned char)flags;
                }
            }
        }
        if (d.bc[0] != 0) {
            const int end = c < 0 ? -c0 : min(n - 1 - c0, 63);   // the lane of the end cell
#pragma unroll
            for (int v = 0; v < 9; ++v) {
                const double e = __shfl(q[v], end);
                q[v] = c < 0 || c >= n ? e : q[v];
            }
        }
    }
    if (own) {
#pragma unroll
        for (int v = 0; v < 9; ++v)
            A.Uo[v * d.N + c] = ub[v];
        store_prim(d, A.Pn, cache_index(d, c, 0, 0), c, 0, 0, q);
    }
    count_sums(A.cnt, nfail, natm, npf, nfb, itmax);
}

// The state k_line left beside the caller's (U, and the primitive rows) into it.
__global__ __launch_bounds__(256) void k_line_copy(const double* __restrict__ Us, double* __restrict__ U, long long nu,
                                                   const double* __restrict__ Ps, double* __restrict__ P, long long np)
{
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t < nu)
        U[t] = Us[t];
    if (t < np)
        P[t] = Ps[t];
}

hipError_t launch_line(int ns, const double* a, const double* b, double* P0, double* P1, double* U, double* U1, const Dev& d, double dt,
                       unsigned long long* cnt, double* const* stages, unsigned char* fout, hipStream_t s)
{
    const int own = 64 - 4 * ns, waves = (d.n[0] + own - 1) / own;
    const bool direct = waves <= 4;
    SweepArgs A{};
    A.Pc = P0;
    A.Pn = direct ? P0 : P1;
    A.Un = U;
    A.Uo = direct ? U : U1;
    A.cnt = cnt;
    A.fout = fout;
    A.dt = dt;
    LineStages rk{};
    for (int k = 0; k < ns; ++k) {
        rk.a[k] = a[k];
        rk.b[k] = b[k];
        rk.P[k] = stages ? stages[k] : nullptr;
    }
    const dim3 grid(direct ? 1 : waves), block(direct ? 64 * waves : 64);
    if (ns == 3)
        hipLaunchKernelGGL((k_line<true>), grid, block, 0, s, A, d, rk, (int)direct);
    else
        hipLaunchKernelGGL((k_line<false>), grid, block, 0, s, A, d, rk, (int)direct);
    if (!direct) {
        const long long nu = 9 * d.N, np = 9 * d.sv;
        hipLaunchKernelGGL(k_line_copy, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, s, U1, U, nu, P1, P0, np);
    }
    return hipGetLastError();
}

hipError_t launch_sweep(int kind, const SweepArgs& A, const Dev& d, hipStream_t s)
{
    if (!A.R5 && A.R)
        return A.P ? launch_sweep_r<SWEEP_RHS, true>(kind, A, d, s) : launch_sweep_r<SWEEP_RHS, false>(kind, A, d, s);
    if (!A.R5)
        return launch_sweep_r<SWEEP_STEP, false>(kind, A, d, s);
    SweepArgs B = A;
    B.R = A.R5;
    return A.P ? launch_sweep_r<SWEEP_CT, true>(kind, B, d, s) : launch_sweep_r<SWEEP_CT, false>(kind, B, d, s);
}

}  // namespace grmhd
