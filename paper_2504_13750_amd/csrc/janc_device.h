// janc_device.h -- device helpers shared by the forward and adjoint kernels:
// reduction slots, coarse-fine ring tests, source resolution, primitives,
// Newton for T, WENO5 and the RK combination. Included by .hip files only.
#pragma once

#include "janc_internal.h"

namespace janc {

constexpr double WENO_EPS = 1e-6;

// Read-only tables (domains, mechanism) viewed through the constant address
// space: the compiler may then serve workgroup-uniform reads from scalar loads,
// also after the kernel's own global stores.
typedef __attribute__((address_space(4))) const DevMech CMech;
typedef __attribute__((address_space(4))) const DevDomain CDom;
__device__ __forceinline__ CMech* cmech(const DevMech* p) { return (CMech*)p; }
__device__ __forceinline__ CDom& cdom(const DevDomain* p, int d) { return ((CDom*)p)[d]; }
typedef __attribute__((address_space(4))) const int CInt;
template <class T>
__device__ __forceinline__ T cload(const T* p) {
    static_assert(sizeof(T) % 4 == 0, "whole words");
    CInt* w = (CInt*)(const int*)p;
    union { int i[sizeof(T) / 4]; T t; } v;
#pragma unroll
    for (int k = 0; k < (int)(sizeof(T) / 4); ++k) v.i[k] = w[k];
    return v.t;
}
__device__ __forceinline__ DevBlock cblock(const DevBlock* p, int b) { return cload(p + b); }
__device__ __forceinline__ Tile ctile(const Tile* p, int t) { return cload(p + t); }

// ------------------------------------------------------------------ small helpers
__device__ __forceinline__ double sq(double x) { return x * x; }

// Word of slot idx of buffer buf (each slot alone in a 128-byte line).
__device__ __forceinline__ size_t slot_word(int stride, int buf, int idx) {
    return ((size_t)buf * stride + idx) * SLOT_WORDS;
}

__device__ __forceinline__ double slot_get(const Reduce& r, int buf, int idx) {
    return __longlong_as_double((long long)r.buf[slot_word(r.stride, buf, idx)]);
}

__device__ __forceinline__ void slot_max(const Reduce& r, int buf, int idx, double v) {
    // v >= 0: the bit pattern orders like the value
    atomicMax(&r.buf[slot_word(r.stride, buf, idx)], (unsigned long long)__double_as_longlong(v));
}

// n / d where d is a normal number and so is its reciprocal: hardware reciprocal (relative
// error 2^-24 over 1.3e8 random values), one Newton step (2^-48) and one residual step
// (2^-96 before the last rounding: the rounded quotient, equal to n / d on all of them).
// Six instructions for the eleven of the general division.
__device__ __forceinline__ double quotient(double n, double d) {
    double y = __builtin_amdgcn_rcp(d);
    y = __builtin_fma(__builtin_fma(-d, y, 1.0), y, y);
    const double q = n * y;
    return __builtin_fma(__builtin_fma(-d, q, n), y, q);
}

// Makes `next` available only once `done` is computed: keeps the compiler from starting the
// arithmetic on `next` early, whose registers cost more than its parallelism gives.
__device__ __forceinline__ void after(double& done, double& next) {
    asm volatile("" : "+v"(done), "+v"(next));
}

// LDS accesses of one wave are executed in order; this keeps the compiler from moving them
// across the point where lanes read what other lanes of their wave wrote.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// A value that is the same in every lane, moved to scalar registers.
__device__ __forceinline__ double uniform(double v) {
    union { double d; int i[2]; } x;
    x.d = v;
    x.i[0] = __builtin_amdgcn_readfirstlane(x.i[0]);
    x.i[1] = __builtin_amdgcn_readfirstlane(x.i[1]);
    return x.d;
}

// Value of another lane by a DPP row operation; lanes without a source keep `v`.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp(double v) {
    union { double d; int i[2]; } x, y;
    x.d = v;
    y.i[0] = __builtin_amdgcn_update_dpp(x.i[0], x.i[0], CTRL, ROWS, 0xf, false);
    y.i[1] = __builtin_amdgcn_update_dpp(x.i[1], x.i[1], CTRL, ROWS, 0xf, false);
    return y.d;
}

// Maximum over a wavefront, in every lane: row shifts by 1, 2, 4, 8 leave a row's maximum in
// its last lane, two broadcasts carry it on to lane 63 (register moves; the exchanges by
// __shfl_xor went through the LDS pipeline, six dependent trips).
__device__ __forceinline__ double wave_max(double v) {
    v = fmax(v, dpp<0x111, 0xf>(v));
    v = fmax(v, dpp<0x112, 0xf>(v));
    v = fmax(v, dpp<0x114, 0xf>(v));
    v = fmax(v, dpp<0x118, 0xf>(v));
    v = fmax(v, dpp<0x142, 0xa>(v));
    v = fmax(v, dpp<0x143, 0xc>(v));
    union { double d; int i[2]; } x;
    x.d = v;
    x.i[0] = __builtin_amdgcn_readlane(x.i[0], 63);
    x.i[1] = __builtin_amdgcn_readlane(x.i[1], 63);
    return x.d;
}

// Workgroup max of three values over NW waves; thread 0 publishes them.
template <int NW>
__device__ __forceinline__ void publish_max3(const Reduce& r, int buf, int i0, int i1, int i2,
                                             double v0, double v1, double v2, double* scratch) {
    v0 = wave_max(v0);
    v1 = wave_max(v1);
    v2 = wave_max(v2);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) {
        scratch[3 * w + 0] = v0;
        scratch[3 * w + 1] = v1;
        scratch[3 * w + 2] = v2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double m0 = scratch[0], m1 = scratch[1], m2 = scratch[2];
        for (int q = 1; q < NW; ++q) {
            m0 = fmax(m0, scratch[3 * q]);
            m1 = fmax(m1, scratch[3 * q + 1]);
            m2 = fmax(m2, scratch[3 * q + 2]);
        }
        if (m0 > 0.0) slot_max(r, buf, i0, m0);
        if (m1 > 0.0) slot_max(r, buf, i1, m1);
        if (m2 > 0.0) slot_max(r, buf, i2, m2);
    }
}

// The same for one wave.
__device__ __forceinline__ void publish_wave3(const Reduce& r, int buf, int i0, int i1, int i2, double v0,
                                              double v1, double v2) {
    v0 = wave_max(v0);
    v1 = wave_max(v1);
    v2 = wave_max(v2);
    if ((threadIdx.x & 63) == 0) {
        if (v0 > 0.0) slot_max(r, buf, i0, v0);
        if (v1 > 0.0) slot_max(r, buf, i1, v1);
        if (v2 > 0.0) slot_max(r, buf, i2, v2);
    }
}

// The same for values that the W waves staged in LDS (v[k * 64 W + thread], k = 0..2): wave k
// takes quantity k (and k + W) of all threads, so that one sixth of the exchanges remain.
template <int W>
__device__ __forceinline__ void publish_staged(const Reduce& r, int buf, int i0, int i1, int i2,
                                               const double* v) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
#pragma unroll
    for (int q = w; q < 3; q += W) {
        const double* x = v + 64 * W * q + l;
        double m = fmax(x[0], x[64]);
        if constexpr (W == 4) m = fmax(m, fmax(x[128], x[192]));
        m = wave_max(m);
        if (l == 0 && m > 0.0) slot_max(r, buf, q == 0 ? i0 : q == 1 ? i1 : i2, m);
    }
}

// Coarse-fine ring test for block-local cell (li, lj) (segment masks per side).
__device__ __forceinline__ bool ring_at(const DevBlock& B, int li, int lj) {
    const unsigned sx = (unsigned)(lj >> 3) & 31u, sy = (unsigned)(li >> 3) & 31u;
    return (li < 3 && ((B.ring[0] >> sx) & 1u)) || (li >= B.nx - 3 && ((B.ring[1] >> sx) & 1u)) ||
           (lj < 3 && ((B.ring[2] >> sy) & 1u)) || (lj >= B.ny - 3 && ((B.ring[3] >> sy) & 1u));
}

// Effective source of level-`lev` cell (I, J) of domain D: boundary rule first,
// then the covering block of that level, or the coarser level where the cell is
// uncovered or a ring cell. Returns a pool cell (>= 0) or -(1 + Dirichlet row);
// fl gets bit 0 / bit 1 when x / y momentum must be mirrored.
__device__ long long resolve(const StageArgs& a, CDom& D, int lev, int I, int J,
                             unsigned& fl) {
    const int W = D.nx0 << lev, H = D.twod ? (D.ny0 << lev) : 1;
    if (I < 0 || I >= W) {
        const int side = (I < 0) ? 0 : 1;
        switch (D.bc[side]) {
            case BC_PERIODIC: I = (I < 0) ? I + W : I - W; break;
            case BC_ZEROGRAD: I = (I < 0) ? 0 : W - 1; break;
            case BC_SLIPWALL: I = (I < 0) ? -I - 1 : 2 * W - 1 - I; fl ^= 1u; break;
            default: return -(1ll + D.dir[side]);
        }
    }
    if (J < 0 || J >= H) {
        const int side = (J < 0) ? 2 : 3;
        switch (D.bc[side]) {
            case BC_PERIODIC: J = (J < 0) ? J + H : J - H; break;
            case BC_ZEROGRAD: J = (J < 0) ? 0 : H - 1; break;
            case BC_SLIPWALL: J = (J < 0) ? -J - 1 : 2 * H - 1 - J; fl ^= 2u; break;
            default: return -(1ll + D.dir[side]);
        }
    }
    for (;;) {
        const int b = a.maps[D.map_off[lev] + (J >> 3) * D.map_w[lev] + (I >> 3)];
        if (b >= 0) {
            const DevBlock& B = a.blk[b];
            const int li = I - B.i0, lj = J - B.j0;
            if (!ring_at(B, li, lj)) return B.offset + (long long)lj * B.nx + li;
        }
        // level 0 tiles the domain and has no ring cells, so this ends; bit 2 of fl
        // marks a source on a coarser level than the one asked for
        --lev;
        I >>= 1;
        J >>= 1;
        fl |= 4u;
    }
}

template <int NU>
__device__ __forceinline__ void fetch(const StageArgs& a, long long src, unsigned fl,
                                      const double* Uarr, const double* Tarr, double (&u)[NU],
                                      double& T) {
    if (src >= 0) {
#pragma unroll
        for (int f = 0; f < NU; ++f) u[f] = Uarr[(size_t)f * a.pool + src];
        T = Tarr[src];
    } else {
        const double* r = a.dirU + (size_t)(-src - 1) * (MAXF + 1);
#pragma unroll
        for (int f = 0; f < NU; ++f) u[f] = r[f];
        T = r[MAXF];
    }
    if (fl & 1u) u[1] = -u[1];
    if (fl & 2u) u[2] = -u[2];
}

// Velocities and pressure of a stencil cell (Eq. 4.2; T from storage for NASA-7).
template <int M, int NU, class Dom, class Mech>
__device__ __forceinline__ void halo_prims(const double (&u)[NU], double T, const Dom& D,
                                           Mech mech, double& vx, double& vy,
                                           double& p) {
    const double ir = quotient(1.0, u[0]);
    vx = u[1] * ir;
    vy = u[2] * ir;
    if constexpr (M == DETAILED) {
        double s = 0.0, r = 0.0;
#pragma unroll
        for (int k = 0; k < NU - 4; ++k) {
            s += u[4 + k];
            r += u[4 + k] * mech->invM[k];
        }
        r += (u[0] - s) * mech->invM[NU - 4];
        p = RU * r * T;
    } else {
        double e = u[3] * ir - 0.5 * (vx * vx + vy * vy);
        if constexpr (M == ONESTEP) e -= u[4] * ir * D.Q;
        p = (D.gamma - 1.0) * u[0] * e;
    }
}

// Mixture NASA-7 polynomials (Y fixed, so the species sums are formed once), per mass:
// e(T) = T (c0 + T (c1 + ..)) + e0 and c_v(T) = c0 + T (v1 + T (v2 + ..)) of one range.
struct MixPoly {
    double c0, c1, c2, c3, c4, e0, v1, v2, v3, v4;
};

__device__ __forceinline__ void poly_eval(const MixPoly& x, double T, double& e, double& cv) {
    e = T * (x.c0 + T * (x.c1 + T * (x.c2 + T * (x.c3 + T * x.c4)))) + x.e0;
    cv = x.c0 + T * (x.v1 + T * (x.v2 + T * (x.v3 + T * x.v4)));
}

// Mixture R and the polynomials of one table of coefficients. The coefficients are scalar
// loads; they are taken three species at a time (all at once they spilled).
template <int NS, class Tab>
__device__ __forceinline__ void mix_poly(const double (&Y)[NS], CMech* m, Tab* tab, MixPoly& x, double& Rmix) {
    double b0 = 0.0, b1 = 0.0, b2 = 0.0, b3 = 0.0, b4 = 0.0, b5 = 0.0, R = 0.0;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        const double w = Y[k] * m->Rk[k];
        R += w;
        b0 += w * tab[k][0];
        b1 += w * tab[k][1];
        b2 += w * tab[k][2];
        b3 += w * tab[k][3];
        b4 += w * tab[k][4];
        b5 += w * tab[k][5];
        if (k % 3 == 2 && k + 1 < NS) asm volatile("" : "+v"(b5), "+s"(m), "+s"(tab));
    }
    Rmix = R;
    x.c0 = b0 - R;
    x.c1 = 0.5 * b1;
    x.c2 = b2 * (1.0 / 3.0);
    x.c3 = 0.25 * b3;
    x.c4 = 0.2 * b4;
    x.e0 = b5;
    x.v1 = b1;
    x.v2 = b2;
    x.v3 = b3;
    x.v4 = b4;
}

typedef __attribute__((address_space(4))) const double CNasa[7];

// e(T) and c_v(T) by the range of T.
__device__ __forceinline__ void range_eval(const MixPoly& lo, const MixPoly& hi, double tm, double T, double& e,
                                           double& cv) {
    const bool h = T >= tm;
    const MixPoly x = {h ? hi.c0 : lo.c0, h ? hi.c1 : lo.c1, h ? hi.c2 : lo.c2, h ? hi.c3 : lo.c3,
                       h ? hi.c4 : lo.c4, h ? hi.e0 : lo.e0, h ? hi.v1 : lo.v1, h ? hi.v2 : lo.v2,
                       h ? hi.v3 : lo.v3, h ? hi.v4 : lo.v4};
    poly_eval(x, T, e, cv);
}

// Newton for T: eval(T, e, cv) is the mixture's; cv returns c_v at the root.
template <class Eval>
__device__ __forceinline__ unsigned newton_loop(double e, double& T, double& cv, Eval&& eval) {
    unsigned st = STB_NEWTON;
    double ec;
    for (int it = 0; it < 50; ++it) {
        double cvv;
        eval(T, ec, cvv);
        const double dT = quotient(ec - e, cvv);
        T -= dT;
        if (!(fabs(dT) <= 1e-12 * fabs(T))) {
            if (!isfinite(T)) { st = STB_NONFINITE; break; }
            continue;
        }
        st = 0u;
        break;
    }
    eval(T, ec, cv);
    return st;
}

// Newton for T from the internal energy on the mixture coefficients (Sec. 4.2). With two
// NASA-7 ranges (one t_mid for all species) both sets are formed and an evaluation uses the
// set of its temperature.
template <int NS>
__device__ __forceinline__ unsigned newton_T(const double (&Y)[NS], double e, CMech* m,
                                             double& T, double& cv, double& Rmix) {
    MixPoly lo;
    mix_poly<NS>(Y, m, (CNasa*)m->nasa, lo, Rmix);
    if (m->two_range) {
        MixPoly hi;
        double R;
        const double tm = m->tmid[0];
        mix_poly<NS>(Y, m, (CNasa*)m->nasa_hi, hi, R);
        return newton_loop(e, T, cv, [&](double Tc, double& ec, double& c) { range_eval(lo, hi, tm, Tc, ec, c); });
    }
    return newton_loop(e, T, cv, [&](double Tc, double& ec, double& c) { poly_eval(lo, Tc, ec, c); });
}

// Mixture R and c_v at a stored temperature, the forward's own sums.
template <int NS>
__device__ __forceinline__ void mix_cv(const double (&Y)[NS], CMech* m, double T, double& cv, double& Rmix) {
    MixPoly lo;
    double e;
    mix_poly<NS>(Y, m, (CNasa*)m->nasa, lo, Rmix);
    if (m->two_range) {
        MixPoly hi;
        double R;
        mix_poly<NS>(Y, m, (CNasa*)m->nasa_hi, hi, R);
        range_eval(lo, hi, m->tmid[0], T, e, cv);
    } else {
        poly_eval(lo, T, e, cv);
    }
}

// State of an owned cell after an update: T (closed form or Newton from Tprev),
// sound speed and velocities; returns status bits.
template <int M, int NU, class Dom, class Mech>
__device__ __forceinline__ unsigned owner_state(const double (&u)[NU], double Tprev,
                                                const Dom& D, Mech mech,
                                                double& T, double& c, double& vx, double& vy) {
    const double rho = u[0];
    if (!isfinite(rho)) return STB_NONFINITE;
    if (!(rho > 0.0)) return STB_NEGATIVE;
    const double ir = quotient(1.0, rho);
    vx = u[1] * ir;
    vy = u[2] * ir;
    const double e = u[3] * ir - 0.5 * (vx * vx + vy * vy);
    double p, gam;
    unsigned st = 0u;
    if constexpr (M == DETAILED) {
        constexpr int NS = NU - 3;
        double Y[NS];
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < NS - 1; ++k) {
            Y[k] = u[4 + k] * ir;
            s += Y[k];
        }
        Y[NS - 1] = 1.0 - s;
        T = Tprev;
        double cv, Rmix;
        st = newton_T<NS>(Y, e, mech, T, cv, Rmix);
        p = rho * Rmix * T;
        gam = quotient(cv + Rmix, cv);
    } else {
        double ee = e;
        if constexpr (M == ONESTEP) ee -= u[4] * ir * D.Q;
        p = (D.gamma - 1.0) * rho * ee;
        T = p / (rho * D.R);
        gam = D.gamma;
    }
    if (!isfinite(p) || !isfinite(T)) return st | STB_NONFINITE;
    if (!(p > 0.0) || !(T > 0.0)) return st | STB_NEGATIVE;
    c = sqrt(gam * p * ir);
    return st;
}

// WENO5-JS at i+1/2 from f_{i-2..i+2} (a..e), written in first differences
// d1..d4: the candidate values are c + r_k / 6, the smoothness indicators times 12
// are 13 (second difference)^2 + 3 (one-sided slope)^2 (the common factor 144 of
// the squared (eps + beta) cancels in the normalized weights), and the weighted
// average is c + sum w_k r_k / (6 sum w_k) with the weights in common-denominator
// form (one division). Algebraically the textbook form; fewer operations.
__device__ __forceinline__ double weno5(double a, double b, double c, double d, double e) {
    const double d1 = b - a, d2 = c - b, d3 = d - c, d4 = e - d;
    const double r0 = 5.0 * d2 - 2.0 * d1, r1 = d2 + 2.0 * d3, r2 = 4.0 * d3 - d4;
    const double t0 = d2 - d1, t1 = d3 - d2, t2 = d4 - d3;
    const double u0 = 3.0 * d2 - d1, u1 = d2 + d3, u2 = d4 - 3.0 * d3;
    const double s0 = sq((12.0 * WENO_EPS + 13.0 * t0 * t0) + 3.0 * u0 * u0);
    const double s1 = sq((12.0 * WENO_EPS + 13.0 * t1 * t1) + 3.0 * u1 * u1);
    const double s2 = sq((12.0 * WENO_EPS + 13.0 * t2 * t2) + 3.0 * u2 * u2);
    const double w0 = 0.1 * (s1 * s2), w1 = 0.6 * (s0 * s2), w2 = 0.3 * (s0 * s1);
    return c + quotient(w0 * r0 + w1 * r1 + w2 * r2, 6.0 * (w0 + w1 + w2));
}

// The split fluxes of the detailed model are kept at a sixth of their value, so that the
// factors 6 of the reconstruction below fall on constants; the other models keep the form
// above, whose rounding their long runs are compared with.
template <int M>
constexpr double SPLIT_SCALE = (M == DETAILED) ? 1.0 / 12.0 : 0.5;

// weno5_flux of the detailed model divides by the product of two sums of squared smoothness
// indicators, the sixteenth power of a flux difference: in range while the split fluxes stay
// below 2^59 (5.8e17) in magnitude, for every shape of a stencil. The reconstruction is
// homogeneous, so tiles beyond that are reconstructed at WENO_SHRINK times their fluxes, which
// holds to differences of 2e33, as far as a division for each side alone did (1.6e33). The
// smallest denominator, of equal fluxes, is 2^-994 then; the numerator above it is exact to
// 2^-1074, 2e-9 of a flux.
constexpr double WENO_C1 = 12.0 * WENO_EPS / 108.0, WENO_SHRINK = 0x1p-51;

// One-sided WENO5-JS from a..e (a sixth of the split fluxes) as c + num / den: weno5()'s
// form with everything over 36 * 3 in the smoothness indicators (their common factor
// cancels in the weights) and the linear weights 1 : 6 : 3. c1: WENO_C1, or for fluxes
// multiplied by WENO_SHRINK its square times that.
__device__ __forceinline__ void weno5_parts(double a, double b, double c, double d, double e,
                                            double& num, double& den, double c1) {
    constexpr double C2 = 13.0 / 3.0;
    const double d1 = b - a, d2 = c - b, d3 = d - c, d4 = e - d;
    const double t0 = d2 - d1, t1 = d3 - d2, t2 = d4 - d3;
    const double u0 = 3.0 * d2 - d1, u1 = d2 + d3, u2 = 3.0 * d3 - d4;
    const double b0 = c1 + (C2 * t0) * t0, b1 = c1 + (C2 * t1) * t1, b2 = c1 + (C2 * t2) * t2;
    const double s0 = sq(b0 + u0 * u0), s1 = sq(b1 + u1 * u1), s2 = sq(b2 + u2 * u2);
    const double w0 = s1 * s2, w1 = 6.0 * (s0 * s2), w2 = 3.0 * (s0 * s1);
    const double r0 = 2.0 * u0 - d2, r1 = u1 + d3, r2 = d3 + u2;
    num = w0 * r0 + (w1 * r1 + w2 * r2);
    den = w0 + (w1 + w2);
}

// Numerical flux at an interface: WENO5 of F+ from p0..p4 plus WENO5 of F- from m0..m4
// (its stencil mirrored). The detailed model takes both over one denominator.
template <int M>
__device__ __forceinline__ double weno5_flux(double p0, double p1, double p2, double p3, double p4,
                                             double& m0, double m1, double m2, double m3, double m4,
                                             double c1) {
    if constexpr (M == DETAILED) {
        double np, dp, nm, dm;
        weno5_parts(p0, p1, p2, p3, p4, np, dp, c1);
        after(dp, m0);
        weno5_parts(m0, m1, m2, m3, m4, nm, dm, c1);
        const double q = quotient(np * dm + nm * dp, dp * dm);
        return 6.0 * (p2 + m2) + q;
    } else {
        double h = weno5(p0, p1, p2, p3, p4);
        after(h, m0);
        return h + weno5(m0, m1, m2, m3, m4);
    }
}

template <int M>
__device__ __forceinline__ double weno5_pair(const double (&P)[5], double (&N)[5], double c1) {
    return weno5_flux<M>(P[0], P[1], P[2], P[3], P[4], N[0], N[1], N[2], N[3], N[4], c1);
}

// R consecutive interfaces from LDS strips of stride STR: F+ from p[k .. k+4], F- from
// n[k+4 .. k]. Neighbouring stencils share their differences, second differences and their
// squares. The strips are read as the run advances and the interfaces kept in order, so
// that one interface's working set is live at a time (all R at once took 60 more registers).
template <int M, int R, int STR>
__device__ __forceinline__ void weno5_runs(const double* p, const double* n, double (&h)[R], double c1) {
    double P[R + 4], N[R + 4];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        P[k] = p[k * STR];
        N[k] = n[k * STR];
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
        if (k + 1 < R) {
            P[k + 5] = p[(k + 5) * STR];
            N[k + 5] = n[(k + 5) * STR];
        }
        h[k] = weno5_flux<M>(P[k], P[k + 1], P[k + 2], P[k + 3], P[k + 4],
                             N[k + 4], N[k + 3], N[k + 2], N[k + 1], N[k], c1);
        if (k + 1 < R) after(h[k], P[k + 5]);
    }
}

// One interface; `wide` (the same in every lane): at WENO_SHRINK times its fluxes.
template <int M, int STR>
__device__ __forceinline__ double weno5_one(const double* p, const double* n, bool wide) {
    double P[5], N[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        P[k] = p[k * STR];
        N[k] = n[(4 - k) * STR];
    }
    if (M == DETAILED && __builtin_expect(wide, 0)) {
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            P[k] *= WENO_SHRINK;
            N[k] *= WENO_SHRINK;
        }
        return weno5_pair<M>(P, N, WENO_C1 * WENO_SHRINK * WENO_SHRINK) * (1.0 / WENO_SHRINK);
    }
    return weno5_pair<M>(P, N, WENO_C1);
}

// Magnitudes compared by their high words, read as FP32 numbers: ordered as the values are (up
// to 2^1017). raise(): the largest of m, |x| and |y| (one instruction; fmaxf() would first
// quiet its operands).
__device__ __forceinline__ float high_float(double x) {
    return __uint_as_float((unsigned)(__double_as_longlong(x) >> 32));
}
__device__ __forceinline__ void raise(float& m, double x, double y) {
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(high_float(x)), "v"(high_float(y)));
}
// Whether fluxes of values up to mu (the pressure among them) at speeds up to mv (one at
// least), so raised, need WENO_SHRINK. Split fluxes are within 1.5 mu mv; the sum of the high
// words is the logarithm of the product to 0.18, and 2^58.18 * 1.5 < 2^59.
__device__ __forceinline__ bool flux_wide(float mu, float mv) {
    return __float_as_uint(mu) + __float_as_uint(mv) >= (2u * 1023u + 58u) << 20;
}

// dt of domain d for this step from the CFL slot of buffer `bin`; in the crossover
// advance dt_0, from the largest bound over every level's slot triple.
__device__ __forceinline__ double step_dt(const StageArgs& a, int d, int bin) {
    double dt;
    if (a.tm.dt_fixed > 0.0) {
        dt = a.tm.dt_fixed;
    } else if (a.cross) {
        double m = 0.0;
        for (int l = 0; l < a.xlevels; ++l)
            m = fmax(m, __longlong_as_double((long long)a.xred[slot_word(a.red.stride, l * RED_BUFS + bin,
                                                                         2 * a.red.nunits + d)]));
        dt = a.tm.cfl / m;
    } else {
        dt = a.tm.cfl / slot_get(a.red, bin, 2 * a.red.nunits + d);
    }
    if (a.tm.t_end > 0.0) {
        const double rem = a.tm.t_end - a.t[d];
        if (!(rem > 0.0)) dt = 0.0;
        else if (dt > rem) dt = rem;
    }
    return dt;
}

// Is level-`lev` cell (I, J) of D under a valid block of level lev+1?
__device__ __forceinline__ bool covered_by_finer(const StageArgs& a, CDom& D, int lev,
                                                 int I, int J) {
    if (lev + 1 >= D.nlevels) return false;
    const int I2 = 2 * I, J2 = 2 * J;
    return a.maps[D.map_off[lev + 1] + (J2 >> 3) * D.map_w[lev + 1] + (I2 >> 3)] >= 0;
}

// Level-lev cell (I, J) lies under a finer valid block and none of its four children is
// a coarse-fine ring cell of that block: the restriction replaces it by the mean of its
// children without reading it. (Fine blocks sit on even cells, so the 2 x 2 children
// belong to one block.)
__device__ __forceinline__ bool restricted_over(const StageArgs& a, CDom& D, int lev, int I, int J) {
    if (lev + 1 >= D.nlevels || !D.twod) return false;
    const int I2 = 2 * I, J2 = 2 * J;
    const int b = a.maps[D.map_off[lev + 1] + (J2 >> 3) * D.map_w[lev + 1] + (I2 >> 3)];
    if (b < 0) return false;
    const DevBlock& F = a.blk[b];
    const int li = I2 - F.i0, lj = J2 - F.j0;
    return !ring_at(F, li, lj) && !ring_at(F, li + 1, lj) && !ring_at(F, li, lj + 1) &&
           !ring_at(F, li + 1, lj + 1);
}

// The dispatcher deals the workgroups of a launch round-robin over the 8 XCDs,
// each with its own L2. Workgroup b of n is given tile chunk(b) so that each XCD
// walks one contiguous run of tiles: neighbouring tiles, whose halos overlap,
// then read them through the same L2. The map is a bijection of [0, n).
__device__ __forceinline__ int xcd_chunk(int b, int n) {
    const int q = n >> 3, r = n & 7, x = b & 7;
    return x * q + min(x, r) + (b >> 3);
}

// CFL bound of a cell with wave speeds sx, sy at the spacing of its level (1/dx, 1/dy);
// in the crossover advance at the spacing of level 0, so that dt_0 bounds every level.
__device__ __forceinline__ double cfl_bound(const StageArgs& a, CDom& D, int lev, double sx,
                                            double sy, double idx, double idy) {
    if (a.cross) {
        idx = ldexp(idx, -lev);
        idy = ldexp(idy, -lev);
    }
    return sx * idx + (D.twod ? sy * idy : 0.0);
}

// Per-launch bookkeeping done by workgroup 0: rotate reduction buffers, dt and t.
// This step's dt per domain (from buffer 0's CFL slots) into a.dt and the dt log.
__device__ void record_dt(const StageArgs& a) {
    const int step = *a.step;
    for (int d = threadIdx.x; d < a.ndom; d += (int)blockDim.x) {
        const double dt = step_dt(a, d, 0);
        a.dt[d] = dt;
        if (a.dt_log && step < a.dt_log_cap) a.dt_log[(size_t)step * a.ndom + d] = dt;
    }
}

__device__ void stage_bookkeeping(const StageArgs& a, int owner_launch) {
    const int s = a.stage;
    const int bclear = (s + 1) % 3;
    for (int q = threadIdx.x; q < a.red.stride; q += (int)blockDim.x) a.red.buf[slot_word(a.red.stride, bclear, q)] = 0ull;
    if (a.cross) owner_launch = a.xfirst;
    if (!owner_launch) return;
    if (s == 1 && !a.strang) record_dt(a);   // under Strang splitting the first chemistry launch does
}

__device__ void step_finish(const StageArgs& a) {
    for (int d = threadIdx.x; d < a.ndom; d += (int)blockDim.x) a.t[d] = a.t[d] + a.dt[d];
    if (threadIdx.x == 0) *a.step = *a.step + 1;
}


}  // namespace janc
