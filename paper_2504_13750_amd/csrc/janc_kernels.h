// janc_kernels.h -- gfx950 kernels of the JANC per-time-step update (templates over the
// model and the field count; instantiated by janc_kernels.hip and, for the detailed model,
// one species count per translation unit, by janc_species.hip).
//
// One RK stage is one launch over a list of tiles (a tile is up to 16x16,
// 32x8 or 64x4 cells of one block, or 256 cells of a one-dimensional block),
// one workgroup of four wavefronts per tile. Per tile:
//   phase 0  every cell of the tile plus 3 halo layers (cross-shaped; corners
//            are not needed by the dimension-by-dimension sweeps) is fetched
//            from its source -- the same block, a neighbouring block, the
//            coarser level for coarse-fine ring cells, or a boundary rule --
//            and its velocities and pressure go to LDS;
//   phase 1  each wavefront takes whole conserved components and, without any
//            workgroup barrier, re-reads the component (L1/L2), forms the
//            Lax-Friedrichs split fluxes F+/F- and then G+/G- (Eq. 4.11) in an
//            LDS buffer of its own, reconstructs runs of four consecutive WENO5
//            interfaces per lane (Sec. 4.2), and forms the conservative
//            difference (Eq. 4.10) and the Shu-Osher RK stage of four cells a lane;
//   phase 2  T of the new state (Newton warm-started from the previous stage
//            for the NASA-7 model, Sec. 4.2), status checks, and the maxima of
//            |u|+c, |v|+c and the CFL bound for the next stage, reduced per
//            workgroup and published with one 64-bit atomic max each.
// Bound: FP64 VALU issue and the latency between the phases. Runs of four share the
// differences and smoothness terms of neighbouring stencils (62 FP64 instructions per
// interface of the 9-species model for 113 when every interface stood alone), and waves
// that meet at two barriers per tile instead of twelve keep three workgroups per CU
// apart in phase. 9 species, 1.92 M cells in 661 blocks: 0.305 -> 0.24 ms per stage,
// 4,225 -> 3,080 VALU instructions per 64 cells; one-step, 131 k cells: 19.1 -> 16.6 us.
// Four workgroups per CU (128 registers) spilled and were slower (0.29 ms).
// Nothing here is a dense contraction, so there is no MFMA: the work is FP64
// VALU arithmetic on values staged through LDS.
#pragma once

#include "janc_device.h"

namespace janc {

// ------------------------------------------------------------------ the stage tile
// A tile of TX x TY cells is swept by waves that each take whole conserved components
// (wave w: components w, w + W, ..). A lane reconstructs runs of R = TX TY / 64
// consecutive interfaces, along x in one pass and along y in the next, so that
// neighbouring stencils share their differences and smoothness terms in registers.
// Points of a tile: the owned cells first (point 64 q + l is cell q of lane l's y run, or
// cell 64 q + l of a 1-D tile), then the x halo (3 columns each side of every row) and,
// for 2-D tiles, the y halo (3 rows below and above every column).
template <int TX, int TY>
struct Geom {
    static constexpr bool TWO = TY > 1;
    static constexpr int NC = TX * TY, R = NC / 64;
    static constexpr int NHX = 6 * TY, NHY = TWO ? 6 * TX : 0;
    static constexpr int NP = NC + NHX + NHY;
    static constexpr int NPL = (NP + 63) / 64, NPP = 64 * NPL;   // points per lane of a wave
    // split fluxes of one component in a wave's LDS buffer. x pass: rows of PX doubles, F+ of
    // cell i at i + 3 and F- at i + 2 (a run's stencils of both start 16-byte aligned; the
    // slots that this shift leaves unused take the F- of the first halo column). y pass: rows
    // of PY doubles (16-wide tiles are padded so that the four y runs of a column fall on
    // different banks). Then the numerical fluxes: x rows of HX, and the lowest y interface
    // of every run plus the top row.
    static constexpr int PX = TX + 6, PY = TX + (TX == 16 ? 2 : 0), HX = TX + 4;
    static constexpr int NX = PX * TY, NY = TWO ? PY * (TY + 6) : 0, NH = HX * TY;
    static constexpr int XR = TX / R;                 // x runs per row
    static constexpr int NEXT = TY + (TWO ? TX : 0);  // right column / top row interfaces
    static constexpr int NHT = NH + (TWO ? (TY / R + 1) * TX : 0);
    static constexpr int BUF0 = 2 * (NX > NY ? NX : NY);
    static constexpr int BUF = BUF0 > NHT ? BUF0 : NHT;
    static_assert(BUF % 2 == 0 && NX % 2 == 0, "16-byte alignment");
    static_assert(NC % 64 == 0 && (R == 1 || R == 2 || R == 4), "tile shape");

    // tile-local position (li, lj) of point p
    __device__ static void point(int p, int& li, int& lj) {
        if (p < NC) {
            const unsigned q = (unsigned)p >> 6, l = (unsigned)p & 63u;
            li = TWO ? l % TX : p;
            lj = TWO ? (l / TX) * R + q : 0;
        } else if (p < NC + NHX) {
            const int h = p - NC, side = h >= 3 * TY, r = h - side * 3 * TY;
            lj = (r * 171) >> 9;   // r / 3 for r < 256
            li = side ? TX + (r - lj * 3) : (r - lj * 3) - 3;
        } else {
            const int h = p - NC - NHX, side = h >= 3 * TX, r = h - side * 3 * TX;
            const int row = (unsigned)r / TX;
            li = r - row * TX;
            lj = side ? TY + row : row - 3;
        }
    }
};

// Four waves sweep a 256-cell tile, one component each per round. One or two components
// left over after whole rounds are swept by all four waves together, an interface of every
// run each (a round of their own would leave three or two waves idle; workgroups of five
// waves left the two of each CU that fit resident, half as many waves as four of four).
constexpr int STAGE_W = 4;
constexpr int stage_left(int nu, int w) { return 2 * (nu % w) <= w ? nu % w : 0; }
// Plans of few tiles cut every tile into four of 64 cells (8 x 8, or 64 of a 1-D block), each
// swept by one wave per component with one interface per lane: a tile's chain of dependent
// phases is shorter and four times as many CUs work on it, for 2.5 points fetched and 3
// interfaces formed per cell and direction pair where whole tiles take 1.75 and 2.25. (9
// species, 128 x 64 cells: 15.5 -> 10 us per stage.)
constexpr int SMALL_SPLIT = 4;
constexpr int HALF_W = 2;   // waves of a tile of 128 cells

// LDS doubles of a stage workgroup: u, v, p (detailed model: times SPLIT_SCALE), source and
// flags (32 bits each) of every point, one split-flux buffer and one word (wide) per wave.
template <int TX, int TY>
constexpr int stage_lds(int waves) {
    return 3 * Geom<TX, TY>::NPP + Geom<TX, TY>::NPP + waves * Geom<TX, TY>::BUF +
           (Geom<TX, TY>::R == 1 ? 64 : 0) + (waves + 1) / 2;
}

// Point p of a tile of tw x th valid cells: its tile-local position and whether the x
// and the y sweep read it (the halo is cross-shaped).
template <int TX, int TY>
__device__ __forceinline__ void point_needs(int p, int tw, int th, int& li, int& lj, bool& nx,
                                            bool& ny) {
    Geom<TX, TY>::point(p, li, lj);
    nx = (lj >= 0 && lj < th) && (li >= -3 && li < tw + 3);
    ny = Geom<TX, TY>::TWO && (li >= 0 && li < tw) && (lj >= -3 && lj < th + 3);
}

// Block-local cell (bi, bj) is its own source: inside the block and not a ring cell.
__device__ __forceinline__ bool own_source(const DevBlock& B, int bi, int bj) {
    return bi >= 0 && bi < B.nx && bj >= 0 && bj < B.ny && !ring_at(B, bi, bj);
}

// Flags of a point besides resolve()'s: its source is a row of the Dirichlet table; it is a
// solved cell of the tile. Halo table word of a point that no sweep reads.
constexpr unsigned PT_DIR = 8u, PT_OWN = 16u;
constexpr int HALO_NONE = (int)0x80000000;
template <bool WIDE> struct FlagWord { using type = unsigned; };
template <> struct FlagWord<true> { using type = unsigned long long; };

// Source (pool cell, or -(1 + Dirichlet row)) and flags of point p of a tile; false if no
// sweep reads it.
template <int TX, int TY>
__device__ __forceinline__ bool point_source(const StageArgs& a, const DevBlock& B, CDom& D, const Tile& tile, int p,
                                             int tw, int th, long long& s, unsigned& fl) {
    int li, lj;
    bool nx, ny;
    point_needs<TX, TY>(p, tw, th, li, lj, nx, ny);
    if (!(nx || ny)) return false;
    const int bi = tile.x0 + li, bj = tile.y0 + lj;
    if (own_source(B, bi, bj)) s = B.offset + (long long)bj * B.nx + bi;
    else s = resolve(a, D, B.level, B.i0 + bi, B.j0 + bj, fl);
    return true;
}

// Split fluxes F+- = (F +- alpha u) / 2 (Eq. 4.11) of a conserved value u, F = ue v + add,
// at the scale they are kept in. Detailed model: v, alpha and add come scaled.
template <int M>
__device__ __forceinline__ void split_flux(double u, double v, double al, double add, double& Fp, double& Fm,
                                           double ue) {
    if constexpr (M == DETAILED) {
        const double F = u * v + add, t = u * al;
        Fp = F + t;
        Fm = F - t;
    } else {
        double F = ue * v;
        F += add;
        Fp = SPLIT_SCALE<M> * (F + al * u);
        Fm = SPLIT_SCALE<M> * (F - al * u);
    }
}

template <int M, int NU, int TX, int TY, int W>
__device__ __forceinline__ void stage_tile(const StageArgs& a, const int ti, const Tile tile, double* smem) {
    using G = Geom<TX, TY>;
    constexpr int R = G::R, NPL = G::NPL, NPP = G::NPP;
    constexpr int LEFT = (R == W && W < NU) ? stage_left(NU, W) : 0, NR = NU - LEFT;   // components of whole rounds
    static_assert(LEFT == 0 || (R == W && 2 * LEFT <= W),
                  "left-over components: one interface of a run per wave, two buffers each");
    static_assert(64 * W >= G::NC && (R == 1 || R == W), "phase 2: wave w has cell w of every run");
    constexpr bool DET = M == DETAILED;
    constexpr double scale = DET ? SPLIT_SCALE<M> : 1.0;
    double* pu = smem;                 // u, v, p of every point, times scale
    double* pv = pu + NPP;
    double* pp = pv + NPP;
    double* bufs = pp + NPP;
    unsigned* psrc = (unsigned*)(bufs + W * G::BUF);
    unsigned* pfl = psrc + NPP;   // flags, and in the high half the place of a halo point in its strip
    unsigned* pwide = (unsigned*)(bufs + W * G::BUF + NPP + (R == 1 ? 64 : 0));   // one word per wave
    double* psr = bufs + W * G::BUF + NPP;   // (R == 1) explicit source of the cells

    // ---------------- phase 0: source and primitives of every point of the tile and its halo
    // Everything a thread loads is on its way before it waits: the table words of its NT
    // points first (they need the tile number alone), then all fields of the points.
    constexpr int NT = (NPP + 64 * W - 1) / (64 * W);
    const int tid = threadIdx.x;
    // the loads of a new tile go ahead of the arithmetic of the tiles beside it (64 one-step
    // domains of uneven sizes, 949 k cells: 58 -> 55 us per stage; other plans +-0.5 %)
    __builtin_amdgcn_s_setprio(2);
    int hv[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const int p = tid + 64 * W * k;
        hv[k] = (a.hsrc && p < G::NP) ? a.hsrc[(size_t)ti * a.hstride + p] : HALO_NONE;
    }
    const DevBlock B = cblock(a.blk, tile.block);
    CDom& D = cdom(a.dom, B.domain);
    const int lev = B.level;
    const int stage = a.stage;
    const int bin = (stage == 1 && a.strang) ? 3 : stage - 1, bout = stage % 3;
    const int slot = D.slot0 + lev;
    const int tw = min(TX, B.nx - tile.x0), th = min(TY, B.ny - tile.y0);
    if (R == 1 && (tw <= 0 || th <= 0)) return;   // a quarter beyond its block's edge
    double ur[NT][NU], Tr[NT];
    unsigned src[NT], pfl0[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const int p = tid + 64 * W * k;
        long long s = (long long)(hv[k] >> 3);
        unsigned fl = (unsigned)(hv[k] & 7);
        bool needed = hv[k] != HALO_NONE;
        if (!a.hsrc) {
            fl = 0u;
            needed = p < G::NP && point_source<TX, TY>(a, B, D, tile, p, tw, th, s, fl);
        }
        // points that no sweep reads stand on the block's first cell; crossover: coarser
        // levels are read at their current state
        if (!needed) {
            s = B.offset;
            fl = 0u;
        }
        const bool base = a.cross && (fl & 4u);
        src[k] = (unsigned)(s < 0 ? -s - 1 : s);
        pfl0[k] = (base ? fl : (fl & 3u)) | (s < 0 ? PT_DIR : 0u);
        if (k == 0) {   // a valid cell of the tile is solved unless it is a ring cell
            int li, lj; // (a coarser source)
            G::point(tid, li, lj);
            if (needed && tid < G::NC && li < tw && lj < th && !(fl & 4u)) pfl0[k] |= PT_OWN;
        }
        const size_t c = s < 0 ? 0 : (size_t)s;
        const double* U = (base ? a.U0 : a.Uin) + c;
#pragma unroll
        for (int f = 0; f < NU; ++f) ur[k][f] = U[(size_t)f * a.pool];
        Tr[k] = (base ? a.Tbase : a.Tin)[c];
    }
#pragma unroll
    for (int k = 0; k < NT; ++k)
        if (pfl0[k] & PT_DIR) {
            const double* r = a.dirU + (size_t)src[k] * (MAXF + 1);
#pragma unroll
            for (int f = 0; f < NU; ++f) ur[k][f] = r[f];
            Tr[k] = r[MAXF];
        }
    // crossover advance: dt_l = dt_0 / 2^l, dt_0 formed by the first launch of the step
    const double dt = uniform(a.cross ? ldexp((a.xfirst && stage == 1) ? step_dt(a, B.domain, 0)
                                                                       : a.dt[B.domain], -lev)
                                      : (stage == 1) ? step_dt(a, B.domain, 0) : a.dt[B.domain]);
    if (!(dt > 0.0)) return;   // finished domain: state unchanged
    // scaling by a power of two is exact
    double idx = uniform(ldexp(D.idx0, lev)), idy = uniform(ldexp(D.idy0, lev));
    const double ax = uniform(slot_get(a.red, bin, 2 * slot));
    const double ay = uniform(slot_get(a.red, bin, 2 * slot + 1));
    double sax = uniform(scale * ax), say = uniform(scale * ay);
    const double Town = Tr[0];   // T of the cell this thread solves in phase 2
    double src_e = 0.0;          // its explicit source, one-step model (Sec. 4.3)
    float mu = 0.0f, mv = high_float(1.0);   // largest values and speeds (flux_wide)
    double uleft[LEFT + 1];      // its left-over components
#pragma unroll
    for (int k = 0; k < LEFT; ++k) uleft[k] = ur[0][NR + k];
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const int p = tid + 64 * W * k;
        if (p >= NPP) continue;
        if (pfl0[k] & 1u) ur[k][1] = -ur[k][1];
        if (pfl0[k] & 2u) ur[k][2] = -ur[k][2];
        double vx, vy, pr;
        halo_prims<M, NU>(ur[k], Tr[k], D, cmech(a.mech), vx, vy, pr);
#pragma unroll
        for (int j = 0; j < LEFT; ++j) {   // species rows: no pressure term
            double* X = bufs + 2 * j * G::BUF;
            double* Y = X + G::BUF;
            const double uk = ur[k][NR + j];
            int li, lj;
            G::point(p, li, lj);
            if (p < G::NC + G::NHX) {
                const int o = lj * G::PX + li + 3;
                split_flux<M>(uk, scale * vx, sax, 0.0, X[o], X[G::NX - 1 + o], uk);
            }
            if (G::TWO && (p < G::NC || (p >= G::NC + G::NHX && p < G::NP))) {
                const int o = (lj + 3) * G::PY + li;
                split_flux<M>(uk, scale * vy, say, 0.0, Y[o], Y[G::NY + o], uk);
            }
        }
        if constexpr (DET) {
#pragma unroll
            for (int f = 0; f < NU; f += 2) raise(mu, ur[k][f], f + 1 < NU ? ur[k][f + 1] : pr);
            if (NU % 2 == 0) raise(mu, pr, pr);
            raise(mv, vx, vy);
        }
        if constexpr (M == ONESTEP) {
            if (k == 0) {
                const double Tc = pr / (ur[k][0] * D.R);
                src_e = -D.k * ur[k][4] * exp(-D.Ea / Tc);
                if (LEFT == 0 && tid < G::NC) psr[tid] = src_e;
            }
        }
        pu[p] = scale * vx;
        pv[p] = scale * vy;
        pp[p] = scale * pr;
        psrc[p] = src[k];
        unsigned place = 0u;
        if (p >= G::NC) {
            int li, lj;
            G::point(p, li, lj);
            place = (unsigned)(p < G::NC + G::NHX ? lj * G::PX + li + 3 : (lj + 3) * G::PY + li);
        }
        pfl[p] = pfl0[k] | place << 16;
    }
    if constexpr (DET) {
        raise(mv, ax, ay);
        const bool any = __any(flux_wide(mu, mv));
        if ((tid & 63) == 0) pwide[tid >> 6] = any ? 1u : 0u;
    }
    __syncthreads();

    // ---------------- phase 1: per component split fluxes, WENO5, RK update
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    double* S = bufs + w * G::BUF;
    double* SM = S + G::NX - 1;          // F- of the x pass: cell i at PX row + i + 2
    double* SY = S + G::NY;              // F- of the y pass
    double* SH = S + G::NH;              // lowest y fluxes of the runs
    // sources and flags (4 bits a point) of the lane's points
    using Flags = typename FlagWord<(NPL > 8)>::type;
    unsigned sp[NPL];
    Flags pf = 0;
    unsigned own = 0u;                    // bit q: cell q of this lane is solved
    int hoff[NPL];                        // LDS offset of a halo point in its pass
#pragma unroll
    for (int q = 0; q < NPL; ++q) {
        sp[q] = psrc[64 * q + l];
        const unsigned fl = pfl[64 * q + l];
        pf |= (Flags)(fl & 15u) << (4 * q);
        if (q < R) own |= (fl & PT_OWN) ? 1u << q : 0u;
        hoff[q] = (int)(fl >> 16);
    }
    const bool special = __any((pf & (Flags)0xccccccccccccccccull) != 0);
    const int oli = G::TWO ? l % TX : l, olj = G::TWO ? (l / TX) * R : 0;
    const int xbase = (l / G::XR) * G::PX + (l % G::XR) * R;
    const int ybase = G::TWO ? olj * G::PY + oli : 0;
    // RK stage (Shu-Osher): ca U^n + cb (U + dt L)
    const double ca = (stage == 1) ? 0.0 : (stage == 2) ? 0.75 : 1.0 / 3.0;
    const double cb = (stage == 1) ? 1.0 : (stage == 2) ? 0.25 : 2.0 / 3.0;
    // The tile's fluxes are reconstructed at WENO_SHRINK times their value.
    // (Cost against no test at all: 9 species, 0 to 1 % of the steps; 2 species, 700 k cells, 3 %.
    // A test of every denominator took 1.4 % of the former and 7 % where launches are short.)
    bool wide = false;
    if constexpr (DET) {
        unsigned h = 0u;
#pragma unroll
        for (int q = 0; q < W; ++q) h |= pwide[q];
        wide = __builtin_amdgcn_readfirstlane(h) != 0u;
    }
    if constexpr (LEFT > 0) {   // components left over: wave w takes interface w of every run
        double hx[LEFT], hy[LEFT], he[LEFT];
#pragma unroll
        for (int k = 0; k < LEFT; ++k) {
            const double* X = bufs + 2 * k * G::BUF;
            const double* Y = X + G::BUF;
            hx[k] = weno5_one<M, 1>(X + xbase + w, X + G::NX + xbase + w, wide);
            hy[k] = he[k] = 0.0;
            if constexpr (G::TWO)
                hy[k] = weno5_one<M, G::PY>(Y + ybase + w * G::PY, Y + G::NY + ybase + (w + 1) * G::PY, wide);
            if (tid < G::NEXT) {   // right column, top row
                if (tid < TY) he[k] = weno5_one<M, 1>(X + tid * G::PX + TX, X + G::NX + tid * G::PX + TX, wide);
                else he[k] = weno5_one<M, G::PY>(Y + TY * G::PY + tid - TY, Y + G::NY + (TY + 1) * G::PY + tid - TY, wide);
            }
            // one component after the other: both at once took 191 registers, two waves per SIMD
            // where one takes three (3 species, 700 k cells: 261 -> 221 us per step)
            asm volatile("" : "+v"(hx[k]), "+v"(hy[k]), "+v"(he[k]) : : "memory");
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < LEFT; ++k) {
            double* X = bufs + 2 * k * G::BUF;
            double* Y = X + G::BUF;
            X[(l / G::XR) * G::HX + (l % G::XR) * R + w] = hx[k];
            if (G::TWO) Y[(olj + w) * TX + oli] = hy[k];
            if (tid < TY) X[tid * G::HX + TX] = he[k];
            else if (tid < G::NEXT) Y[TY * TX + tid - TY] = he[k];
        }
        __syncthreads();
        if ((own >> w) & 1u) {
            const unsigned c = psrc[tid];
#pragma unroll
            for (int k = 0; k < LEFT; ++k) {
                const double* X = bufs + 2 * k * G::BUF;
                const double* Y = X + G::BUF;
                const int o = G::TWO ? (olj + w) * G::HX + oli : tid;
                double L = -(X[o + 1] - X[o]) * idx;
                if constexpr (G::TWO) L -= (Y[(olj + w + 1) * TX + oli] - Y[(olj + w) * TX + oli]) * idy;
                if constexpr (M == ONESTEP) L += src_e;
                const double u0 = (stage != 1) ? a.U0[(size_t)(NR + k) * a.pool + c] : 0.0;
                a.Uout[(size_t)(NR + k) * a.pool + c] = ca * u0 + cb * (uleft[k] + dt * L);
            }
        }
        __syncthreads();
    }
    double c1 = WENO_C1, escale = 1.0 / scale;
    if (DET && __builtin_expect(wide, 0)) {
#pragma unroll
        for (int k = 0; k < NT; ++k) {
            const int p = tid + 64 * W * k;
            if (p >= NPP) continue;
            pu[p] *= WENO_SHRINK;
            pv[p] *= WENO_SHRINK;
            pp[p] *= WENO_SHRINK;
        }
        sax = uniform(sax * WENO_SHRINK);
        say = uniform(say * WENO_SHRINK);
        c1 = WENO_C1 * WENO_SHRINK * WENO_SHRINK;
        escale = 1.0 / (scale * WENO_SHRINK);
        idx = uniform(idx * (1.0 / WENO_SHRINK));
        idy = uniform(idy * (1.0 / WENO_SHRINK));
        __syncthreads();
    }
    // component f of the lane's points
    auto load = [&](int f, double (&u)[NPL]) {
        const double* Uf = a.Uin + (size_t)f * a.pool;
        if (!special) {
#pragma unroll
            for (int q = 0; q < NPL; ++q) u[q] = Uf[sp[q]];
        } else {
            const double* U0f = a.U0 + (size_t)f * a.pool;
#pragma unroll
            for (int q = 0; q < NPL; ++q) {
                const unsigned fl = (unsigned)(pf >> (4 * q)) & 15u;
                const double* F = (fl & PT_DIR) ? a.dirU + f : (fl & 4u) ? U0f : Uf;
                u[q] = F[(fl & PT_DIR) ? sp[q] * (unsigned)(MAXF + 1) : sp[q]];
            }
        }
    };
    __builtin_amdgcn_s_setprio(0);
    double u[NPL], un[NPL];   // this component and, on its way, the wave's next one
    load(w, un);
    for (int f = w; f < NR; f += W) {
        // opaque in every pass: values derived from these are formed where they are used
        // (hoisted out of the loop they took 70 registers)
        asm volatile("" : "+v"(pf), "+v"(own));
#pragma unroll
        for (int q = 0; q < NPL; ++q) asm volatile("" : "+v"(sp[q]), "+v"(hoff[q]));
        const double* U0f = a.U0 + (size_t)f * a.pool;
        double u0[R];
#pragma unroll
        for (int q = 0; q < NPL; ++q) u[q] = un[q];
#pragma unroll
        for (int q = 0; q < R; ++q) u0[q] = 0.0;
        if (stage != 1) {
#pragma unroll
            for (int q = 0; q < R; ++q) u0[q] = U0f[((own >> q) & 1u) ? sp[q] : (unsigned)B.offset];
        }
        if (f == 1 || f == 2) {
#pragma unroll
            for (int q = 0; q < NPL; ++q) u[q] = ((unsigned)(pf >> (4 * q)) & (unsigned)f) ? -u[q] : u[q];
        }
        // split fluxes of point q along x or y; `plain`: neither the momentum along the sweep
        // nor the energy, which carry the pressure
        auto split = [&](int q, const double* pn, double al, bool plain, double& Fp, double& Fm) {
            const double vn = pn[64 * q + l];
            double F = 0.0, ue = u[q];   // pressure terms of the flux
            if (!plain) {
                const double p = pp[64 * q + l];
                if constexpr (DET) {
                    F = (f == 3) ? (p * vn) * escale : p;
                } else {
                    ue += (f == 3) ? p : 0.0;
                    F = (f == 3) ? 0.0 : p;
                }
            }
            split_flux<M>(u[q], vn, al, F, Fp, Fm, ue);
        };
        auto xfluxes = [&](bool plain) {
#pragma unroll
            for (int q = 0; q < NPL; ++q) {
                if (64 * q >= G::NC + G::NHX) continue;
                const int o = (q < R) ? (G::TWO ? (olj + q) * G::PX + oli + 3 : 64 * q + l + 3) : hoff[q];
                if (64 * q + 64 <= G::NC + G::NHX || 64 * q + l < G::NC + G::NHX) {
                    double Fp, Fm;
                    split(q, pu, sax, plain, Fp, Fm);
                    S[o] = Fp;
                    SM[o] = Fm;
                }
            }
        };
        auto yfluxes = [&](bool plain) {
#pragma unroll
            for (int q = 0; q < NPL; ++q) {
                if (q >= R && 64 * q + 64 <= G::NC + G::NHX) continue;
                const int o = (q < R) ? (olj + q + 3) * G::PY + oli : hoff[q];
                if (q < R || ((64 * q >= G::NC + G::NHX || 64 * q + l >= G::NC + G::NHX) &&
                              (64 * q + 64 <= G::NP || 64 * q + l < G::NP))) {
                    double Fp, Fm;
                    split(q, pv, say, plain, Fp, Fm);
                    S[o] = Fp;
                    SY[o] = Fm;
                }
            }
        };
        double eP[5], eM[5];   // stencils of the right column / top row interface of this lane
#pragma unroll
        for (int k = 0; k < 5; ++k) eP[k] = eM[k] = 0.0;
        // x pass
        double hx[R];
        if (f == 1 || f == 3) xfluxes(false);
        else xfluxes(true);
        if (f + W < NR) load(f + W, un);
        wave_sync();
        {
            if (l < TY) {
                const int o = l * G::PX + TX;
#pragma unroll
                for (int k = 0; k < 5; ++k) {
                    eP[k] = S[o + k];
                    eM[k] = S[G::NX + o + 4 - k];
                }
            }
            weno5_runs<M, R, 1>(S + xbase, S + G::NX + xbase, hx, c1);
        }
        wave_sync();
        // y pass
        double hy[R + 1];
        if constexpr (G::TWO) {
            if (f == 2 || f == 3) yfluxes(false);
            else yfluxes(true);
            wave_sync();
            double h[R];
            const int e = l - (G::NEXT <= 64 ? TY : 0);   // top row, column e
            if (e >= 0 && e < TX && G::NEXT <= 64) {
                const int o = TY * G::PY + e;
#pragma unroll
                for (int k = 0; k < 5; ++k) {
                    eP[k] = S[o + k * G::PY];
                    eM[k] = SY[o + (5 - k) * G::PY];
                }
            }
            double tP[5], tM[5];
            if constexpr (G::NEXT > 64) {
#pragma unroll
                for (int k = 0; k < 5; ++k) {
                    tP[k] = S[TY * G::PY + l + k * G::PY];
                    tM[k] = SY[TY * G::PY + l + (5 - k) * G::PY];
                }
            }
            weno5_runs<M, R, G::PY>(S + ybase, SY + G::PY + ybase, h, c1);
#pragma unroll
            for (int k = 0; k < R; ++k) hy[k] = h[k];
            wave_sync();
            SH[(l / TX) * TX + oli] = h[0];
            if constexpr (G::NEXT > 64) SH[(TY / R) * TX + l] = weno5_pair<M>(tP, tM, c1);
        }
        // numerical fluxes to LDS, the right column and top row with them
#pragma unroll
        for (int k = 0; k < R; ++k) S[(l / G::XR) * G::HX + (l % G::XR) * R + k] = hx[k];
        if (G::NEXT > 64 ? l < TY : l < G::NEXT) {
            const double he = weno5_pair<M>(eP, eM, c1);
            if (l < TY) S[l * G::HX + TX] = he;
            else SH[(TY / R) * TX + l - TY] = he;
        }
        wave_sync();
        if constexpr (G::TWO) hy[R] = SH[(l / TX + 1) * TX + oli];
        // flux difference (Eq. 4.10), source and RK stage
        double L[R];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int o = G::TWO ? (olj + q) * G::HX + oli : 64 * q + l;
            L[q] = -(S[o + 1] - S[o]) * idx;
            if constexpr (G::TWO) L[q] -= (hy[q + 1] - hy[q]) * idy;
        }
        if constexpr (M == ONESTEP && LEFT == 0) {
            static_assert(R == 1 || LEFT > 0, "the source is kept for one cell per lane");
            if (f == 4) L[0] += psr[l];
        }
        double* out = a.Uout + (size_t)f * a.pool;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const double unew = ca * u0[q] + cb * (u[q] + dt * L[q]);
            if ((own >> q) & 1u) out[sp[q]] = unew;
        }
        wave_sync();
    }
    if (DET && __builtin_expect(wide, 0)) {
        idx = uniform(idx * WENO_SHRINK);
        idy = uniform(idy * WENO_SHRINK);
    }
    __syncthreads();   // the new state of the tile is complete (in the caches)

    __builtin_amdgcn_s_setprio(2);
    // ---------------- phase 2: T, checks, maxima for the next stage
    double sx = 0.0, sy = 0.0, sc = 0.0;
    if (w < R && ((own >> w) & 1u)) {   // cell tid = 64 w + l
        const long long oc = psrc[tid];
        const double* Uo = a.Uout + oc;
        double unew[NU];
#pragma unroll
        for (int f = 0; f < NU; ++f) unew[f] = Uo[(size_t)f * a.pool];
        double T, c, vx, vy;
        const unsigned st = owner_state<M, NU>(unew, Town, D, cmech(a.mech), T, c, vx, vy);
        a.Tout[oc] = T;
        if (st) atomicOr(a.status, st);
        bool skip = false;
        if (stage == 3 && B.fine_child && (!a.cross || a.xskip_cov)) {
            int li, lj;
            G::point(tid, li, lj);
            skip = covered_by_finer(a, D, lev, B.i0 + tile.x0 + li, B.j0 + tile.y0 + lj);
        }
        if (a.reduce_out && !st && !skip) {
            sx = fabs(vx) + c;
            sy = fabs(vy) + c;
            sc = cfl_bound(a, D, lev, sx, sy, idx, idy);
        }
    }
    if (!a.reduce_out) return;
    const int i0 = 2 * slot, i2 = 2 * a.red.nunits + B.domain;
    if constexpr (R == 1) {   // one wave holds every cell
        if (w == 0) publish_wave3(a.red, bout, i0, i0 + 1, i2, sx, sy, sc);
    } else {
        bufs[tid] = sx;
        bufs[64 * W + tid] = sy;
        bufs[128 * W + tid] = sc;
        __syncthreads();
        publish_staged<W>(a.red, bout, i0, i0 + 1, i2, bufs);
    }
}

// Waves per SIMD that the registers have to leave room for: with 2 and 3 species the 16 x 16
// kernel takes about 128 registers, and one more costs the fourth wave.
template <int M, int NU, int TX>
constexpr int stage_waves() { return (M == DETAILED && NU <= 6 && TX == 16) ? 4 : 1; }
template <int M, int NU, int TX, int TY, bool HAS1D, bool HAS2D>
__global__ __launch_bounds__(64 * STAGE_W, (stage_waves<M, NU, TX>())) void stage_kernel(StageArgs a, int first_tile, int owner_launch) {
    constexpr int L2 = HAS2D ? stage_lds<TX, TY>(STAGE_W) : 0, L1 = HAS1D ? stage_lds<256, 1>(STAGE_W) : 0;
    __shared__ __align__(16) double smem[(L2 > L1) ? L2 : L1];
    if (blockIdx.x == 0) stage_bookkeeping(a, owner_launch);
    const int ti = first_tile + (a.linear_sched ? (int)blockIdx.x : xcd_chunk(blockIdx.x, gridDim.x));
    const Tile tile = ctile(a.tiles, ti);
    if (HAS1D && tile.kind == 1) {
        if constexpr (HAS1D) stage_tile<M, NU, 256, 1, STAGE_W>(a, ti, tile, smem);
    } else {
        if constexpr (HAS2D) stage_tile<M, NU, TX, TY, STAGE_W>(a, ti, tile, smem);
    }
    if (a.stage == 3 && (a.cross ? a.xlast : owner_launch) && blockIdx.x == 0) {
        // t and the step counter are read by the next step's first stage only
        if (M != DETAILED) step_finish(a);
    }
}

// Quarter `sub` of a tile.
__device__ __forceinline__ Tile quarter(Tile t, int sub) {
    if (t.kind == 1) {
        t.x0 += 64 * sub;
    } else {
        const int n = t.kind >> 11;   // quarters side by side (tile width / 8)
        t.y0 += 8 * (sub / n);
        t.x0 += 8 * (sub % n);
    }
    return t;
}

// The stage on tiles of 8 x 8 or 64 x 1 cells, W waves each. SPLIT = SMALL_SPLIT: quarter tiles,
// one wave per component; workgroup b takes quarter b % 4 of tile b / 4. SPLIT = 1: plans of many
// tiles whose valid cells all fit into the first quarter (blocks of up to 8 x 8 or 64 x 1 cells),
// four waves, as many workgroups as a CU holds; the whole tiles sweep 256 cells for at most 64 of
// them (us per step, whole / these: 9 species 1000 x 50 cells 105 / 75, 4000 x 8 x 8 446 / 287, 3
// species 4000 x 50 167 / 115, one-step 4000 x 8 x 8 211 / 124).
// Two waves: tiles of 16 x 8 or 128 x 1 cells (runs of two interfaces per lane), for plans of
// still more tiles whose valid cells fit into the first half (whole / these: 9 species 4000 x 100
// cells 350 / 276, 4000 x 20 x 5 837 / 623, 3 species 4000 x 100 184 / 135, one-step 4000 x 20 x
// 5 372 / 279, gas without chemistry 301 / 226).
template <int M, int NU, int W, int SPLIT, bool HAS1D, bool HAS2D>
__global__ __launch_bounds__(64 * W) void stage_small_kernel(StageArgs a, int first_tile, int owner_launch) {
    constexpr int TX = W == HALF_W ? 16 : 8, N1 = 8 * TX;
    constexpr int L2 = HAS2D ? stage_lds<TX, 8>(W) : 0, L1 = HAS1D ? stage_lds<N1, 1>(W) : 0;
    __shared__ __align__(16) double smem[(L2 > L1) ? L2 : L1];
    if (blockIdx.x == 0) stage_bookkeeping(a, owner_launch);
    const int ti = SPLIT * first_tile + (a.linear_sched ? (int)blockIdx.x : xcd_chunk(blockIdx.x, gridDim.x));
    const Tile tile = quarter(ctile(a.tiles, ti / SPLIT), ti % SPLIT);
    if (HAS1D && tile.kind == 1) {
        if constexpr (HAS1D) stage_tile<M, NU, N1, 1, W>(a, ti, tile, smem);
    } else {
        if constexpr (HAS2D) stage_tile<M, NU, TX, 8, W>(a, ti, tile, smem);
    }
    if (a.stage == 3 && (a.cross ? a.xlast : owner_launch) && blockIdx.x == 0) {
        if (M != DETAILED) step_finish(a);
    }
}

// ------------------------------------------------------------------ halo source table
// Workgroup t fills row t of the table: for each point of tile t that a sweep reads,
// 8 * source + flags (bit 0 / 1: mirrored x / y momentum, bit 2: a coarser level);
// HALO_NONE elsewhere.
template <int TX, int TY>
__device__ void halo_table_tile(const StageArgs& a, int ti, const Tile& tile, int* row) {
    const DevBlock B = a.blk[tile.block];
    CDom& D = cdom(a.dom, B.domain);
    const int tw = min(TX, B.nx - tile.x0), th = min(TY, B.ny - tile.y0);
    for (int p = threadIdx.x; p < Geom<TX, TY>::NP; p += WG) {
        long long s = 0;
        unsigned fl = 0u;
        const bool needed = point_source<TX, TY>(a, B, D, tile, p, tw, th, s, fl);
        row[p] = needed ? (int)(s * 8 + (long long)fl) : HALO_NONE;
    }
}

template <int TX, int TY>
__global__ __launch_bounds__(WG) void halo_table_kernel(StageArgs a, int* out, int stride) {
    const int ti = blockIdx.x;
    const Tile tile = a.tiles[ti];
    int* row = out + (size_t)ti * stride;
    if (tile.kind == 1) halo_table_tile<WG, 1>(a, ti, tile, row);
    else halo_table_tile<TX, TY>(a, ti, tile, row);
}

// ------------------------------------------------------------------ per-cell kernels
// Cell of a tile owned by this thread (same mapping as the stage kernel).
struct CellRef {
    long long c;
    int I, J;     // level coordinates
    bool own;
};

__device__ __forceinline__ CellRef tile_cell(const StageArgs& a, const Tile& tile, const DevBlock& B) {
    (void)a;
    CellRef r;
    int tw, th, li, lj;
    if (tile.kind == 1) {
        li = threadIdx.x;
        lj = 0;
        tw = min(WG, B.nx - tile.x0);
        th = 1;
    } else {
        // 2-D tile shapes encode their width in kind >> 8
        const int TXs = tile.kind >> 8;
        li = threadIdx.x % TXs;
        lj = threadIdx.x / TXs;
        tw = min(TXs, B.nx - tile.x0);
        th = min(WG / TXs, B.ny - tile.y0);
    }
    const int bi = tile.x0 + li, bj = tile.y0 + lj;
    r.own = (li < tw) && (lj < th) && !ring_at(B, bi, bj);
    r.c = B.offset + (long long)bj * B.nx + bi;
    r.I = B.i0 + bi;
    r.J = B.j0 + bj;
    return r;
}

// Call entry: T re-solved from U (warm start = stored T) and the maxima for stage 1.
//
// A workgroup takes `per` tiles in turn and publishes when the slots change: one address takes
// an atomic every 13 ns, and three per tile were the length of this launch at many tiles (9
// species, everything before the first step: 7,750 tiles 256 -> 190 us, 15,750 tiles 326 ->
// 187 us). Below INIT_MANY tiles the launch is short and one each fills the chip better.
constexpr int INIT_MANY = 4096, INIT_PER = 4;
inline int init_per(int ntiles) { return ntiles >= INIT_MANY ? INIT_PER : 1; }
template <int M, int NU>
__global__ __launch_bounds__(WG) void init_kernel(StageArgs a, int per) {
    __shared__ double scratch[16];
    double sx = 0.0, sy = 0.0, sc = 0.0;
    const int t0 = blockIdx.x * per, t1 = min(t0 + per, a.ntiles);
    for (int ti = t0; ti < t1; ++ti) {
        const Tile tile = a.tiles[ti];
        const DevBlock B = a.blk[tile.block];
        CDom& D = cdom(a.dom, B.domain);
        const CellRef r = tile_cell(a, tile, B);
        const int lev = B.level, slot = D.slot0 + lev;
        const double idx = ldexp(D.idx0, lev), idy = ldexp(D.idy0, lev);
        if (r.own) {
            double u[NU];
#pragma unroll
            for (int f = 0; f < NU; ++f) u[f] = a.Uin[(size_t)f * a.pool + r.c];
            double T, c, vx, vy;
            const unsigned st = owner_state<M, NU>(u, a.Tin[r.c], D, cmech(a.mech), T, c, vx, vy);
            a.Tout[r.c] = T;
            if (st) atomicOr(a.status, st);
            else {
                sx = fmax(sx, fabs(vx) + c);
                sy = fmax(sy, fabs(vy) + c);
                sc = fmax(sc, cfl_bound(a, D, lev, fabs(vx) + c, fabs(vy) + c, idx, idy));
            }
        }
        bool last = ti + 1 == t1;
        if (!last) {
            const DevBlock N = a.blk[a.tiles[ti + 1].block];
            last = N.level != lev || N.domain != B.domain;
        }
        if (last) {
            publish_max3<WG / 64>(a.red, 0, 2 * slot, 2 * slot + 1, 2 * a.red.nunits + B.domain, sx, sy, sc, scratch);
            sx = sy = sc = 0.0;
        }
    }
}

// (I - dt J) dU = dt w of the point-implicit step (Eq. 4.12-4.13) for the Jacobian J of
// rho Y_1 .. rho Y_{Ns-1} and the production rates w: Gaussian elimination with partial
// pivoting in registers; w returns the increment. One reciprocal per pivot serves its column
// and its row of the back substitution (both rounded as the divisions they replace; with the
// terms a mechanism leaves out, 4617 -> 4272 instructions at 9 species and 19 reactions).
template <int NS>
__device__ __forceinline__ void chem_solve(double (&J)[NS - 1][NS - 1], double (&w)[NS - 1],
                                           double dt, unsigned& st) {
    constexpr int NT = NS - 1;
    double ipiv[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) {
#pragma unroll
        for (int q = 0; q < NT; ++q) J[k][q] = (k == q ? 1.0 : 0.0) - dt * J[k][q];
        w[k] = w[k] * dt;
    }
#pragma unroll
    for (int c = 0; c < NT; ++c) {
        // pivot row: the first row at or below c with the largest |entry| in column c;
        // rows are exchanged by selects so that the matrix stays in registers, and only
        // in wavefronts where some cell needs an exchange
        int p = c;
        double amax = fabs(J[c][c]);
#pragma unroll
        for (int r = c + 1; r < NT; ++r) {
            const double ar = fabs(J[r][c]);
            if (ar > amax) { amax = ar; p = r; }
        }
        if (__any(p != c)) {
#pragma unroll
            for (int r = c + 1; r < NT; ++r) {
                const bool sw = (r == p);
#pragma unroll
                for (int q = c; q < NT; ++q) {
                    const double top = J[c][q], row = J[r][q];
                    J[c][q] = sw ? row : top;
                    J[r][q] = sw ? top : row;
                }
                const double wt = w[c], wr = w[r];
                w[c] = sw ? wr : wt;
                w[r] = sw ? wt : wr;
            }
        }
        const double piv = J[c][c];
        if (!(fabs(piv) > 0.0) || !isfinite(piv)) st |= STB_NONFINITE;
        const double ip = quotient(1.0, piv);
        ipiv[c] = ip;
#pragma unroll
        for (int r = c + 1; r < NT; ++r) {
            const double fct = J[r][c] * ip;
#pragma unroll
            for (int q = c + 1; q < NT; ++q) J[r][q] -= fct * J[c][q];
            w[r] -= fct * w[c];
        }
    }
#pragma unroll
    for (int r = NT - 1; r >= 0; --r) {
        double sacc = w[r];
#pragma unroll
        for (int q = r + 1; q < NT; ++q) sacc -= J[r][q] * w[q];
        // the rounded quotient by the pivot: product with its reciprocal and one residual step
        const double q0 = sacc * ipiv[r];
        w[r] = __builtin_fma(__builtin_fma(-J[r][r], q0, sacc), ipiv[r], q0);
    }
}


// Point-implicit chemistry (Eq. 4.12-4.13) on rho Y_1 .. rho Y_{Ns-1} of each
// solved cell, then Newton for the new T and the maxima for the next step.
// Mechanism tables are read as wave-uniform scalar loads. Per-thread columns in
// LDS hold X, the species Gibbs terms and the derivative row dq/dX of the
// current reaction (indexed by wave-uniform species numbers); the (Ns-1)^2
// Jacobian, the production rates and the LU factorization live in registers.
template <int NS, bool FULLJ>
__device__ __forceinline__ void chem_cell(CMech* m, double* Xs, double* gts, double* dqs,
                                          double rho, double T, const double (&rY)[NS - 1],
                                          double dt, double (&w)[NS - 1], unsigned& st) {
    constexpr int NT = NS - 1;
    const int tid = threadIdx.x;
    // LDS column per thread: X[0..NS-1], X[NS] = 1 (padding of the molecule lists)
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        Xs[j * WG + tid] = rY[j] * m->invM[j];
        s += rY[j];
    }
    Xs[NT * WG + tid] = (rho - s) * m->invM[NT];
    Xs[NS * WG + tid] = 1.0;
    const double lnT = log(T), invT = 1.0 / T;
    const double lnC = log(PATM / RU) - lnT;      // ln(p_atm / (R_u T))
#pragma unroll
    for (int j = 0; j < NS; ++j) {                 // h/(R T) - s/R per species
        const bool hi = m->two_range && T >= m->tmid[j];
        double a[7];
#pragma unroll
        for (int q = 0; q < 7; ++q) a[q] = hi ? m->nasa_hi[j][q] : m->nasa[j][q];
        gts[j * WG + tid] = a[0] * (1.0 - lnT) -
                T * (0.5 * a[1] + T * (a[2] * (1.0 / 6.0) + T * (a[3] * (1.0 / 12.0) + T * (a[4] * 0.05)))) +
                a[5] * invT - a[6];
    }
    gts[NS * WG + tid] = 0.0;   // padding slot of the molecule lists
    // species + T Jacobian: T follows the composition at fixed rho and e, so
    // J += (dS/dT) (dT/d rho Y)^T with dT/d rho Y_m = -(e_m - e_last) / (rho c_v);
    // hm1[j] = h_j/(R_u T) - 1 = e_j / (R_u T) per mole, cvs = rho c_v / R_u
    double hm1[NS], dSdT[NT];
    double cvs = 0.0;
    if constexpr (FULLJ) {
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            const bool hi = m->two_range && T >= m->tmid[j];
            double a[7];
#pragma unroll
            for (int q = 0; q < 7; ++q) a[q] = hi ? m->nasa_hi[j][q] : m->nasa[j][q];
            hm1[j] = a[0] + T * (0.5 * a[1] + T * (a[2] * (1.0 / 3.0) + T * (0.25 * a[3] + T * (0.2 * a[4])))) +
                     a[5] * invT - 1.0;
            cvs += Xs[j * WG + tid] * (a[0] + T * (a[1] + T * (a[2] + T * (a[3] + T * a[4]))) - 1.0);
        }
#pragma unroll
        for (int k = 0; k < NT; ++k) dSdT[k] = 0.0;
    }
    double J[NT][NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        w[k] = 0.0;
#pragma unroll
        for (int q = 0; q < NT; ++q) J[k][q] = 0.0;
    }
    const int nr = m->nr;
    for (int i = 0; i < nr; ++i) {
        const double lnkf = m->lnA[i] + m->b[i] * lnT - m->EaR[i] * invT;
        const double kf = exp(lnkf);
        const int f0 = m->lf[i][0], f1 = m->lf[i][1], f2 = m->lf[i][2];
        const int r0 = m->lb[i][0], r1 = m->lb[i][1], r2 = m->lb[i][2];
        double kb = 0.0;
        if (m->rev[i]) {
            // sum_j dnu_j g_j, g = h/(RT) - s/R: products minus reactants, one entry per
            // molecule (the padding slot holds 0)
            const double sg = (gts[r0 * WG + tid] + gts[r1 * WG + tid] + gts[r2 * WG + tid]) -
                              (gts[f0 * WG + tid] + gts[f1 * WG + tid] + gts[f2 * WG + tid]);
            // K_eq = exp(-sum dnu g) (p_atm/(R_u T))^(sum dnu), Eq. 4.9
            kb = exp(lnkf + sg - (double)m->dnsum[i] * lnC);
        }
        const double xf0 = Xs[f0 * WG + tid], xf1 = Xs[f1 * WG + tid], xf2 = Xs[f2 * WG + tid];
        const double xb0 = Xs[r0 * WG + tid], xb1 = Xs[r1 * WG + tid], xb2 = Xs[r2 * WG + tid];
        const double Rf = kf * (xf0 * xf1 * xf2), Rb = kb * (xb0 * xb1 * xb2);
        const bool tbr = m->has_tb[i] != 0;
        double ctb = 1.0;
        if (tbr) {
            ctb = 0.0;
#pragma unroll
            for (int j = 0; j < NS; ++j) ctb += m->tb[i][j] * Xs[j * WG + tid];
        }
        const double net = Rf - Rb;
        const double q = ctb * net;
#pragma unroll
        for (int k = 0; k < NT; ++k) w[k] += m->Mdnu[i][k] * q;
        if constexpr (FULLJ) {
            // d ln kf/dT = (b + Ea/(R T))/T; d ln kb/dT = d ln kf/dT - sum_j dnu_j (H_j - 1)/T
            const double dlf = (m->b[i] + m->EaR[i] * invT) * invT;
            double dlb = dlf;
            if (m->rev[i]) {
                double sh = 0.0;
#pragma unroll
                for (int j = 0; j < NS; ++j) sh += (double)m->dnu[i][j] * hm1[j];
                dlb = dlf - sh * invT;
            }
            const double dqT = ctb * (Rf * dlf - Rb * dlb);
#pragma unroll
            for (int k = 0; k < NT; ++k) dSdT[k] += m->Mdnu[i][k] * dqT;
        }
        // dq/dX_j into LDS (padding slot NS absorbs the entries of missing molecules)
#pragma unroll
        for (int j = 0; j <= NS; ++j) dqs[j * WG + tid] = (tbr && j < NS) ? m->tb[i][j] * net : 0.0;
        const double cf = ctb * kf, cb = ctb * kb;
        dqs[f0 * WG + tid] += cf * (xf1 * xf2);
        dqs[f1 * WG + tid] += cf * (xf0 * xf2);
        dqs[f2 * WG + tid] += cf * (xf0 * xf1);
        dqs[r0 * WG + tid] -= cb * (xb1 * xb2);
        dqs[r1 * WG + tid] -= cb * (xb0 * xb2);
        dqs[r2 * WG + tid] -= cb * (xb0 * xb1);
        // d(rho Y_m): dX_j/d(rho Y_m) = delta_jm / M_m - delta_{j,last} / M_last
        const double dlast = dqs[NT * WG + tid] * m->invM[NT];
        double Dm[NT];
#pragma unroll
        for (int mm = 0; mm < NT; ++mm) Dm[mm] = dqs[mm * WG + tid] * m->invM[mm] - dlast;
#pragma unroll
        for (int k = 0; k < NT; ++k) {
            if (m->dnu[i][k] != 0) {
                const double ck = m->Mdnu[i][k];
#pragma unroll
                for (int mm = 0; mm < NT; ++mm) J[k][mm] += ck * Dm[mm];
            }
        }
    }
    if constexpr (FULLJ) {
        const double ilast = hm1[NT] * m->invM[NT];
#pragma unroll
        for (int mm = 0; mm < NT; ++mm) {
            const double dTm = -T * (hm1[mm] * m->invM[mm] - ilast) / cvs;
#pragma unroll
            for (int k = 0; k < NT; ++k) J[k][mm] += dSdT[k] * dTm;
        }
    }
    chem_solve<NS>(J, w, dt, st);
}

// One chemistry launch over the tiles (one cell per thread): the dt of the phase, the
// point-implicit step `cell(mech, rho, T, rho Y, dt, dY, status)` on each solved cell,
// Newton for the new T, and the maxima for the next stage. Shared by the generic kernel
// below and the kernel specialised at run time to a mechanism's structure.
template <int NS, class Cell>
__device__ __forceinline__ void chem_body(const StageArgs& a, double* scratch, Cell&& cell) {
    constexpr int NU = NS + 3;
    const Tile tile = a.tiles[blockIdx.x];
    const DevBlock B = a.blk[tile.block];
    CDom& D = cdom(a.dom, B.domain);
    CMech* mech = cmech(a.mech);
    const CellRef r = tile_cell(a, tile, B);
    const int lev = B.level, slot = D.slot0 + lev;
    // phase 0: the whole dt after the stages (Lie); phase 1: dt/2 before stage 1, this
    // launch forms the step's dt; phase 2: dt/2 after stage 3 (Strang, Sec. 4.2)
    const int phase = a.chem_phase;
    const double dstep = a.cross ? ldexp((phase == 1 && a.xfirst) ? step_dt(a, B.domain, 0)
                                                                   : a.dt[B.domain], -lev)
                                 : (phase == 1) ? step_dt(a, B.domain, 0) : a.dt[B.domain];
    const double dt = (phase == 0) ? dstep : 0.5 * dstep;
    const double idx = ldexp(D.idx0, lev), idy = ldexp(D.idy0, lev);
    if (blockIdx.x == 0) {
        if (phase == 1) {
            if (!a.cross || a.xfirst) record_dt(a);
        } else if (!a.cross || a.xlast) {
            step_finish(a);
        }
    }
    if (phase == 2)   // buffer 3 was read by stage 1; clean for the next step's first half
        for (int q = threadIdx.x; q < a.red.stride; q += WG) a.red.buf[slot_word(a.red.stride, 3, q)] = 0ull;
    if (!(dt > 0.0)) return;
    // A cell under a finer block is overwritten by the restriction that follows this
    // launch (the Lie step, or the second half of the Strang split; in the crossover
    // advance, the level's last step) and leaves the maxima (the restriction publishes
    // the restricted cell's instead). Where none of its four children is a ring cell,
    // the restriction does not read it either: its chemistry is dead work.
    const bool covered = r.own && phase != 1 && B.fine_child && (!a.cross || a.xskip_cov) &&
                         covered_by_finer(a, D, lev, r.I, r.J);
    const bool dead = covered && restricted_over(a, D, lev, r.I, r.J);
    const bool work = r.own && !dead;
    double sx = 0.0, sy = 0.0, sc = 0.0;
    unsigned st = 0u;
    double dY[NS - 1];
    double T = 1.0;
    {
        // inactive lanes run the same arithmetic on a harmless state
        double rho = 1.0;
        double rY[NS - 1];
#pragma unroll
        for (int k = 0; k < NS - 1; ++k) rY[k] = 0.0;
        if (work) {
            rho = a.Uout[r.c];
#pragma unroll
            for (int k = 0; k < NS - 1; ++k) rY[k] = a.Uout[(size_t)(4 + k) * a.pool + r.c];
            T = a.Tout[r.c];
        }
        if (__any(work)) cell(mech, rho, T, rY, dt, dY, st);   // wavefronts with no work skip it
    }
    if (work) {
        double u[NU];
#pragma unroll
        for (int f = 0; f < NU; ++f) u[f] = a.Uout[(size_t)f * a.pool + r.c];
#pragma unroll
        for (int k = 0; k < NS - 1; ++k) {
            u[4 + k] += dY[k];
            a.Uout[(size_t)(4 + k) * a.pool + r.c] = u[4 + k];
        }
        double Tn, c, vx, vy;
        st |= owner_state<DETAILED, NU>(u, T, D, mech, Tn, c, vx, vy);
        a.Tout[r.c] = Tn;
        if (st) atomicOr(a.status, st);
        // the first half's maxima are stage 1's alpha over all solved cells
        if (!st && !covered) {
            sx = fabs(vx) + c;
            sy = fabs(vy) + c;
            sc = cfl_bound(a, D, lev, sx, sy, idx, idy);
        }
    }
    publish_max3<WG / 64>(a.red, (phase == 1) ? 3 : 0, 2 * slot, 2 * slot + 1, 2 * a.red.nunits + B.domain, sx,
                 sy, sc, scratch);
}

#ifndef CHEM_WAVES
#define CHEM_WAVES 1
#endif
template <int NS, bool FULLJ>
__global__ __launch_bounds__(WG, CHEM_WAVES) void chem_kernel(StageArgs a) {
    __shared__ double Xs[(NS + 1) * WG];
    __shared__ double gts[(NS + 1) * WG];
    __shared__ double dqs[(NS + 1) * WG];
    __shared__ double scratch[16];
    chem_body<NS>(a, scratch, [&](CMech* m, double rho, double T, const double (&rY)[NS - 1],
                                  double dt, double (&dY)[NS - 1], unsigned& st) {
        chem_cell<NS, FULLJ>(m, Xs, gts, dqs, rho, T, rY, dt, dY, st);
    });
}

// Four-to-one restriction (Sec. 3.1.4 coarsening): each coarse cell under a
// valid block of this level becomes the mean of its four children (ring
// children count with their effective value, the coarse cell itself); T is
// re-solved; the coarse cell enters the maxima of the next step. Workgroup
// (b, y) takes coarse cells y*WG, y*WG + gridDim.y*WG, ... of fine block b.
template <int M, int NU>
__global__ __launch_bounds__(WG) void restrict_kernel(StageArgs a, const int* fine_blocks) {
    __shared__ double scratch[16];
    const DevBlock B = a.blk[fine_blocks[blockIdx.x]];
    CDom& D = cdom(a.dom, B.domain);
    const int lev = B.level;
    const double dt = a.dt[B.domain];
    const int cw = B.nx / 2, ch = B.ny / 2;
    if (!(dt > 0.0) || (int)blockIdx.y * WG >= cw * ch) return;
    const int cslot = D.slot0 + lev - 1;
    const double idx = ldexp(D.idx0, lev - 1), idy = ldexp(D.idy0, lev - 1);
    double sx = 0.0, sy = 0.0, sc = 0.0;
    for (int cc = blockIdx.y * WG + threadIdx.x; cc < cw * ch; cc += gridDim.y * WG) {
        const int cj = cc / cw, ci = cc - cj * cw;
        unsigned fl = 0u;
        const long long cpar = resolve(a, D, lev - 1, (B.i0 >> 1) + ci, (B.j0 >> 1) + cj, fl);
        double mean[NU];
        double ch4[4][NU];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int li = 2 * ci + (q & 1), lj = 2 * cj + (q >> 1);
            long long s;
            unsigned f2 = 0u;
            if (!ring_at(B, li, lj)) s = B.offset + (long long)lj * B.nx + li;
            else s = resolve(a, D, lev - 1, (B.i0 + li) >> 1, (B.j0 + lj) >> 1, f2);
            double Tq;
            fetch<NU>(a, s, f2, a.Uout, a.Tout, ch4[q], Tq);
        }
#pragma unroll
        for (int f = 0; f < NU; ++f) mean[f] = ((ch4[0][f] + ch4[1][f]) + (ch4[2][f] + ch4[3][f])) * 0.25;
        // all children are read before any coarse value changes: a ring child of this
        // coarse cell resolves to the cell itself, which only this thread writes
#pragma unroll
        for (int f = 0; f < NU; ++f) a.Uout[(size_t)f * a.pool + cpar] = mean[f];
        double T, c, vx, vy;
        const unsigned st = owner_state<M, NU>(mean, a.Tout[cpar], D, cmech(a.mech), T, c, vx, vy);
        a.Tout[cpar] = T;
        if (st) atomicOr(a.status, st);
        else {
            sx = fmax(sx, fabs(vx) + c);
            sy = fmax(sy, fabs(vy) + c);
            sc = fmax(sc, cfl_bound(a, D, lev - 1, fabs(vx) + c, fabs(vy) + c, idx, idy));
        }
    }
    publish_max3<WG / 64>(a.red, 0, 2 * cslot, 2 * cslot + 1, 2 * a.red.nunits + B.domain, sx, sy, sc,
                 scratch);
}

// Ring cells take the injection (one-to-four) of the coarser level after restriction.
// Only the 3-cell bands along the four sides can hold ring cells: workgroup (b, y)
// walks the band cells y*WG, y*WG + gridDim.y*WG, ... of block b (W, E, S, N bands;
// a corner cell lies in two bands and is written twice with the same value).
template <int NU>
__global__ __launch_bounds__(WG) void ring_fill_kernel(StageArgs a, const int* ring_blocks) {
    const DevBlock B = a.blk[ring_blocks[blockIdx.x]];
    CDom& D = cdom(a.dom, B.domain);
    const int nband = 6 * B.ny + 6 * B.nx;
    if (!(a.dt[B.domain] > 0.0) || (int)blockIdx.y * WG >= nband) return;
    for (int q = blockIdx.y * WG + threadIdx.x; q < nband; q += gridDim.y * WG) {
        int li, lj;
        if (q < 6 * B.ny) {
            const int r = (q < 3 * B.ny) ? q : q - 3 * B.ny;
            lj = r / 3;
            li = (q < 3 * B.ny) ? r - 3 * lj : B.nx - 3 + (r - 3 * lj);
        } else {
            const int h = q - 6 * B.ny, r = (h < 3 * B.nx) ? h : h - 3 * B.nx;
            const int row = r / B.nx;
            li = r - row * B.nx;
            lj = (h < 3 * B.nx) ? row : B.ny - 3 + row;
        }
        if (!ring_at(B, li, lj)) continue;
        unsigned fl = 0u;
        const long long s = resolve(a, D, B.level - 1, (B.i0 + li) >> 1, (B.j0 + lj) >> 1, fl);
        double u[NU], T;
        fetch<NU>(a, s, fl, a.Uout, a.Tout, u, T);
        const long long c = B.offset + (long long)lj * B.nx + li;
#pragma unroll
        for (int f = 0; f < NU; ++f) a.Uout[(size_t)f * a.pool + c] = u[f];
        a.Tout[c] = T;
    }
}

// The same of the models without NASA-7 thermodynamics: w = rho, u, v, p (, Y).
template <int M, int NU>
__device__ __forceinline__ void gas_to_cons(const double (&w)[NU], double gamma, double Q, double (&U)[NU]) {
    const double rho = w[0], u = w[1], v = w[2], p = w[3];
    U[0] = rho;
    U[1] = rho * u;
    U[2] = rho * v;
    double E = p / (gamma - 1.0) + 0.5 * rho * (u * u + v * v);
    if constexpr (M == ONESTEP) {
        E += rho * w[4] * Q;
        U[4] = rho * w[4];
    }
    U[3] = E;
}

// Conserved state from primitives (Eq. 4.2), one thread per cell.
template <int M, int NU>
__global__ void prim_to_cons_kernel(const DevMech* mech, double gamma, double R, double Q,
                                    long long n, const double* W, double* U, double* T,
                                    long long sin, long long sout) {
    const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    double w[NU];
#pragma unroll
    for (int f = 0; f < NU; ++f) w[f] = W[(size_t)f * sin + c];
    if constexpr (M == DETAILED) {
        constexpr int NS = NU - 3;
        const double p = w[0], u = w[1], v = w[2], Tt = w[3];
        double Y[NS], s = 0.0;
#pragma unroll
        for (int k = 0; k < NS - 1; ++k) {
            Y[k] = w[4 + k];
            s += Y[k];
        }
        Y[NS - 1] = 1.0 - s;
        double Rm = 0.0, e = 0.0;
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            const double* a = (mech->two_range && Tt >= mech->tmid[k]) ? mech->nasa_hi[k] : mech->nasa[k];
            const double h = Tt * (a[0] + Tt * (0.5 * a[1] + Tt * (a[2] * (1.0 / 3.0) +
                             Tt * (0.25 * a[3] + Tt * (0.2 * a[4]))))) + a[5];
            Rm += Y[k] * mech->Rk[k];
            e += Y[k] * mech->Rk[k] * (h - Tt);
        }
        const double rho = p / (Rm * Tt);
        U[c] = rho;
        U[(size_t)sout + c] = rho * u;
        U[(size_t)2 * sout + c] = rho * v;
        U[(size_t)3 * sout + c] = rho * e + 0.5 * rho * (u * u + v * v);
#pragma unroll
        for (int k = 0; k < NS - 1; ++k) U[(size_t)(4 + k) * sout + c] = rho * Y[k];
        T[c] = Tt;
    } else {
        double q[NU];
        gas_to_cons<M, NU>(w, gamma, Q, q);
#pragma unroll
        for (int f = 0; f < NU; ++f) U[(size_t)f * sout + c] = q[f];
        T[c] = w[3] / (w[0] * R);
    }
}

// ------------------------------------------------------------------ whole runs of tiny domains
// One workgroup runs all steps of a one-dimensional domain of up to RUN_CELLS cells (one
// block, one level; the models without chemistry solves): cell c on thread c, whose state
// stays in registers from the first step to the last; split fluxes and interface fluxes
// pass through LDS, the interfaces of different components on different groups of waves; the
// wave speeds and dt through LDS. The arithmetic is the stage kernel's (the same functions on
// the same operands), so the results are bitwise the same.
// Bound: the latency of a stage's dependent arithmetic and LDS trips, where one launch per
// stage paid for a launch and a chain of table reads each time (400-cell shock tube: 8.0 -> 4.2
// us per stage; 10.7 us with 256-cell tiles).
constexpr int RUN_CELLS = 1023;   // one thread per interface

// LDS bytes of a run over up to `cap` cells: RUN_CELLS takes 99 and 124 KB, one workgroup per
// CU. Kernels of half, a quarter and an eighth of that let shorter domains share a CU.
constexpr int run_lds(int nu, int cap) { return 8 * (nu * (2 * (cap + 6) + cap + 1) + 96 + 2 * (nu + 3)); }

template <int M, int NU, int CAP>
__global__ __launch_bounds__(1024) void run_kernel(RunArgs A) {
    constexpr int NS = CAP + 6, NH = CAP + 1;
    __shared__ double fp[NU * NS], fm[NU * NS], hf[NU * NH];
    __shared__ double smax[2][3][16];             // |u|+c, |v|+c, CFL bound of each wave
    __shared__ double dirs[2][NU + 3];            // Dirichlet sides: state, u, v, p
    const int d = A.order ? A.order[blockIdx.x] : (int)blockIdx.x, tid = threadIdx.x, l = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the scalars of the domain
    DevDomain D{};
    int bc[2] = {0, 0}, dir[2] = {-1, -1};
    {
        const auto take = [&](const auto& S) {
            D.nx0 = S.nx0;
            D.idx0 = S.idx0;
            D.gamma = S.gamma;
            D.R = S.R;
            D.Q = S.Q;
            D.Ea = S.Ea;
            D.k = S.k;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                bc[s] = S.bc[s];
                dir[s] = S.dir[s];
            }
        };
        if (A.dom) take(cdom(A.dom, d));
        else take(A.dom0);
    }
    const int n = D.nx0;
    const long long c = (A.blk ? A.blk[d].offset : 0) + tid;
    const bool own = tid < n;
    // interfaces: group g of m threads takes components g, g + groups, ..
    const int m = (n + 64) / 64 * 64, groups = max(1, (int)blockDim.x / m);
    const int g0 = tid / m, k0 = tid - g0 * m;
    const bool ifc = g0 < groups && k0 <= n;
    const double idx = D.idx0;
    if (tid < 2 && bc[tid] == BC_DIRICHLET) {
        double u[NU], vx, vy, pr;
        if (A.dirU) {
#pragma unroll
            for (int f = 0; f < NU; ++f) u[f] = A.dirU[(size_t)dir[tid] * (MAXF + 1) + f];
        } else {
            double q[NU];
#pragma unroll
            for (int f = 0; f < NU; ++f) q[f] = A.prim[tid][f];
            gas_to_cons<M, NU>(q, D.gamma, D.Q, u);
        }
        halo_prims<M, NU>(u, 0.0, D, (CMech*)nullptr, vx, vy, pr);
#pragma unroll
        for (int f = 0; f < NU; ++f) dirs[tid][f] = u[f];
        dirs[tid][NU] = vx;
        dirs[tid][NU + 2] = pr;
    }
    // ghosts (bit 3 side + k) that copy or mirror this cell
    unsigned gh = 0u;
    if (own)
#pragma unroll
        for (int side = 0; side < 2; ++side)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int from = bc[side] == BC_PERIODIC ? (side ? k : n - 1 - k)
                                 : bc[side] == BC_SLIPWALL ? (side ? n - 1 - k : k) : (side ? n - 1 : 0);
                if (tid == from) gh |= 1u << (3 * side + k);
            }
    double u[NU], un[NU], T = 0.0;
    auto solve = [&](int buf) {   // T and the wave speeds of the cell
        double sx = 0.0, sy = 0.0, sc = 0.0;
        if (own) {
            double cs, vx, vy;
            const unsigned st = owner_state<M, NU>(u, T, D, (CMech*)nullptr, T, cs, vx, vy);
            if (st) {
                atomicOr(A.status, st);
            } else {
                sx = fabs(vx) + cs;
                sy = fabs(vy) + cs;
                sc = sx * idx + 0.0;
            }
        }
        if (64 * w < n) {
            sx = wave_max(sx);
            sc = wave_max(sc);
            if (l == 0) {
                smax[buf][0][w] = sx;
                smax[buf][2][w] = sc;
            }
        }
    };
    const int nown = (n + 63) / 64;
    auto top = [&](int buf, int k) { return wave_max(l < nown ? smax[buf][k][l] : 0.0); };
#pragma unroll
    for (int f = 0; f < NU; ++f) u[f] = own ? A.U[(size_t)f * A.pool + c] : 1.0;
    if (own) T = A.T[c];
    solve(0);
    __syncthreads();
    double t = A.t[d];
    int cur = 0;   // buffer of the maxima of the present state
    for (int step = 0; step < A.nsteps; ++step) {
        double dt = A.tm.dt_fixed > 0.0 ? A.tm.dt_fixed : A.tm.cfl / top(cur, 2);
        if (A.tm.t_end > 0.0) {
            const double rem = A.tm.t_end - t;
            if (!(rem > 0.0)) dt = 0.0;
            else if (dt > rem) dt = rem;
        }
        t = t + dt;
        if (tid == 0 && A.dt_log && A.step0 + step < A.dt_log_cap) A.dt_log[(size_t)(A.step0 + step) * A.ndom + d] = dt;
        if (!(dt > 0.0)) continue;   // finished: state unchanged
#pragma unroll
        for (int f = 0; f < NU; ++f) un[f] = u[f];
        for (int stage = 1; stage <= 3; ++stage) {
            const double ax = top(cur, 0);
            const double ca = (stage == 1) ? 0.0 : (stage == 2) ? 0.75 : 1.0 / 3.0;
            const double cb = (stage == 1) ? 1.0 : (stage == 2) ? 0.25 : 2.0 / 3.0;
            double src_e = 0.0;
            if (own) {
                double vx, vy, pr;
                halo_prims<M, NU>(u, T, D, (CMech*)nullptr, vx, vy, pr);
                if constexpr (M == ONESTEP) {
                    const double Tc = pr / (u[0] * D.R);
                    src_e = -D.k * u[4] * exp(-D.Ea / Tc);
                }
                auto flux = [&](int f, double uf, double vn, double p, int at) {
                    split_flux<M>(uf, vn, ax, f == 1 ? p : 0.0, fp[f * NS + at], fm[f * NS + at], f == 3 ? uf + p : uf);
                };
#pragma unroll
                for (int f = 0; f < NU; ++f) flux(f, u[f], vx, pr, tid + 3);
                for (unsigned b = gh; b; b &= b - 1) {
                    const int q = __ffs(b) - 1, side = q >= 3, k = q - 3 * side, at = (side ? n + k : -1 - k) + 3;
                    const int kind = side ? bc[1] : bc[0];
#pragma unroll
                    for (int f = 0; f < NU; ++f) {
                        if (kind == BC_DIRICHLET) flux(f, dirs[side][f], dirs[side][NU], dirs[side][NU + 2], at);
                        else if (kind == BC_SLIPWALL) flux(f, f == 1 ? -u[f] : u[f], -vx, pr, at);
                        else flux(f, u[f], vx, pr, at);
                    }
                }
            }
            __syncthreads();
            if (ifc)
                for (int f = g0; f < NU; f += groups) {
                    const double* P = fp + f * NS + k0;
                    const double* Q = fm + f * NS + k0;
                    hf[f * NH + k0] = weno5(P[0], P[1], P[2], P[3], P[4]) + weno5(Q[5], Q[4], Q[3], Q[2], Q[1]);
                }
            __syncthreads();
            if (own) {
#pragma unroll
                for (int f = 0; f < NU; ++f) {
                    const double* H = hf + f * NH + tid;
                    double L = -(H[1] - H[0]) * idx;
                    if (M == ONESTEP && f == 4) L += src_e;
                    const double u0 = stage == 1 ? 0.0 : un[f];
                    u[f] = ca * u0 + cb * (u[f] + dt * L);
                }
            }
            cur ^= 1;
            solve(cur);
            __syncthreads();
        }
    }
    if (own) {
#pragma unroll
        for (int f = 0; f < NU; ++f) A.U[(size_t)f * A.pool + c] = u[f];
        A.T[c] = T;
    }
    if (tid == 0) A.t[d] = t;
}

// ------------------------------------------------------------------ launch shapes
// Workgroups per block of the restriction and ring-fill launches (a 64 x 64 fine
// block has 1024 coarse cells and 768 band cells: four workgroups of 256 threads).
constexpr int RESTRICT_SPLIT = 4;

}  // namespace janc
