// janc_kernels.hip -- launchers of the JANC step kernels (janc_kernels.h): the
// calorically perfect and one-step models here, the detailed model through the
// per-species-count launch tables of janc_species.hip.
#include <algorithm>

#include "janc_launch.h"

namespace janc {

__global__ void clear_kernel(unsigned long long* buf, int n) {
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < n; q += gridDim.x * blockDim.x) buf[q] = 0ull;
}

__global__ void zero_int_kernel(int* p) {
    if (threadIdx.x == 0) *p = 0;
}

template <int TX>
__global__ __launch_bounds__(WG) void halo_table_small_kernel(StageArgs a, int* out, int stride, int split) {
    const int ti = blockIdx.x;
    const Tile tile = quarter(a.tiles[ti / split], ti % split);
    int* row = out + (size_t)ti * stride;
    if (tile.kind == 1) halo_table_tile<8 * TX, 1>(a, ti, tile, row);
    else halo_table_tile<TX, 8>(a, ti, tile, row);
}

// ------------------------------------------------------------------ launchers
// The per-species-count tables (janc_species.hip, one translation unit per count).
const SpeciesOps* species_ops_2();
const SpeciesOps* species_ops_3();
const SpeciesOps* species_ops_4();
const SpeciesOps* species_ops_5();
const SpeciesOps* species_ops_6();
const SpeciesOps* species_ops_7();
const SpeciesOps* species_ops_8();
const SpeciesOps* species_ops_9();
const SpeciesOps* species_ops_10();
const SpeciesOps* species_ops_11();
const SpeciesOps* species_ops_12();
static_assert(JANC_NS_FIRST == 2 && JANC_NS_LAST == 12, "species tables 2 .. 12");

const SpeciesOps* species_ops(int ns) {
    switch (ns) {
        case 2: return species_ops_2();
        case 3: return species_ops_3();
        case 4: return species_ops_4();
        case 5: return species_ops_5();
        case 6: return species_ops_6();
        case 7: return species_ops_7();
        case 8: return species_ops_8();
        case 9: return species_ops_9();
        case 10: return species_ops_10();
        case 11: return species_ops_11();
        case 12: return species_ops_12();
        default: return nullptr;
    }
}

bool model_supported(int model, int ns) {
    if (model == CPG || model == ONESTEP) return true;
    return model == DETAILED && species_ops(ns) != nullptr;
}

hipError_t launch_zero_int(int* p, hipStream_t s) {
    zero_int_kernel<<<1, 64, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_clear_reduce(const Reduce& r, int which, hipStream_t s) {
    const int n = ((which < 0) ? RED_BUFS * r.stride : r.stride) * SLOT_WORDS;
    unsigned long long* p = (which < 0) ? r.buf : r.buf + (size_t)which * r.stride * SLOT_WORDS;
    clear_kernel<<<1, WG, 0, s>>>(p, n);
    return hipGetLastError();
}


hipError_t launch_stage(int model, int ns, int kind_mask, int tile_w, const StageArgs& a,
                        int first_tile, int ntiles, hipStream_t s) {
    const int owner = (first_tile == 0) ? 1 : 0;
    if (ntiles <= 0) return hipSuccess;
    if (model == CPG) return launch_stage_m<CPG, 4>(kind_mask, tile_w, a, first_tile, ntiles, owner, s);
    if (model == ONESTEP) return launch_stage_m<ONESTEP, 5>(kind_mask, tile_w, a, first_tile, ntiles, owner, s);
    const SpeciesOps* o = species_ops(ns);
    return o ? o->stage(kind_mask, tile_w, a, first_tile, ntiles, owner, s) : hipErrorInvalidValue;
}

int halo_table_stride(int tile_w, int kind_mask) {
    if (tile_w == QUARTER_TILES || tile_w == TINY_TILES) return (kind_mask & 1) ? Geom<8, 8>::NP : Geom<64, 1>::NP;
    if (tile_w == HALF_TILES) return (kind_mask & 1) ? Geom<16, 8>::NP : Geom<128, 1>::NP;
    int np2 = Geom<16, 16>::NP;
    if (tile_w == 32) np2 = Geom<32, 8>::NP;
    else if (tile_w == 64) np2 = Geom<64, 4>::NP;
    const int np1 = Geom<WG, 1>::NP;
    int n = (kind_mask & 1) ? np2 : 0;
    if (kind_mask & 2) n = max(n, np1);
    return n > 0 ? n : np2;
}

hipError_t launch_halo_table(int tile_w, const StageArgs& a, int* out, int stride, hipStream_t s) {
    if (a.ntiles <= 0) return hipSuccess;
    if (tile_w == QUARTER_TILES) halo_table_small_kernel<8><<<SMALL_SPLIT * a.ntiles, WG, 0, s>>>(a, out, stride, SMALL_SPLIT);
    else if (tile_w == TINY_TILES) halo_table_small_kernel<8><<<a.ntiles, WG, 0, s>>>(a, out, stride, 1);
    else if (tile_w == HALF_TILES) halo_table_small_kernel<16><<<a.ntiles, WG, 0, s>>>(a, out, stride, 1);
    else if (tile_w == 32) halo_table_kernel<32, 8><<<a.ntiles, WG, 0, s>>>(a, out, stride);
    else if (tile_w == 64) halo_table_kernel<64, 4><<<a.ntiles, WG, 0, s>>>(a, out, stride);
    else halo_table_kernel<16, 16><<<a.ntiles, WG, 0, s>>>(a, out, stride);
    return hipGetLastError();
}

// Largest 1-D domain that runs in one workgroup. Measured, us per step of launches per stage /
// of the run. 64 domains: gas without chemistry 50 cells 21.4 / 7.7, 400 cells 21.6 / 13.1, 1023
// cells 22.3 / 20.2; one-step 256 cells 19.8 / 12.8, 511 cells 25.4 / 16.0, 704 cells 25.3 / 21.2.
// One domain alone, in long calls: 400 cells 19.2 / 12.8, 700 cells 18.8 / 16.9, 1023 cells
// 17.9 / 19.7; one-step 511 cells 20.5 / 15.7, 700 cells 19.3 / 20.7. There the largest sizes
// are 4 to 12 % faster in launches per stage, but a call of one step is not (1023 cells 44 / 37,
// allocation-free 67 / 34; one-step 700 cells 48 / 38; even at 8 to 16 steps).
// (Two-dimensional domains were slower from 16 x 16 cells on.)
int run_cells(int model) { return model == CPG ? RUN_CELLS : model == ONESTEP ? 704 : 0; }

// LDS capacity (cells) of the kernel for the largest domain. (511 only with more domains than
// CUs: alone, a 400-cell tube took 1279 us in place of 1268.)
int run_cap(int cells, bool many) { return cells <= 127 ? 127 : cells <= 255 ? 255 : cells <= 511 && many ? 511 : RUN_CELLS; }

// Threads of a workgroup: whole groups of waves for the interfaces of up to all components, and
// no more groups than the chip's wave slots (16 per CU at these registers) have room for: with
// fewer slots than groups, the components of one domain in turn and more domains at once.
RunShape run_shape(int model, int cells, int ndom, int cus) {
    const int nu = model == CPG ? 4 : 5, m = (cells + 64) / 64 * 64;
    RunShape r;
    r.cap = run_cap(cells, ndom > cus);
    const int fit = 160 * 1024 / run_lds(nu, r.cap);   // workgroups of a CU by their LDS
    int groups = std::min(nu, 1024 / m);
    while (groups > 1 && std::min(fit, 1024 / (m * groups)) < fit &&
           (long long)ndom > (long long)cus * std::min(fit, 1024 / (m * groups)))
        --groups;
    r.threads = std::max((cells + 63) / 64 * 64, m * groups);
    const long long at_once = (long long)cus * std::min(fit, 1024 / r.threads);
    r.rounds = (int)((ndom + at_once - 1) / at_once);
    return r;
}

template <int M, int NU>
void launch_run_m(const RunArgs& a, int count, const RunShape& r, hipStream_t s) {
    switch (r.cap) {
        case 127: run_kernel<M, NU, 127><<<count, r.threads, 0, s>>>(a); break;
        case 255: run_kernel<M, NU, 255><<<count, r.threads, 0, s>>>(a); break;
        case 511: run_kernel<M, NU, 511><<<count, r.threads, 0, s>>>(a); break;
        default: run_kernel<M, NU, RUN_CELLS><<<count, r.threads, 0, s>>>(a);
    }
}

hipError_t launch_run(int model, const RunArgs& a, int count, const RunShape& r, hipStream_t s) {
    if (run_cells(model) == 0) return hipErrorInvalidValue;
    if (model == CPG) launch_run_m<CPG, 4>(a, count, r, s);
    else launch_run_m<ONESTEP, 5>(a, count, r, s);
    return hipGetLastError();
}

hipError_t launch_init(int model, int ns, const StageArgs& a, hipStream_t s) {
    if (a.ntiles <= 0) return hipSuccess;
    const int per = init_per(a.ntiles), n = (a.ntiles + per - 1) / per;
    if (model == CPG) init_kernel<CPG, 4><<<n, WG, 0, s>>>(a, per);
    else if (model == ONESTEP) init_kernel<ONESTEP, 5><<<n, WG, 0, s>>>(a, per);
    else {
        const SpeciesOps* o = species_ops(ns);
        return o ? o->init(a, s) : hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_chem(int model, int ns, int tile_w, const StageArgs& a, hipStream_t s) {
    (void)tile_w;
    if (model != DETAILED || a.ntiles <= 0) return hipSuccess;
    const SpeciesOps* o = species_ops(ns);
    return o ? o->chem(a, s) : hipErrorInvalidValue;
}


hipError_t launch_restrict(int model, int ns, const StageArgs& a, const int* fine_blocks, int nfine,
                           hipStream_t s) {
    if (nfine <= 0) return hipSuccess;
    const dim3 grid(nfine, RESTRICT_SPLIT);
    if (model == CPG) restrict_kernel<CPG, 4><<<grid, WG, 0, s>>>(a, fine_blocks);
    else if (model == ONESTEP) restrict_kernel<ONESTEP, 5><<<grid, WG, 0, s>>>(a, fine_blocks);
    else {
        const SpeciesOps* o = species_ops(ns);
        return o ? o->restrict_fine(a, fine_blocks, nfine, s) : hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_ring_fill(int model, int ns, const StageArgs& a, const int* ring_blocks, int nring,
                            hipStream_t s) {
    if (nring <= 0) return hipSuccess;
    const dim3 grid(nring, RESTRICT_SPLIT);
    if (model == CPG) ring_fill_kernel<4><<<grid, WG, 0, s>>>(a, ring_blocks);
    else if (model == ONESTEP) ring_fill_kernel<5><<<grid, WG, 0, s>>>(a, ring_blocks);
    else {
        const SpeciesOps* o = species_ops(ns);
        return o ? o->ring_fill(a, ring_blocks, nring, s) : hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_prim_to_cons(int model, int ns, const DevMech* mech, double gamma, double R,
                               double Q, long long n, const double* W, double* U, double* T,
                               long long sin, long long sout, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int nb = (int)((n + WG - 1) / WG);
    if (model == CPG) prim_to_cons_kernel<CPG, 4><<<nb, WG, 0, s>>>(mech, gamma, R, Q, n, W, U, T, sin, sout);
    else if (model == ONESTEP) prim_to_cons_kernel<ONESTEP, 5><<<nb, WG, 0, s>>>(mech, gamma, R, Q, n, W, U, T, sin, sout);
    else {
        const SpeciesOps* o = species_ops(ns);
        return o ? o->prim_to_cons(mech, n, W, U, T, sin, sout, s) : hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace janc
