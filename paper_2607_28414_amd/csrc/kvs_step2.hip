// Two FDTD steps per launch for one context (the tile code is in
// kvs_step2_tile.hpp).  The first pblocks blocks copy the launch's input state
// (the previous step's result) at the probe cells, as in the one-step kernel;
// the remaining blocks are the tiles, numbered XCD by XCD.
#include <hip/hip_ext.h>

#include <cmath>

#include "kvs_step2_tile.hpp"

namespace {

template <typename T, bool HET, bool VISC, bool FORCE, bool PEAK, int WX, int R>
__global__ __launch_bounds__(64 * WX * R) void step2_kernel(const Step2Args<T> A2, const Step2Peaks<T> pk) {
    __shared__ __align__(16) T lds[Step2Tile<T, HET, VISC, WX, R>::LDS];
    const StepArgs<T>& a = A2.a;
    if ((int)blockIdx.x < a.pblocks) {
        step2_probe(A2, (long long)blockIdx.x * (64 * WX * R) + threadIdx.y * (64 * WX) + threadIdx.x);
        return;
    }
    const int B = a.gx * a.gy * a.gz;
    const int b = (int)blockIdx.x - a.pblocks;
    const int t = a.remap ? tile_of(b, B) : b;
    step2_tile<T, HET, VISC, FORCE, PEAK, WX, R>(A2, &pk, lds, t % a.gx, (t / a.gx) % a.gy, t / (a.gx * a.gy));
}

// Tile and z segment of a launch: the ones whose blocks finish first by a model
// of the march, rounds of resident blocks x (planes + 3 to fill the queues) x the
// time of a plane, the larger of a floor (the latency of loads, barrier and LDS)
// and the wavefronts' work on a CU, one unit per wavefront and update.  Unit 80 ns
// (256^3 heterogeneous: 28 units, 2.2 us a plane), floor 9 units (0.7 us: small
// grids).  Shapes whose march is short (kShortMarch planes) are compared with
// kPlaneStart units added to the work of a plane instead: without, 64 x 8 was taken
// at 128^3 heterogeneous (21 + 3 planes of 14 units, 22.0 us a step) where 128 x 8
// (11 + 3 planes of 28) takes 19.7 and 64 x 16 (9 + 3 of 30) 20.1; 90 x 65 x 269
// 21.9 / 18.0 (128 x 8); 100 x 165 x 71 uniform 13.1 / 10.0 (64 x 16).  Over 252
// viscous grids up to 256^3 6 to 9 units gave 1.036 to 1.039x in the geometric
// mean and none slower, 12 and more made some slower.  In a long march the start
// is hidden: 384 x 384 x 512 with force, 513 planes of 192 x 5 or 420 of 64 x 16,
// takes 0.75 ms a step with the former and 0.85 with the latter, which the added
// units would choose.
constexpr double kPlaneFloor = 9.0, kPlaneStart = 6.0;
constexpr long long kShortMarch = 100;

struct Step2Plan {
    double cost = 1e300, short_cost = 1e300;
    long long march = 0;
    int shape = -1, gx = 1, gy = 1, kchunk = 1;
};

// The plans of the shapes offered so far: the best by either cost.
struct Step2Plans {
    Step2Plan by_work, by_start;
    const Step2Plan& best() const { return by_work.march <= kShortMarch ? by_start : by_work; }
};

// only: the shape asked for, where the context offers it, else -1
void consider(Step2Plans& plans, int shape, int only, const kvs_grid& g, int cap, int zchunk) {
    if (!step2_offers(shape, g.ny) || (only >= 0 && shape != only)) return;
    const int planes = (int)g.nz - 2;
    const int gx = overlap_tiles((int)g.nx, 64 * kStep2Wx[shape]), gy = overlap_tiles((int)g.ny, kStep2Rows[shape]);
    const double units = step2_units(shape);
    const int per_cu = std::max(1, cap / 256);
    const int max_seg = std::max(1, planes / 2);
    Step2Plan p;
    for (int seg = 1; seg <= max_seg; ++seg) {
        int chunk = (planes + seg - 1) / seg;
        if (zchunk > 0) chunk = std::min(zchunk, planes);
        const long long blocks = (long long)gx * gy * ((planes + chunk - 1) / chunk);
        const long long rounds = (blocks + cap - 1) / cap;
        const double work = units * (double)std::min<long long>(per_cu, (blocks + 255) / 256);
        const long long march = rounds * (chunk + 3);
        const double cost = (double)march * std::max(kPlaneFloor, work);
        if (cost < p.cost * 0.999) p = {cost, (double)march * (kPlaneStart + work), march, shape, gx, gy, chunk};
        if (zchunk > 0) break;
    }
    if (p.cost < plans.by_work.cost * 0.999) plans.by_work = p;
    if (p.short_cost < plans.by_start.short_cost * 0.999) plans.by_start = p;
}

template <typename T, bool HET, bool VISC, bool FORCE, int S, bool PEAK = false>
hipError_t launch_shape(kvs_ctx* c, Step2Args<T>& A2, const Step2Peaks<T>& pk) {
    constexpr int WX = kStep2Wx[S], R = kStep2Rows[S];
    StepArgs<T>& a = A2.a;
    auto kern = step2_kernel<T, HET, VISC, FORCE, PEAK, WX, R>;
    a.gz = (a.nz - 2 + a.kchunk - 1) / a.kchunk;
    a.pblocks = a.np > 0 && (a.pout || A2.pmid) ? (int)((a.np + 64 * WX * R - 1) / (64 * WX * R)) : 0;
    c->launched_tile[0] = 64 * WX;
    c->launched_tile[1] = R;
    c->launched_tile[2] = a.kchunk;
    const int blocks = a.gx * a.gy * a.gz + a.pblocks;
    if (c->launch_ev[0])
        hipExtLaunchKernelGGL(kern, dim3(blocks), dim3(64 * WX, R), 0, c->stream, c->launch_ev[0], c->launch_ev[1], 0,
                              A2, pk);
    else
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(64 * WX, R), 0, c->stream, A2, pk);
    return hipGetLastError();
}

template <typename T, bool HET, bool VISC, bool FORCE, int S>
int shape_cap() {
    constexpr int WX = kStep2Wx[S], R = kStep2Rows[S];
    static const int cap = resident_blocks(step2_kernel<T, HET, VISC, FORCE, false, WX, R>, 64 * WX * R);
    return cap;
}

template <typename T, bool HET, bool VISC, bool FORCE>
hipError_t launch_medium(kvs_ctx* c, Step2Args<T>& A2, const Step2Peaks<T>& pk) {
    const kvs_grid& g = c->grid;
    Step2Plans plans;
    const int want = c->step2_tile;
    const bool has = sizeof(T) == 8 ? want == 2 : want >= 0 && (pk.n == 0 || want == 1 || want == 2);
    const int only = has && step2_offers(want, g.ny) ? want : -1;
    // peak maps: the shape that fits most row lengths (FP32: 64 x 16), compiled
    // for them alone; 64 x 8 where the grid's rows rule that out.  Resident blocks
    // as without maps, which holds but for 64 x 8 heterogeneous viscous (one block
    // on a CU for two); rounds x blocks on a CU come out the same there
    if constexpr (sizeof(T) == 4) {
        if (pk.n > 0) consider(plans, 1, only, g, shape_cap<T, HET, VISC, FORCE, 1>(), c->step2_zchunk);
    }
    if (pk.n > 0 && plans.by_work.shape < 0) consider(plans, 2, only, g, shape_cap<T, HET, VISC, FORCE, 2>(), c->step2_zchunk);
    if (pk.n > 0) {
        const Step2Plan& p = plans.best();
        A2.a.gx = p.gx;
        A2.a.gy = p.gy;
        A2.a.kchunk = p.kchunk;
        if constexpr (sizeof(T) == 4) {
            if (p.shape == 1) return launch_shape<T, HET, VISC, FORCE, 1, true>(c, A2, pk);
        }
        return launch_shape<T, HET, VISC, FORCE, 2, true>(c, A2, pk);
    }
    if constexpr (sizeof(T) == 4) {
        consider(plans, 0, only, g, shape_cap<T, HET, VISC, FORCE, 0>(), c->step2_zchunk);
        consider(plans, 1, only, g, shape_cap<T, HET, VISC, FORCE, 1>(), c->step2_zchunk);
        consider(plans, 3, only, g, shape_cap<T, HET, VISC, FORCE, 3>(), c->step2_zchunk);
    }
    consider(plans, 2, only, g, shape_cap<T, HET, VISC, FORCE, 2>(), c->step2_zchunk);
    const Step2Plan& p = plans.best();
    A2.a.gx = p.gx;
    A2.a.gy = p.gy;
    A2.a.kchunk = p.kchunk;
    if constexpr (sizeof(T) == 4) {
        if (p.shape == 0) return launch_shape<T, HET, VISC, FORCE, 0>(c, A2, pk);
        if (p.shape == 1) return launch_shape<T, HET, VISC, FORCE, 1>(c, A2, pk);
        if (p.shape == 3) return launch_shape<T, HET, VISC, FORCE, 3>(c, A2, pk);
    }
    return launch_shape<T, HET, VISC, FORCE, 2>(c, A2, pk);
}

template <typename T, bool HET, bool VISC>
hipError_t launch_force(kvs_ctx* c, Step2Args<T>& A2, const Step2Peaks<T>& pk) {
    return A2.a.gn != T(0) || A2.gn2 != T(0) ? launch_medium<T, HET, VISC, true>(c, A2, pk)
                                             : launch_medium<T, HET, VISC, false>(c, A2, pk);
}

template <typename T>
hipError_t launch_t(kvs_ctx* c, double gn, double gn2) {
    const kvs_grid& g = c->grid;
    Step2Args<T> A2{};
    StepArgs<T>& a = A2.a;
    const int nb = 1 - c->cur;
    a.u = static_cast<const T*>(c->u[c->cur]);
    a.w = static_cast<const T*>(c->w[c->cur]);
    a.un = static_cast<T*>(c->u[nb]);
    a.wn = static_cast<T*>(c->w[nb]);
    a.G = static_cast<const T*>(c->G);
    a.eta = static_cast<const T*>(c->eta);
    a.crho = static_cast<const T*>(c->crho);
    a.FS = static_cast<const T*>(c->FS);
    a.N = c->N;
    a.nx = (int)g.nx;
    a.ny = (int)g.ny;
    a.nz = (int)g.nz;
    a.L = c->sponge_cells;
    a.invL = a.L > 0 ? T(1.0 / a.L) : T(0);
    a.ihx2 = T(1.0 / (g.hx * g.hx));
    a.ihy2 = T(1.0 / (g.hy * g.hy));
    a.ihz2 = T(1.0 / (g.hz * g.hz));
    a.G0 = T(c->G0);
    a.eta_dt0 = T(c->eta0 / c->dt);
    a.crho0 = T(c->dt * c->dt / c->rho0);
    a.inv_dt = T(1.0 / c->dt);
    a.gn = T(gn);
    A2.gn2 = T(gn2);
    a.half_dt_smax = T(0.5 * c->sigma_max * c->dt);
    a.remap = c->step_remap;
    if (c->nprobes > 0) {
        a.pcells = reinterpret_cast<const long long*>(c->probe_cells);
        a.pout = c->probe_fused_out;
        a.np = c->nprobes;
        a.pcomp = c->probe_comp;
        A2.rowtab = c->probe_rowtab;
        A2.ptab = c->probe_ptab;
        A2.pmid = c->probe_mid_out;
    }
    Step2Peaks<T> pk{};
    pk.n = c->npeak;
    pk.mid = c->npeak > 0 ? static_cast<T*>(c->peak) + c->peak_cells : nullptr;
    for (int p = 0; p < c->npeak; ++p) {
        pk.axis[p] = c->peak_axis[p];
        pk.index[p] = (int)c->peak_index[p];
        pk.n1[p] = c->peak_axis[p] == 0 ? a.ny : a.nx;
        pk.off[p] = c->peak_off[p];
    }
    if (c->hetero) return c->viscous ? launch_force<T, true, true>(c, A2, pk) : launch_force<T, true, false>(c, A2, pk);
    return c->viscous ? launch_force<T, false, true>(c, A2, pk) : launch_force<T, false, false>(c, A2, pk);
}

}  // namespace

bool kvs_step2_supported(const kvs_ctx* c) {
    // wherever the launch can be made: cell offsets within a field are 32-bit, byte
    // offsets within a plane too; FP64 has one tile shape.  us per step against
    // the tuned one-step kernel, heterogeneous viscous FP32, without and with three
    // peak planes: 500 x 500 x 640 1322 / 2266, 1366 / 2276; 512 x 512 x 640, whose
    // planes are 1 MiB apart, 1813 / 1830, 1845 / 1863; 512 x 256 x 512 684 / 744,
    // 692 / 753; of 340 contexts of every medium, precision, with and without
    // force, none slower than before two steps shared a launch
    const int64_t plane = c->grid.nx * c->grid.ny * (c->prec == KVS_FP32 ? 4 : 8);
    return c->pml_cells == 0 && c->N < ((int64_t)1 << 31) && plane < ((int64_t)1 << 32) - 4096 &&
           (c->nprobes == 0 || c->probe_rows_ok) && (c->prec == KVS_FP32 || step2_offers(2, c->grid.ny));
}

bool kvs_step2_reported(const kvs_ctx* c) {
    return kvs_step2_supported(c) && c->prec == KVS_FP32 && c->viscous && c->npeak == 0 && c->grid.nx <= 256;
}

hipError_t kvs_launch_step2(kvs_ctx* c, double gn, double gn2) {
    return c->prec == KVS_FP32 ? launch_t<float>(c, gn, gn2) : launch_t<double>(c, gn, gn2);
}
