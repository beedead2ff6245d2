// One FDTD step per launch with the march of the two-step tile
// (kvs_step2_tile.hpp) cut down to its first stage, for the contexts whose
// steps cannot be paired: those with an absorbing layer.  The same operations
// in the same order as kvs_step_tile.hpp: bitwise the same state.
//
// A block of 64 WX x R threads covers that many cells of every plane of a z
// segment (tiles side by side from the row's first node on, so that rows of
// whole lines are stored as whole lines, walls as the 0 they hold; the input
// staged in LDS with one more cell on each side, fields of a cell together), z
// neighbours in rings of registers (the march is unrolled by three: nothing is
// moved and plane k + 2 is loaded into the registers that plane k - 1 leaves),
// one barrier per plane, one copy of the march for wavefronts with and without
// halo work.  60 B per cell and step (heterogeneous viscous) bound it: 190 x
// 161 x 175 69 us a step (4.7 TB/s) against 96 us for the tiled kernel.  With
// the layer pass, us per step, tiled kernel and this one: 190 x 161 x 175
// heterogeneous 197 / 171, uniform 173 / 147; 128^3 92.0 / 82.3; 101 x 90 x 160
// 72.6 / 60.5; 60^3 28.3 / 26.7; 230 x 150 x 150 195 / 170; 256^3 443 / 434.
#include <hip/hip_ext.h>

#include "kvs_step2_tile.hpp"

namespace {

template <typename T, bool HET, bool VISC, bool FORCE, int WX, int R>
__device__ __forceinline__ void step1_tile(const StepArgs<T>& a, T* lds, int bx, int by, int bz) {
    using S = Step2Tile<T, HET, VISC, WX, R>;
    static_assert(R >= 4 && 2 * R <= 64 && 64 * WX * R <= 1024, "halo rows, columns by a row of their own");
    constexpr int TX = S::TX, W = S::W, NU = S::NU, NQ = S::NQ, QG = NU, P = S::CELLS;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int kb = 1 + bz * a.kchunk;
    const int ke = min(nz - 1, kb + a.kchunk);  // planes kb .. ke - 1
    const int tx = threadIdx.x, ty = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int i = bx * TX + tx, j = 1 + by * R + ty;
    const bool act = i >= 1 && i <= nx - 2 && j <= ny - 2;
    const int sxy = nx * ny;
    // a lane beyond the grid reads cell 0 of the plane, which no cell uses
    const unsigned col = i < nx && j < ny ? (unsigned)(i + nx * j) * (unsigned)sizeof(T) : 0u;  // bytes
    // Halo: the rows below and above the tile by its first and last row, the
    // columns (2 R cells) by the first wavefront of row 1.
    const int hj = ty == 0 ? j - 1 : j + 1;
    const int hpos = ty == 0 ? tx + 1 : (R + 1) * W + tx + 1;
    const unsigned hcol = i < nx && hj < ny ? (unsigned)(i + nx * hj) * (unsigned)sizeof(T) : 0u;
    const bool right = tx >= R, creal = tx < 2 * R;
    const int crow = right ? tx - R : tx;
    const int ci = right ? bx * TX + TX : bx * TX - 1, cj = 1 + by * R + crow;
    const int cpos = creal ? (crow + 1) * W + (right ? TX + 1 : 0) : 0;  // 0: a corner, never read
    const unsigned ccol = creal && ci >= 0 && ci < nx && cj < ny ? (unsigned)(ci + nx * cj) * (unsigned)sizeof(T) : 0u;
    const int pos = (ty + 1) * W + tx + 1;

    auto stride = [&]() {  // opaque, see step2_tile
        long long n = a.N;
        asm volatile("" : "+s"(n));
        return n;
    };
    auto field = [&](int f, long long n, size_t o) {
        return glob(f == QG && HET ? a.G + o : f < 3 ? a.u + f * n + o : a.w + (f - 3) * n + o);
    };
    const gptr<const T> crho_g = glob(a.crho), eta_g = glob(a.eta);
    auto plane_of = [&](int k) { return (size_t)min(k, nz - 1) * (size_t)sxy; };
    const T rxy = a.L > 0 ? max(ramp<T>(i, nx, a.L, a.invL), ramp<T>(j, ny, a.L, a.invL)) : T(0);
    const T ihx2 = a.ihx2, ihy2 = a.ihy2, ihz2 = a.ihz2;
    const T h2x = T(2) * ihx2, h2y = T(2) * ihy2, h2z = T(2) * ihz2;
    const T gx0 = HET ? T(0) : a.G0 * ihx2, gy0 = HET ? T(0) : a.G0 * ihy2, gz0 = HET ? T(0) : a.G0 * ihz2;

    auto march = [&](auto halo_tag) {
        constexpr bool HALO = decltype(halo_tag)::value;  // row or column cells to stage
        const unsigned hoff = ty == 1 ? ccol : hcol;
        const int hp = ty == 1 ? cpos : hpos;
        T z0[NQ], z1[NQ], z2[NQ], h[NQ];
        T wv[3] = {T(0), T(0), T(0)}, fs[3] = {T(0), T(0), T(0)};
        T crho = a.crho0, eta = T(0), fz = T(0);  // fz: z- face of the plane to come
#pragma unroll
        for (int f = 0; f < NQ; ++f) {
            z0[f] = *at_byte(field(f, a.N, plane_of(kb - 1)), col);
            z1[f] = *at_byte(field(f, a.N, plane_of(kb)), col);
            z2[f] = *at_byte(field(f, a.N, plane_of(kb + 1)), col);
        }
        auto load_halo = [&](int k) {
            if constexpr (HALO) {
                const size_t o = plane_of(k);
                const long long n = stride();
                const unsigned l = lane_byte(hoff);
#pragma unroll
                for (int f = 0; f < NQ; ++f) h[f] = *at_byte(field(f, n, o), l);
            }
        };
        auto load_cell = [&](int k, unsigned l) {  // what is read at the cell itself only
            const size_t o = plane_of(k);
            const long long n = stride();
            if constexpr (HET) {
                crho = __builtin_nontemporal_load(at_byte(crho_g + o, l));
                if constexpr (VISC) eta = __builtin_nontemporal_load(at_byte(eta_g + o, l));
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                if constexpr (!VISC) wv[c] = *at_byte(glob(a.w) + c * n + o, l);
                if constexpr (FORCE) fs[c] = __builtin_nontemporal_load(at_byte(glob(a.FS) + c * n + o, l));
            }
        };
        load_cell(kb, col);
        load_halo(kb);
        if constexpr (HET) fz = face_modulus(z1[QG], z0[QG], h2z);
        auto plane = [&](const int k, T(&zm)[NQ], T(&zc)[NQ], T(&zp)[NQ]) {
            T* const b0 = lds + (k & 1) * S::SN;
            lds_put<T, NQ>(b0, P, pos, zc);
            if constexpr (HALO) lds_put<T, NQ>(b0, P, hp, h);
            load_halo(k + 1);
            lds_barrier();
            T c1 = T(1), c2 = crho;
            if (a.L > 0) {
                const T s = a.half_dt_smax * max(rxy, ramp<T>(k, nz, a.L, a.invL));
                const T inv1ps = rcp_fast<T>(T(1) + s);
                c1 = (T(1) - s) * inv1ps;
                c2 = crho * inv1ps;
            }
            const T e = !VISC ? T(0) : HET ? eta * a.inv_dt : a.eta_dt0;
            T acc[3], lap[3];
            {
                T m[NQ], p[NQ];
                lds_get<T, NQ>(b0, P, pos - 1, m);
                lds_get<T, NQ>(b0, P, pos + 1, p);
                const T fm = HET ? face_modulus(zc[HET ? QG : 0], m[HET ? QG : 0], h2x) : gx0;
                const T fp = HET ? face_modulus(zc[HET ? QG : 0], p[HET ? QG : 0], h2x) : gx0;
                first_axis<T, VISC>(zc, m, p, fm, fp, acc, lap);
            }
            {
                T m[NQ], p[NQ];
                lds_get<T, NQ>(b0, P, pos - W, m);
                lds_get<T, NQ>(b0, P, pos + W, p);
                const T fm = HET ? face_modulus(zc[HET ? QG : 0], m[HET ? QG : 0], h2y) : gy0;
                const T fp = HET ? face_modulus(zc[HET ? QG : 0], p[HET ? QG : 0], h2y) : gy0;
                second_axis<T, VISC>(zc, m, p, fm, fp, ihx2, ihy2, acc, lap);
            }
            const T fn = HET ? face_modulus(zc[HET ? QG : 0], zp[HET ? QG : 0], h2z) : gz0;
            third_axis<T, VISC>(zc, zm, zp, HET ? fz : gz0, fn, ihz2, acc, lap);
            fz = fn;
            T uo[3], wo[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const T uc = zc[c];
                T wc = wv[c];
                if constexpr (VISC) {
                    wc = zc[3 + c];
                    acc[c] = fma_t(e, lap[c], acc[c]);
                }
                if constexpr (FORCE) acc[c] = fma_t(a.gn, fs[c], acc[c]);
                const T wnew = fma_t(c1, wc, c2 * acc[c]);
                wo[c] = act ? wnew : T(0);
                uo[c] = act ? uc + wnew : T(0);
            }
            {
                const size_t o = plane_of(k + 2);
                const long long st = stride();
                const unsigned l = lane_byte(col);
                load_cell(k + 1, l);
#pragma unroll
                for (int n = 0; n < NQ; ++n) zm[n] = *at_byte(field(n, st, o), l);
            }
            const size_t o = (size_t)k * (size_t)sxy;
            const long long n = stride();
            const unsigned bytes = (unsigned)sxy * (unsigned)sizeof(T), l = i < nx && j <= ny - 2 ? col : kNoStore;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                store_plane(a.wn + c * n + o, bytes, l, wo[c]);
                store_plane(a.un + c * n + o, bytes, l, uo[c]);
            }
        };
        for (int k = kb;;) {
            plane(k, z0, z1, z2);
            if (++k >= ke) break;
            plane(k, z1, z2, z0);
            if (++k >= ke) break;
            plane(k, z2, z0, z1);
            if (++k >= ke) break;
        }
    };
    if (ty == 0 || ty == R - 1 || (ty == 1 && tx < 64))
        march(std::integral_constant<bool, true>{});
    else
        march(std::integral_constant<bool, false>{});
}

template <typename T, bool HET, bool VISC, bool FORCE, int WX, int R>
__global__ __launch_bounds__(64 * WX * R) void step1_kernel(const StepArgs<T> a) {
    __shared__ __align__(16) T lds[2 * Step2Tile<T, HET, VISC, WX, R>::SN];
    if ((int)blockIdx.x < a.pblocks) {
        Step2Args<T> A2{};
        A2.a = a;
        step2_probe(A2, (long long)blockIdx.x * (64 * WX * R) + threadIdx.y * (64 * WX) + threadIdx.x);
        return;
    }
    const int B = a.gx * a.gy * a.gz;
    const int b = (int)blockIdx.x - a.pblocks;
    const int t = a.remap ? tile_of(b, B) : b;
    step1_tile<T, HET, VISC, FORCE, WX, R>(a, lds, t % a.gx, (t / a.gx) % a.gy, t / (a.gx * a.gy));
}

template <bool HET, bool VISC, bool FORCE, int WX, int R>
hipError_t launch(kvs_ctx* c, StepArgs<float> a) {
    auto kern = step1_kernel<float, HET, VISC, FORCE, WX, R>;
    static const int cap = resident_blocks(kern, 64 * WX * R);
    a.gx = (a.nx - 1 + 64 * WX - 1) / (64 * WX);  // the last node, a wall, needs no tile of its own
    a.gy = (a.ny - 2 + R - 1) / R;
    a.kchunk = choose_kchunk(a.gx * a.gy, a.nz - 2, cap);
    a.gz = (a.nz - 2 + a.kchunk - 1) / a.kchunk;
    a.pblocks = a.pout ? (int)((a.np + 64 * WX * R - 1) / (64 * WX * R)) : 0;
    c->launched_tile[0] = 64 * WX;
    c->launched_tile[1] = R;
    c->launched_tile[2] = a.kchunk;
    const int blocks = a.gx * a.gy * a.gz + a.pblocks;
    if (c->launch_ev[0])
        hipExtLaunchKernelGGL(kern, dim3(blocks), dim3(64 * WX, R), 0, c->stream, c->launch_ev[0], c->launch_ev[1], 0, a);
    else
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(64 * WX, R), 0, c->stream, a);
    return hipGetLastError();
}

// Large grids: the narrowest tile that spans the row (its last node needs no
// thread): such a tile has no column halo.  190 x 161 x 175, us per step with the
// layer pass: 192 x 5 171, 256 x 4 176, 64 x 8 179, 128 x 8 192; 128^3: 128 x 8 82,
// 64 x 8 83, 256 x 4 86; 256^3: 256 x 4 427, 128 x 8 437, 64 x 8 461.  Below
// kRowNodes nodes there are too few such blocks, and blocks of 1024 threads
// march slower than those of 512: 64 x 8.  138 x 65 x 15: 192 x 5 35.0, 64 x 8
// 27.7; 120 x 98 x 31: 128 x 8 31.0, 25.8; 203 x 97 x 29: 256 x 4 40.3, 34.4;
// 171 x 114 x 71 (1.4 M nodes): 192 x 5 45.2, 47.2; 96 x 193 x 93: 52.7, 55.2.
constexpr long long kRowNodes = 1200000;
template <bool HET, bool VISC, bool FORCE>
hipError_t launch_rows(kvs_ctx* c, const StepArgs<float>& a) {
    const int by_rule = a.N < kRowNodes || a.nx <= 65 ? 1 : a.nx <= 129 ? 2 : a.nx <= 193 ? 3 : 4;
    switch (c->march_tile > 0 ? c->march_tile : by_rule) {
        case 1: return launch<HET, VISC, FORCE, 1, 8>(c, a);
        case 2: return launch<HET, VISC, FORCE, 2, 8>(c, a);
        case 3: return launch<HET, VISC, FORCE, 3, 5>(c, a);
        default: return launch<HET, VISC, FORCE, 4, 4>(c, a);
    }
}

template <bool HET, bool VISC>
hipError_t launch_force(kvs_ctx* c, const StepArgs<float>& a) {
    return a.gn != 0.f ? launch_rows<HET, VISC, true>(c, a) : launch_rows<HET, VISC, false>(c, a);
}

}  // namespace

bool kvs_step1_offered(const kvs_ctx* c) {
    // rows of one tile: 320 x 200 x 200 in two of 256 took 366 us against 333 of
    // the tiled kernel.  Byte offsets within a plane are 32-bit.
    return c->grid.nx <= 257 && c->pml_cells > 0 && c->prec == KVS_FP32 && c->N < ((int64_t)1 << 31) &&
           c->grid.nx * c->grid.ny < ((int64_t)1 << 30) - 1024;
}

// On small grids a step is a short chain of launches, loads and barriers, and
// where a thread has little to do besides, the tiled kernel's smaller blocks
// end first.  us per step with the layer pass, march and tiled kernel: lossless
// 118 x 14 x 61 23.1 / 21.9, 33 x 29 x 104 21.7 / 20.6, 105 x 31 x 51 20.6 / 19.7;
// heterogeneous with force on the step 138 x 65 x 15 27.7 / 26.1, 256 x 24 x 20
// 25.7 / 24.3; viscous without, 186 x 25 x 12 22.8 / 23.8, 100 x 44 x 14 21.7 / 22.6;
// lossless 60 x 90 x 59 21.8 / 24.9.  Of 220 grids of 10^3 to 6 10^6 nodes two are
// more than 2 % slower with the march than with the tiled kernel by this rule
// (4 and 3 %); with tiles that span the row on all of them 54 were, by up to 25 %.
constexpr int64_t kMarchNodes = 250000;
bool kvs_step1_applies(const kvs_ctx* c, double gn) {
    if (!kvs_step1_offered(c) || c->march_tile == 0) return false;
    if (c->march_tile > 0) return true;
    if (c->step1_use >= 0) return c->step1_use == 1;
    return c->N >= kMarchNodes || (c->viscous && !(c->hetero && gn != 0.0));
}

hipError_t kvs_launch_step1(kvs_ctx* c, double gn) {
    const kvs_grid& g = c->grid;
    StepArgs<float> a{};
    const int nb = 1 - c->cur;
    a.u = static_cast<const float*>(c->u[c->cur]);
    a.w = static_cast<const float*>(c->w[c->cur]);
    a.un = static_cast<float*>(c->u[nb]);
    a.wn = static_cast<float*>(c->w[nb]);
    a.G = static_cast<const float*>(c->G);
    a.eta = static_cast<const float*>(c->eta);
    a.crho = static_cast<const float*>(c->crho);
    a.FS = static_cast<const float*>(c->FS);
    a.N = c->N;
    a.nx = (int)g.nx;
    a.ny = (int)g.ny;
    a.nz = (int)g.nz;
    a.L = c->sponge_cells;
    a.invL = a.L > 0 ? float(1.0 / a.L) : 0.f;
    a.ihx2 = float(1.0 / (g.hx * g.hx));
    a.ihy2 = float(1.0 / (g.hy * g.hy));
    a.ihz2 = float(1.0 / (g.hz * g.hz));
    a.G0 = float(c->G0);
    a.eta_dt0 = float(c->eta0 / c->dt);
    a.crho0 = float(c->dt * c->dt / c->rho0);
    a.inv_dt = float(1.0 / c->dt);
    a.gn = float(gn);
    a.half_dt_smax = float(0.5 * c->sigma_max * c->dt);
    a.remap = c->step_remap;
    if (c->probe_fused_out) {
        a.pcells = reinterpret_cast<const long long*>(c->probe_cells);
        a.pout = c->probe_fused_out;
        a.np = c->nprobes;
        a.pcomp = c->probe_comp;
    }
    if (c->hetero) return c->viscous ? launch_force<true, true>(c, a) : launch_force<true, false>(c, a);
    return c->viscous ? launch_force<false, true>(c, a) : launch_force<false, false>(c, a);
}
