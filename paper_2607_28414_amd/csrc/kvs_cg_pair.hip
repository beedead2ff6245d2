// Two CG iterations per pair of sweeps (Sec. 3.2.3 with constant-diagonal
// Jacobi or no preconditioner) for FP32 storage of the direction and the
// residual: the iterates, the stop test after every iteration and the scalars
// are those of the one-iteration sweeps of kvs_cg.hip in exact arithmetic.
//
// With p the direction, r the residual, q = A p and z = zs r, two steps are
//   r1 = r - a0 q,          p1 = zs r1 + b0 p,   A p1 = zs (A r - a0 A q) + b0 q,
//   r2 = r1 - a1 A p1,      phi += a0 p + a1 p1,
// so every inner product that a0, b0, a1 need is one of p.q, r.q, q.q, r.Ar,
// q.Ar, q.Aq of the vectors at hand:
//   a0 = r.z / p.q,  r1.r1 = r.r - 2 a0 r.q + a0^2 q.q,  b0 = r1.r1 / r.r,
//   p1.A p1 = zs^2 (r.Ar - 2 a0 q.Ar + a0^2 q.Aq) + 2 zs b0 (r.q - a0 q.q) + b0^2 p.q,
//   a1 = zs r1.r1 / p1.A p1,
// and b1 = r2.r2 / r1.r1 with r2.r2 summed from r2 as it is stored.
//
// Sweep "sums" reads r and the last stored direction, forms p = z + b p_old
// (rounded to FP32 once, as stored directions are), q, A r and A q on chip and
// writes nothing but six partial sums per block: 8 B per cell.  Sweep "update"
// forms the same values again and writes phi, r2 and p1: 32 B per cell.  40 B
// per cell and two iterations, where two sweeps per iteration move 40 B for
// each.  All arithmetic and sums are FP64; r2 is rounded once per pair, phi is
// updated with the same unrounded p1 as r2, and only the direction kept for
// the next pair is rounded.
//
// When the first of the two iterations already ends the solve (tolerance, a
// fixed or the largest count), takes the residual so far down that r1.r1 has no
// digits left (kPairFall), or p1.A p1 is not positive, the update applies that
// iteration alone (phi += a0 p, r = r1, p stays p); the next pair then
// meets the breakdown itself.
//
// Tiles: 64 WX x R threads, all forming q, the inner ones (and those next to
// a wall) owning their cells (overlap_tiles); z is marched with A q one plane
// behind q, so one barrier per plane orders both stages.  Loads are issued two
// planes ahead into two named register sets (the march is unrolled by two), so
// that no wait is for a load of the plane before.  The tiles are held to 64
// registers, so that two blocks of 1024 threads share a CU: without the limit the
// update takes 68 to 72 and both sweeps are planned for one, 65 + 129 us at 256^3
// instead of 60 + 120, 27 + 50 instead of 29 + 48 at 160 x 144 x 208, 37 + 83 instead
// of 39 + 77 at 240 x 200 x 200; but 238 + 680 instead of 260 + 722 at 384 x 384 x 512.
//
// Measured at 256^3: 60 us (sums; 134 MB algorithmic, 156 MB fetched, mostly from
// the 256 MB cache: LDS and FP64 issue bound it) + 120 us (update; 537 MB
// algorithmic, 342 MB fetched and 266 MB written, 5.1 TB/s: HBM bounds it) for two
// iterations, where two pairs of one-iteration sweeps with their scalar kernels
// took 262 us; 1e-8 in 904 iterations: 82 instead of 118 ms.
#include <type_traits>

#include "kvs_cg_pair.hpp"
#include "kvs_cg_scalars.hpp"

namespace {

using kvs_tiling::lds_barrier;
using kvs_tiling::overlap_owns;
using kvs_tiling::overlap_tiles;
using kvs_tiling::tile_of;

struct PairGeom {
    int nx, ny, nz, gx, gy, gz, kchunk;
    double ihx2, ihy2, ihz2, diag;
    double dinv;
};

__device__ __forceinline__ double pair_wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

template <int WX, int R, bool UPD>
__global__ __launch_bounds__(64 * WX * R) __attribute__((amdgpu_waves_per_eu(8))) void cg_pair_kernel(const PairGeom g, const float* r_in, const float* p_in,
                                                              float* r_out, float* p_out, double* phi,
                                                              const CgFold fold, double* partials, int npart) {
    static_assert(R >= 3 && 2 * R <= 64 && 64 * WX * R <= 1024, "halo lanes: 3 <= R <= 32");
    constexpr int TX = 64 * WX, W = TX + 2, NW = WX * R;
    const CgState* st = cg_fold<UPD ? CG_PAIR : CG_PAIR_END, 64 * WX * R>(fold, threadIdx.y * TX + threadIdx.x);
    if (st->done) return;
    __shared__ float sp[2][R + 3][W], sr[2][R + 3][W];  // rows 0 .. R + 1, and a row for lanes without halo work
    __shared__ double sq[2][R + 2][W];                  // first stage, with a border that stays 0 (walls)
    const int tx = threadIdx.x, ty = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int B = g.gx * g.gy * g.gz;
    const int t = tile_of(blockIdx.x, B);
    const int bx = t % g.gx, by = (t / g.gx) % g.gy, bz = t / (g.gx * g.gy);
    const int i = 1 + bx * (TX - 2) + tx, j = 1 + by * (R - 2) + ty;
    const int kb = 1 + bz * g.kchunk, ke = min(g.nz - 1, kb + g.kchunk);
    const bool act = i <= g.nx - 2 && j <= g.ny - 2;
    const bool own = act && overlap_owns(tx, bx, TX, i, g.nx) && overlap_owns(ty, by, R, j, g.ny);
    const int sxy = g.nx * g.ny;
    const int col = act ? i + g.nx * j : 0;  // cell 0 of every plane is a wall: 0
    // halo slot: the rows below and above the tile (thread rows 0 and R - 1),
    // the columns left and right of it (the first 2 R lanes of row 1)
    const bool hload = ty == 0 || ty == R - 1 || (ty == 1 && tx < 64);
    int hoff = 0, hrow = R + 2, hcol = tx + 1;
    if (ty == 0 || ty == R - 1) {
        const int hj = ty == 0 ? j - 1 : j + 1;
        hrow = ty == 0 ? 0 : R + 1;
        if (i <= g.nx - 1 && hj <= g.ny - 1) hoff = i + g.nx * hj;
    } else if (ty == 1 && tx < 2 * R) {
        const bool right = tx >= R;
        const int row = right ? tx - R : tx;
        const int hi = right ? 1 + bx * (TX - 2) + TX : bx * (TX - 2), hj = 1 + by * (R - 2) + row;
        hrow = row + 1;
        hcol = right ? TX + 1 : 0;
        if (hi <= g.nx - 1 && hj <= g.ny - 1) hoff = hi + g.nx * hj;
    }
    // the border of the first stage
    for (int q = ty * TX + tx; q < 2 * (R + 2) * W; q += TX * R) (&sq[0][0][0])[q] = 0.0;

    const double beta = cg_uniform(st->beta), zs = cg_uniform(st->jacobi ? g.dinv : 1.0);
    const bool first = beta == 0.0;
    const double a0 = UPD ? cg_uniform(st->pair_a0) : 0.0, b0 = UPD ? cg_uniform(st->pair_b0) : 0.0;
    const double a1 = UPD ? cg_uniform(st->pair_a1) : 0.0;
    const bool two = UPD && __builtin_amdgcn_readfirstlane(st->pair_m) == 2;
    auto dir = [&](float rv, float po) {
        return (float)(first ? (double)rv * zs : (double)rv * zs + beta * (double)po);
    };
    const int k0 = kb - 1;
    const int km = max(k0 - 1, 0), zl = g.nz - 1;
    float rm = r_in[km * sxy + col], rc = r_in[k0 * sxy + col];
    float pm = dir(rm, p_in[km * sxy + col]), pc = dir(rc, p_in[k0 * sxy + col]);
    // raw values in flight, two iterations ahead of their use (two named sets,
    // so that no register move waits for a load): plane k + 1 of the cell,
    // plane k of the halo slot and plane k - 1 of phi are used at iteration k
    float rq[2], oq[2], hrq[2] = {0.f, 0.f}, hoq[2] = {0.f, 0.f};
    double phq[2] = {0.0, 0.0};
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        const int kc = min(k0 + 1 + d, zl) * sxy, kh = min(k0 + d, zl) * sxy;
        rq[d] = r_in[kc + col];
        oq[d] = p_in[kc + col];
        if (hload) {
            hrq[d] = r_in[kh + hoff];
            hoq[d] = p_in[kh + hoff];
        }
        if (UPD && d == 1) phq[1] = __builtin_nontemporal_load(phi + k0 * sxy + col);
    }
    double qm = 0.0, qc = 0.0, arc = 0.0;  // q of planes k - 2, k - 1 and A r of plane k - 1
    double s0 = 0, s1 = 0, s2 = 0, s3 = 0, s4 = 0, s5 = 0;
    __syncthreads();  // the zeroed border, before the first planes land in it
    auto plane = [&](int k, auto set) {
        constexpr int S = decltype(set)::value;
        sp[S][ty + 1][tx + 1] = pc;
        sr[S][ty + 1][tx + 1] = rc;
        if (hload) {
            sp[S][hrow][hcol] = dir(hrq[S], hoq[S]);
            sr[S][hrow][hcol] = hrq[S];
        }
        const float rp = rq[S], pp = dir(rq[S], oq[S]);
        const double phc = phq[S];
        const int k3 = min(k + 3, zl) * sxy, k2 = min(k + 2, zl) * sxy, k1 = min(k + 1, zl) * sxy;
        rq[S] = r_in[k3 + col];
        oq[S] = p_in[k3 + col];
        if (hload) {
            hrq[S] = r_in[k2 + hoff];
            hoq[S] = p_in[k2 + hoff];
        }
        if (UPD) phq[S] = __builtin_nontemporal_load(phi + k1 + col);
        lds_barrier();
        const bool in = act && k >= 1 && k <= g.nz - 2;
        const double pcd = pc, rcd = rc;
        double q = g.diag * pcd
                 - ((double)sp[S][ty + 1][tx + 2] + (double)sp[S][ty + 1][tx]) * g.ihx2
                 - ((double)sp[S][ty + 2][tx + 1] + (double)sp[S][ty][tx + 1]) * g.ihy2
                 - ((double)pp + (double)pm) * g.ihz2;
        q = in ? q : 0.0;
        const double ar = g.diag * rcd
                        - ((double)sr[S][ty + 1][tx + 2] + (double)sr[S][ty + 1][tx]) * g.ihx2
                        - ((double)sr[S][ty + 2][tx + 1] + (double)sr[S][ty][tx + 1]) * g.ihy2
                        - ((double)rp + (double)rm) * g.ihz2;
        sq[S][ty + 1][tx + 1] = q;
        if (!UPD && own && k >= kb && k < ke) {
            s0 += pcd * q;
            s1 += rcd * q;
            s2 += q * q;
            s3 += rcd * ar;
            s4 += q * ar;
        }
        // second stage, plane k - 1 (its q neighbours were written before this plane's barrier)
        const int kk = k - 1;
        if (own && kk >= kb) {
            const double aq = g.diag * qc
                            - (sq[1 - S][ty + 1][tx + 2] + sq[1 - S][ty + 1][tx]) * g.ihx2
                            - (sq[1 - S][ty + 2][tx + 1] + sq[1 - S][ty][tx + 1]) * g.ihy2
                            - (q + qm) * g.ihz2;
            if (UPD) {
                const int o = kk * sxy + col;
                const double pd = pm, r1 = (double)rm - a0 * qc;
                double rv = r1, pv = pd, ph = phc + a0 * pd;
                if (two) {
                    const double ap1 = zs * (arc - a0 * aq) + b0 * qc;
                    pv = zs * r1 + b0 * pd;
                    rv = r1 - a1 * ap1;
                    ph += a1 * pv;
                }
                const float rs = (float)rv;
                __builtin_nontemporal_store(ph, phi + o);
                r_out[o] = rs;
                p_out[o] = (float)pv;
                s0 += (double)rs * (double)rs;
            } else {
                s5 += qc * aq;
            }
        }
        qm = qc;
        qc = q;
        arc = ar;
        rm = rc;
        rc = rp;
        pm = pc;
        pc = pp;
    };
    for (int k = k0; k <= ke; k += 2) {
        plane(k, std::integral_constant<int, 0>{});
        if (k + 1 <= ke) plane(k + 1, std::integral_constant<int, 1>{});
    }
    // block sums in wave order
    __shared__ double sh[6][NW];
    const int wv = ty * WX + tx / 64;
    constexpr int NS = UPD ? 1 : 6;
    double s[6] = {s0, s1, s2, s3, s4, s5};
#pragma unroll
    for (int n = 0; n < NS; ++n) {
        const double v = pair_wave_sum(s[n]);
        if ((tx & 63) == 0) sh[n][wv] = v;
    }
    __syncthreads();
    if (ty == 0 && tx < NS) {
        double v = 0.0;
        for (int w = 0; w < NW; ++w) v += sh[tx][w];
        partials[tx * npart + blockIdx.x] = v;
    }
}

struct PairShape {
    int wx, rows;
};

// The tile with the fewest threads over the grid's rows, whole tiles counted
// (the first stage is formed by all of them).  Measured, us per update sweep:
// 256 x 256 x 256 120 (2 x 8), 149 (1 x 16), 170 (1 x 8); 160 x 144 x 208 54,
// 48, 51; 240 x 200 x 200 84, 77, 89.
PairShape pair_shape(int nx, int ny) {
    constexpr PairShape shapes[] = {{2, 8}, {1, 16}, {1, 8}};
    PairShape best = shapes[0];
    double cost = 1e300;
    for (const PairShape& s : shapes) {
        const double c = (double)overlap_tiles(nx, 64 * s.wx) * 64 * s.wx * overlap_tiles(ny, s.rows) * s.rows;
        if (c < cost * 0.98) {
            cost = c;
            best = s;
        }
    }
    return best;
}

template <int WX, int R>
int pair_cap() {
    static const int cap = kvs_tiling::resident_blocks(cg_pair_kernel<WX, R, true>, 64 * WX * R);
    return cap;
}

template <int WX, int R>
void launch_pair(const CgPair& c, const PairGeom& g, int blocks) {
    constexpr int SUMS_END = 6;  // partial array of the update (0 .. 5: the sums)
    const bool fold = blocks <= kFoldMax;
    const dim3 grid(blocks), block(64 * WX, R);
    double* upd_part = c.partials + (size_t)SUMS_END * c.npart;
    const CgFold f0{c.st, fold ? c.st + 1 : nullptr, upd_part, blocks, c.npart};
    hipLaunchKernelGGL((cg_pair_kernel<WX, R, false>), grid, block, 0, c.stream, g, c.r_in, c.p_in, c.r_out, c.p_out,
                       c.phi, f0, c.partials, c.npart);
    if (!fold)
        hipLaunchKernelGGL(cg_scalars_kernel<CG_PAIR>, dim3(1), dim3(256), 0, c.stream, c.partials, blocks, c.npart, 0,
                           c.st);
    const CgFold f1{fold ? c.st + 1 : c.st, fold ? c.st : nullptr, c.partials, blocks, c.npart};
    hipLaunchKernelGGL((cg_pair_kernel<WX, R, true>), grid, block, 0, c.stream, g, c.r_in, c.p_in, c.r_out, c.p_out,
                       c.phi, f1, upd_part, c.npart);
    if (!fold || c.last)
        hipLaunchKernelGGL(cg_scalars_kernel<CG_PAIR_END>, dim3(1), dim3(256), 0, c.stream, upd_part, blocks, c.npart,
                           fold ? 1 : 0, c.st);
}

}  // namespace

int64_t kvs_cg_pair_blocks_max(const kvs_grid& gr) {
    const PairShape s = pair_shape((int)gr.nx, (int)gr.ny);
    return kvs_tiling::max_tiled_blocks(overlap_tiles((int)gr.nx, 64 * s.wx) * overlap_tiles((int)gr.ny, s.rows),
                                        (int)gr.nz - 2);
}

void kvs_cg_pair_launch(const kvs_grid& gr, const CgPair& c) {
    PairGeom g{};
    g.nx = (int)gr.nx;
    g.ny = (int)gr.ny;
    g.nz = (int)gr.nz;
    g.ihx2 = 1.0 / (gr.hx * gr.hx);
    g.ihy2 = 1.0 / (gr.hy * gr.hy);
    g.ihz2 = 1.0 / (gr.hz * gr.hz);
    g.diag = 2.0 * g.ihx2 + 2.0 * g.ihy2 + 2.0 * g.ihz2;
    g.dinv = 1.0 / g.diag;
    const PairShape s = pair_shape(g.nx, g.ny);
    g.gx = overlap_tiles(g.nx, 64 * s.wx);
    g.gy = overlap_tiles(g.ny, s.rows);
    const int cap = s.rows == 16 ? pair_cap<1, 16>() : s.wx == 2 ? pair_cap<2, 8>() : pair_cap<1, 8>();
    g.kchunk = kvs_tiling::cg_kchunk(g.gx * g.gy, g.nz - 2, cap);
    g.gz = (g.nz - 2 + g.kchunk - 1) / g.kchunk;
    const int blocks = g.gx * g.gy * g.gz;
    if (s.rows == 16)
        launch_pair<1, 16>(c, g, blocks);
    else if (s.wx == 2)
        launch_pair<2, 8>(c, g, blocks);
    else
        launch_pair<1, 8>(c, g, blocks);
}
