// Two FDTD steps per pass over the state (temporal blocking): the Sec. 3.1
// update of kvs_step_tile.hpp applied twice, with the same operations in the
// same order, so the result is bitwise that of two one-step launches.  The
// per-tile code, shared by the single-context kernel (kvs_step2.hip) and the
// batched one (kvs_batch.hip).
//
// A block of 64 WX x R threads covers that many interior cells of every plane
// of a z segment.  All its threads form the intermediate state (step n + 1)
// of their cell from the input state, staged in LDS with one more cell on
// each side (z neighbours in a per-thread register queue); the threads that
// own their cell then advance it to step n + 2 from the intermediate state
// staged in LDS (z neighbours again in registers).  A thread owns its cell
// unless it is the first or last of its row or column of threads with more
// tiles beyond (overlap_owns): next to a wall the intermediate state beyond
// is 0, the Dirichlet layer, so the tiles' end threads there own theirs too.
// 256 interior cells in x take two tiles of 128 and 254 rows 42 tiles of 8
// exactly.  The march forms the intermediate state one plane ahead of the
// second step: at iteration k plane k of step n + 1 and plane k - 1 of step
// n + 2, so one barrier per plane orders both.  Per two cell-updates the
// input is read and the output written once; the cells at the tiles' inner
// edges and the planes at the segments' ends form the intermediate state
// twice (8 x 128 tiles: 7/6 x 64/63 updates of arithmetic per update).
//
// The march is unrolled by three with the register queues (input planes
// k - 1, k, k + 1; intermediate planes k - 2, k - 1, k; face moduli of the
// same) as rings, so nothing is moved between registers and plane k + 2 is
// loaded straight into the registers that plane k - 1 leaves after the first
// step.  Each field's plane address is uniform, the lane's cell a constant
// offset.
//
// Measured, us per step with two steps per launch, against rows of 256 x 4
// threads in one copy of the march (FP32 viscous rows up to 256 cells only,
// else one step per launch): 256^3 heterogeneous 118 against 135, with force
// on every step 159 / 254; 240 x 200 x 200 homogeneous 66 / 79; 384 x 320 x 352
// heterogeneous 397 / 540, with force 457 / 632, with three peak planes
// 419 / 552; 181^3 lossless 35 / 85; 48^3 FP64 lossless 4.8 / 11.3.  The
// vector-ALU instructions of a 256^3 launch fell from 137 to 70 million; what
// is left is the latency of a plane (one block of 16 wavefronts on a CU meets
// at a barrier per plane) and, lossless, HBM (256^3: 805 MB in 167 us).
//
// Face moduli: harm(G, G') / h^2 = 2 G G' / (G + G') / h^2 is formed as
// (G G') / (G + G') (2 / h^2).  Scaling by 2 is exact, so this is the same
// rounded value as the one-step kernel's, and it does not depend on the
// operand order: the z- face of plane k is the z+ face of plane k - 1, and
// the second step reuses the faces and the sponge factors of the first.
//
// Probe values of the intermediate step: written by the thread that owns
// their cell, found through a table with one entry per grid row that is
// fetched a plane ahead (a lookup per plane would drain the loads in flight).
// Cells of the Dirichlet layer have no thread; the probe blocks write their
// zeros.  On peak planes |u| of the intermediate step is stored beside the
// maps, for the fold after the launch, which takes both steps' values: an
// atomic maximum into the maps from here held up the loads behind it (450
// against 400 us per step at 384 x 320 x 352).
#pragma once

#include <type_traits>

#include "kvs_step_tile.hpp"

namespace {

using kvs_tiling::overlap_owns;
using kvs_tiling::overlap_tiles;

template <typename T>
struct Step2Args {
    StepArgs<T> a;      // a.gn: envelope of the first step
    T gn2;              // envelope of the second
    const int* rowtab;  // [nz][ny]: offset of row (j, k) in ptab where it holds a probe, else -1
    const int* ptab;    // per probed row, nx entries: probe index or -1
    double* pmid;       // trace slot of the intermediate state
};

// Peak planes, as the kernels take them (n = 0: none); mid: the intermediate
// |u| on them, laid out like the maps.
template <typename T>
struct Step2Peaks {
    int n;
    int axis[KVS_MAX_PEAK_PLANES];
    int index[KVS_MAX_PEAK_PLANES];
    int n1[KVS_MAX_PEAK_PLANES];
    long long off[KVS_MAX_PEAK_PLANES];
    T* mid;
};

// Global-memory views of the argument pointers: a pointer read from a table
// in memory (the batched launch) is otherwise generic, and flat accesses also
// count against the LDS wait counter, so the wait before each barrier would
// drain the plane-ahead loads.
template <typename T>
using gptr = __attribute__((address_space(1))) T*;
template <typename T>
__device__ __forceinline__ gptr<T> glob(T* p) {
    return (gptr<T>)p;
}

// base + off bytes: a uniform base and a lane's 32-bit byte offset, the form
// that a global access takes without address arithmetic in vector registers.
// The empty asm keeps the base a scalar of its own: otherwise base and lane
// offset are added outside the march, two vector registers per field, and the
// plane's offset to that by vector arithmetic at every access.  lane_byte
// does the same for the lane's offset, once for a group of accesses: a copy
// that is seen to be 32 bits wide where it is used.
__device__ __forceinline__ unsigned lane_byte(unsigned off) {
    asm volatile("" : "+v"(off));
    return off;
}
template <typename T>
__device__ __forceinline__ gptr<T> at_byte(gptr<T> base, unsigned off) {
    using byte = __attribute__((address_space(1))) char;
    unsigned long long b = (unsigned long long)base;
    asm("" : "+s"(b));
    return (gptr<T>)((byte*)b + off);
}

// Streamed store of v at byte l of a plane of `bytes` bytes, nothing where l is
// kNoStore: a buffer store, which drops what is out of its bounds.  Stores
// under a branch would leave the number of accesses in flight open, and every
// wait for a load would wait for them as well.
constexpr unsigned kNoStore = 0xffffff00u;
__device__ __forceinline__ void store_plane(float* base, unsigned bytes, unsigned l, float v) {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00027000);
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, l, 0, 0);
}
__device__ __forceinline__ void store_plane(double* base, unsigned bytes, unsigned l, double v) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00027000);
    const u2 d = {(unsigned)__double2loint(v), (unsigned)__double2hiint(v)};
    __builtin_amdgcn_raw_buffer_store_b64(d, r, l, 0, 0);
}

__device__ __forceinline__ float face_modulus(float g, float gn, float h2) {
    return g * gn * __builtin_amdgcn_rcpf(g + gn) * h2;
}
__device__ __forceinline__ double face_modulus(double g, double gn, double h2) { return g * gn / (g + gn) * h2; }

// The update's sums, with the fused multiply-adds that the one-step kernel's
// expressions compile to written out: left to the compiler, the flux through
// a z face would be formed once for the planes on its two sides (the march is
// unrolled, so it sees both), rounded there and no longer fused.
__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }
// For each component: acc, the sum over the faces of modulus x difference, and
// lap, the Laplacian of w; one axis after the other, c the cell's values, m and
// p its neighbours', gm and gp the moduli of the faces between.
template <typename T, bool VISC, int N>
__device__ __forceinline__ void first_axis(const T (&c)[N], const T* m, const T* p, T gm, T gp, T (&acc)[3], T (&lap)[3]) {
#pragma unroll
    for (int n = 0; n < 3; ++n) {
        acc[n] = fma_t(gp, p[n] - c[n], -(gm * (c[n] - m[n])));
        if constexpr (VISC) lap[n] = fma_t(T(-2), c[3 + n], p[3 + n] + m[3 + n]);
    }
}
template <typename T, bool VISC, int N>
__device__ __forceinline__ void second_axis(const T (&c)[N], const T* m, const T* p, T gm, T gp, T ihx2, T ihy2, T (&acc)[3],
                                            T (&lap)[3]) {
#pragma unroll
    for (int n = 0; n < 3; ++n) {
        acc[n] = fma_t(-gm, c[n] - m[n], fma_t(gp, p[n] - c[n], acc[n]));
        if constexpr (VISC) lap[n] = fma_t(lap[n], ihx2, fma_t(T(-2), c[3 + n], p[3 + n] + m[3 + n]) * ihy2);
    }
}
template <typename T, bool VISC, int N>
__device__ __forceinline__ void third_axis(const T (&c)[N], const T* m, const T* p, T gm, T gp, T ihz2, T (&acc)[3],
                                           T (&lap)[3]) {
#pragma unroll
    for (int n = 0; n < 3; ++n) {
        acc[n] = fma_t(-gm, c[n] - m[n], fma_t(gp, p[n] - c[n], acc[n]));
        if constexpr (VISC) lap[n] = fma_t(fma_t(T(-2), c[3 + n], p[3 + n] + m[3 + n]), ihz2, lap[n]);
    }
}

// The staged fields of a cell lie together in LDS, in chunks of up to 16 bytes
// (FP32: u and the first of w, the rest of w and G), each chunk an array over
// the plane's cells: a neighbour's fields take one or two wide reads instead
// of one narrow read each (28 and 24 reads for the two steps of an FP32
// heterogeneous viscous cell become 8 and 8, and the march waits for LDS a few
// times per plane instead of at every field).
template <typename T, int N>
struct Chunks {
    static constexpr int V = N <= 4 ? 1 : 16 / sizeof(T);  // values of a full chunk
    static constexpr int count = (N + V - 1) / V;
    static constexpr int width(int c) {                    // values of chunk c
        const int left = N - c * V;
        return left >= V ? V : left == 3 ? 4 : left;
    }
    static constexpr int cell = (count - 1) * V + width(count - 1);  // values per cell
};
template <typename T, int W>
struct ChunkVec {
    typedef T type __attribute__((ext_vector_type(W)));
};
template <typename T>
struct ChunkVec<T, 1> {
    typedef T type;
};
template <typename T, int N, int C = 0>
__device__ __forceinline__ void lds_put(T* plane, int cells, int pos, const T (&v)[N]) {
    using K = Chunks<T, N>;
    if constexpr (C < K::count) {
        constexpr int w = K::width(C);
        typename ChunkVec<T, w>::type x;
        if constexpr (w == 1) {
            x = v[C * K::V];
        } else {
#pragma unroll
            for (int n = 0; n < w; ++n) x[n] = C * K::V + n < N ? v[C * K::V + n < N ? C * K::V + n : 0] : T(0);
        }
        *reinterpret_cast<typename ChunkVec<T, w>::type*>(plane + C * K::V * cells + pos * w) = x;
        lds_put<T, N, C + 1>(plane, cells, pos, v);
    }
}
template <typename T, int N, int C = 0>
__device__ __forceinline__ void lds_get(const T* plane, int cells, int pos, T (&v)[N]) {
    using K = Chunks<T, N>;
    if constexpr (C < K::count) {
        constexpr int w = K::width(C);
        const typename ChunkVec<T, w>::type x =
            *reinterpret_cast<const typename ChunkVec<T, w>::type*>(plane + C * K::V * cells + pos * w);
        if constexpr (w == 1) {
            v[C * K::V] = x;
        } else {
#pragma unroll
            for (int n = 0; n < w; ++n)
                if (C * K::V + n < N) v[C * K::V + n] = x[n];
        }
        lds_get<T, N, C + 1>(plane, cells, pos, v);
    }
}

// one field of a cell
template <typename T, int N, int F>
__device__ __forceinline__ void lds_put_one(T* plane, int cells, int pos, T v) {
    using K = Chunks<T, N>;
    constexpr int c = F / K::V;
    plane[c * K::V * cells + pos * K::width(c) + F % K::V] = v;
}

// Sizes of a tile: staged input fields NQ (u, w where neighbours of w are
// needed, G), staged intermediate fields NM, LDS row W, LDS elements.
template <typename T, bool HET, bool VISC, int WX, int R>
struct Step2Tile {
    static constexpr int TX = 64 * WX, W = TX + 2, NU = VISC ? 6 : 3, NQ = NU + (HET ? 1 : 0), NM = NU;
    static constexpr int CELLS = (R + 2) * W;
    static constexpr int SN = Chunks<T, NQ>::cell * CELLS, S1 = Chunks<T, NM>::cell * CELLS;  // one plane of each
    static constexpr int LDS = 2 * (SN + S1);
};

// Tile shapes (threads per row / 64, rows): 128 x 8, 64 x 16, 64 x 8, 192 x 5.
// FP64, whose state takes twice the LDS and registers, uses 64 x 8 only.
constexpr int kStep2Shapes = 4;
constexpr int kStep2Wx[kStep2Shapes] = {2, 1, 1, 3}, kStep2Rows[kStep2Shapes] = {8, 16, 8, 5};

// Whether a shape is offered for a grid of ny rows (see the halo cells below).
constexpr bool step2_offers(int shape, int64_t ny) { return ny != kStep2Rows[shape] + 2; }

// Wavefront-updates per plane of a tile: R first and R - 2 second steps a row.
constexpr int step2_units(int shape) { return kStep2Wx[shape] * (2 * kStep2Rows[shape] - 2); }

// One tile; lds holds Step2Tile::LDS elements.
template <typename T, bool HET, bool VISC, bool FORCE, bool PEAK, int WX, int R>
__device__ __forceinline__ void step2_tile(const Step2Args<T>& A2, const Step2Peaks<T>* pk, T* lds, int bx, int by, int bz) {
    using S = Step2Tile<T, HET, VISC, WX, R>;
    static_assert(R >= 3 && 2 * R <= 64 && 64 * WX * R <= 1024, "halo lanes of row 1, threads of a block");
    constexpr int TX = S::TX, W = S::W, NU = S::NU, NQ = S::NQ, NM = S::NM, QG = NU;
    constexpr int P = S::CELLS;
    const StepArgs<T>& a = A2.a;
    T* const sn = lds;               // input planes, two buffers
    T* const s1 = lds + 2 * S::SN;   // intermediate planes, two buffers, with a border that stays 0

    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int kb = 1 + bz * a.kchunk;
    const int ke = min(nz - 1, kb + a.kchunk);  // output planes kb .. ke - 1
    // a wavefront is 64 threads of one thread row (blockDim.x = 64 WX), so the
    // row index is uniform across it: kept in a scalar register, the row tests
    // below are scalar branches
    const int tx = threadIdx.x, ty = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int i = 1 + bx * (TX - 2) + tx, j = 1 + by * (R - 2) + ty;
    const bool act = i <= nx - 2 && j <= ny - 2;
    const bool own = act && overlap_owns(tx, bx, TX, i, nx);            // with ownrow
    const bool ownrow = j <= ny - 2 && overlap_owns(ty, by, R, j, ny);  // uniform
    // the rows that carry both steps: issued first, they reach the second
    // step while the others still form the first, instead of running it alone
    // at the end of each plane
    if (ownrow) __builtin_amdgcn_s_setprio(1);
    const int sxy = nx * ny;
    // a lane beyond the grid reads cell 0 of the plane (a wall) and forms 0
    const unsigned col = i < nx && j < ny ? (unsigned)(i + nx * j) * (unsigned)sizeof(T) : 0u;  // bytes
    // Halo cells, all loaded by thread rows that do not own theirs (the
    // registers of the second step are free there): the rows below and above
    // the tile by thread rows 0 and R - 1; where one of these owns its cells,
    // the row beyond is a wall, of which only G is not 0, loaded by the other;
    // the columns left and right of the tile (2 R cells) by one wavefront of
    // row 0 or else R - 1.  (Both own in a grid of R + 2 rows: not offered.)
    const bool hrow = ty == 0 || ty == R - 1;
    const bool cols = tx < 64 && ty == (by > 0 ? 0 : R - 1);
    const int dummy = 0;  // a corner: staged, never read
    const int hj = ty == 0 ? j - 1 : j + 1;
    const int hpos = ty == 0 ? tx + 1 : ty == R - 1 ? (R + 1) * W + tx + 1 : dummy;
    const unsigned hcol = hrow && i < nx && hj < ny ? (unsigned)(i + nx * hj) * (unsigned)sizeof(T) : 0u;
    const int wj = ty == 0 && j + R - 1 == ny - 2 ? ny - 1 : ty == R - 1 && by == 0 ? 0 : -1;  // the wall row
    const int wpos = wj < 0 ? dummy : wj == 0 ? tx + 1 : (R + 1) * W + tx + 1;
    const unsigned wcol = wj >= 0 && i < nx ? (unsigned)(i + nx * wj) * (unsigned)sizeof(T) : 0u;
    const bool right = tx >= R, creal = tx < 2 * R;
    const int crow = right ? tx - R : tx;
    const int ci = right ? 1 + bx * (TX - 2) + TX : bx * (TX - 2), cj = 1 + by * (R - 2) + crow;
    const int cpos = creal ? (crow + 1) * W + (right ? TX + 1 : 0) : dummy;
    const unsigned ccol = creal && ci < nx && cj < ny ? (unsigned)(ci + nx * cj) * (unsigned)sizeof(T) : 0u;
    const int pos = (ty + 1) * W + tx + 1;

    // Staged field f at element o.  The stride between components is made
    // opaque at each group of accesses (scalar adds), so that not every field's
    // address is kept in scalar registers, which then spill into vector ones.
    auto stride = [&]() {
        long long n = a.N;
        asm volatile("" : "+s"(n));
        return n;
    };
    auto field = [&](int f, long long n, size_t o) {
        return glob(f == QG && HET ? a.G + o : f < 3 ? a.u + f * n + o : a.w + (f - 3) * n + o);
    };
    const gptr<const T> crho_g = glob(a.crho), eta_g = glob(a.eta);
    auto plane_of = [&](int k) { return (size_t)min(max(k, 0), nz - 1) * (size_t)sxy; };
    const T rx = a.L > 0 ? ramp<T>(i, nx, a.L, a.invL) : T(0);
    const T rxy = a.L > 0 ? max(rx, ramp<T>(j, ny, a.L, a.invL)) : T(0);
    const T ihx2 = a.ihx2, ihy2 = a.ihy2, ihz2 = a.ihz2;
    const T h2x = T(2) * ihx2, h2y = T(2) * ihy2, h2z = T(2) * ihz2;
    const T gx0 = HET ? T(0) : a.G0 * ihx2, gy0 = HET ? T(0) : a.G0 * ihy2, gz0 = HET ? T(0) : a.G0 * ihz2;
    const bool probes = A2.pmid != nullptr && ownrow;  // uniform across a wavefront
    // read-only for the launch and uniform across the wavefront: scalar loads
    using tab_t = __attribute__((address_space(4))) const int*;
    const tab_t rowtab_j = (tab_t)(probes ? A2.rowtab + j : nullptr);
    auto rowoff = [&](int k) { return k >= kb && k < ke ? rowtab_j[ny * k] : -1; };

    for (int q = ty * TX + tx; q < S::LDS; q += TX * R) lds[q] = T(0);

    const int k0 = kb - 1;  // first intermediate plane
    auto probe = [&](int p, T x, T y, T z) {
        const gptr<double> out = glob(A2.pmid);
        if (a.pcomp == 3) {
            out[3 * p] = (double)x;
            out[3 * p + 1] = (double)y;
            out[3 * p + 2] = (double)z;
        } else {
            out[p] = (double)(a.pcomp == 0 ? x : a.pcomp == 1 ? y : z);
        }
    };
    // the wavefront's peak planes: whether some x or y plane crosses it, and the
    // z plane (more than one: every plane is looked at)
    bool pkxy = false;
    int pkz = -1;
    const int iw = __builtin_amdgcn_readfirstlane(i);  // the wavefront's first cell
    if constexpr (PEAK) {
        int nz_planes = 0;
        for (int p = 0; p < pk->n; ++p) {
            const int ax = pk->axis[p], idx = pk->index[p];
            pkxy = pkxy || (ax == 0 && idx >= iw && idx <= iw + 63) || (ax == 1 && idx == j);
            if (ax == 2) {
                pkz = idx;
                ++nz_planes;
            }
        }
        pkxy = pkxy || nz_planes > 1;
    }
    auto peaks = [&](T x, T y, T z, int k) {
        if (!pkxy && k != pkz) return;
        for (int p = 0; p < pk->n; ++p) {
            const int ax = pk->axis[p], idx = pk->index[p];
            if (ax == 0 ? (idx < iw || idx > iw + 63) : ax == 1 ? idx != j : idx != k) continue;
            const T v = sqrt(fma_t(z, z, fma_t(x, x, y * y)));
            const int c = ax == 0 ? j + pk->n1[p] * k : ax == 1 ? i + pk->n1[p] * k : i + pk->n1[p] * j;
            if (own && (ax != 0 || i == idx)) glob(pk->mid)[pk->off[p] + c] = v;
        }
    };
    __syncthreads();  // the zeroes, before the first plane lands among them

    // The march, once for each kind of wavefront (owning; halo rows; halo rows
    // and columns), which meet at the barriers of their own copies.  In one copy
    // for all, the loads and stores that some wavefronts skip made the compiler
    // wait, at every use of a loaded value, for all that was issued after it
    // too (halo values just asked for, stores).
    auto march = [&](auto own_tag, auto cols_tag) {
        constexpr bool OWN = decltype(own_tag)::value, COLS = decltype(cols_tag)::value;
        // rings: input planes, intermediate planes, face moduli (x-, x+, y-, y+, z+)
        T z0[NQ], z1[NQ], z2[NQ], q0[NM], q1[NM], q2[NM], f0[5], f1[5], f2[5];
        T hr[NQ], hs[NQ], hw = T(0);     // halo row, column and wall values of the plane to come
        T wv[3] = {T(0), T(0), T(0)};    // lossless: w of the cell at that plane ...
        T wq[3] = {T(0), T(0), T(0)};    // ... and the intermediate w of the plane before
        T fs[3] = {T(0), T(0), T(0)}, fsp[3] = {T(0), T(0), T(0)};
        T crho = a.crho0, eta = T(0);
        T c1p = T(0), c2p = T(0), ep = T(0);  // sponge factors and eta / dt of the plane before
#pragma unroll
        for (int f = 0; f < NQ; ++f) {
            z0[f] = *at_byte(field(f, a.N, plane_of(k0 - 1)), col);
            z1[f] = *at_byte(field(f, a.N, plane_of(k0)), col);
            z2[f] = *at_byte(field(f, a.N, plane_of(k0 + 1)), col);
            hr[f] = hs[f] = T(0);
        }
        auto load_halo = [&](int k) {
            const size_t o = plane_of(k);
            const long long n = stride();
            if constexpr (!OWN) {
                const unsigned l = lane_byte(hcol);
#pragma unroll
                for (int f = 0; f < NQ; ++f) hr[f] = *at_byte(field(f, n, o), l);
                if constexpr (HET) hw = *at_byte(glob(a.G) + o, lane_byte(wcol));
            }
            if constexpr (COLS) {
                const unsigned l = lane_byte(ccol);
#pragma unroll
                for (int f = 0; f < NQ; ++f) hs[f] = *at_byte(field(f, n, o), l);
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
        load_cell(k0, col);
#pragma unroll
        for (int f = 0; f < NM; ++f) q0[f] = q1[f] = q2[f] = T(0);
#pragma unroll
        for (int f = 0; f < 5; ++f) f0[f] = f1[f] = f2[f] = T(0);
        if constexpr (HET) f0[4] = face_modulus(z1[QG], z0[QG], h2z);
        int poff = probes ? rowoff(k0) : -1, poff_n = -1;
        load_halo(k0);
        // zm, zc, zp: input planes k - 1, k, k + 1 (zm leaves as k + 2); qm, qc, q:
        // intermediate planes k - 2, k - 1, k (formed here); fm, fc, f: their faces
        auto plane = [&](const int k, T(&zm)[NQ], T(&zc)[NQ], T(&zp)[NQ], T(&qm)[NM], T(&qc)[NM], T(&q)[NM], T(&fm)[5],
                         T(&fc)[5], T(&f)[5]) {
            T* const b0 = sn + (k & 1) * S::SN;
            T* const b1 = s1 + (k & 1) * S::S1;
            const T* const b2 = s1 + ((k + 1) & 1) * S::S1;  // plane k - 1
            lds_put<T, NQ>(b0, P, pos, zc);
            if constexpr (!OWN) {
                lds_put<T, NQ>(b0, P, hpos, hr);
                if constexpr (HET) lds_put_one<T, NQ, QG>(b0, P, wpos, hw);
            }
            if constexpr (COLS) lds_put<T, NQ>(b0, P, cpos, hs);
            load_halo(k + 1);
            if constexpr (OWN) {
                if (probes) poff_n = rowoff(k + 1);
            }
            lds_barrier();

            // ---- step n + 1 at (i, j, k) ----
            T c1 = T(1), c2 = crho;
            if (a.L > 0) {
                const T s = a.half_dt_smax * max(rxy, ramp<T>(k, nz, a.L, a.invL));
                const T inv1ps = rcp_fast<T>(T(1) + s);
                c1 = (T(1) - s) * inv1ps;
                c2 = crho * inv1ps;
            }
            const T e = !VISC ? T(0) : HET ? eta * a.inv_dt : a.eta_dt0;
            T acc[3], lap[3], wn[3];
            {
                T m[NQ], p[NQ];
                lds_get<T, NQ>(b0, P, pos - 1, m);
                lds_get<T, NQ>(b0, P, pos + 1, p);
                if constexpr (HET) {
                    f[0] = face_modulus(zc[QG], m[QG], h2x);
                    f[1] = face_modulus(zc[QG], p[QG], h2x);
                }
                first_axis<T, VISC>(zc, m, p, HET ? f[0] : gx0, HET ? f[1] : gx0, acc, lap);
            }
            {
                T m[NQ], p[NQ];
                lds_get<T, NQ>(b0, P, pos - W, m);
                lds_get<T, NQ>(b0, P, pos + W, p);
                if constexpr (HET) {
                    f[2] = face_modulus(zc[QG], m[QG], h2y);
                    f[3] = face_modulus(zc[QG], p[QG], h2y);
                }
                second_axis<T, VISC>(zc, m, p, HET ? f[2] : gy0, HET ? f[3] : gy0, ihx2, ihy2, acc, lap);
            }
            if constexpr (HET) f[4] = face_modulus(zc[QG], zp[QG], h2z);
            third_axis<T, VISC>(zc, zm, zp, HET ? fc[4] : gz0, HET ? f[4] : gz0, ihz2, acc, lap);
            const bool in = act && k >= 1 && k <= nz - 2;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const T uc = zc[c];
                T wc = wv[c];
                if constexpr (VISC) {
                    wc = zc[3 + c];
                    acc[c] = fma_t(e, lap[c], acc[c]);
                }
                if constexpr (FORCE) {
                    if (a.gn != T(0)) acc[c] = fma_t(a.gn, fs[c], acc[c]);
                }
                const T wnew = fma_t(c1, wc, c2 * acc[c]);
                wn[c] = in ? wnew : T(0);
                q[c] = in ? uc + wnew : T(0);
                if constexpr (VISC) q[3 + c] = wn[c];
            }
            // the force and (lossless) the intermediate w, for the second step a plane later
            T fo[3], wo[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                fo[c] = fsp[c];
                wo[c] = wq[c];
                fsp[c] = fs[c];
                wq[c] = wn[c];
            }
            {
                const size_t o = plane_of(k + 2);
                const long long st = stride();
                const unsigned l = lane_byte(col);
                load_cell(k + 1, l);
#pragma unroll
                for (int n = 0; n < NQ; ++n) zm[n] = *at_byte(field(n, st, o), l);
            }
            lds_put<T, NM>(b1, P, pos, q);
            if (OWN && k >= kb && k < ke) {
                if (poff >= 0 && own) {
                    const int p = glob(A2.ptab)[poff + i];
                    if (p >= 0) probe(p, q[0], q[1], q[2]);
                }
                if constexpr (PEAK) peaks(q[0], q[1], q[2], k);
            }

            // ---- step n + 2 at (i, j, k - 1) ----
            const int k2 = k - 1;
            if constexpr (OWN) {
                T uo[3], vo[3];
                {
                    T m[NM], p[NM];
                    lds_get<T, NM>(b2, P, pos - 1, m);
                    lds_get<T, NM>(b2, P, pos + 1, p);
                    first_axis<T, VISC>(qc, m, p, HET ? fc[0] : gx0, HET ? fc[1] : gx0, acc, lap);
                }
                {
                    T m[NM], p[NM];
                    lds_get<T, NM>(b2, P, pos - W, m);
                    lds_get<T, NM>(b2, P, pos + W, p);
                    second_axis<T, VISC>(qc, m, p, HET ? fc[2] : gy0, HET ? fc[3] : gy0, ihx2, ihy2, acc, lap);
                }
                third_axis<T, VISC>(qc, qm, q, HET ? fm[4] : gz0, HET ? fc[4] : gz0, ihz2, acc, lap);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const T uc = qc[c];
                    T wc = wo[c];
                    if constexpr (VISC) {
                        wc = qc[3 + c];
                        acc[c] = fma_t(ep, lap[c], acc[c]);
                    }
                    if constexpr (FORCE) {
                        if (A2.gn2 != T(0)) acc[c] = fma_t(A2.gn2, fo[c], acc[c]);
                    }
                    vo[c] = fma_t(c1p, wc, c2p * acc[c]);
                    uo[c] = uc + vo[c];
                }
                // planes kb - 1 and kb have no second step before them
                const bool keep = own && k2 >= kb;
                const size_t o = (size_t)k2 * (size_t)sxy;
                const long long n = stride();
                const unsigned bytes = (unsigned)sxy * (unsigned)sizeof(T), l = keep ? col : kNoStore;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    store_plane(a.wn + c * n + o, bytes, l, vo[c]);
                    store_plane(a.un + c * n + o, bytes, l, uo[c]);
                }
                // the walls at the row's ends, 0 as they are, with their neighbours: whole lines
                if (keep && (i == 1 || i == nx - 2)) {
                    const unsigned lw = i == 1 ? l - (unsigned)sizeof(T) : l + (unsigned)sizeof(T);
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        store_plane(a.wn + c * n + o, bytes, lw, T(0));
                        store_plane(a.un + c * n + o, bytes, lw, T(0));
                    }
                }
            }
            c1p = c1;
            c2p = c2;
            ep = e;
            poff = poff_n;
        };
        for (int k = k0;;) {  // left from between the planes: no values merge there
            plane(k, z0, z1, z2, q1, q2, q0, f2, f0, f1);
            if (++k > ke) break;
            plane(k, z1, z2, z0, q2, q0, q1, f0, f1, f2);
            if (++k > ke) break;
            plane(k, z2, z0, z1, q0, q1, q2, f1, f2, f0);
            if (++k > ke) break;
        }
    };
    constexpr std::integral_constant<bool, false> no{};
    constexpr std::integral_constant<bool, true> yes{};
    if (ownrow)
        march(yes, no);
    else if (cols)
        march(no, yes);
    else
        march(no, no);
}

// Probe blocks of a two-step launch: copy the launch's input state (the result
// of the step before) at the probe cells into a.pout, and write the zeros of
// the probes on the Dirichlet layer into the intermediate state's slot.
template <typename T>
__device__ __forceinline__ void step2_probe(const Step2Args<T>& A2, long long p) {
    const StepArgs<T>& a = A2.a;
    if (p >= a.np) return;
    const long long q = a.pcells[p];
    if (a.pout) {
        if (a.pcomp == 3) {
            a.pout[3 * p] = (double)a.u[q];
            a.pout[3 * p + 1] = (double)a.u[a.N + q];
            a.pout[3 * p + 2] = (double)a.u[2 * a.N + q];
        } else {
            a.pout[p] = (double)a.u[a.pcomp * a.N + q];
        }
    }
    const int i = (int)(q % a.nx), j = (int)((q / a.nx) % a.ny);
    if (A2.pmid && (i == 0 || i == a.nx - 1 || j == 0 || j == a.ny - 1)) {
        const int nc = a.pcomp == 3 ? 3 : 1;
        for (int c = 0; c < nc; ++c) A2.pmid[nc * p + c] = 0.0;
    }
}

}  // namespace
