// Tiling helpers shared by the stencil kernels (FDTD step and CG sweeps).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

namespace kvs_tiling {

// Tiles are numbered x fastest, then y, then z.  The hardware hands block b
// to XCD b % 8; remapping so that each XCD receives a contiguous range of
// tile numbers keeps y-adjacent tiles (which share halo rows) in one L2.
__device__ __forceinline__ int tile_of(int b, int B) {
    const int xcd = b & 7, pos = b >> 3;
    const int per = B >> 3, rem = B & 7;
    return xcd * per + min(xcd, rem) + pos;
}

// Workgroup barrier that orders LDS only.  __syncthreads() also fences
// global memory, which makes every wave drain its outstanding global loads
// (the plane-ahead prefetch) at each barrier; the stencils only share LDS.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Blocks of one kernel instance that fit on the chip at once.
template <typename K>
int resident_blocks(K kernel, int threads) {
    int dev = 0, per_cu = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return 1024;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess || per_cu <= 0)
        per_cu = 1;
    return per_cu * prop.multiProcessorCount;
}

// Tiles of a two-stage stencil (the value of the second stage needs the first
// stage's values one cell around it) along one axis of n nodes: a tile covers
// T consecutive interior nodes with the first stage and owns the T - 2 inner
// ones, plus its end nodes where they sit next to a wall (whose first-stage
// value is 0 and needs no thread).  Tile t covers nodes 1 + t (T - 2) ..
// t (T - 2) + T, so one tile spans n - 2 <= T interior nodes and every further
// one adds T - 2.
inline int overlap_tiles(int n, int T) {
    const int m = n - 2;
    return m <= T ? 1 : (m - 2 + T - 3) / (T - 2);
}

// Whether local position l of tile t (T wide, of nt) owns its node i of n.
__device__ __forceinline__ bool overlap_owns(int l, int t, int T, int i, int n) {
    return (l >= 1 || t == 0) && (l <= T - 2 || i == n - 2);
}

// Split z into segments so that (xy tiles) x (segments) fills whole rounds of
// resident blocks; fewer, longer segments re-read fewer halo planes.
inline int choose_kchunk(int xytiles, int planes, int cap) {
    int best_seg = 1;
    double best = -1.0;
    const int max_seg = std::max(1, planes / 8);
    for (int seg = 1; seg <= max_seg; ++seg) {
        const int chunk = (planes + seg - 1) / seg;
        const int nseg = (planes + chunk - 1) / chunk;
        const long long blocks = (long long)xytiles * nseg;
        const long long rounds = (blocks + cap - 1) / cap;
        const double fill = (double)blocks / (double)(rounds * cap);
        const double halo = 2.0 / (double)chunk;
        const double score = fill / (1.0 + halo);
        if (score > best + 1e-9) {
            best = score;
            best_seg = seg;
        }
    }
    return (planes + best_seg - 1) / best_seg;
}

// Shortest z segments of the CG sweeps.  Where segments of 8 planes leave the
// chip short of blocks, a sweep's time is its blocks' serial march, not their
// halo planes, so segments of 2 planes are allowed: while 8-plane segments are
// 1024 blocks or fewer.  us per iteration with segments of 8 planes and more, and
// with short ones (blocks at 8 planes): FP32 48^3 (24) 17.4, 11.9; 96^3 (168) 18.1,
// 16.0; 128^3 (288) 20.3, 20.4; FP64 64^3 (64) 20.9, 14.0; 96^3 (288) 28.2, 22.9;
// 144^3 (972) 55.5, 50.9.  Beyond the line halo planes begin to count, but by the
// model below short segments still are no slower up to 3500 blocks: FP64 160 x 144 x
// 208 (1404) 75.6, 70.3; 192^3 (1728) 96.3, 90.6; FP32 320 x 256 x 256 (3456) 157,
// 147; 240 x 200 x 200, 224^3, 256^3 the same.
inline int cg_min_planes(int xytiles, int planes) { return (long long)xytiles * ((planes + 7) / 8) <= 1024 ? 2 : 8; }

// z segment of a CG sweep.  Where short segments are allowed: the one with the
// least rounds x (planes + 3 to start) x the time of a plane, which with one
// block on a CU is the latency of its loads and barriers and grows by 0.8 of
// that for each block more (us per iteration, FP32 pairs: 93 x 70 x 101 with
// segments of 2, 4, 8 planes, 500, 250, 130 blocks: 17.0, 14.2, 17.0; 96^3 with
// 3, 6, 12, 448, 224, 112 blocks: 18.7, 16.0, 20.3; 160 x 144 x 208 with 14, 24,
// 495, 297 blocks: 39, 51).
inline int cg_kchunk(int xytiles, int planes, int cap) {
    if (cg_min_planes(xytiles, planes) == 8) return choose_kchunk(xytiles, planes, cap);
    const int per_cu = std::max(1, cap / 256);
    int best = planes;
    double least = 1e300;
    for (int seg = 1; seg <= std::max(1, planes / 2); ++seg) {
        const int chunk = (planes + seg - 1) / seg;
        const long long blocks = (long long)xytiles * ((planes + chunk - 1) / chunk);
        const long long rounds = (blocks + cap - 1) / cap;
        const double on_cu = (double)std::min<long long>(per_cu, (blocks + 255) / 256);
        const double cost = (double)rounds * (chunk + 3) * std::max(1.0, 0.8 * on_cu);
        if (cost < least * 0.999) {
            least = cost;
            best = chunk;
        }
    }
    return best;
}

// Upper bound on the blocks a CG sweep over `planes` z planes uses.
inline long long max_tiled_blocks(int xytiles, int planes) {
    const int m = cg_min_planes(xytiles, planes);
    return (long long)xytiles * std::max(1, (planes + m - 1) / m);
}

}  // namespace kvs_tiling
