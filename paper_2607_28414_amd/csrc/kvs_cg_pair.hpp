// Two CG iterations per pair of sweeps for FP32 storage of direction and
// residual (kvs_cg_pair.hip), as the projection's host loop launches them.
#pragma once

#include "kvs_internal.hpp"
#include "kvs_tiling.hpp"

// One pair on explicit buffers: r_in, p_in (the residual and the direction
// that the last pair stored) are read, r_out, p_out written, phi updated;
// outer layers of all of them are 0 and are not written.
struct CgPair {
    hipStream_t stream;
    const float* r_in;
    const float* p_in;
    float* r_out;
    float* p_out;
    double* phi;
    CgState* st;       // two copies (folded scalars alternate); current before and, with `last`, after
    double* partials;  // KVS_CG_SUMS npart
    int npart;
    bool last;         // the host reads the control block next
};

// Largest number of blocks a pair's sweeps use on a grid (partials per sum).
int64_t kvs_cg_pair_blocks_max(const kvs_grid& g);
void kvs_cg_pair_launch(const kvs_grid& g, const CgPair& c);
