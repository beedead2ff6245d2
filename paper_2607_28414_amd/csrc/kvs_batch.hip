// Batched sweeps: many homogeneous instances advanced together, either one
// launch per step over every instance's tiles (captured once as a hipGraph
// and replayed), or, when every instance's state fits one workgroup's LDS,
// one persistent launch for the whole run.
#include <algorithm>
#include <functional>

#include "kvs_step2_tile.hpp"
#include "kvs_step_tile.hpp"

namespace {

// Batched homogeneous instances: one launch covers every instance's tiles
// through a work list (instance, bx, by, bz).  `parity` (launches since the
// table was built, mod 2) selects which ping-pong buffers are current; the
// absolute step n indexes each instance's envelope.
template <typename T>
struct BatchInst {
    StepArgs<T> a[2];  // [parity]: u, w current / next swapped
    const double* env;
    long long n_env;
};

template <typename T, bool VISC, bool FORCE, int BY, int VEC, int WX>
__global__ __launch_bounds__(64 * WX * BY) void batch_step_kernel(const BatchInst<T>* inst, const int4* work,
                                                                  int nwork, long long n, int parity) {
    const int t = tile_of(blockIdx.x, nwork);
    const int4 wi = work[t];
    const BatchInst<T>& bi = inst[wi.x];
    StepArgs<T> a = bi.a[parity];
    a.gn = n < bi.n_env ? T(bi.env[n]) : T(0);
    step_tile<T, false, VISC, FORCE, BY, VEC, WX>(a, wi.y, wi.z, wi.w);
}


template <typename T>
StepArgs<T> instance_args(kvs_ctx* c, int cur, int by, int vec, int wx, int zchunk) {
    const kvs_grid& g = c->grid;
    StepArgs<T> a{};
    a.u = static_cast<const T*>(c->u[cur]);
    a.w = static_cast<const T*>(c->w[cur]);
    a.un = static_cast<T*>(c->u[1 - cur]);
    a.wn = static_cast<T*>(c->w[1 - cur]);
    a.FS = static_cast<const T*>(c->FS);
    a.N = c->N;
    a.nx = (int)g.nx;
    a.ny = (int)g.ny;
    a.nz = (int)g.nz;
    a.gx = (a.nx + 64 * wx * vec - 1) / (64 * wx * vec);
    a.gy = (a.ny + by - 1) / by;
    a.kchunk = std::min(zchunk, a.nz - 2);
    a.gz = (a.nz - 2 + a.kchunk - 1) / a.kchunk;
    a.L = c->sponge_cells;
    a.invL = a.L > 0 ? T(1.0 / a.L) : T(0);
    a.ihx2 = T(1.0 / (g.hx * g.hx));
    a.ihy2 = T(1.0 / (g.hy * g.hy));
    a.ihz2 = T(1.0 / (g.hz * g.hz));
    a.G0 = T(c->G0);
    a.eta_dt0 = T(c->eta0 / c->dt);
    a.crho0 = T(c->dt * c->dt / c->rho0);
    a.inv_dt = T(1.0 / c->dt);
    a.gn = T(0);
    a.half_dt_smax = T(0.5 * c->sigma_max * c->dt);
    a.remap = 1;
    return a;
}

// Batch tile shapes: ids 0 .. kNumVariants-1 are the step-kernel variants;
// kShape192 is a 192 x 4 tile (three wavefronts per row), used only by the
// row-fitted tiling.
constexpr int kShape192 = kNumVariants;

void batch_shape_dims(int shape, int* by, int* vec, int* wx) {
    if (shape == kShape192) {
        *by = 4;
        *vec = 1;
        *wx = 3;
        return;
    }
    *by = kVariants[shape].by;
    *vec = kVariants[shape].vec;
    *wx = kVariants[shape].wx;
}

// The narrowest tile spanning an x row of nx cells: the row is then loaded
// once per tile with its Dirichlet ends as the x halo, instead of each tile
// re-reading two halo columns of its neighbours.  FP64 stays within the
// shapes whose two buffered planes fit the LDS (64 x 8, 128 x 4).
int fit_shape(int nx, bool fp64) {
    if (nx <= 64) return 1;  // 64 x 8
    if (fp64) return 5;      // 128 x 4
    if (nx <= 128) return 6; // 128 x 8
    if (nx <= 192) return kShape192;
    return 7;                // 256 x 4 (several per row beyond 256)
}

// The batch's tile shape, narrowed like the single-context launch (two
// cells per lane need every instance's nx even).
int batch_variant(const kvs_batch* b) {
    int v = b->variant;
    if (v < 0 || v >= kNumVariants) v = 1;
    bool even = true;
    for (const kvs_ctx* c : b->inst) even = even && (c->grid.nx % 2 == 0);
    return effective_variant(v, b->prec == KVS_FP64, !even);
}

// Tile shape of instance c in batch b.
int instance_shape(const kvs_batch* b, const kvs_ctx* c) {
    if (b->variant == KVS_BATCH_FIT_ROWS) return fit_shape((int)c->grid.nx, b->prec == KVS_FP64);
    return batch_variant(b);
}

// mid: the intermediate slot of a two-step launch (else null), whose values on
// the Dirichlet layer are written here
template <typename T>
__global__ void batch_probe_kernel(const BatchInst<T>* inst, const long long* probes, int np, int comp, int parity,
                                   double* out, double* mid) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= np) return;
    const StepArgs<T>& a = inst[probes[2 * p]].a[parity];
    const long long q = probes[2 * p + 1];
    out[p] = (double)a.un[comp * a.N + q];  // u after the step
    if (mid) {
        const int i = (int)(q % a.nx), j = (int)((q / a.nx) % a.ny);
        if (i == 0 || i == a.nx - 1 || j == 0 || j == a.ny - 1) mid[p] = 0.0;
    }
}

// The instances' parameter table and envelopes, staged in `host` (kept by the
// caller until the stream has copied it), and the work list.
template <typename T>
hipError_t prepare_t(kvs_batch* b, std::vector<char>& host, std::vector<int4>& work) {
    const int n = (int)b->inst.size();
    bool visc = false;
    size_t env_total = 0;
    for (int i = 0; i < n; ++i) env_total += b->inst[(size_t)i]->env.size();
    const size_t pbytes = sizeof(BatchInst<T>) * (size_t)n;
    const size_t ebytes = sizeof(double) * std::max<size_t>(env_total, 1);
    hipError_t e = hipSuccess;
    if (!b->dev_params || b->params_bytes < pbytes + ebytes) {
        b->mem.put(b->dev_params);  // after the stream's earlier steps (put synchronises)
        b->dev_params = nullptr;
        e = b->mem.get(&b->dev_params, pbytes + ebytes);
        if (e != hipSuccess) return e;
        b->params_bytes = pbytes + ebytes;
        b->graph_valid = false;  // the graph holds the old table's address
    }
    double* env_dev = reinterpret_cast<double*>(static_cast<char*>(b->dev_params) + pbytes);
    host.assign(pbytes + ebytes, 0);
    BatchInst<T>* const params = reinterpret_cast<BatchInst<T>*>(host.data());
    double* const env_host = reinterpret_cast<double*>(host.data() + pbytes);
    size_t off = 0;
    std::vector<int> shape((size_t)n);
    for (int i = 0; i < n; ++i) {
        kvs_ctx* c = b->inst[(size_t)i];
        shape[(size_t)i] = instance_shape(b, c);
        int by = 0, vec = 0, wx = 0;
        batch_shape_dims(shape[(size_t)i], &by, &vec, &wx);
        params[i].a[0] = instance_args<T>(c, c->cur, by, vec, wx, b->zchunk);
        params[i].a[1] = instance_args<T>(c, 1 - c->cur, by, vec, wx, b->zchunk);
        params[i].env = env_dev + off;
        params[i].n_env = (long long)c->env.size();
        std::copy(c->env.begin(), c->env.end(), env_host + off);
        off += c->env.size();
        visc = visc || c->viscous;
    }
    if (!b->dev_work) {
        // the work list grouped by tile shape: one launch per group
        b->groups.clear();
        for (int sh = 0; sh <= kShape192; ++sh) {
            const int first = (int)work.size();
            for (int i = 0; i < n; ++i) {
                if (shape[(size_t)i] != sh) continue;
                const StepArgs<T>& a = params[i].a[0];
                for (int bz = 0; bz < a.gz; ++bz)
                    for (int by = 0; by < a.gy; ++by)
                        for (int bx = 0; bx < a.gx; ++bx) work.push_back(make_int4(i, bx, by, bz));
            }
            if ((int)work.size() > first) b->groups.push_back({sh, first, (int)work.size() - first});
        }
    }
    e = hipMemcpyAsync(b->dev_params, host.data(), pbytes + ebytes, hipMemcpyHostToDevice, b->stream);
    if (e == hipSuccess && !b->dev_work) {
        e = b->mem.get(&b->dev_work, sizeof(int4) * work.size());
        if (e == hipSuccess)
            e = hipMemcpyAsync(b->dev_work, work.data(), sizeof(int4) * work.size(), hipMemcpyHostToDevice,
                               b->stream);
        b->nwork = (int)work.size();
    }
    if (visc != b->viscous) b->graph_valid = false;
    b->viscous = visc;
    return e;
}

template <typename T, bool VISC, bool FORCE, int BY, int VEC, int WX>
void launch_batch_shape(kvs_batch* b, long long n, int parity, const kvs_batch::Group& g) {
    hipLaunchKernelGGL((batch_step_kernel<T, VISC, FORCE, BY, VEC, WX>), dim3(g.count), dim3(64 * WX, BY), 0,
                       b->stream, static_cast<const BatchInst<T>*>(b->dev_params),
                       static_cast<const int4*>(b->dev_work) + g.off, g.count, n, parity);
}

// One launch per tile-shape group (a single group unless the tiling is
// fitted to each instance's rows).
template <typename T, bool VISC, bool FORCE>
void launch_batch_step(kvs_batch* b, long long n, int parity) {
    for (const kvs_batch::Group& g : b->groups) {
        if constexpr (sizeof(T) == 8) {
            switch (g.shape) {
                case 1: launch_batch_shape<T, VISC, FORCE, 8, 1, 1>(b, n, parity, g); break;
                case 5: launch_batch_shape<T, VISC, FORCE, 4, 1, 2>(b, n, parity, g); break;
                default: launch_batch_shape<T, VISC, FORCE, 4, 1, 1>(b, n, parity, g); break;
            }
        } else {
            switch (g.shape) {
                case 1: launch_batch_shape<T, VISC, FORCE, 8, 1, 1>(b, n, parity, g); break;
                case 2: launch_batch_shape<T, VISC, FORCE, 4, 2, 1>(b, n, parity, g); break;
                case 3: launch_batch_shape<T, VISC, FORCE, 8, 2, 1>(b, n, parity, g); break;
                case 4: launch_batch_shape<T, VISC, FORCE, 16, 1, 1>(b, n, parity, g); break;
                case 5: launch_batch_shape<T, VISC, FORCE, 4, 1, 2>(b, n, parity, g); break;
                case 6: launch_batch_shape<T, VISC, FORCE, 8, 1, 2>(b, n, parity, g); break;
                case 7: launch_batch_shape<T, VISC, FORCE, 4, 1, 4>(b, n, parity, g); break;
                case kShape192: launch_batch_shape<T, VISC, FORCE, 4, 1, 3>(b, n, parity, g); break;
                default: launch_batch_shape<T, VISC, FORCE, 4, 1, 1>(b, n, parity, g); break;
            }
        }
    }
}

// Per step of the run starting at b->step: 1 when any instance's envelope is
// non-zero there (that step launches the kernel that reads f_S).
std::vector<uint8_t> batch_force_mask(const kvs_batch* b, int64_t nsteps) {
    std::vector<uint8_t> m((size_t)nsteps, 0);
    for (int64_t q = 0; q < nsteps; ++q) {
        const int64_t n = b->step + q;
        for (const kvs_ctx* c : b->inst)
            if (n < (int64_t)c->env.size() && c->env[(size_t)n] != 0.0) {
                m[(size_t)q] = 1;
                break;
            }
    }
    return m;
}

// ---- two steps per launch ----------------------------------------------------
//
// Pairs of steps are advanced by one launch of the two-step tile
// (kvs_step2_tile.hpp, homogeneous form) over a work list of (instance, tile,
// z segment), one launch per tile shape; the result is bitwise that of two
// one-step launches.  The intermediate state's probe values are written by the
// kernel into their trace slot; the gather after the launch records the second
// step's (and the intermediate zeros of probes on the Dirichlet layer).

struct BatchInst2 {
    Step2Args<float> a2[2];  // [parity], buffers as in BatchInst::a
    const double* env;
    long long n_env;
    long long probe0;  // the instance's first probe in the flat probe list
};

// An instance's z segments: equal ones of at most `most` planes.
inline int step2_chunk(int64_t nz, int most) {
    const int planes = (int)nz - 2, seg = (planes + most - 1) / most;
    return (planes + seg - 1) / seg;
}

// A group's work list and its launch order.  Block b runs on XCD b mod 8, so
// the list is cut into eight runs of neighbouring tiles with equal work (planes
// to march and 3 to fill the queues), one per XCD, each issued longest block
// first; entries -1 fill the shorter runs.  span: when the last block ends if
// every CU marches one block at a time.
struct Step2List {
    std::vector<int4> order;
    long long span = 0;
};
Step2List step2_list(const kvs_batch* b, const std::vector<int>& members, int shape, int most) {
    std::vector<int4> work;
    std::vector<int> planes;
    long long total = 0, sum = 0;
    for (int i : members) {
        const kvs_grid& g = b->inst[(size_t)i]->grid;
        const int gx = overlap_tiles((int)g.nx, 64 * kStep2Wx[shape]), gy = overlap_tiles((int)g.ny, kStep2Rows[shape]);
        const int chunk = step2_chunk(g.nz, most), np = (int)g.nz - 2;
        for (int bz = 0; bz * chunk < np; ++bz)
            for (int by = 0; by < gy; ++by)
                for (int bx = 0; bx < gx; ++bx) {
                    work.push_back(make_int4(i, bx, by, bz));
                    planes.push_back(std::min(chunk, np - bz * chunk) + 3);
                    total += planes.back();
                }
    }
    std::vector<std::vector<int>> run(8);
    size_t longest = 0;
    for (size_t q = 0; q < work.size(); ++q) {
        run[(size_t)std::min<long long>(7, 8 * sum / std::max(1LL, total))].push_back((int)q);
        sum += planes[q];
    }
    Step2List out;
    for (auto& r : run) {
        std::stable_sort(r.begin(), r.end(), [&](int x, int y) { return planes[(size_t)x] > planes[(size_t)y]; });
        longest = std::max(longest, r.size());
        std::vector<long long> cu(32, 0);  // min-heap: when each CU of the XCD is free
        for (int q : r) {
            std::pop_heap(cu.begin(), cu.end(), std::greater<long long>());
            cu.back() += planes[(size_t)q];
            out.span = std::max(out.span, cu.back());
            std::push_heap(cu.begin(), cu.end(), std::greater<long long>());
        }
    }
    out.order.assign(8 * longest, make_int4(-1, 0, 0, 0));
    for (size_t x = 0; x < 8; ++x)
        for (size_t q = 0; q < run[x].size(); ++q) out.order[8 * q + x] = work[(size_t)run[x][q]];
    return out;
}

// The list's work in planes, spread evenly over the 256 CUs (no span is less).
long long step2_even_span(const kvs_batch* b, const std::vector<int>& members, int shape, int most) {
    long long total = 0;
    for (int i : members) {
        const kvs_grid& g = b->inst[(size_t)i]->grid;
        const long long xy = (long long)overlap_tiles((int)g.nx, 64 * kStep2Wx[shape]) * overlap_tiles((int)g.ny, kStep2Rows[shape]);
        const int chunk = step2_chunk(g.nz, most), np = (int)g.nz - 2;
        total += xy * (np + 3 * ((np + chunk - 1) / chunk));
    }
    return (total + 255) / 256;
}

// FORCE: some instance's envelope is non-zero in one of the two steps; the
// others take the tile without force.
template <bool VISC, bool FORCE, int WX, int R>
__global__ __launch_bounds__(64 * WX * R) void batch_step2_kernel(const BatchInst2* inst, const int4* work, long long n,
                                                                  int parity, double* slot) {
    __shared__ __align__(16) float lds[Step2Tile<float, false, VISC, WX, R>::LDS];
    const int4 wi = work[blockIdx.x];
    if (wi.x < 0) return;  // an XCD's list shorter than the longest
    const BatchInst2& bi = inst[wi.x];
    Step2Args<float> A = bi.a2[parity];
    A.pmid = slot != nullptr && A.rowtab != nullptr ? slot + bi.probe0 : nullptr;
    if constexpr (FORCE) {
        A.a.gn = n < bi.n_env ? (float)bi.env[n] : 0.f;
        A.gn2 = n + 1 < bi.n_env ? (float)bi.env[n + 1] : 0.f;
        if (A.a.gn != 0.f || A.gn2 != 0.f) {
            step2_tile<float, false, VISC, true, false, WX, R>(A, nullptr, lds, wi.y, wi.z, wi.w);
            return;
        }
    }
    step2_tile<float, false, VISC, false, false, WX, R>(A, nullptr, lds, wi.y, wi.z, wi.w);
}

// The tile shape with the least work over the instance's rows and columns,
// whole tiles counted.  Edges 64, 96, 128, 160 take 64 x 16 threads, 192 takes
// 192 x 5.
int step2_shape(const kvs_grid& g) {
    int best = -1;
    long long least = 0;
    for (int s = 0; s < kStep2Shapes; ++s) {
        if (!step2_offers(s, g.ny)) continue;
        const long long w = (long long)overlap_tiles((int)g.nx, 64 * kStep2Wx[s]) *
                            overlap_tiles((int)g.ny, kStep2Rows[s]) * step2_units(s);
        if (best < 0 || w < least) {
            best = s;
            least = w;
        }
    }
    return best;
}

// What the launches of a pair of steps take, us: the tile shapes follow one
// another, each with a start (code, arguments, first planes) and its span of
// planes.  Fitted to 360 ragged batches of 1 to 40 instances with the instances
// in one shape, 7 % rms.
constexpr double kStep2StartUs[kStep2Shapes] = {3.0, 1.0, 6.0, 3.0}, kStep2PlaneUs[kStep2Shapes] = {1.4, 1.7, 0.75, 1.2};

// The work list of the two-step launches: instances by tile shape, per shape
// the segment length whose launch ends first.  Measured, us per step, 24
// instances of edges 64 to 160: segments of 64 planes in XCD-contiguous order
// 375, 32 planes in this order 320; 64 instances of edges 96 to 192: 1521, and
// 1455 with 96 planes.
//
// Each instance takes the shape with the least work (step2_shape), or all of
// them one shape where by the model that ends by a fifth earlier: small
// instances in several shapes are several short launches, one after the other.
// us per step, each its own shape and all 64 x 8: lossless with force on every
// step, 28 x 79 x 6 and 105 x 11 x 7 13.2 and 7; three instances of up to
// 80 000 cells 20.2 and 6.4; 12 of up to 10^6 cells 27.8 and 7.8.  Above
// kStep2MergeUs launches are long enough to hide it (24 instances of edges 64 to
// 160: 600 us, one shape).
constexpr double kStep2MergeUs = 200.0;

void step2_plan_work(kvs_batch* b, std::vector<int4>& work) {
    struct Part {
        int shape, most;
        std::vector<int> members;
        Step2List list;
    };
    const int n = (int)b->inst.size();
    auto plan = [&](int only, double* us) {
        std::vector<Part> parts;
        *us = 0.0;
        for (int sh = 0; sh < kStep2Shapes; ++sh) {
            Part p{sh, 0, {}, {}};
            for (int i = 0; i < n; ++i) {
                const kvs_grid& g = b->inst[(size_t)i]->grid;
                if ((only >= 0 && step2_offers(only, g.ny) ? only : step2_shape(g)) == sh) p.members.push_back(i);
            }
            if (p.members.empty()) continue;
            // shorter segments have more planes to start and can only end earlier
            // while their work spread evenly does: not even listed otherwise (the
            // lists of 64 instances of edges 96 to 192 took 4 ms)
            for (int m : {128, 96, 64, 48, 32, 24, 16, 12, 8}) {
                if (p.most > 0 && step2_even_span(b, p.members, sh, m) > p.list.span) break;
                Step2List l = step2_list(b, p.members, sh, m);
                if (p.most == 0 || l.span <= p.list.span) {
                    p.list = std::move(l);
                    p.most = m;
                }
            }
            *us += kStep2StartUs[sh] + kStep2PlaneUs[sh] * (double)p.list.span;
            parts.push_back(std::move(p));
        }
        return parts;
    };
    double own = 0.0;
    std::vector<Part> best = plan(-1, &own);
    double least = 0.8 * own;
    for (int only = 0; own < kStep2MergeUs && only < kStep2Shapes; ++only) {
        double us = 0.0;
        std::vector<Part> p = plan(only, &us);
        if (us >= least) continue;
        best = std::move(p);
        least = us;
    }
    b->groups2.clear();
    b->chunk2.assign((size_t)n, 1);
    for (const Part& p : best) {
        for (int i : p.members) b->chunk2[(size_t)i] = step2_chunk(b->inst[(size_t)i]->grid.nz, p.most);
        b->groups2.push_back({p.shape, (int)work.size(), (int)p.list.order.size()});
        work.insert(work.end(), p.list.order.begin(), p.list.order.end());
    }
}

// The two-step launches' parameter table and work list, staged as above.
hipError_t prepare2(kvs_batch* b, std::vector<BatchInst2>& params, std::vector<int4>& work) {
    const int n = (int)b->inst.size();
    if (!b->dev_work2) step2_plan_work(b, work);
    params.resize((size_t)n);
    const double* env = reinterpret_cast<const double*>(static_cast<const char*>(b->dev_params) +
                                                        sizeof(BatchInst<float>) * (size_t)n);
    for (int i = 0; i < n; ++i) {
        kvs_ctx* c = b->inst[(size_t)i];
        const int64_t roff = i < (int)b->rowtab2_off.size() ? b->rowtab2_off[(size_t)i] : -1;
        const int64_t poff = i < (int)b->ptab2_off.size() ? b->ptab2_off[(size_t)i] : -1;
        for (int par = 0; par < 2; ++par) {
            Step2Args<float>& A = params[(size_t)i].a2[par];
            A = Step2Args<float>{};
            A.a = instance_args<float>(c, par == 0 ? c->cur : 1 - c->cur, 4, 1, 1, b->chunk2[(size_t)i]);
            A.a.pcomp = b->comp;
            A.rowtab = roff >= 0 ? b->dev_ptabs2 + roff : nullptr;
            A.ptab = poff >= 0 ? b->dev_ptabs2 + poff : nullptr;
        }
        params[(size_t)i].env = env;
        params[(size_t)i].n_env = (long long)c->env.size();
        env += c->env.size();
        params[(size_t)i].probe0 = b->probe_first.empty() ? 0 : (long long)b->probe_first[(size_t)i];
    }
    const size_t bytes = sizeof(BatchInst2) * (size_t)n;
    hipError_t e = hipSuccess;
    if (!b->dev_params2 || b->params2_bytes < bytes) {
        b->mem.put(b->dev_params2);
        b->dev_params2 = nullptr;
        e = b->mem.get(&b->dev_params2, bytes);
        if (e != hipSuccess) return e;
        b->params2_bytes = bytes;
        b->graph_valid = false;
    }
    e = hipMemcpyAsync(b->dev_params2, params.data(), bytes, hipMemcpyHostToDevice, b->stream);
    if (e == hipSuccess && !b->dev_work2) {
        e = b->mem.get(&b->dev_work2, sizeof(int4) * work.size());
        if (e == hipSuccess)
            e = hipMemcpyAsync(b->dev_work2, work.data(), sizeof(int4) * work.size(), hipMemcpyHostToDevice,
                               b->stream);
        b->nwork2 = (int)work.size();
    }
    return e;
}

template <bool VISC, bool FORCE, int S>
void launch_batch_step2_shape(kvs_batch* b, const kvs_batch::Group& g, long long n, int parity, double* slot) {
    hipLaunchKernelGGL((batch_step2_kernel<VISC, FORCE, kStep2Wx[S], kStep2Rows[S]>), dim3(g.count),
                       dim3(64 * kStep2Wx[S], kStep2Rows[S]), 0, b->stream, static_cast<const BatchInst2*>(b->dev_params2),
                       static_cast<const int4*>(b->dev_work2) + g.off, n, parity, slot);
}

template <bool VISC, bool FORCE>
void launch_batch_step2(kvs_batch* b, long long n, int parity, double* slot) {
    for (const kvs_batch::Group& g : b->groups2) {
        switch (g.shape) {
            case 0: launch_batch_step2_shape<VISC, FORCE, 0>(b, g, n, parity, slot); break;
            case 1: launch_batch_step2_shape<VISC, FORCE, 1>(b, g, n, parity, slot); break;
            case 2: launch_batch_step2_shape<VISC, FORCE, 2>(b, g, n, parity, slot); break;
            default: launch_batch_step2_shape<VISC, FORCE, 3>(b, g, n, parity, slot); break;
        }
    }
}

// The launches of a run: per step 0 (one-step launch), 1 (one-step launch
// reading f_S), 2 (first step of a two-step launch), 4 (the same reading f_S),
// 3 (the second step of either).
std::vector<uint8_t> batch_plan(const kvs_batch* b, int64_t nsteps, int64_t* launches) {
    std::vector<uint8_t> plan = batch_force_mask(b, nsteps);
    const bool two = b->two_ok && b->step_block == 2;
    int64_t nl = 0;
    for (int64_t q = 0; q < nsteps; ++nl) {
        if (two && q + 1 < nsteps) {
            plan[(size_t)q] = plan[(size_t)q] || plan[(size_t)(q + 1)] ? 4 : 2;
            plan[(size_t)(q + 1)] = 3;
            q += 2;
        } else {
            q += 1;
        }
    }
    *launches = nl;
    return plan;
}

template <typename T>
hipError_t capture_t(kvs_batch* b, int64_t nsteps, const std::vector<uint8_t>& plan) {
    const int np = (int)b->probe_inst.size();
    int64_t launch = 0;
    for (int64_t q = 0; q < nsteps; ++launch) {
        const int64_t n = b->step + q;
        const int parity = (int)(launch & 1);  // every launch swaps the buffers once
        int adv = 1;
        double* mid = nullptr;
        if (plan[(size_t)q] == 2 || plan[(size_t)q] == 4) {
            mid = np > 0 ? b->traces + (b->trace_steps + q) * np : nullptr;
            if constexpr (sizeof(T) == 4) {
                const bool force = plan[(size_t)q] == 4;
                if (b->viscous)
                    force ? launch_batch_step2<true, true>(b, n, parity, mid) : launch_batch_step2<true, false>(b, n, parity, mid);
                else
                    force ? launch_batch_step2<false, true>(b, n, parity, mid) : launch_batch_step2<false, false>(b, n, parity, mid);
            }
            adv = 2;
        } else {
            const bool force = plan[(size_t)q] == 1;
            if (b->viscous)
                force ? launch_batch_step<T, true, true>(b, n, parity) : launch_batch_step<T, true, false>(b, n, parity);
            else
                force ? launch_batch_step<T, false, true>(b, n, parity) : launch_batch_step<T, false, false>(b, n, parity);
        }
        if (np > 0)
            hipLaunchKernelGGL(batch_probe_kernel<T>, dim3((np + 255) / 256), dim3(256), 0, b->stream,
                               static_cast<const BatchInst<T>*>(b->dev_params),
                               static_cast<const long long*>(b->dev_probes), np, b->comp, parity,
                               b->traces + (b->trace_steps + q + adv - 1) * np, mid);
        q += adv;
    }
    return hipGetLastError();
}

// ---- persistent path for small instances -----------------------------------
//
// When every instance's whole state (u and w, three components each) fits in
// one workgroup's LDS, a batch run is one launch of one block per instance
// that advances its instance through all the steps in the kernel: the state
// lives in LDS for the whole run, the block's threads own fixed interior
// cells, and block barriers separate reading the old state from writing the
// new one; probe values are written after every step.  The per-cell arithmetic
// is the step kernel's (same operand order, sponge factors and FP32
// reciprocal), so one launch replaces two launches per step and the run is
// bound by the latency of a step, not by launches.
//
// A step is one chain: LDS reads, the update of a thread, LDS writes, barrier.
// Where three times the threads fit a block, each component of a cell has its
// own thread (SPLIT): the update is a third as long and the SIMDs are evenly
// filled (299 cells are five wavefronts on four SIMDs, as components fifteen).
// A line keeps only its own nodes in LDS, twice, and needs one barrier a step.
// 16 lines of 301 nodes, 16000 steps: 6.70 -> 5.07 ms (0.32 us a step).
constexpr int kSmallMaxThreads = 1024;
constexpr int kSmallChunk = 64;  // steps whose envelope and probe values are staged in LDS at a time
constexpr size_t kSmallMaxLds = 150 * 1024;

// LINE: every instance is a line (ny = nz = 3): the y and z neighbours of an
// interior node lie on the Dirichlet layer and are exactly 0, so they are
// taken as the constant 0 instead of read (the same arithmetic).
template <typename T, bool VISC, int CPT, bool LINE, bool SPLIT>
__global__ __launch_bounds__(kSmallMaxThreads) void batch_small_kernel(const BatchInst<T>* inst, const long long* probes,
                                                                       const long long* probe_first, int np, int comp,
                                                                       double* traces, long long step0,
                                                                       long long nsteps) {
    extern __shared__ __align__(16) unsigned char small_lds[];
    constexpr int NC = SPLIT ? 1 : 3;    // components of a thread, from cb on
    constexpr int NB = LINE ? 2 : 1;     // copies of the state
    const int nthr = blockDim.x, ncell = SPLIT ? nthr / 3 : nthr;
    const int cb = SPLIT ? __builtin_amdgcn_readfirstlane(threadIdx.x / (unsigned)ncell) : 0;
    const int tcell = (int)threadIdx.x - cb * ncell;
    // everything the step loop needs is read once: the loop's stores to the
    // traces would otherwise make the compiler re-read it every step
    const StepArgs<T> a = inst[blockIdx.x].a[0];  // parity 0: the buffers current at the start of the run
    // the envelope through a global-memory pointer: a generic (flat) load
    // could alias LDS, which would order every LDS access behind it
    typedef const __attribute__((address_space(1))) double* genv_t;
    const genv_t env = (genv_t)inst[blockIdx.x].env;
    const long long n_env = inst[blockIdx.x].n_env;
    const int N = (int)a.N;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int S = LINE ? nx : N;                // nodes of a component in LDS
    T* su = reinterpret_cast<T*>(small_lds);    // [NB][3][S]
    T* sw = su + NB * 3 * S;                    // [NB][3][S]
    T* senv = sw + NB * 3 * S;                  // [kSmallChunk]: the chunk's envelope values; LINE: and a 0
    const long long pf = np > 0 ? probe_first[blockIdx.x] : 0;
    const int npi = np > 0 ? (int)(probe_first[blockIdx.x + 1] - pf) : 0;
    T* strace = senv + kSmallChunk + (LINE ? 1 : 0);                    // [kSmallChunk][npi]: probe values
    int* sprobe = reinterpret_cast<int*>(strace + kSmallChunk * npi);  // this instance's probe cells
    const int row = LINE ? nx * (1 + ny) : 0;  // node 0 of the row kept
    if constexpr (LINE) {
        for (int c = 0; c < 3; ++c)
            for (int i = threadIdx.x; i < S; i += nthr) {
                su[c * S + i] = su[(3 + c) * S + i] = a.u[c * N + row + i];
                sw[c * S + i] = sw[(3 + c) * S + i] = a.w[c * N + row + i];
            }
    } else {
        for (int q = threadIdx.x; q < 3 * N; q += nthr) {
            su[q] = a.u[q];
            sw[q] = a.w[q];
        }
    }
    if (LINE && threadIdx.x == 0) senv[kSmallChunk] = T(0);
    for (int p = threadIdx.x; p < npi; p += nthr) {
        const int q = (int)probes[2 * (pf + p) + 1];
        // off the row kept: a node of the Dirichlet layer, 0
        sprobe[p] = !LINE ? comp * N + q : q >= row && q < row + nx ? comp * S + q - row : -1;
    }
    const int nxi = nx - 2, nyi = ny - 2, nint = nxi * nyi * (nz - 2);
    const int sy = nx, sz = nx * ny;
    // owned cells: their index, sponge factors, f_S and own u, w (registers)
    int cell[CPT];
    T a1[CPT], a2[CPT], fs[CPT][NC], ur[CPT][NC], wr[CPT][NC];
#pragma unroll
    for (int m = 0; m < CPT; ++m) {
        const int t = tcell + m * ncell;
        cell[m] = -1;
        a1[m] = a2[m] = T(0);
#pragma unroll
        for (int c = 0; c < NC; ++c) fs[m][c] = ur[m][c] = wr[m][c] = T(0);
        if (t < nint) {
            const int i = 1 + t % nxi, j = 1 + (t / nxi) % nyi, k = 1 + t / (nxi * nyi);
            const int q = i + nx * (j + ny * k);
            cell[m] = q - row;
            const T r = a.L > 0 ? max(max(ramp<T>(i, nx, a.L, a.invL), ramp<T>(j, ny, a.L, a.invL)),
                                      ramp<T>(k, nz, a.L, a.invL))
                                : T(0);
            const T s = a.half_dt_smax * r;
            const T inv1ps = rcp_fast<T>(T(1) + s);
            a1[m] = (T(1) - s) * inv1ps;
            a2[m] = a.crho0 * inv1ps;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                fs[m][c] = a.FS[(cb + c) * a.N + q];
                ur[m][c] = a.u[(cb + c) * a.N + q];
                wr[m][c] = a.w[(cb + c) * a.N + q];
            }
        }
    }
    const T gx = a.G0 * a.ihx2, gy = a.G0 * a.ihy2, gz = a.G0 * a.ihz2;
    const T ihx2 = a.ihx2, ihy2 = a.ihy2, ihz2 = a.ihz2, eta_dt = a.eta_dt0;
    for (long long st0 = 0; st0 < nsteps; st0 += kSmallChunk) {
        const int cn = (int)min((long long)kSmallChunk, nsteps - st0);
        // the chunk's envelope values: global memory is touched only here and
        // in the flush of the chunk's probe values below, so the step loop
        // itself waits on LDS alone
        for (int q = threadIdx.x; q < cn; q += nthr) {
            const long long n = step0 + st0 + q;
            senv[q] = n < n_env ? T(env[n]) : T(0);
        }
        lds_barrier();
        for (int sc = 0; sc < cn; ++sc) {
            const T gn = senv[sc];
            const T* ru = su + (LINE ? (sc & 1) * 3 * S : 0);  // chunks are of even length but the last
            const T* rw = sw + (LINE ? (sc & 1) * 3 * S : 0);
            T* nu = su + (LINE ? (~sc & 1) * 3 * S : 0);
            T* nw = sw + (LINE ? (~sc & 1) * 3 * S : 0);
#pragma unroll
            for (int m = 0; m < CPT; ++m) {
                if (cell[m] < 0) continue;
                const int c0 = cell[m];
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const T* u = ru + (cb + c) * S;
                    const T uc = ur[m][c];
                    const T uyp = LINE ? T(0) : u[c0 + sy], uym = LINE ? T(0) : u[c0 - sy];
                    const T uzp = LINE ? T(0) : u[c0 + sz], uzm = LINE ? T(0) : u[c0 - sz];
                    T acc = gx * (u[c0 + 1] - uc) - gx * (uc - u[c0 - 1]) + gy * (uyp - uc) - gy * (uc - uym)
                          + gz * (uzp - uc) - gz * (uc - uzm);
                    const T wc = wr[m][c];
                    if constexpr (VISC) {
                        const T* w = rw + (cb + c) * S;
                        const T wyp = LINE ? T(0) : w[c0 + sy], wym = LINE ? T(0) : w[c0 - sy];
                        const T wzp = LINE ? T(0) : w[c0 + sz], wzm = LINE ? T(0) : w[c0 - sz];
                        const T lw = (w[c0 + 1] + w[c0 - 1] - T(2) * wc) * ihx2 + (wyp + wym - T(2) * wc) * ihy2
                                   + (wzp + wzm - T(2) * wc) * ihz2;
                        acc += eta_dt * lw;
                    }
                    if (gn != T(0)) acc += gn * fs[m][c];
                    const T wnew = a1[m] * wc + a2[m] * acc;
                    wr[m][c] = wnew;
                    ur[m][c] = uc + wnew;
                }
            }
            if constexpr (!LINE) lds_barrier();  // every read of the old state is done
#pragma unroll
            for (int m = 0; m < CPT; ++m)
                if (cell[m] >= 0)
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        nu[(cb + c) * S + cell[m]] = ur[m][c];
                        if constexpr (VISC) nw[(cb + c) * S + cell[m]] = wr[m][c];
                    }
            lds_barrier();  // the new state is complete
            for (int p = threadIdx.x; p < npi; p += nthr)
                strace[sc * npi + p] = *(!LINE || sprobe[p] >= 0 ? nu + sprobe[p] : senv + kSmallChunk);
        }
        lds_barrier();  // the chunk's probe values are complete
        for (int r = threadIdx.x >> 6; r < cn; r += nthr >> 6)
            for (int p = threadIdx.x & 63; p < npi; p += 64)
                traces[(st0 + r) * (long long)np + pf + p] = (double)strace[r * npi + p];
        // the next chunk writes senv and strace only after the barrier that
        // follows its envelope load, i.e. after these reads
    }
    // the run leaves the instance's state in the buffers current after nsteps
    T* du = (nsteps & 1) ? a.un : const_cast<T*>(a.u);
    T* dw = (nsteps & 1) ? a.wn : const_cast<T*>(a.w);
    if constexpr (LINE) {
        // the cells from the registers; the Dirichlet layer of both buffers is 0
#pragma unroll
        for (int m = 0; m < CPT; ++m)
            if (cell[m] >= 0)
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    du[(cb + c) * a.N + row + cell[m]] = ur[m][c];
                    dw[(cb + c) * a.N + row + cell[m]] = wr[m][c];
                }
    } else {
        // w in LDS is stale without viscosity: the registers hold it
#pragma unroll
        for (int m = 0; m < CPT; ++m)
            if (cell[m] >= 0)
#pragma unroll
                for (int c = 0; c < NC; ++c) sw[(cb + c) * N + cell[m]] = wr[m][c];
        lds_barrier();
        for (int q = threadIdx.x; q < 3 * N; q += nthr) {
            du[q] = su[q];
            dw[q] = sw[q];
        }
    }
}

// LDS of the persistent kernel: the state (6 N values), a chunk's envelope
// and probe values, and the probe cells, for the instance with the most
// probes.  (A line takes less: two copies of a ninth of that state, and a 0.)
template <typename T>
size_t small_lds_bytes(const kvs_batch* b, const kvs_ctx* c) {
    int64_t most = 0;
    for (size_t i = 0; i + 1 < b->probe_first.size(); ++i)
        most = std::max<int64_t>(most, b->probe_first[i + 1] - b->probe_first[i]);
    return (6 * (size_t)c->N + kSmallChunk * (1 + (size_t)most)) * sizeof(T) + sizeof(int) * (size_t)most;
}

// Threads per workgroup (a multiple of 64, at most 1024, enough for one
// interior cell each where possible) and cells per thread.
template <typename T>
bool small_fits(const kvs_batch* b, int* cpt, int* threads) {
    long long most = 1;
    for (const kvs_ctx* c : b->inst) {
        const kvs_grid& g = c->grid;
        if (small_lds_bytes<T>(b, c) > kSmallMaxLds) return false;
        most = std::max<long long>(most, (g.nx - 2) * (g.ny - 2) * (g.nz - 2));
    }
    const int thr = (int)std::min<long long>(kSmallMaxThreads, 64 * ((most + 63) / 64));
    const long long need = (most + thr - 1) / thr;
    if (need > 8) return false;
    *threads = thr;
    *cpt = need <= 1 ? 1 : need <= 2 ? 2 : need <= 4 ? 4 : 8;
    return true;
}

template <typename T, bool VISC, int CPT, bool LINE, bool SPLIT = false>
hipError_t launch_small_shape(kvs_batch* b, int64_t nsteps, int threads) {
    size_t lds = 0;
    for (const kvs_ctx* c : b->inst) lds = std::max(lds, small_lds_bytes<T>(b, c));
    static bool attr_set = false;  // one attribute call per instantiation
    if (!attr_set) {
        const hipError_t e = hipFuncSetAttribute((const void*)batch_small_kernel<T, VISC, CPT, LINE, SPLIT>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSmallMaxLds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int np = (int)b->probe_inst.size();
    const long long* pr = static_cast<const long long*>(b->dev_probes);
    double* tr = np > 0 ? b->traces + b->trace_steps * np : nullptr;
    hipLaunchKernelGGL((batch_small_kernel<T, VISC, CPT, LINE, SPLIT>), dim3((unsigned)b->inst.size()), dim3(SPLIT ? 3 * threads : threads), lds,
                       b->stream, static_cast<const BatchInst<T>*>(b->dev_params), pr, np > 0 ? pr + 2 * np : nullptr,
                       np, b->comp, tr, (long long)b->step, (long long)nsteps);
    return hipGetLastError();
}

template <typename T, bool VISC>
hipError_t launch_small(kvs_batch* b, int64_t nsteps, int cpt, int threads) {
    bool line = true;
    for (const kvs_ctx* c : b->inst) line = line && c->grid.ny == 3 && c->grid.nz == 3;
    const bool split = cpt == 1 && 3 * threads <= kSmallMaxThreads;
    if (line) {
        if (split) return launch_small_shape<T, VISC, 1, true, true>(b, nsteps, threads);
        switch (cpt) {
            case 1: return launch_small_shape<T, VISC, 1, true>(b, nsteps, threads);
            case 2: return launch_small_shape<T, VISC, 2, true>(b, nsteps, threads);
            case 4: return launch_small_shape<T, VISC, 4, true>(b, nsteps, threads);
            default: return launch_small_shape<T, VISC, 8, true>(b, nsteps, threads);
        }
    }
    switch (cpt) {
        case 1: return launch_small_shape<T, VISC, 1, false>(b, nsteps, threads);
        case 2: return launch_small_shape<T, VISC, 2, false>(b, nsteps, threads);
        case 4: return launch_small_shape<T, VISC, 4, false>(b, nsteps, threads);
        default: return launch_small_shape<T, VISC, 8, false>(b, nsteps, threads);
    }
}

template <typename T>
hipError_t run_small_t(kvs_batch* b, int64_t nsteps, int cpt, int threads) {
    return b->viscous ? launch_small<T, true>(b, nsteps, cpt, threads) : launch_small<T, false>(b, nsteps, cpt, threads);
}

}  // namespace

bool kvs_batch_small_path(const kvs_batch* b) {
    int cpt = 0, thr = 0;
    return b->small_ok && (b->prec == KVS_FP32 ? small_fits<float>(b, &cpt, &thr) : small_fits<double>(b, &cpt, &thr));
}

// One uncaptured step launch that only rewrites the next buffers (parity 0,
// no force): used to time tile shapes without advancing the state.
hipError_t kvs_batch_trial_launch(kvs_batch* b) {
    if (b->prec == KVS_FP32) {
        b->viscous ? launch_batch_step<float, true, false>(b, b->step, 0)
                   : launch_batch_step<float, false, false>(b, b->step, 0);
    } else {
        b->viscous ? launch_batch_step<double, true, false>(b, b->step, 0)
                   : launch_batch_step<double, false, false>(b, b->step, 0);
    }
    return hipGetLastError();
}

bool kvs_batch_step2_supported(const kvs_batch* b) {
    if (b->prec != KVS_FP32 || !b->probes2_ok || b->inst.empty()) return false;
    for (const kvs_ctx* c : b->inst)
        if (!c->have_material || c->N >= ((int64_t)1 << 31) || c->grid.nx * c->grid.ny >= ((int64_t)1 << 30) - 1024 ||
            c->npeak > 0 || c->pml_cells > 0)
            return false;
    return true;
}

bool kvs_batch_two_step_supported(const kvs_batch* b) {
    if (!kvs_batch_step2_supported(b)) return false;
    bool visc = false;
    for (const kvs_ctx* c : b->inst) {
        if (c->grid.nx > 256) return false;
        visc = visc || c->viscous;
    }
    return visc;
}

hipError_t kvs_batch_prepare(kvs_batch* b, int64_t nsteps) {
    std::vector<char> host;
    std::vector<BatchInst2> params2;
    std::vector<int4> work, work2;
    hipError_t e = b->prec == KVS_FP32 ? prepare_t<float>(b, host, work) : prepare_t<double>(b, host, work);
    // tables of two-step launches only for a run that has some: made and copied
    // for every run of a persistent batch too, they took 10 to 25 of its 50 to 80 us
    b->two_ok = nsteps > 1 && b->step_block == 2 && !kvs_batch_small_path(b) && kvs_batch_step2_supported(b);
    if (e == hipSuccess && b->two_ok) e = prepare2(b, params2, work2);
    const hipError_t s = hipStreamSynchronize(b->stream);  // the staging vectors end here
    return e != hipSuccess ? e : s;
}

hipError_t kvs_batch_run(kvs_batch* b, int64_t nsteps, int64_t* flips) {
    int cpt = 0, thr = 0;
    *flips = nsteps;
    if (b->small_ok && (b->prec == KVS_FP32 ? small_fits<float>(b, &cpt, &thr) : small_fits<double>(b, &cpt, &thr)))
        return b->prec == KVS_FP32 ? run_small_t<float>(b, nsteps, cpt, thr) : run_small_t<double>(b, nsteps, cpt, thr);
    // Replay the cached graph when it was captured for the same start step,
    // step count, trace slot and launch plan (which steps read f_S, which are
    // paired into two-step launches; the parameter tables and envelopes it
    // reads were refreshed in place by kvs_batch_prepare); otherwise capture a
    // new one.
    std::vector<uint8_t> force_mask = batch_plan(b, nsteps, flips);
    const bool hit = b->graph_valid && b->graph && b->graph_start == b->step && b->graph_steps == nsteps &&
                     b->graph_trace0 == b->trace_steps && b->graph_force == force_mask;
    hipError_t e = hipSuccess;
    if (!hit) {
        if (b->graph) (void)hipGraphExecDestroy(b->graph);
        b->graph = nullptr;
        b->graph_valid = false;
        hipGraph_t graph = nullptr;
        e = hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal);
        if (e == hipSuccess) {
            const hipError_t le = b->prec == KVS_FP32 ? capture_t<float>(b, nsteps, force_mask)
                                                      : capture_t<double>(b, nsteps, force_mask);
            e = hipStreamEndCapture(b->stream, &graph);
            if (e == hipSuccess) e = le;
        }
        if (e == hipSuccess) e = hipGraphInstantiate(&b->graph, graph, nullptr, nullptr, 0);
        if (graph) (void)hipGraphDestroy(graph);
        if (e != hipSuccess) return e;
        b->graph_valid = true;
        b->graph_start = b->step;
        b->graph_steps = nsteps;
        b->graph_trace0 = b->trace_steps;
        b->graph_force.swap(force_mask);
    }
    return hipGraphLaunch(b->graph, b->stream);
}
