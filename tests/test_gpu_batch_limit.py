"""Batches whose LDS is just what the persistent kernel takes: 6 N values of
state, 64 of the envelope and 64 per probe, and 4 bytes per probe, at most
150 KB = 153600 bytes.  Both grids come to 153596 bytes in FP64; with a probe
more they are over."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kvs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2607_28414_amd import kvs as k
    k.lib()
    return k


def run(kvs, dims, nprobes, persistent):
    nx, ny, nz = dims
    h = 0.25e-3
    b = kvs.kvs_batch_create([dims + (h, h, h)], precision=kvs.KVS_FP64, sponge_cells=2)
    try:
        kvs.kvs_batch_set_persistent(b, persistent)
        ctx = kvs.kvs_batch_instance(b, 0)
        kvs.kvs_set_material_uniform(ctx, 4e3, 1000.0, 0.4)
        kvs.kvs_set_dt(ctx, 0.4 * kvs.kvs_stable_dt(ctx))
        rng = np.random.default_rng(nx)
        fs = np.zeros((3, nz, ny, nx))
        fs[:, 1:-1, 1:-1, 1:-1] = 1e3 * rng.standard_normal((3, nz - 2, ny - 2, nx - 2))
        kvs.kvs_set_projected_force(ctx, fs)
        kvs.kvs_set_envelope(ctx, rng.standard_normal(70))
        kvs.kvs_batch_set_probes(b, 0, [[nx - 2 - p % (nx - 2), 1 + p % (ny - 2), nz - 2] for p in range(nprobes)])
        uses = kvs.kvs_batch_uses_persistent(b)
        for m in (63, 66, 5):
            kvs.kvs_batch_step(b, m)
        return uses, kvs.kvs_batch_read_traces(b, 0, nprobes), kvs.kvs_get_state(ctx, (nz, ny, nx))[:2]
    finally:
        kvs.kvs_batch_destroy(b)


@pytest.mark.parametrize("dims,nprobes", [((7, 11, 41), 3), ((346, 3, 3), 7)], ids=str)
def test_fullest_accepted_instance(kvs, dims, nprobes):
    """The persistent path is taken and agrees with the per-step launches, whose
    arithmetic is the same up to contraction (FP64, 1e-12 of the largest value)."""
    N = dims[0] * dims[1] * dims[2]
    assert 8 * (6 * N + 64 * (1 + nprobes)) + 4 * nprobes == 153596
    print(f"case fullest persistent instance {dims} probes {nprobes}", flush=True)
    uses, tr, st = run(kvs, dims, nprobes, True)
    assert uses
    assert not run(kvs, dims, nprobes + 1, True)[0]
    uses0, tr0, st0 = run(kvs, dims, nprobes, False)
    assert not uses0 and np.abs(tr0).max() > 0
    assert np.abs(tr - tr0).max() <= 1e-12 * np.abs(tr0).max()
    for a, a0 in zip(st, st0):
        assert np.abs(a - a0).max() <= 1e-12 * np.abs(a0).max()


@pytest.mark.parametrize("persistent,blocking,steps,tables", [
    (True, 2, 40, 2),    # the run is one launch: parameters and the one-step work list
    (False, 1, 40, 2),
    (False, 2, 1, 2),
    (False, 2, 2, 4),    # and those of the two-step launches
])
@pytest.mark.parametrize("eta", [0.5, 0.0], ids=["viscous", "lossless"])
def test_two_step_tables_only_where_they_are_used(kvs, persistent, blocking, steps, tables, eta):
    """Device buffers that the first run takes from the batch's allocator."""
    import torch
    h = 0.25e-3
    print(f"case batch tables persistent {persistent} blocking {blocking} steps {steps}", flush=True)
    stream = torch.cuda.Stream()
    mem = kvs.TorchAllocator(0, stream.cuda_stream)
    b = kvs.kvs_batch_create([(40, 3, 3, h, h, h), (9, 8, 7, h, h, h)], precision=kvs.KVS_FP32, sponge_cells=2,
                             stream=stream.cuda_stream, allocator=mem)
    try:
        kvs.kvs_batch_set_persistent(b, persistent)
        kvs.kvs_batch_set_step_blocking(b, blocking)
        for i in range(2):
            c = kvs.kvs_batch_instance(b, i)
            kvs.kvs_set_material_uniform(c, 4e3, 1000.0, eta)
            kvs.kvs_set_dt(c, 0.4 * kvs.kvs_stable_dt(c))
        before = mem.allocs
        kvs.kvs_batch_step(b, steps)
        assert mem.allocs - before == tables
    finally:
        kvs.kvs_batch_destroy(b)
