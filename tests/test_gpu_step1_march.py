"""The one-step kernel of contexts with an absorbing layer against the tiled
one-step kernel (reached by a z split of one's own): the same operations in the
same order, so the states, memories and traces are the same bits.  Rows at
the edges of each tile width and beyond the widest, whole and broken tiles of
rows, few planes and several segments."""
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


def run(kvs, dims, hetero, eta, zchunk):
    nx, ny, nz = dims
    h = 0.25e-3
    rng = np.random.default_rng([nx, ny, nz])
    ctx = kvs.kvs_create((nx, ny, nz, h, h, h), precision=kvs.KVS_FP32, sponge_cells=0)
    try:
        if hetero:
            shape = (nz, ny, nx)
            kvs.kvs_set_material(ctx, 1e3 * (1 + 5 * rng.random(shape)), 950 + 100 * rng.random(shape),
                                 eta * rng.random(shape))
        else:
            kvs.kvs_set_material_uniform(ctx, 3e3, 1000.0, eta)
        kvs.kvs_set_dt(ctx, 0.4 * kvs.kvs_stable_dt(ctx))
        fs = np.zeros((3, nz, ny, nx))
        fs[:, 1:-1, 1:-1, 1:-1] = 1e3 * rng.standard_normal((3, nz - 2, ny - 2, nx - 2))
        kvs.kvs_set_projected_force(ctx, fs)
        kvs.kvs_set_envelope(ctx, np.array([1.0, 0.5, 0.0, 0.25]))
        kvs.kvs_set_pml(ctx, 3)
        kvs.kvs_set_probes(ctx, [[i, ny // 2, nz // 2] for i in range(nx)] + [[0, 0, 0]], 3)
        if zchunk:
            kvs.kvs_set_step_tuning(ctx, 0, zchunk, 1)
        kvs.kvs_step(ctx, 5)
        kvs.kvs_step(ctx, 4)
        u, w, step = kvs.kvs_get_state(ctx, (nz, ny, nx))
        return u, w, step, kvs.kvs_read_traces(ctx, nx + 1, 3)
    finally:
        kvs.kvs_destroy(ctx)


@pytest.mark.parametrize("hetero", [True, False], ids=["maps", "uniform"])
@pytest.mark.parametrize("eta", [0.8, 0.0], ids=["viscous", "lossless"])
@pytest.mark.parametrize("dims", [(9, 9, 9), (65, 9, 17), (66, 10, 11), (129, 37, 64), (130, 12, 30), (193, 42, 29), (194, 14, 9), (257, 15, 33), (258, 10, 9)], ids=str)
def test_same_bits_as_tiled_kernel(kvs, dims, eta, hetero):
    print(f"case one-step march {dims} eta {eta} hetero {hetero}", flush=True)
    a, b = run(kvs, dims, hetero, eta, 0), run(kvs, dims, hetero, eta, 5)
    assert a[2] == b[2] == 9 and np.abs(a[0]).max() > 0
    for x, y in zip((a[0], a[1], np.asarray(a[3])), (b[0], b[1], np.asarray(b[3]))):
        assert np.array_equal(x, y)
