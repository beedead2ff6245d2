"""Two-step launches beyond the contexts that kvs_step_blocking_applies names:
FP64, lossless media, peak maps, force on both steps, rows of several
overlapping tiles and grids at the tiles' edges.  The state, the traces (probes
on the Dirichlet layer included) and the peak maps are bitwise those of
one-step launches."""
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


def run(kvs, grid, precision, het, visc, peaks, blocking, zchunk):
    nx, ny, nz = grid[:3]
    shape = (nz, ny, nx)
    rng = np.random.default_rng(nx + ny + nz)
    ctx = kvs.kvs_create(grid, precision=precision, sponge_cells=2 if min(shape) > 6 else 0)
    try:
        eta = 0.7 if visc else 0.0
        if het:
            kvs.kvs_set_material(ctx, rng.uniform(1e3, 1e4, shape), rng.uniform(900, 1100, shape),
                                 eta * rng.uniform(0.2, 1.0, shape))
        else:
            kvs.kvs_set_material_uniform(ctx, 3e3, 1030.0, eta)
        kvs.kvs_set_dt(ctx, 0.4 * kvs.kvs_stable_dt(ctx))
        kvs.kvs_set_projected_force(ctx, 1e2 * rng.standard_normal((3,) + shape))
        kvs.kvs_set_envelope(ctx, [1.0, 0.5, 0.0, -0.7, 0.0, 0.0, 0.3])  # pairs with force in either step, both, none
        probes = [[i, ny // 2, nz // 2] for i in range(nx)] + [[nx // 2, j, 1] for j in range(ny)]
        kvs.kvs_set_probes(ctx, probes, 3)
        planes = [(0, nx // 2), (1, 1), (2, nz // 2), (2, 1), (0, nx - 1)] if peaks else []
        planes = list(dict.fromkeys(planes))
        if peaks:
            kvs.kvs_set_peak_planes(ctx, planes)
        if zchunk:
            kvs.kvs_set_step_tuning(ctx, 0, zchunk)
        kvs.kvs_set_step_blocking(ctx, blocking)
        kvs.kvs_set_state(ctx, 1e-6 * rng.standard_normal((3,) + shape), 1e-8 * rng.standard_normal((3,) + shape), 0)
        for n in (4, 1, 6):
            kvs.kvs_step(ctx, n)
        u, w, step = kvs.kvs_get_state(ctx, shape)
        tr = kvs.kvs_read_traces(ctx, len(probes), 3)
        return [u, w, tr] + [kvs.kvs_peak_map(ctx, a, i, grid) for a, i in planes] + [np.array(step)]
    finally:
        kvs.kvs_destroy(ctx)


@pytest.mark.parametrize("nx,ny,nz,zchunk", [
    (3, 3, 3, 0),       # one interior cell
    (66, 18, 5, 0),     # 64 x 16 interior cells: one tile wall to wall
    (67, 19, 12, 3),    # one cell more, short z segments
    (130, 10, 9, 0),    # 128 interior cells; eight rows
    (131, 11, 8, 0),
    (194, 7, 10, 4),    # 192 and five
    (195, 40, 9, 0),
    (257, 21, 7, 0),    # longer than any tile
    (390, 12, 20, 7),
])
@pytest.mark.parametrize("het", [True, False])
@pytest.mark.parametrize("visc", [True, False])
@pytest.mark.parametrize("fp64,peaks", [(False, False), (False, True), (True, False), (True, True)])
def test_two_step_tiles_match_one_step_bitwise(kvs, nx, ny, nz, zchunk, het, visc, fp64, peaks):
    grid = (nx, ny, nz, 0.25e-3, 0.3e-3, 0.2e-3)
    prec = kvs.KVS_FP64 if fp64 else kvs.KVS_FP32
    print(f"case two-step tiles {grid[:3]} zchunk {zchunk} het {het} visc {visc} fp64 {fp64} peaks {peaks}", flush=True)
    ref = run(kvs, grid, prec, het, visc, peaks, 1, zchunk)
    got = run(kvs, grid, prec, het, visc, peaks, 2, zchunk)
    assert len(ref) == len(got)
    for n, (a, b) in enumerate(zip(ref, got)):
        assert np.array_equal(a, b), n
    assert np.max(np.abs(ref[0])) > 0


def test_lossless_and_wide_batches_match_one_step_bitwise(kvs):
    """Batches of lossless instances, and of rows longer than a tile, with
    pushes of different lengths and probes on the Dirichlet layer."""
    h = 0.25e-3
    for eta, shapes in ((0.0, [(40, 20, 12), (66, 18, 9)]), (0.6, [(300, 10, 8), (131, 7, 20), (194, 30, 6)])):
        out = []
        for blocking in (1, 2):
            b = kvs.kvs_batch_create([s + (h, h, h) for s in shapes], precision=kvs.KVS_FP32, sponge_cells=2,
                                     sponge_sigma_max=500.0)
            try:
                kvs.kvs_batch_set_persistent(b, False)
                for i, s in enumerate(shapes):
                    c = kvs.kvs_batch_instance(b, i)
                    rng = np.random.default_rng(i)
                    kvs.kvs_set_material_uniform(c, 3e3 + 500 * i, 1000.0, eta)
                    kvs.kvs_set_dt(c, 0.4 * kvs.kvs_stable_dt(c))
                    kvs.kvs_set_projected_force(c, 1e2 * rng.standard_normal((3,) + s[::-1]))
                    kvs.kvs_set_envelope(c, np.ones(2 + 3 * i))
                    kvs.kvs_batch_set_probes(b, i, [[x, s[1] // 2, 2] for x in range(s[0])])
                kvs.kvs_batch_set_component(b, 1)
                kvs.kvs_batch_set_step_blocking(b, blocking)
                res = []
                for _ in range(2):  # the second run replays the captured launches
                    kvs.kvs_batch_reset(b)
                    kvs.kvs_batch_step(b, 9)
                    kvs.kvs_batch_step(b, 4)
                    res += [kvs.kvs_batch_read_traces(b, i, s[0]) for i, s in enumerate(shapes)]
                    res += [a for i, s in enumerate(shapes)
                            for a in kvs.kvs_get_state(kvs.kvs_batch_instance(b, i), s[::-1])[:2]]
                out.append(res)
            finally:
                kvs.kvs_batch_destroy(b)
        for n, (x, y) in enumerate(zip(*out)):
            assert np.array_equal(x, y), (eta, n)
        assert max(np.max(np.abs(x)) for x in out[0]) > 0
