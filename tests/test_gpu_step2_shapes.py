"""Every tile of the two-step kernel at its own edges, and which kernel and
tile a step takes.  The tile is asked for and what was launched is checked, so
that a lost dispatch cannot pass by comparing one-step launches with
themselves.  Large grids take 128 x 8 and 64 x 16, the small grids of the other
tests mostly 64 x 8."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TILES = [(128, 8), (64, 16), (64, 8), (192, 5)]


@pytest.fixture(scope="module")
def kvs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2607_28414_amd import kvs as k
    k.lib()
    return k


def run(kvs, dims, prec, het, visc, peaks, blocking, tile, zchunk):
    nx, ny, nz = dims
    shape = (nz, ny, nx)
    rng = np.random.default_rng([nx, ny, nz])
    ctx = kvs.kvs_create(dims + (0.25e-3, 0.3e-3, 0.2e-3), precision=prec, sponge_cells=2)
    try:
        eta = 0.7 if visc else 0.0
        if het:
            kvs.kvs_set_material(ctx, rng.uniform(1e3, 1e4, shape), rng.uniform(900, 1100, shape),
                                 eta * rng.uniform(0.2, 1.0, shape))
        else:
            kvs.kvs_set_material_uniform(ctx, 3e3, 1030.0, eta)
        kvs.kvs_set_dt(ctx, 0.4 * kvs.kvs_stable_dt(ctx))
        kvs.kvs_set_projected_force(ctx, 1e2 * rng.standard_normal((3,) + shape))
        # pairs with force on both steps, on the second, on none
        kvs.kvs_set_envelope(ctx, [1.0, 0.5, 0.0, -0.7, 0.3])
        probes = [[i, ny // 2, nz // 2] for i in range(nx)] + [[nx // 2, j, 1] for j in range(ny)]
        kvs.kvs_set_probes(ctx, probes, 3)
        planes = list(dict.fromkeys([(0, nx // 2), (1, 1), (2, nz // 2), (2, 1), (0, nx - 1)])) if peaks else []
        if peaks:
            kvs.kvs_set_peak_planes(ctx, planes)
        if zchunk:
            kvs.kvs_set_step_tuning(ctx, 0, zchunk)
        kvs.kvs_set_step_blocking(ctx, blocking)
        kvs.kvs_set_two_step_tile(ctx, tile)
        kvs.kvs_set_state(ctx, 1e-6 * rng.standard_normal((3,) + shape), 1e-8 * rng.standard_normal((3,) + shape), 0)
        kvs.kvs_enable_kernel_timing(ctx, True)
        kvs.kvs_step(ctx, 5)
        kvs.kvs_step(ctx, 6)
        last = kvs.kvs_last_step_launch(ctx)
        (_, one), (_, two) = kvs.kvs_kernel_time_split(ctx)
        u, w, _ = kvs.kvs_get_state(ctx, shape)
        out = [u, w, kvs.kvs_read_traces(ctx, len(probes), 3)]
        return last, (one, two), out + [kvs.kvs_peak_map(ctx, a, i, dims) for a, i in planes]
    finally:
        kvs.kvs_destroy(ctx)


def edges(tile):
    """One tile with a lane to spare, one wall to wall in x, one cell more, two
    tiles that end at the walls, one cell more; a row more than one tile (R + 2
    rows are not offered), two tiles, one row more; segments of 1, 3 and 4 planes
    and the model's."""
    X, R = tile
    return [(X + 1, R + 1, 5, 0), (X + 2, R + 3, 12, 3), (X + 3, 2 * R, 9, 1), (2 * X, 2 * R + 1, 7, 4),
            (2 * X + 1, 3 * R - 1, 14, 0)]


CASES = [(t, e, False, p) for t in range(4) for e in range(5) for p in (False, True) if not p or t in (1, 2)]
CASES += [(2, e, True, p) for e in range(5) for p in (False, True)]


@pytest.mark.parametrize("tile,edge,fp64,peaks", CASES)
@pytest.mark.parametrize("het", [True, False], ids=["maps", "uniform"])
@pytest.mark.parametrize("visc", [True, False], ids=["viscous", "lossless"])
def test_every_tile_matches_one_step_bitwise(kvs, tile, edge, fp64, peaks, het, visc):
    nx, ny, nz, zchunk = edges(TILES[tile])[edge]
    prec = kvs.KVS_FP64 if fp64 else kvs.KVS_FP32
    print(f"case tile {TILES[tile]} grid {nx}x{ny}x{nz} zchunk {zchunk} fp64 {fp64} peaks {peaks} het {het} visc {visc}",
          flush=True)
    last1, n1, ref = run(kvs, (nx, ny, nz), prec, het, visc, peaks, 1, tile, zchunk)
    last2, n2, got = run(kvs, (nx, ny, nz), prec, het, visc, peaks, 2, tile, zchunk)
    assert last1[0] == kvs.KVS_STEP_TILED and n1 == (11, 0)
    assert last2[0] == kvs.KVS_STEP_TWO and last2[1][:2] == TILES[tile] and n2 == (1, 5)
    if zchunk:
        assert last2[1][2] == zchunk
    assert np.max(np.abs(ref[0])) > 0
    for n, (a, b) in enumerate(zip(ref, got)):
        assert np.array_equal(a, b), n


MARCH = [(64, 8), (128, 8), (192, 5), (256, 4)]


@pytest.mark.parametrize("tile", [1, 2, 3, 4])
@pytest.mark.parametrize("edge", range(4))
@pytest.mark.parametrize("het", [True, False], ids=["maps", "uniform"])
@pytest.mark.parametrize("visc", [True, False], ids=["viscous", "lossless"])
def test_every_march_tile_matches_the_tiled_kernel_bitwise(kvs, tile, edge, het, visc):
    """The one-step march of contexts with a layer: each tile on rows it spans, on
    rows one node longer (a second tile of few cells) and on the longest, with
    whole and broken tiles of rows, force and probes."""
    X, R = MARCH[tile - 1]
    nx, ny, nz = [(X, R + 2, 9), (min(X + 1, 257), 2 * R + 2, 13), (min(X + 2, 257), 2 * R + 3, 9), (257, 3 * R + 1, 10)][edge]
    ny = max(ny, 9)
    shape = (nz, ny, nx)
    print(f"case march tile {MARCH[tile - 1]} grid {nx}x{ny}x{nz} het {het} visc {visc}", flush=True)
    out = []
    for t in (0, tile):
        rng = np.random.default_rng([nx, ny, nz])
        ctx = kvs.kvs_create((nx, ny, nz) + (0.25e-3,) * 3, precision=kvs.KVS_FP32, sponge_cells=0)
        try:
            eta = 0.8 if visc else 0.0
            if het:
                kvs.kvs_set_material(ctx, 1e3 * (1 + 5 * rng.random(shape)), 950 + 100 * rng.random(shape),
                                     eta * rng.random(shape))
            else:
                kvs.kvs_set_material_uniform(ctx, 3e3, 1000.0, eta)
            kvs.kvs_set_dt(ctx, 0.4 * kvs.kvs_stable_dt(ctx))
            kvs.kvs_set_projected_force(ctx, 1e3 * rng.standard_normal((3,) + shape))
            kvs.kvs_set_envelope(ctx, [1.0, 0.5, 0.0, 0.25])
            kvs.kvs_set_pml(ctx, 3)
            kvs.kvs_set_probes(ctx, [[i, ny // 2, nz // 2] for i in range(nx)] + [[0, 0, 0]], 3)
            kvs.kvs_set_march_tile(ctx, t)
            kvs.kvs_step(ctx, 5)
            kvs.kvs_step(ctx, 4)
            kernel, launched = kvs.kvs_last_step_launch(ctx)
            assert kernel == (kvs.KVS_STEP_MARCH if t else kvs.KVS_STEP_TILED)
            assert not t or launched[:2] == (X, R)
            out.append(list(kvs.kvs_get_state(ctx, shape)[:2]) + [kvs.kvs_read_traces(ctx, nx + 1, 3)])
        finally:
            kvs.kvs_destroy(ctx)
    assert np.abs(out[0][0]).max() > 0
    for n, (a, b) in enumerate(zip(*out)):
        assert np.array_equal(a, b), n


def last_launch(kvs, dims, prec=None, pml=0, steps=2, tile=-1, zchunk=None, probe=None, eta=0.5, het=False, force=False,
                march=-1):
    ctx = kvs.kvs_create(dims + (0.3e-3,) * 3, precision=kvs.KVS_FP32 if prec is None else prec, sponge_cells=0)
    try:
        assert kvs.kvs_last_step_launch(ctx)[0] == kvs.KVS_STEP_NONE
        if het:
            one = np.ones(dims[::-1])
            one[0] *= 2
            kvs.kvs_set_material(ctx, 3e3 * one, 1000.0 * one, eta * one)
        else:
            kvs.kvs_set_material_uniform(ctx, 3e3, 1000.0, eta)
        kvs.kvs_set_dt(ctx, 0.4 * kvs.kvs_stable_dt(ctx))
        if force:
            kvs.kvs_set_projected_force(ctx, np.ones((3,) + dims[::-1]))
            kvs.kvs_set_envelope(ctx, np.ones(steps))
        kvs.kvs_set_march_tile(ctx, march)
        if pml:
            kvs.kvs_set_pml(ctx, pml)
        if probe:
            kvs.kvs_set_probes(ctx, [probe], 0)
        if zchunk is not None:
            kvs.kvs_set_step_tuning(ctx, 0, zchunk)
        kvs.kvs_set_two_step_tile(ctx, tile)
        kvs.kvs_step(ctx, steps)
        return kvs.kvs_last_step_launch(ctx)
    finally:
        kvs.kvs_destroy(ctx)


def test_which_kernel_steps(kvs):
    print("case step dispatch", flush=True)
    two, march, tiled = kvs.KVS_STEP_TWO, kvs.KVS_STEP_MARCH, kvs.KVS_STEP_TILED
    assert last_launch(kvs, (40, 30, 20))[0] == two
    assert last_launch(kvs, (40, 30, 20), steps=3)[0] == tiled           # the odd last step
    assert last_launch(kvs, (40, 30, 20), probe=[3, 3, 0])[0] == tiled   # a probe on the plane k = 0
    assert last_launch(kvs, (40, 30, 20), probe=[3, 0, 3])[0] == two
    assert last_launch(kvs, (300, 30, 20), prec=kvs.KVS_FP64) == (two, last_launch(kvs, (300, 30, 20), kvs.KVS_FP64, tile=0)[1])
    assert last_launch(kvs, (40, 10, 20), prec=kvs.KVS_FP64)[0] == tiled  # 64 x 8 is the only FP64 tile
    assert last_launch(kvs, (40, 10, 20))[0] == two
    assert last_launch(kvs, (40, 10, 20), tile=2)[1][:2] in [(64, 16), (192, 5)]  # eight rows are not offered
    # 22.0 us a step with 64 x 8, 19.7 and 20.1 with these
    assert last_launch(kvs, (128, 128, 128), het=True)[1][:2] in [(128, 8), (64, 16)]
    # a long march: 0.75 ms a step with force against 0.85 with 64 x 16
    assert last_launch(kvs, (384, 384, 512))[1][:2] == (192, 5)
    # contexts with an absorbing layer: 64 x 8 on small grids, else a tile that spans the row
    assert last_launch(kvs, (130, 12, 11), pml=2)[1][:2] == (64, 8)
    for nx, tile in ((100, (128, 8)), (130, (192, 5)), (194, (256, 4)), (257, (256, 4))):
        dims = (nx, 110, 1 + 1200000 // (110 * nx))
        k, t = last_launch(kvs, dims, pml=2)
        assert k == march and t[:2] == tile, nx
        assert last_launch(kvs, dims, pml=2, eta=0.0, het=True, force=True)[0] == march
    small = (60, 40, 104)  # 249600 nodes
    for dims, kernel in ((small, tiled), ((60, 40, 105), march)):
        assert last_launch(kvs, dims, pml=2, eta=0.0)[0] == kernel
        assert last_launch(kvs, dims, pml=2, het=True, force=True)[0] == kernel
    assert last_launch(kvs, small, pml=2, het=True)[0] == march
    assert last_launch(kvs, small, pml=2, force=True)[0] == march
    assert last_launch(kvs, small, pml=2, eta=0.0, march=3) == (march, last_launch(kvs, small, pml=2, march=3)[1])
    assert last_launch(kvs, (130, 12, 11), pml=2, march=0)[0] == tiled
    assert last_launch(kvs, (258, 12, 11), pml=2, march=1)[0] == tiled   # longer than any tile
    assert last_launch(kvs, (66, 12, 11), prec=kvs.KVS_FP64, pml=2)[0] == tiled
    assert last_launch(kvs, (66, 12, 11), pml=2, zchunk=5) == (tiled, (64, 4, 5))  # the caller's own tuning
    with pytest.raises(kvs.KvsError):
        last_launch(kvs, (9, 9, 9), tile=4)
    with pytest.raises(kvs.KvsError):
        last_launch(kvs, (9, 9, 9), march=5)
