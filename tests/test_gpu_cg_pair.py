"""Two CG iterations per pair of sweeps (FP32 direction and residual) against
the one-iteration sweeps in FP64 storage: the potential after a fixed number
of iterations, odd and even, on grids at the edges of the overlapping tiles
(one wall-to-wall tile, one cell more, several, rows shorter than a tile), and
the count at which max_iter ends the solve."""
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


@pytest.mark.parametrize("nx,ny,nz", [
    (3, 3, 3),        # one interior cell
    (66, 10, 5),      # one tile exactly (64 x 8 interior cells)
    (67, 11, 7),      # one cell more on both axes
    (130, 18, 9),     # two wavefronts a row, wall to wall; sixteen rows
    (131, 19, 24),    # one more
    (192, 33, 40),    # three overlapping tiles, several z segments
    (300, 8, 6),      # long rows, few of them
    (5, 70, 31),
])
@pytest.mark.parametrize("jacobi", [True, False])
def test_pairs_match_single_iterations(kvs, nx, ny, nz, jacobi):
    """After k iterations each stored FP32 vector (r, p) has been rounded at
    most k times at 2^-24 relative; with an amplification of at most 64 per
    iteration count over these few iterations, phi agrees with the FP64 one to
    64 k 2^-24 in relative L2 (k = 7: 2.7e-5)."""
    h = (0.3e-3, 0.25e-3, 0.4e-3)
    grid = (nx, ny, nz) + h
    rng = np.random.default_rng(nx + ny + nz)
    F = rng.standard_normal((3, nz, ny, nx))
    pc = kvs.KVS_PC_JACOBI if jacobi else kvs.KVS_PC_NONE
    shape = (nz, ny, nx)
    print(f"case cg pair {grid[:3]} jacobi {jacobi}", flush=True)
    ctx = kvs.kvs_create(grid, precision=kvs.KVS_FP32)
    try:
        kvs.kvs_set_force(ctx, F)
        cells = (nx - 2) * (ny - 2) * (nz - 2)
        for k in (1, 2, 3, 6, 7):
            if cells == 1 and k > 1:
                break
            phi = []
            for st in (kvs.KVS_FP32, kvs.KVS_FP64):
                kvs.kvs_set_direction_precision(ctx, st)
                kvs.kvs_set_residual_precision(ctx, st)
                rep = kvs.kvs_project(ctx, fixed_iters=k, precond=pc)
                assert rep["iters"] == k and rep["status"] == 0
                phi.append(kvs.kvs_get_phi(ctx, shape))
            assert np.linalg.norm(phi[0] - phi[1]) <= 64 * k * 2.0 ** -24 * np.linalg.norm(phi[1]), k
        kvs.kvs_set_direction_precision(ctx, kvs.KVS_FP32)
        kvs.kvs_set_residual_precision(ctx, kvs.KVS_FP32)
        for m in (1, 2, 3):
            if cells == 1:
                break
            rep = kvs.kvs_project(ctx, tol=1e-14, max_iter=m, precond=pc, raise_on_status=False)
            assert rep["status"] == kvs.KVS_ENOTCONV and rep["iters"] == m
    finally:
        kvs.kvs_destroy(ctx)
