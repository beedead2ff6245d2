"""The control flow of the paired CG iterations (FP32 direction and residual):
grids of a few unknowns, where one iteration takes the residual to rounding."""
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


def system(F, h):
    """A = -lap_h and -b = -div F on the interior nodes, in FP64."""
    n = [s - 2 for s in F.shape[1:]]  # z, y, x
    b = np.zeros(n)
    A = np.zeros((b.size, b.size))
    at = np.arange(b.size).reshape(n)
    for ax, hh in ((2, h[0]), (1, h[1]), (0, h[2])):
        mid = [slice(1, -1)] * 3
        up, dn = list(mid), list(mid)
        up[ax], dn[ax] = slice(2, None), slice(0, -2)
        f = F[2 - ax]
        b += (f[tuple(up)] - f[tuple(dn)]) / (2 * hh)
        A[at.ravel(), at.ravel()] += 2 / hh ** 2
        i = np.take(at, range(n[ax] - 1), ax).ravel()
        j = np.take(at, range(1, n[ax]), ax).ravel()
        A[i, j] -= 1 / hh ** 2
        A[j, i] -= 1 / hh ** 2
    return A, -b.ravel()


@pytest.mark.parametrize("dims", [(3, 3, 3), (5, 3, 3), (4, 4, 3), (3, 5, 3)], ids=str)
@pytest.mark.parametrize("h", [(0.3e-3, 0.25e-3, 0.4e-3), (1e-3, 1e-3, 1e-3)], ids=["oblong", "cubic"])
@pytest.mark.parametrize("jacobi", [True, False])
def test_few_unknowns(kvs, dims, h, jacobi):
    """CG of N unknowns ends after N iterations within FP32 rounding of the
    solution; a second cycle from the true residual reaches 1e-12.  The true
    residual of phi meets tol to FP64 rounding, and so does its distance from
    the direct solution times the condition number.  One iteration more than N
    leaves phi within 64 cond 2^-24 (each vector is rounded a few times at
    2^-24), whether or not it ends at a residual of 0."""
    nx, ny, nz = dims
    N = (nx - 2) * (ny - 2) * (nz - 2)
    pc = kvs.KVS_PC_JACOBI if jacobi else kvs.KVS_PC_NONE
    print(f"case few unknowns {dims} h {h} jacobi {jacobi}", flush=True)
    ctx = kvs.kvs_create(dims + h, precision=kvs.KVS_FP32)
    try:
        for seed in range(24):
            F = np.random.default_rng(seed).standard_normal((3, nz, ny, nx))
            A, c = system(F, h)
            exact, cond = np.linalg.solve(A, c), np.linalg.cond(A)
            kvs.kvs_set_force(ctx, F)
            for tol in (1e-8, 1e-12):
                rep = kvs.kvs_project(ctx, tol=tol, max_iter=200, precond=pc, raise_on_status=False)
                phi = kvs.kvs_get_phi(ctx, (nz, ny, nx))[1:-1, 1:-1, 1:-1].ravel()
                what = (seed, tol, rep)
                assert rep["status"] == 0, what
                assert rep["iters"] <= 6 * N + 6, what
                assert np.linalg.norm(c - A @ phi) <= (tol + 1e-14) * np.linalg.norm(c), what
                assert np.linalg.norm(phi - exact) <= cond * (tol + 1e-14) * np.linalg.norm(exact), what
            rep = kvs.kvs_project(ctx, fixed_iters=N + 1, precond=pc, raise_on_status=False)
            phi = kvs.kvs_get_phi(ctx, (nz, ny, nx))[1:-1, 1:-1, 1:-1].ravel()
            assert rep["status"] in (0, kvs.KVS_EBREAKDOWN), (seed, rep)
            assert np.linalg.norm(phi - exact) <= 64 * cond * 2.0 ** -24 * np.linalg.norm(exact), (seed, rep)
    finally:
        kvs.kvs_destroy(ctx)
