"""The control flow of the paired CG iterations (FP32 direction and residual):
grids of a few unknowns, where one iteration takes the residual to rounding;
solves that end at either iteration of a pair; breakdown inside a sweep; warm
starts; scalars in kernels of their own, where the partial sums are many."""
import numpy as np
import pytest

from workloads import gaussian_push

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


def storage(kvs, ctx, prec):
    kvs.kvs_set_direction_precision(ctx, prec)
    kvs.kvs_set_residual_precision(ctx, prec)


@pytest.mark.parametrize("jacobi", [True, False])
@pytest.mark.parametrize("dims", [(40, 30, 25), (131, 19, 24)], ids=str)
def test_tolerance_met_by_either_iteration_of_a_pair(kvs, dims, jacobi):
    """tol between the residuals after k - 1 and k iterations of FP64 storage, for
    odd and even k: the solve ends after k, with phi within 64 k 2^-24 of the
    FP64 one (each stored vector is rounded at most k times at 2^-24).  Only k
    whose residual lies 5 % and more below all before it are asked for: the
    FP32 residuals are off by about k 2^-24 of them."""
    nx, ny, nz = dims
    pc = kvs.KVS_PC_JACOBI if jacobi else kvs.KVS_PC_NONE
    F = np.random.default_rng(nx).standard_normal((3, nz, ny, nx))
    print(f"case tolerance inside a pair {dims} jacobi {jacobi}", flush=True)
    ctx = kvs.kvs_create(dims + (0.3e-3, 0.25e-3, 0.4e-3), precision=kvs.KVS_FP32)
    try:
        kvs.kvs_set_force(ctx, F)
        storage(kvs, ctx, kvs.KVS_FP64)
        res, phi = [1.0], [None]
        for k in range(1, 25):
            res.append(kvs.kvs_project(ctx, fixed_iters=k, precond=pc)["relres_recursive"])
            phi.append(kvs.kvs_get_phi(ctx, (nz, ny, nx)))
        asked = [k for k in range(1, 25) if res[k] < 0.95 * min(res[:k])]
        assert len([k for k in asked if k % 2]) >= 3 and len([k for k in asked if k % 2 == 0]) >= 3
        storage(kvs, ctx, kvs.KVS_FP32)
        for k in asked:
            rep = kvs.kvs_project(ctx, tol=(res[k] * min(res[:k])) ** 0.5, precond=pc)
            assert rep["status"] == 0 and rep["iters"] == k, (k, rep)
            got = kvs.kvs_get_phi(ctx, (nz, ny, nx))
            assert np.linalg.norm(got - phi[k]) <= 64 * k * 2.0 ** -24 * np.linalg.norm(phi[k]), k
    finally:
        kvs.kvs_destroy(ctx)


def test_overflow_of_the_stored_residual_is_a_breakdown(kvs):
    """b just inside FP32's range, and the residual of plain CG grows in its first
    iterations: the stored values become infinite inside a pair.  FP64 storage
    solves it.  The solve after it is that of a new context, bit for bit."""
    dims = (20, 18, 16)
    shape, h = dims[::-1], 0.3e-3
    F = gaussian_push(dims + (h, h, h), 0.6e-3, 1.2e-3, 1.0)
    b = sum(np.gradient(F[c], h, axis=2 - c)[1:-1, 1:-1, 1:-1] for c in range(3))  # centred inside
    big = F * (0.999 * float(np.finfo(np.float32).max) / np.abs(b).max())
    print("case breakdown inside a pair", flush=True)
    ctx, new = (kvs.kvs_create(dims + (h, h, h), precision=kvs.KVS_FP32) for _ in range(2))
    try:
        kvs.kvs_set_force(ctx, big)
        storage(kvs, ctx, kvs.KVS_FP64)
        assert kvs.kvs_project(ctx, precond=kvs.KVS_PC_NONE)["status"] == 0
        storage(kvs, ctx, kvs.KVS_FP32)
        rep = kvs.kvs_project(ctx, precond=kvs.KVS_PC_NONE, raise_on_status=False)
        assert rep["status"] == kvs.KVS_EBREAKDOWN and 0 <= rep["iters"] <= 2, rep
        out = []
        for c in (ctx, new):
            kvs.kvs_set_force(c, F)
            rep = kvs.kvs_project(c, precond=kvs.KVS_PC_NONE)
            out.append((rep["iters"], kvs.kvs_get_phi(c, shape)))
        assert out[0][0] == out[1][0] > 10 and np.array_equal(out[0][1], out[1][1])
    finally:
        kvs.kvs_destroy(ctx)
        kvs.kvs_destroy(new)


@pytest.mark.parametrize("jacobi", [True, False])
def test_warm_starts(kvs, jacobi):
    """From the potential of another force (odd and even counts before it, so that
    the residual was left in either half of its buffer), from its own, and with
    b = 0; a cold solve after them is that of a new context."""
    dims = (47, 33, 29)
    shape, h = dims[::-1], (0.3e-3, 0.25e-3, 0.4e-3)
    pc = kvs.KVS_PC_JACOBI if jacobi else kvs.KVS_PC_NONE
    rng = np.random.default_rng(2)
    F1, F2 = (rng.standard_normal((3,) + shape) for _ in range(2))
    print(f"case warm starts jacobi {jacobi}", flush=True)
    ctx, new = (kvs.kvs_create(dims + h, precision=kvs.KVS_FP32) for _ in range(2))
    try:
        kvs.kvs_set_force(new, F2)
        rep2 = kvs.kvs_project(new, tol=1e-9, precond=pc)
        cold = kvs.kvs_get_phi(new, shape)
        for before in (1, 2, 3, 4):
            kvs.kvs_set_force(ctx, F1)
            kvs.kvs_project(ctx, fixed_iters=before, precond=pc)
            kvs.kvs_set_force(ctx, F2)
            rep = kvs.kvs_project(ctx, tol=1e-9, precond=pc, warm_start=True)
            assert rep["status"] == 0 and rep["relres_true"] <= 1e-9, rep
            # both residuals are within tol |b|: phi within twice that over the
            # least eigenvalue of A, the sum over the axes of (pi / ((n - 1) h))^2
            # less its discretisation error
            lmin = sum((np.pi / (n * d)) ** 2 for n, d in zip(dims, h)) * 0.9
            b = sum(np.gradient(F2[c], h[c], axis=2 - c)[1:-1, 1:-1, 1:-1] for c in range(3))
            assert np.linalg.norm(kvs.kvs_get_phi(ctx, shape) - cold) <= 2e-9 * np.linalg.norm(b) / lmin, before
            again = kvs.kvs_project(ctx, tol=1e-9, precond=pc, warm_start=True)
            assert again["status"] == 0 and again["relres_true"] <= 1e-9, again
        kvs.kvs_set_force(ctx, np.zeros_like(F1))
        rep = kvs.kvs_project(ctx, tol=1e-9, precond=pc, warm_start=True)
        assert rep["status"] == 0 and rep["iters"] == 0 and not kvs.kvs_get_phi(ctx, shape).any()
        kvs.kvs_set_force(ctx, F2)
        rep = kvs.kvs_project(ctx, tol=1e-9, precond=pc)
        assert rep["iters"] == rep2["iters"] and np.array_equal(kvs.kvs_get_phi(ctx, shape), cold)
    finally:
        kvs.kvs_destroy(ctx)
        kvs.kvs_destroy(new)


def test_many_partials(kvs):
    """1000 x 1000 x 4 nodes take 1224 blocks, more than are folded into the
    sweeps: the scalars are kernels of their own.  Against FP64 storage, with the
    bound of the fixed counts above, and the tolerance on the true residual."""
    dims = (1000, 1000, 4)
    shape = dims[::-1]
    F = np.random.default_rng(1).standard_normal((3,) + shape)
    print("case many partials", flush=True)
    ctx = kvs.kvs_create(dims + (0.3e-3, 0.25e-3, 0.4e-3), precision=kvs.KVS_FP32)
    try:
        kvs.kvs_set_force(ctx, F)
        for k in (1, 2, 7):
            phi = []
            for st in (kvs.KVS_FP32, kvs.KVS_FP64):
                storage(kvs, ctx, st)
                rep = kvs.kvs_project(ctx, fixed_iters=k, precond=kvs.KVS_PC_JACOBI)
                assert rep["iters"] == k and rep["status"] == 0
                phi.append(kvs.kvs_get_phi(ctx, shape))
            assert np.linalg.norm(phi[0] - phi[1]) <= 64 * k * 2.0 ** -24 * np.linalg.norm(phi[1]), k
        reps = []
        for st in (kvs.KVS_FP32, kvs.KVS_FP64):
            storage(kvs, ctx, st)
            reps.append(kvs.kvs_project(ctx, tol=1e-6, precond=kvs.KVS_PC_JACOBI))
        assert reps[0]["status"] == reps[1]["status"] == 0 and reps[0]["relres_true"] <= 1e-6
        assert abs(reps[0]["iters"] - reps[1]["iters"]) <= 2, reps
    finally:
        kvs.kvs_destroy(ctx)
