"""Lines in the persistent batch kernel, at the sizes where its threads and
its two LDS copies can go wrong: fewer cells than a wavefront, a last thread
without a cell, the largest line with a thread per component and the next, one
near what LDS holds, instances of different lengths, odd and even step
counts and ones around the 64 steps staged at a time, probes off the line."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
TOL = {0: 1e-12, 1: 2e-5}


@pytest.fixture(scope="module")
def kvs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2607_28414_amd import kvs as k
    k.lib()
    return k


def run(kvs, lengths, precision, calls, eta, persistent):
    h = 0.25e-3
    b = kvs.kvs_batch_create([(n, 3, 3, h, h, h) for n in lengths], precision=precision, sponge_cells=2)
    try:
        kvs.kvs_batch_set_persistent(b, persistent)
        probes = []
        for q, n in enumerate(lengths):
            ctx = kvs.kvs_batch_instance(b, q)
            kvs.kvs_set_material_uniform(ctx, 4e3, 1000.0, eta)
            kvs.kvs_set_dt(ctx, 0.4 * kvs.kvs_stable_dt(ctx))
            rng = np.random.default_rng([n, q])
            kvs.kvs_set_envelope(ctx, rng.standard_normal(40))
            fs = np.zeros((3, 3, 3, n))
            fs[:, 1, 1, 1:-1] = 1e3 * rng.standard_normal((3, n - 2))
            kvs.kvs_set_projected_force(ctx, fs)
            p = [[i, 1, 1] for i in range(0, n, max(1, n // 9))] + [[n // 2, 0, 1], [n // 2, 1, 2], [n - 1, 1, 1]]
            kvs.kvs_batch_set_probes(b, q, p)
            probes.append(p)
        kvs.kvs_batch_set_component(b, 1)
        assert kvs.kvs_batch_uses_persistent(b) == persistent
        for m in calls:
            kvs.kvs_batch_step(b, m)
        tr = [kvs.kvs_batch_read_traces(b, q, len(p)) for q, p in enumerate(probes)]
        st = [kvs.kvs_get_state(kvs.kvs_batch_instance(b, q), (3, 3, n)) for q, n in enumerate(lengths)]
    finally:
        kvs.kvs_batch_destroy(b)
    return tr, st


@pytest.mark.parametrize("eta", [0.5, 0.0], ids=["viscous", "lossless"])
@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("lengths", [(3, 66, 67, 322), (323, 5), (690, 9)], ids=str)
def test_lines_match_per_step_launches(kvs, lengths, precision, eta):
    """Traces and the final state against the per-step launches of the same
    batch, whose arithmetic is the same up to contraction (FP64 1e-12, FP32
    2e-5 of the largest value, the bars of the line sweep)."""
    print(f"case lines {lengths} precision {precision} eta {eta}", flush=True)
    if precision == 0 and max(lengths) > 340:
        lengths = tuple(n for n in lengths if n <= 340) + (300,)  # LDS
    calls = (1, 63, 64, 65, 2)
    tr, st = run(kvs, lengths, precision, calls, eta, True)
    tr0, st0 = run(kvs, lengths, precision, calls, eta, False)
    for q, n in enumerate(lengths):
        assert tr[q].shape[0] == sum(calls)
        scale = np.abs(tr0[q]).max()
        assert scale > 0
        assert np.abs(tr[q] - tr0[q]).max() <= TOL[precision] * scale, n
        for f, f0 in zip(st[q][:2], st0[q][:2]):
            assert np.abs(f - f0).max() <= TOL[precision] * np.abs(f0).max(), n
