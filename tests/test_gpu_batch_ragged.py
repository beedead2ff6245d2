"""Ragged batches of small instances whose own best tiles differ in shape."""
import time

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


H = 0.5e-3
BATCHES = [
    ([(28, 79, 6), (105, 11, 7)], 0.0),                         # 64 x 16 and 128 x 8 by their own
    ([(9, 14, 7), (100, 36, 12), (133, 27, 7)], 0.0),           # three shapes
    ([(7, 54, 8), (36, 53, 7)], 0.5),                           # one shape, two short launches' worth
    ([(40, 10, 30), (90, 18, 12), (190, 7, 9), (60, 66, 20)], 0.5),  # rows that rule a shape out (R + 2)
]


def run(kvs, dims, eta, blocking, calls):
    """Traces, states and the best time of the calls (after a first pass)."""
    import torch
    b = kvs.kvs_batch_create([d + (H, H, H) for d in dims], precision=kvs.KVS_FP32, sponge_cells=3)
    try:
        kvs.kvs_batch_set_persistent(b, False)
        kvs.kvs_batch_set_step_blocking(b, blocking)
        for i, d in enumerate(dims):
            c = kvs.kvs_batch_instance(b, i)
            kvs.kvs_set_material_uniform(c, 3e3 + 10 * i, 1000.0, eta)
            kvs.kvs_set_dt(c, 0.4 * kvs.kvs_stable_dt(c))
            fs = np.random.default_rng(i).standard_normal((3,) + d[::-1])
            kvs.kvs_set_projected_force(c, fs)
            kvs.kvs_set_envelope(c, np.ones(sum(calls)))
            kvs.kvs_batch_set_probes(b, i, [[x, d[1] // 2, d[2] // 2] for x in range(d[0])])
        best = 1e9
        for _ in range(5):
            kvs.kvs_batch_reset(b)
            torch.cuda.synchronize()
            t = time.perf_counter()
            for n in calls:
                kvs.kvs_batch_step(b, n)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        out = [kvs.kvs_batch_read_traces(b, i, d[0]) for i, d in enumerate(dims)]
        for i, d in enumerate(dims):
            out += list(kvs.kvs_get_state(kvs.kvs_batch_instance(b, i), d[::-1])[:2])
        return out, best
    finally:
        kvs.kvs_batch_destroy(b)


@pytest.mark.parametrize("dims,eta", BATCHES, ids=lambda v: str(v))
def test_ragged_batches_match_one_step_bitwise(kvs, dims, eta):
    print(f"case ragged batch {dims} eta {eta}", flush=True)
    one, _ = run(kvs, dims, eta, 1, (7, 8))
    two, _ = run(kvs, dims, eta, 2, (7, 8))
    assert max(np.abs(x).max() for x in one) > 0
    for n, (x, y) in enumerate(zip(one, two)):
        assert np.array_equal(x, y), n


@pytest.mark.parametrize("dims,eta", BATCHES[:2], ids=lambda v: str(v))
def test_pairs_of_small_ragged_batches_are_no_slower(kvs, dims, eta):
    """Measured 0.77 and 0.55 of the one-step launches; with a launch per shape it
    was 1.67 and 1.06."""
    print(f"case ragged batch timing {dims}", flush=True)
    _, one = run(kvs, dims, eta, 1, (200,))
    _, two = run(kvs, dims, eta, 2, (200,))
    print(f"one step a launch {one / 200 * 1e6:.2f} us, two {two / 200 * 1e6:.2f} us a step", flush=True)
    assert two <= 1.0 * one, (one, two)
