"""The step autotuner and the one-step march of contexts with an absorbing layer
(190 x 161 x 175: 69 us against 88 us and more of the tiled variants): a tuned
context steps with the faster kernel, whenever the layer was set."""
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


def context(kvs, nx=190):
    ctx = kvs.kvs_create((nx, 161, 175) + (0.25e-3,) * 3, precision=kvs.KVS_FP32, sponge_cells=0)
    rng = np.random.default_rng(5)
    shape = (175, 161, nx)
    kvs.kvs_set_material(ctx, 1e3 * (1 + 5 * rng.random(shape)), 950 + 100 * rng.random(shape), rng.random(shape))
    kvs.kvs_set_dt(ctx, 0.4 * kvs.kvs_stable_dt(ctx))
    kvs.kvs_set_state(ctx, 1e-6 * rng.standard_normal((3,) + shape), np.zeros((3,) + shape), 0)
    return ctx


@pytest.mark.parametrize("when", ["before", "after", "after a split of the caller's"])
def test_tuned_layer_context_keeps_the_march(kvs, when):
    print(f"case autotune, layer set: {when}", flush=True)
    out = []
    for tune in (False, True):
        ctx = context(kvs)
        try:
            if tune and when == "before":
                kvs.kvs_autotune_step(ctx, 5)
            kvs.kvs_set_pml(ctx, 10)
            if tune and when == "after a split of the caller's":
                kvs.kvs_set_step_tuning(ctx, 0, 5)
            if tune and when != "before":
                variant, ms = kvs.kvs_autotune_step(ctx, 5)
                assert 0 <= variant < kvs.kvs_num_step_variants() and ms[variant] == ms.min() > 0
            kvs.kvs_step(ctx, 3)
            assert kvs.kvs_last_step_launch(ctx)[0] == kvs.KVS_STEP_MARCH
            out.append(kvs.kvs_get_state(ctx, (175, 161, 190)))
            if tune:  # what the caller chooses afterwards holds
                kvs.kvs_set_step_tuning(ctx, 3)
                kvs.kvs_step(ctx, 1)
                assert kvs.kvs_last_step_launch(ctx)[0] == kvs.KVS_STEP_TILED
        finally:
            kvs.kvs_destroy(ctx)
    for a, b in zip(out[0][:2], out[1][:2]):
        assert np.array_equal(a, b)


def test_rows_longer_than_the_march_keep_the_tuned_variant(kvs):
    print("case autotune, rows beyond the march", flush=True)
    ctx = context(kvs, 260)
    try:
        kvs.kvs_set_pml(ctx, 10)
        kvs.kvs_autotune_step(ctx, 3)
        kvs.kvs_step(ctx, 2)
        assert kvs.kvs_last_step_launch(ctx)[0] == kvs.KVS_STEP_TILED
    finally:
        kvs.kvs_destroy(ctx)
