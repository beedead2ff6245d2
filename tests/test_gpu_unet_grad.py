"""Weight gradients of the U-Net at the sizes where their row march can go
wrong: rows shorter than a step of four voxels, rows that end inside a step,
fewer rows than wavefronts, more rows than wavefronts; also accumulated."""
import numpy as np
import pytest

from oracle import unet

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kvs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2607_28414_amd import kvs as k
    k.lib()
    return k


@pytest.mark.parametrize("nbott", [2, 5])
@pytest.mark.parametrize("dims", [(3, 3, 3), (5, 4, 9), (66, 7, 12), (17, 31, 6), (37, 52, 45)])
def test_weight_gradient_matches_oracle(kvs, dims, nbott):
    """Per layer within 2e-2 relative L2: at most five BF16 roundings of an
    activation gradient stand between a layer and the output on either side,
    each able to fall on the other side of a tie by 2^-8 (5 x 2^-8 = 2e-2); a
    wrong voxel, tap or channel is off by O(1).  A second accumulated pass adds
    the same FP32 sums: exactly twice the gradient."""
    import torch
    nx, ny, nz = dims
    print(f"case weight gradient {dims} {nbott}", flush=True)
    rng = np.random.default_rng([nx, ny, nz, nbott])
    shapes = unet.layer_shapes(16, 32, 64, nbott)
    w = np.concatenate([rng.standard_normal(unet.layer_size(ci, co, dl)) / np.sqrt(unet.layer_taps(dl) * ci)
                        for ci, co, dl in shapes]).astype(np.float32)
    r, dz = np.zeros((nz, ny, nx)), np.zeros((nz, ny, nx))
    r[1:-1, 1:-1, 1:-1] = rng.standard_normal((nz - 2, ny - 2, nx - 2))
    dz[1:-1, 1:-1, 1:-1] = rng.standard_normal((nz - 2, ny - 2, nx - 2))
    net = kvs.kvs_unet_create((16, 32, 64), nbott)
    try:
        kvs.kvs_unet_set_weights(net, w)
        rd, dzd = torch.from_numpy(r).cuda(), torch.from_numpy(dz).cuda()
        zd = torch.zeros_like(rd)
        st = torch.cuda.current_stream().cuda_stream
        kvs.kvs_unet_forward(net, rd.data_ptr(), 0.8, 1.0, zd.data_ptr(), dims, st)
        kvs.kvs_unet_backward(net, rd.data_ptr(), 0.8, dzd.data_ptr(), 1.5, dims, False, st)
        g = kvs.kvs_unet_get_grad(net)
        kvs.kvs_unet_backward(net, rd.data_ptr(), 0.8, dzd.data_ptr(), 1.5, dims, True, st)
        g2 = kvs.kvs_unet_get_grad(net)
    finally:
        kvs.kvs_unet_destroy(net)
    assert np.array_equal(g2, 2 * g)
    go = unet.backward(r, 0.8, w.astype(np.float64), dz, 1.5, nbott=nbott)
    off = 0
    for li, (ci, co, dl) in enumerate(shapes):
        n = unet.layer_size(ci, co, dl)
        ref = np.linalg.norm(go[off:off + n])
        err = np.linalg.norm(g[off:off + n] - go[off:off + n])
        print(f"layer {li} ({ci}->{co}): grad rel L2 {err / max(ref, 1e-300):.2e}", flush=True)
        assert err <= 2e-2 * ref, (li, err, ref)
        off += n
