"""Back-propagation multiplies no more of a transposed weight copy than its
layer has: with sixteen outputs the FP32 copy has no padding, so the auxiliary
buffer may hold anything before nbvh_sync_shadow writes the copies."""
import pytest

torch = pytest.importorskip("torch")

from nbvh_synth import configs, scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_16237_amd as P
    P.load()
    return P


@pytest.mark.parametrize("width", [32, 256])
def test_fp32_gradient_over_an_unset_auxiliary_buffer(lib, width):
    net = configs.NetConfig(8, 2, 12, 2, 16, 1.5, width, 2, 16, [4, 6, 9, 14, 21, 32, 48, 72])
    sc = configs.make_scene(20480, 64)
    params = configs.init_params(net, "uniform", 1.0, seed_features=95, seed_mlp=96)
    probes = torch.from_numpy(scene.leaf_probes(sc.boxes, 2, seed=97)[0][:64].copy()).cuda()
    dz = torch.randn((64, 16), generator=torch.Generator("cuda").manual_seed(98), device="cuda")
    grads = []
    for fill in (0, 255):  # 255: every float NaN
        m = lib.NBVH(net, sc.boxes, sc.lo, sc.side, precision="fp32")
        m.set_params(params)
        m.aux.fill_(fill)
        m.sync_shadow()
        m.backward(probes, dz)
        grads.append(m.unscaled_grad().clone())
    assert torch.isfinite(grads[1]).all()
    # an entry's at most 64 x 2 x 8 terms may be added in another order
    tol = 1024 * 2.0 ** -24 * float(grads[0].abs().max())
    assert (grads[1] - grads[0]).abs().max() <= tol
