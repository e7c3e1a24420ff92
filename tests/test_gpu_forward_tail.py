"""A forward pass's last tile of up to 32 probes has 32 or 16 rows: each probe's
outputs are those it has in the middle of a full tile, bit for bit."""
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


NETS = {"two features": configs.NetConfig(3, 2, 14, 16, 16, 1.5, 64, 2, 16, [7, 40, 200]),
        "four features, odd samples": configs.NetConfig(8, 4, 12, 5, 16, 1.5, 128, 2, 8, [4, 6, 9, 14, 21, 32, 48, 72])}


@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("net", sorted(NETS))
def test_last_tiles_match_full_ones(lib, net, precision):
    net = NETS[net]
    sc = configs.make_scene(20480, 64)
    m = lib.NBVH(net, sc.boxes, sc.lo, sc.side, precision=precision)
    m.set_params(configs.init_params(net, "uniform", 1.0, seed_features=41, seed_mlp=42))
    probes = torch.from_numpy(scene.leaf_probes(sc.boxes, 4, seed=43)[0][:192].copy()).cuda()
    if precision == "fp8":
        m.calibrate_fp8(probes)
    full = m.forward(probes).view(torch.int32)
    for n in (1, 15, 16, 17, 31, 32, 33, 65, 80, 81, 96, 97, 129):
        print("last tile", precision, n, flush=True)
        assert torch.equal(m.forward(probes[:n].contiguous()).view(torch.int32), full[:n])
