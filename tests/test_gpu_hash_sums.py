"""Table gradients of the levels that a tile of 256 probes sums in its LDS hash
table. Contributions that find a slot are added exactly (64-bit fixed point),
so the order of a tile's probes does not show; what finds none goes to memory
in FP32. Probes of unrelated places, which share no corners, against FP64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from nbvh_synth import configs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_16237_amd as P
    P.load()
    return P


LO, SIDE = np.zeros(3, np.float32), np.float32(1.0)
BOX = np.array([[0, 0, 0, 1, 1, 1]], np.float32)


def _chords(n, seed):
    """Segments between random points of the unit cube."""
    rng = np.random.default_rng(seed)
    a, b = rng.uniform(0, 1, (n, 3)), rng.uniform(0, 1, (n, 3))
    length = np.linalg.norm(b - a, axis=1)
    p = np.zeros((n, 8), np.float32)
    p[:, 0:3], p[:, 4:7], p[:, 7] = a, (b - a) / length[:, None], length
    return p


def _model(lib, net, params):
    m = lib.NBVH(net, BOX, LO, SIDE, precision="fp32", loss_scale=1.0)
    m.set_params(params)
    return m


def test_sums_of_a_tile_do_not_depend_on_the_order_of_its_probes(lib):
    """2,744 entries, of which the tile meets more than 2,048, few enough for each
    to find one of 4,096 slots (consecutive entries spread evenly over them)."""
    net = configs.NetConfig(1, 2, 12, 16, 16, 1.5, 32, 1, 5, [13])
    params = configs.init_params(net, "uniform", 1.0, seed_features=61, seed_mlp=62)
    probes = _chords(256, 63)
    dz = np.random.default_rng(64).normal(size=(256, 5)).astype(np.float32)
    grads = []
    for seed in (None, 65, 66):
        order = np.arange(256) if seed is None else np.random.default_rng(seed).permutation(256)
        m = _model(lib, net, params)
        m.backward(torch.from_numpy(probes[order]).cuda(), torch.from_numpy(dz[order]).cuda())
        grads.append(m.grad[: m.n_table].clone())
    assert int((grads[0].view(-1, 2).abs().sum(1) > 0).sum()) > 2048
    assert torch.equal(grads[0], grads[1]) and torch.equal(grads[0], grads[2])


@pytest.mark.parametrize("features", [2, 4])
@pytest.mark.parametrize("n", [256, 1000])
def test_overflowing_tiles_against_fp64(lib, features, n):
    """Fine levels: a tile meets up to 256 x 8 x 8 entries, far more than slots.
    An entry's terms are rounded once each on their way to memory, 2^-24 of the
    largest sum apart for each of at most 64 of them; the activations before
    them cost 1e-5 (the tolerance of the other gradient tests)."""
    net = configs.NetConfig(4, features, 15, 8, 16, 1.5, 64, 2, 8, [9, 16, 64, 300])
    params = configs.init_params(net, "uniform", 1.0, seed_features=67, seed_mlp=68)
    cfg = oracle.make_cfg(net, LO, SIDE)
    probes = _chords(3 * n, 69)
    probes = probes[oracle.min_abs_preact(cfg, params.astype(np.float64), probes) > 1e-4][:n]
    assert probes.shape[0] == n
    dz = (np.random.default_rng(70).normal(size=(n, 8)) / n).astype(np.float32)
    print("overflowing tiles", features, n, flush=True)
    m = _model(lib, net, params)
    m.backward(torch.from_numpy(probes).cuda(), torch.from_numpy(dz).cuda())
    nt = net.n_table_params
    g = m.unpad(m.grad)[:nt].astype(np.float64)
    ref = oracle.backward(cfg, params.astype(np.float64), probes, dz.astype(np.float64))[:nt]
    assert np.abs(g - ref).max() <= (1e-5 + 64 * 2.0 ** -24) * np.abs(ref).max()
