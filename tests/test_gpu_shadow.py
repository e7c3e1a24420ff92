"""BF16 calls take table and weights from the shadow as they find it: a caller
may restore it without nbvh_sync_shadow, or write it between two queries."""
import numpy as np
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


NETS = {"c1": configs.C1_NET,
        # input of 5 fragments, output rows short of a tile
        "n_in 160, wide": configs.NetConfig(5, 4, 10, 8, 16, 1.5, 256, 3, 9, [5, 11, 60, 130, 400])}


def _rays(n, seed):
    rng = np.random.default_rng(seed)
    r = np.zeros((n, 8), np.float32)
    r[:, 0:3] = rng.uniform(-2.5, 2.5, (n, 3))
    d = rng.uniform(-0.6, 0.6, (n, 3)) - r[:, 0:3]
    r[:, 4:7] = d / np.linalg.norm(d, axis=1, keepdims=True)
    r[:, 7] = np.inf
    return torch.from_numpy(r).cuda()


@pytest.mark.parametrize("net", sorted(NETS))
def test_calls_follow_a_shadow_written_by_the_caller(lib, net):
    net = NETS[net]
    sc = configs.make_scene(20480, 64)
    pair = []
    for seed in (91, 92):
        m = lib.NBVH(net, sc.boxes, sc.lo, sc.side, precision="bf16")
        m.set_params(configs.init_params(net, "uniform", 1.0, seed_features=seed, seed_mlp=seed + 10))
        w = m.params[m.offsets[-2]: m.offsets[-2] + net.mlp_width]
        w -= w.mean()  # hits and misses
        m.reset_optimizer()
        pair.append(m)
    a, b = pair
    keep = a.params_lp.clone()
    probes = torch.from_numpy(scene.leaf_probes(sc.boxes, 3, seed=93)[0][:150].copy()).cuda()
    labels = torch.rand((150, 8), generator=torch.Generator("cuda").manual_seed(94), device="cuda")
    ws = {m: lib.NBVHBatch([m]) for m in pair}

    def outputs(m):
        out = [m.forward(probes)]
        for n in (100, 300, 20_000):
            rays = _rays(n, n)
            print("shadow", net.mlp_width, n, flush=True)
            off, segs = m.traverse(rays, 8 * n)
            hits, _, _, z, _ = m.query_traced(rays, 8 * n)
            out += [m.query(rays, 8 * n), m.query_segments(rays, off, segs), ws[m].query(rays, 8 * n), hits, z]
        return out

    def same(x, y):
        return all(torch.equal(p.view(torch.int32), q.view(torch.int32)) for p, q in zip(x, y))

    want_a, want_b = outputs(a), outputs(b)
    assert not torch.equal(want_a[1], want_b[1])
    a.params_lp.copy_(b.params_lp)
    assert same(outputs(a), want_b)
    a.params_lp.copy_(keep)
    assert same(outputs(a), want_a)
    # the forward half of a training step
    a.params_lp.copy_(b.params_lp)
    assert torch.equal(a.train_step(probes, labels), b.train_step(probes, labels))
