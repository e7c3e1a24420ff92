"""A context's second stream comes from contexts destroyed before it: models
built one after another, two at once and from two threads train as the first
did."""
import threading

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


def test_second_streams_are_handed_on(lib):
    net = configs.C1_NET
    sc = configs.make_scene(20480, 64)
    params = configs.init_params(net, "uniform", 1.0, seed_features=81, seed_mlp=82)
    probes = torch.from_numpy(scene.leaf_probes(sc.boxes, 4, seed=83)[0][:200].copy()).cuda()
    labels = torch.rand((200, 8), generator=torch.Generator("cuda").manual_seed(84), device="cuda")
    torch.cuda.synchronize()

    def build():
        m = lib.NBVH(net, sc.boxes, sc.lo, sc.side, precision="fp32")
        m.set_params(params)
        return m

    def step(m):
        """(loss, MLP weights) after a step; their sums have a fixed order."""
        loss = m.train_step(probes, labels)
        return torch.cat([loss, m.params[m.offsets[1]:].clone()])

    want = step(build())
    for _ in range(3):  # each takes over the stream of the one before
        assert torch.equal(step(build()), want)
    a, b = build(), build()
    got = [step(a), step(b)]
    assert torch.equal(got[0], want) and torch.equal(got[1], want)
    del a, b
    out = [None, None]

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            out[k] = step(build())
            torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert torch.equal(out[0], want) and torch.equal(out[1], want)
