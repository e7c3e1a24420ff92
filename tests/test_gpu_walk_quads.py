"""The per-lane walk fetches nodes by quads of lanes or lane by lane, whichever
the wave's rays allow: lone rays, equal rays and mixtures of both, for trees in
LDS and in memory, against the walk of the whole wave."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from nbvh_synth import configs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_16237_amd as P
    P.load()
    return P


def _rays(n, kind):
    rng = np.random.default_rng(n)
    r = np.zeros((n, 8), np.float32)
    r[:, 0:3] = rng.uniform(-2.5, 2.5, (n, 3))
    d = rng.uniform(-0.8, 0.8, (n, 3)) - r[:, 0:3]
    r[:, 4:7] = d / np.linalg.norm(d, axis=1, keepdims=True)
    r[:, 7] = np.inf
    if kind == "equal":
        r[:] = r[0]
    elif kind == "one apart":  # a quad of the last wave differs from the rest
        r[:-2] = r[0]
    elif kind == "mostly missing":  # waves thin out to single lanes
        r[np.arange(n) % 17 != 3, 4:7] *= -1.0
    return torch.from_numpy(r).cuda()


@pytest.mark.parametrize("kind", ["equal", "one apart", "mostly missing", "random"])
@pytest.mark.parametrize("leaves", [64, 128, 129, 2000])
@pytest.mark.parametrize("inside", ["clip", "reverse"])
def test_walks_of_lanes_and_waves_agree(lib, leaves, kind, inside):
    rng = np.random.default_rng(leaves)
    lo = rng.uniform(-1, 0.8, (leaves, 3)).astype(np.float32)
    boxes = np.concatenate([lo, lo + np.float32(0.2)], 1)
    m = lib.NBVH(configs.C1_NET, boxes, np.full(3, -1, np.float32), 2.0, inside=inside)
    for n in (1, 2, 63, 65, 300, 16385):
        rays = _rays(n, kind)
        print("walks", leaves, kind, inside, n, flush=True)
        got = []
        for mode in (0, 1, 2):
            m.set_tuning(traverse_mode=mode)
            off, _ = m.traverse(rays, 0)
            m.clear_flags()
            off, segs = m.traverse(rays, int(off[-1]))
            got.append((off, segs[: int(off[-1])]))
        for off, segs in got[1:]:
            assert torch.equal(off, got[0][0]) and torch.equal(segs, got[0][1])
