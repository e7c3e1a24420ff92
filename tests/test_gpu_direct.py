"""Queries of few rays, whose segments are evaluated at once, against the slot
loop that takes a ray's segments one after the other (forced by the knob that
fixes the workgroups per compute unit): the same hits bit for bit, and the same
count of evaluated segments."""
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


NETS = {"c1": configs.C1_NET, "odd samples, albedo": configs.NetConfig(8, 4, 12, 5, 16, 1.5, 128, 2, 8,
                                                                   [4, 6, 9, 14, 21, 32, 48, 72]),
        "frame": configs.NetConfig(16, 2, 15, 8, 16, 1.38, 128, 4, 5)}


def _rays(n, seed):
    rng = np.random.default_rng(seed)
    r = np.zeros((n, 8), np.float32)
    r[:, 0:3] = rng.uniform(-2.5, 2.5, (n, 3))
    d = rng.uniform(-0.6, 0.6, (n, 3)) - r[:, 0:3]
    r[:, 4:7] = d / np.linalg.norm(d, axis=1, keepdims=True)
    r[:, 7] = np.inf
    if n > 4:
        r[2, 4:7] *= -1.0  # a miss between rays with segments
    return torch.from_numpy(r).cuda()


@pytest.mark.parametrize("precision", ["bf16", "fp32", "fp8"])
@pytest.mark.parametrize("name,boxes,inside", [("c1", "shell", "clip"), ("c1", "overlapping", "reverse"),
                                               ("odd samples, albedo", "overlapping", "clip"),
                                               ("frame", "shell", "reverse")])
def test_few_rays_match_the_slot_loop(lib, precision, name, boxes, inside):
    """Run lengths of 0 to 3 segments (shell) and of up to 40 (overlapping
    boxes: longer than a tile of rows, most rays starting inside); numbers of rays around
    the sizes where the traversal and the evaluation change their launches."""
    net = NETS[name]
    if boxes == "shell":
        sc = configs.make_scene(20480, 64)
        b, lo, side = sc.boxes, sc.lo, sc.side
    else:
        rng = np.random.default_rng(6)
        b = np.concatenate([rng.uniform(-1.0, -0.2, (40, 3)), rng.uniform(0.2, 1.0, (40, 3))], 1).astype(np.float32)
        lo, side = np.array([-1.1] * 3, np.float32), np.float32(2.2)
    m = lib.NBVH(net, b, lo, side, precision=precision, inside=inside)
    m.set_params(configs.init_params(net, "uniform", 1.0, seed_features=71, seed_mlp=72))
    # the output layer shifted so that hits and misses both occur
    w = m.params[m.offsets[-2]: m.offsets[-2] + net.mlp_width]
    w -= w.mean()
    m.reset_optimizer()
    if precision == "fp8":
        probes = torch.zeros((64, 8), device="cuda")
        probes[:, 0:3] = torch.rand((64, 3), generator=torch.Generator("cuda").manual_seed(1), device="cuda") - 0.5
        probes[:, 4], probes[:, 7] = 1.0, 0.5
        m.calibrate_fp8(probes)
    base = m.get_tuning()
    for n in (1, 15, 17, 64, 256, 257, 700, 16384):
        rays = _rays(n, n)
        cap = 41 * n
        print("few rays", name, boxes, inside, precision, n, flush=True)
        m.set_tuning(**base)
        e0 = m.read_state()["n_evaluated"]
        got = m.query(rays, cap, torch.full((n, 8), 7.0, device="cuda")).view(torch.int32)
        s1 = m.read_state()
        m.set_tuning(query_wgs_per_cu=1)
        ref = m.query(rays, cap, torch.full((n, 8), 8.0, device="cuda")).view(torch.int32)
        s2 = m.read_state()
        assert torch.equal(got, ref)
        assert s2["n_evaluated"] - s1["n_evaluated"] == s1["n_evaluated"] - e0
        assert s1["last_n_segments"] == s2["last_n_segments"] and s2["flags"] == 0


@pytest.mark.parametrize("precision,net", [("bf16", "frame"), ("fp32", "c1"), ("fp8", "odd samples, albedo")])
@pytest.mark.parametrize("n", [16385, 50_001])
def test_tail_tiles_match_full_tiles(lib, precision, net, n):
    """Once the ray queue is empty the slot loop closes its slots up and works
    on tiles of 32 and 16 rows; with three gathers unrolled it keeps 64."""
    sc = configs.make_scene(20480, 64)
    m = lib.NBVH(NETS[net], sc.boxes, sc.lo, sc.side, precision=precision)
    m.set_params(configs.init_params(NETS[net], "uniform", 1.0, seed_features=73, seed_mlp=74))
    if precision == "fp8":
        m.calibrate_fp8(torch.cat([_rays(64, 1)[:, :7], torch.full((64, 1), 3.0, device="cuda")], 1))
    rays = _rays(n, n)
    print("tail tiles", precision, net, n, flush=True)
    out, counts = [], []
    for k, tune in enumerate([dict(), dict(query_unroll=3)]):
        m.set_tuning(**{"query_unroll": 0, **tune})
        e = m.read_state()["n_evaluated"]
        out.append(m.query(rays, 8 * n, torch.full((n, 8), 7.0 + k, device="cuda")).view(torch.int32))
        counts.append(m.read_state()["n_evaluated"] - e)
    assert torch.equal(out[0], out[1]) and counts[0] == counts[1]


@pytest.mark.parametrize("n", [100, 1000])
def test_overflow_of_few_rays_is_flagged(lib, n):
    """A queue too short for the segments: flagged, rays with segments keep
    what their records held, rays without get their miss record."""
    sc = configs.make_scene(20480, 64)
    m = lib.NBVH(configs.C1_NET, sc.boxes, sc.lo, sc.side)
    m.set_params(configs.init_params(configs.C1_NET))
    rays = _rays(n, 3)
    off, _ = m.traverse(rays, 0)
    m.clear_flags()
    none = (off[1:] == off[:-1])
    assert 0 < int(none.sum()) < n
    hits = torch.full((n, 8), 7.0, device="cuda")
    print("overflow", n, flush=True)
    m.query(rays, int(off[-1]) - 1, hits)
    st = m.read_state()
    assert st["flags"] == 1 and st["last_n_segments"] == int(off[-1])
    assert (hits[~none] == 7.0).all()
    assert (hits[none].view(torch.int32)[:, 7] == -1).all() and (hits[none][:, :7] == 0).all()


@pytest.mark.parametrize("n", [7, 300])
def test_first_segment_at_infinity_counts_as_evaluated(lib, n):
    """A ray without direction that begins at infinity crosses the leaves around
    its origin there: its first segment is evaluated (no hit), its others not."""
    b = np.array([[-1, -1, -1, 1, 1, 1], [-0.9, -0.9, -0.9, 0.9, 0.9, 0.9]], np.float32)
    m = lib.NBVH(configs.C1_NET, b, np.full(3, -1.1, np.float32), 2.2)
    m.set_params(configs.init_params(configs.C1_NET))
    rays = _rays(n, 5)
    rays[::3, 0:3] *= 0.2
    rays[::3, 3], rays[::3, 4:7] = np.inf, 0.0
    print("infinity", n, flush=True)
    hits, counts = [], []
    for wgs in (0, 1):
        m.set_tuning(query_wgs_per_cu=wgs)
        e = m.read_state()["n_evaluated"]
        hits.append(m.query(rays, 2 * n).view(torch.int32))
        counts.append(m.read_state()["n_evaluated"] - e)
    assert torch.equal(hits[0], hits[1]) and (hits[0][::3, 7] == -1).all()
    assert counts[0] == counts[1] >= (n + 2) // 3
