"""The sixteen-lanes-per-ray trace kernel against the one-lane-per-ray kernel: a launch that
writes per-ray counters runs the latter, one without them the former, and every output bit
and hit id must be the same. The cases sit where the former's structures change: trees of one
leaf and a few, stacks and hit lists that overflow, rounds cut short, ray bounds and starting
transmittances, waves with idle groups. Needs an MI355X."""
import numpy as np
import pytest

import oracle
from paper_2601_20429_amd import inputs
from tests import parity

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_2601_20429_amd import grtx  # noqa: E402

AMIN = float(np.float32(1.0 / 255.0))


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def scene_of(n, seed, degree=3, spread=0.2, scale=-3.0, opacity=0.0, repeat=1):
    rng = np.random.default_rng(seed)
    m = (n + repeat - 1) // repeat
    means = np.repeat(rng.normal(0.0, spread, (m, 3)), repeat, 0)[:n]
    f = lambda a: np.ascontiguousarray(a, dtype=np.float32)
    q = rng.standard_normal((n, 4))
    return inputs.Scene(f(means), f(np.exp(rng.normal(scale, 0.5, (n, 3)))), f(q / np.linalg.norm(q, axis=1)[:, None]),
                        f(1.0 / (1.0 + np.exp(-rng.normal(opacity, 1.5, n)))),
                        f(rng.normal(0.0, 0.3, (n, (degree + 1) ** 2, 3))), degree)


def rays_of(n, seed, box=0.6):
    return tuple(torch.from_numpy(a).cuda() for a in inputs.incoherent_rays(seed, n, box))


def check(scene, o, d, cap=512, k=16, ref_mode=grtx.CHECKPOINT, **kw):
    bvh = grtx.build(grtx.SceneTensors.from_scene(scene, "cuda"), alpha_min=AMIN)
    ref = grtx.trace(bvh, o, d, k=k, hit_capacity=cap, stats=True, mode=ref_mode, **kw)
    got = grtx.trace(bvh, o, d, k=k, hit_capacity=cap, **kw)
    torch.cuda.synchronize()
    for key in ("rgb", "depth", "opacity", "hit_ids", "hit_counts"):
        assert torch.equal(got[key], ref[key]), key
    return ref


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 16, 17, 65, 257, 1000])
@pytest.mark.parametrize("rays", [1, 3, 5, 63, 257])
def test_small_trees_and_few_rays(n, rays):
    check(scene_of(n, 10 + n, degree=n % 4), *rays_of(rays, n + rays))


@pytest.mark.parametrize("opacity,t_min", [(-6.0, 0.0), (-6.0, 1e-3), (-3.0, 1e-3), (3.0, 1e-3), (6.0, 0.5)])
def test_long_lists_and_cut_rounds(opacity, t_min):
    # faint Gaussians: hundreds of hits a ray, more than a list holds; opaque ones: rays that
    # end after a hit or two
    ref = check(scene_of(20_000, 3, opacity=opacity), *rays_of(700, 4), cap=2048, T_min=t_min)
    assert opacity > -6.0 or int(ref["hit_counts"].max()) > 160


@pytest.mark.parametrize("n,scale,opacity", [(3_000, -2.2, -4.0), (8_000, -3.0, -5.0), (30_000, -3.0, -4.0), (60_000, -3.4, -3.0)])
def test_lists_that_grow_after_a_cut(n, scale, opacity):
    # rays with some 50 to 300 hits, in a launch whose waves take new rays as others end: sorted
    # starts of every length meet from one to 32 new hits, and other groups' first lists
    ref = check(scene_of(n, n, degree=1, scale=scale, opacity=opacity), *rays_of(70_001, 8), cap=2048)
    assert int(ref["hit_counts"].max()) > 64


def test_stacks_beyond_lds():
    # large overlapping Gaussians around the origins: a ray enters most of 60,000 boxes
    check(scene_of(60_000, 5, spread=0.05, scale=-2.0, opacity=-5.0, degree=1), *rays_of(64, 6, box=0.02), cap=4096)


@pytest.mark.parametrize("repeat", [8, 257])
def test_equal_distances(repeat):
    # the same centres many times: keys tie in distance and are told apart by their leaf (more
    # ties than the one-lane kernel's lists hold, so it restarts each round from the root here)
    sc = scene_of(2056, 7, repeat=repeat, opacity=-2.0)
    sc.scales[:] = np.repeat(sc.scales[::repeat], repeat, 0)[:sc.n]
    sc.quats[:] = np.repeat(sc.quats[::repeat], repeat, 0)[:sc.n]
    sc.opacities[:] = np.repeat(sc.opacities[::repeat], repeat, 0)[:sc.n]
    check(sc, *rays_of(300, 8), cap=1024, T_min=0.0, ref_mode=grtx.RESTART)


@pytest.mark.parametrize("kind", [grtx.SPHERE_INSTANCE, grtx.ICO_INSTANCE, grtx.PROXY20])
@pytest.mark.parametrize("k,caps,ties", [(16, (0, 0), 257), (1, (8, 8), 40), (4, (64, 16), 33), (64, (8, 8), 200)])
def test_more_ties_than_the_lists_hold(kind, k, caps, ties):
    """More hits at one distance than the k-buffer and the eviction list hold, in checkpointed
    launches of the one-lane kernel: a round that could blend none of them is followed by one
    without lists, and the ray ends with the hits of restart mode."""
    print("[case] ties", kind, k, caps, ties, flush=True)
    sc = scene_of(4 * ties, 7, degree=1, repeat=ties, opacity=-2.0)
    for a in (sc.scales, sc.quats, sc.opacities):
        a[:] = np.repeat(a[::ties], ties, 0)
    bvh = grtx.build(grtx.SceneTensors.from_scene(sc, "cuda"), kind=kind, alpha_min=AMIN)
    o, d = rays_of(130, 8)
    kw = dict(k=k, T_min=0.0, hit_capacity=1024, stats=True)
    ref = grtx.trace(bvh, o, d, mode=grtx.RESTART, **kw)
    got = grtx.trace(bvh, o, d, defer_capacity=caps[0], evict_capacity=caps[1], **kw)
    torch.cuda.synchronize()
    assert int(ref["hit_counts"].max()) >= ties
    assert int(got["stats"][:, grtx.STAT_FALLBACKS].max()) > 0
    for key in ("rgb", "depth", "opacity", "hit_ids", "hit_counts"):
        assert torch.equal(got[key], ref[key]), key


@pytest.mark.parametrize("degree", [0, 1, 2, 3])
def test_bounds_and_starting_transmittance(degree):
    o, d = rays_of(900, 9)
    g = torch.Generator(device="cuda").manual_seed(degree)
    far = torch.rand(900, device="cuda", generator=g) * 2.0
    far[::7] = float("inf")
    trans = torch.rand(900, device="cuda", generator=g)
    trans[::11] = 0.0
    check(scene_of(5000, 20 + degree, degree), o, d, t_far=far, transmittance=trans, bg=(0.2, 0.5, 0.7), k=4)
    check(scene_of(5000, 30 + degree, degree), o, d, t_near=0.3, bg=(0.2, 0.5, 0.7), cap=3)


@pytest.mark.parametrize("width,height,free", [(1, 1, 0), (7, 9, 0), (33, 17, 5), (64, 64, 130)])
def test_ragged_images_and_continuations(width, height, free):
    cam = inputs.orbit_camera(width, height, eye=(0.0, -1.5, 0.2))
    po, pd = grtx.pinhole_rays(cam)
    fo, fd = rays_of(max(free, 1), 11)
    o, d = torch.cat([fo[:free], po]), torch.cat([fd[:free], pd])
    sc = scene_of(3000, 12)
    check(sc, o, d, image_width=width, image_begin=free)
    ob = grtx.object_rays({"sphere": (0.1, -0.3, 0.0, 0.25, 1.5), "mirror": (-0.2, 0.1, 0.0, 0.3, 0.2, 0, 0, 0, 0.4),
                           "eps": 1e-4}, o, d)
    check(sc, o, d, image_width=width, image_begin=free, t_far=ob["t_far"], continuation=ob)


def test_degenerate_rays():
    o, d = rays_of(64, 13)
    o[::5] = 1e30
    d[1::5] = 0.0
    d[2::5, 0] = 0.0
    o[3::5] = float("nan")
    d[4::20] = float("nan")
    bvh = grtx.build(grtx.SceneTensors.from_scene(scene_of(2000, 14), "cuda"), alpha_min=AMIN)
    ref = grtx.trace(bvh, o, d, stats=True)
    got = grtx.trace(bvh, o, d)
    for key in ("rgb", "depth", "opacity"):
        assert torch.equal(torch.nan_to_num(got[key], 7.0), torch.nan_to_num(ref[key], 7.0)), key


@pytest.mark.parametrize("k", [1, 2, 4, 8, 16, 32, 64])
def test_counting_kernel_at_every_k(k):
    # the rounds of k hits, which only launches with counters, restart mode and proxies take
    cam = inputs.orbit_camera(160, 120)
    o, d = grtx.pinhole_rays(cam)
    ref = check(inputs.cluster_scene(2, 100_000, 3), o, d, cap=128, k=k, image_width=160)
    assert int(ref["stats"][:, grtx.STAT_ROUNDS].max()) * k >= int(ref["hit_counts"].max()) > 16


@pytest.mark.parametrize("what", ["plain frame", "frame", "incoherent"])
def test_against_the_oracle(what):
    """The sixteen-lane kernel itself, by the parity rule, without the detour over the other one."""
    print("[case]", what, flush=True)
    scene = inputs.small_scene(1, 1000) if what == "plain frame" else inputs.cluster_scene(2, 100_000, 3)
    width = {"plain frame": 64, "frame": 800, "incoherent": 0}[what]
    if width:
        o, d = (a.astype(np.float32) for a in oracle.pinhole_rays(inputs.orbit_camera(width, width)))
    else:
        o, d = inputs.incoherent_rays(33, 70_000)
    bvh = grtx.build(grtx.SceneTensors.from_scene(scene, "cuda"), alpha_min=AMIN)
    out = grtx.trace(bvh, torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda(), T_min=1e-3, image_width=width,
                     hit_capacity=512)
    idx = np.arange(len(o)) if what == "plain frame" else inputs.ray_subsample(321, len(o), 768)
    sub = {key: v.cpu().numpy()[idx] for key, v in out.items()}
    ref = oracle.render(scene, o[idx], d[idx], AMIN, 1e-3, cap=512)
    print(parity.compare_render(scene, o[idx], d[idx], sub, ref, AMIN, 1e-3, label=what), flush=True)


def test_largest_launch_equals_the_counting_kernel():
    """3M Gaussians, 2M incoherent rays and the 1920x1080 frame in one launch: rays that start in
    dense clusters, whose stacks leave LDS, and every wave taking new work many times over."""
    print("[case] 3M", flush=True)
    cfg = inputs.SCENE3M
    cam = inputs.orbit_camera(cfg["width"], cfg["height"])
    po, pd = grtx.pinhole_rays(cam)
    fo, fd = (torch.from_numpy(a).cuda() for a in inputs.incoherent_rays(cfg["incoherent_seed"], cfg["incoherent"]))
    check(inputs.cluster_scene(cfg["seed"], cfg["n"], 3), torch.cat([fo, po]), torch.cat([fd, pd]), cap=64,
          image_width=cfg["width"], image_begin=len(fo))
