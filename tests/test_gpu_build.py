"""The build's kernels at the sizes where their work is cut: subtrees of the restructuring pass
(256 leaves, 128 above 2^20), runs of the box tree, tiles of the radix sort. Needs an MI355X."""
import numpy as np
import pytest

from paper_2601_20429_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_2601_20429_amd import grtx  # noqa: E402

AMIN = float(np.float32(1.0 / 255.0))


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def build(n, seed, plain, dups=1, kind=grtx.SPHERE_INSTANCE):
    sc = inputs.cluster_scene(seed, n, 0)
    if dups > 1:
        sc.means[:] = np.repeat(sc.means[::dups], dups, 0)[:n]
    return grtx.build(grtx.SceneTensors.from_scene(sc, "cuda"), alpha_min=AMIN, plain_lbvh=plain, kind=kind)


def check_tree(t, n):
    """Every node has one parent and is reached once; a node's box is its children's union."""
    child = t["child"].cpu().numpy().view(np.uint32)
    parent = t["parent"].cpu().numpy().view(np.uint32)
    boxes = t["boxes"].cpu().numpy()
    node = np.where(child >> 31 != 0, (child & 0x7FFFFFFF) + (n - 1), child).astype(np.int64)
    assert parent[0] == 0xFFFFFFFF
    assert np.array_equal(np.sort(node.ravel()), np.arange(1, 2 * n - 1))
    assert np.array_equal(parent[node[:, 0]], np.arange(n - 1)) and np.array_equal(parent[node[:, 1]], np.arange(n - 1))
    depth, frontier = 0, np.array([0])
    seen = 0
    while frontier.size:
        depth, seen = depth + 1, seen + frontier.size
        nxt = node[frontier].ravel()
        frontier = nxt[nxt < n - 1]
    assert seen == n - 1
    a, b = boxes[node[:, 0]], boxes[node[:, 1]]
    assert np.array_equal(boxes[:n - 1, :3], np.minimum(a[:, :3], b[:, :3]))
    assert np.array_equal(boxes[:n - 1, 3:], np.maximum(a[:, 3:], b[:, 3:]))
    return depth


@pytest.mark.parametrize("n,dups", [(2, 1), (3, 1), (255, 1), (256, 1), (257, 1), (258, 3), (511, 1), (512, 512), (700, 1),
                                    (1025, 1), (4097, 7), (65537, 1), (300_001, 2)])
@pytest.mark.parametrize("plain", [False, True])
def test_trees_at_the_edges(n, dups, plain):
    bvh = build(n, 40 + n % 7, plain, dups)
    t = bvh.export_topology()
    info = bvh.info()
    assert check_tree(t, n) == info["depth"]
    assert info["restructured"] == (0 if plain or n < 3 else 1)
    assert np.array_equal(t["boxes"][0].cpu().numpy(), np.array(info["root_lo"] + info["root_hi"], np.float32))
    codes = t["morton"].cpu().numpy().view(np.uint64)
    assert np.all(codes[1:] >= codes[:-1])
    perm = t["perm"].cpu().numpy()
    assert np.array_equal(np.sort(perm), np.arange(n))
    assert np.all(perm[1:][codes[1:] == codes[:-1]] > perm[:-1][codes[1:] == codes[:-1]])  # stable


@pytest.mark.parametrize("n,dups", [(257, 1), (700, 5), (5000, 1), (40_000, 3)])
def test_restructured_tree_renders_like_the_plain_one(n, dups):
    cam = inputs.orbit_camera(97, 61)
    o, d = grtx.pinhole_rays(cam)
    a, b = (grtx.trace(build(n, 50, p, dups), o, d, image_width=97, hit_capacity=256) for p in (False, True))
    for key in ("rgb", "depth", "opacity", "hit_ids", "hit_counts"):
        assert torch.equal(a[key], b[key]), key


@pytest.mark.parametrize("n", [5, 257, 5000, 1_100_000])
@pytest.mark.parametrize("what", ["scale", "all scales", "mean", "mean and scales"])
def test_trees_over_infinite_gaussians(n, what):
    """Boxes whose surface area is infinite or no number leave a treelet without a cheapest split:
    the build still ends with a tree over all leaves, and so do rays through it, alike in both
    kernels."""
    print("[case] infinite", n, what, flush=True)
    sc = inputs.cluster_scene(61, n, 0)
    odd = np.arange(0, n, 3 if n <= 5000 else 97)
    if what == "scale":  # (unrotated: the box is no number on the other axes, and neither is its area)
        sc.quats[odd] = np.float32([1, 0, 0, 0])
        sc.scales[odd, 0] = np.inf
    if "scales" in what:
        sc.scales[odd] = np.inf
    if "mean" in what:
        sc.means[odd, 1] = np.inf
    bvh = grtx.build(grtx.SceneTensors.from_scene(sc, "cuda"), alpha_min=AMIN)
    child = bvh.export_topology()["child"].cpu().numpy().view(np.uint32)
    node = np.where(child >> 31 != 0, (child & 0x7FFFFFFF) + (n - 1), child).astype(np.int64)
    assert np.array_equal(np.sort(node.ravel()), np.arange(1, 2 * n - 1))  # every node once
    o, d = grtx.pinhole_rays(inputs.orbit_camera(40, 30))
    ref = grtx.trace(bvh, o, d, image_width=40, stats=True)
    got = grtx.trace(bvh, o, d, image_width=40)
    for key in ("rgb", "depth", "opacity"):
        assert torch.equal(torch.nan_to_num(got[key], 7.0), torch.nan_to_num(ref[key], 7.0)), key
