"""The backward pass at the sizes where its work is cut (16 hits of a ray, four rays of a wave,
shares of the sorted hits, Gaussians that reach over many shares), on made-up hit lists, against
the same compositing differentiated in float64. Needs an MI355X."""
import numpy as np
import pytest

import oracle
from paper_2601_20429_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_2601_20429_amd import grtx  # noqa: E402

NAMES = ["means", "scales", "quats", "opacities", "sh"]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def composite(p, o, d, Y, ids, live):
    """Front-to-back compositing of the listed hits, in list order: (rgb, depth, opacity)."""
    i = ids.clamp(0, len(p["means"]) - 1)
    q = p["quats"] / p["quats"].norm(dim=1, keepdim=True)
    w, x, y, z = q.unbind(1)
    R = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                     2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                     2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1).view(-1, 3, 3)
    M = (R.transpose(1, 2) / p["scales"][:, :, None])[i]
    u = (M * (o[:, None] - p["means"][i])[:, :, None, :]).sum(3)
    v = (M * d[:, None, None, :]).sum(3)
    t = -(u * v).sum(2) / (v * v).sum(2)
    c = u + t[..., None] * v
    alpha = torch.where(live, p["opacities"][i] * torch.exp(-0.5 * (c * c).sum(2)), 0.0)
    col = (0.5 + (p["sh"][i] * Y[:, None, :, None]).sum(2)).clamp(min=0)
    T = torch.cumprod(torch.cat([torch.ones_like(alpha[:, :1]), 1 - alpha], 1), 1)
    wgt = T[:, :-1] * alpha
    return (wgt[..., None] * col).sum(1), (wgt * t).sum(1), 1 - T[:, -1]


# rays, Gaussians, list capacity, degree, shortest list, which gradients are given
CASES = [(1, 1, 1, 3, 1, "rdo"), (3, 5, 4, 0, 0, "rdo"), (64, 7, 16, 1, 16, "r"), (77, 300, 33, 2, 0, "do"),
         (1000, 40, 20, 3, 0, "rdo"), (4099, 3, 40, 3, 10, "rdo"), (6000, 500, 60, 3, 50, "rdo"),
         (65, 1, 17, 3, 17, "o"), (3000, 70_000, 24, 0, 0, "rdo"), (15_000, 70_000, 24, 0, 0, "rdo")]


@pytest.mark.parametrize("rays,n,cap,degree,least,given", CASES)
def test_sums_of_made_up_lists(rays, n, cap, degree, least, given):
    """A hit's u has an error of a few float32 steps of |f| / s (at most some 50), so alpha one of
    some 1e-5, which 1 / (1 - alpha) at most trebles: 5e-4 of the gradient and of its group's rms
    leaves a factor of ten. Entries that name no Gaussian of the scene are passed by."""
    print("[case]", rays, n, cap, degree, flush=True)
    g = torch.Generator().manual_seed(rays + n)
    rnd = lambda *s: torch.randn(*s, generator=g)
    uni = lambda *s: torch.rand(*s, generator=g)
    sc = inputs.cluster_scene(1, n, degree)
    p = dict(means=0.5 * rnd(n, 3), scales=0.3 + 0.7 * uni(n, 3), quats=rnd(n, 4), opacities=0.02 + 0.5 * uni(n),
             sh=0.3 * rnd(n, (degree + 1) ** 2, 3))
    p["quats"] += torch.sign(p["quats"]) * 0.1
    for k, v in p.items():
        getattr(sc, k)[...] = v.numpy().reshape(getattr(sc, k).shape)
    o = torch.tensor([0.0, 0.0, -4.0]) + 0.5 * rnd(rays, 3)
    d = torch.tensor([0.0, 0.0, 1.0]) + 0.2 * rnd(rays, 3)
    ids = torch.randint(0, n, (rays, cap), generator=g, dtype=torch.int32)
    ids[uni(rays, cap) < 0.03] = -1
    ids[uni(rays, cap) < 0.03] = n + 2
    counts = torch.randint(least, cap + 1, (rays,), generator=g, dtype=torch.int32)
    live = (torch.arange(cap) < counts[:, None]) & (ids >= 0) & (ids < n)

    p64 = {k: v.double().requires_grad_() for k, v in p.items()}
    dn = (d.double() / d.double().norm(dim=1, keepdim=True)).numpy()
    Y = torch.tensor([[oracle.sh_basis(l, m, x) for l in range(degree + 1) for m in range(-l, l + 1)] for x in dn],
                     dtype=torch.float64)
    out = composite(p64, o.double(), d.double(), Y, ids.long(), live)
    up = dict(r=rnd(rays, 3), d=rnd(rays), o=rnd(rays))
    sum((up[k].double() * x).sum() for k, x in zip("rdo", out) if k in given).backward()

    bvh = grtx.build(grtx.SceneTensors.from_scene(sc, "cuda"))
    cu = lambda x: x.detach().float().contiguous().cuda()
    fwd = dict(rgb=cu(out[0]), depth=cu(out[1]), opacity=cu(out[2]), hit_ids=ids.cuda(), hit_counts=counts.cuda())
    start = {k: torch.full_like(getattr(bvh.scene, k), 1.0) for k in NAMES}  # (the pass adds to what is there)
    runs = []
    for _ in range(2):
        grads, cut = grtx.trace_backward(bvh, o.cuda(), d.cuda(), fwd, *(up[k].cuda() if k in given else None for k in "rdo"),
                                         grads={k: v.clone() for k, v in start.items()})
        assert int(cut.item()) == 0
        runs.append(grads)
    for k in NAMES:
        assert torch.equal(runs[0][k], runs[1][k]), k
        want = (torch.zeros_like(p64[k]) if p64[k].grad is None else p64[k].grad).numpy().reshape(-1)
        got = (runs[0][k].double() - 1.0).cpu().numpy().reshape(-1)
        tol = 5e-4 * (np.abs(want) + np.sqrt((want ** 2).mean())) + 2e-7  # (the last: of the ones)
        bad = np.abs(got - want) > tol
        assert not bad.any(), (k, int(bad.sum()), np.abs(got - want)[bad][:4], want[bad][:4])


@pytest.mark.parametrize("n", [200, 70_000, 300_000])
def test_sums_behind_a_scanned_sort(n):
    """A bound of rays x capacity that gives the sort of the hits a table too large for its workgroups
    to add up themselves (above 16.8M; digits of eight and nine bits), with few hits in it. Tolerance
    as above."""
    rays, cap, most = 300_000, 64, 4
    print("[case] scanned", n, flush=True)
    g = torch.Generator().manual_seed(n)
    rnd = lambda *s: torch.randn(*s, generator=g)
    uni = lambda *s: torch.rand(*s, generator=g)
    sc = inputs.cluster_scene(1, n, 0)
    p = dict(means=0.5 * rnd(n, 3), scales=0.3 + 0.7 * uni(n, 3), quats=rnd(n, 4), opacities=0.02 + 0.5 * uni(n),
             sh=0.3 * rnd(n, 1, 3))
    p["quats"] += torch.sign(p["quats"]) * 0.1
    for k, v in p.items():
        getattr(sc, k)[...] = v.numpy().reshape(getattr(sc, k).shape)
    o = torch.tensor([0.0, 0.0, -4.0]) + 0.5 * rnd(rays, 3)
    d = torch.tensor([0.0, 0.0, 1.0]) + 0.2 * rnd(rays, 3)
    ids = torch.randint(0, n, (rays, most), generator=g, dtype=torch.int32)
    counts = torch.randint(0, most + 1, (rays,), generator=g, dtype=torch.int32)
    live = torch.arange(most) < counts[:, None]

    p64 = {k: v.double().requires_grad_() for k, v in p.items()}
    Y = torch.full((rays, 1), float(oracle.sh_basis(0, 0, np.float64([0, 0, 1]))), dtype=torch.float64)
    out = composite(p64, o.double(), d.double(), Y, ids.long(), live)
    up = (rnd(rays, 3), rnd(rays), rnd(rays))
    sum((u.double() * x).sum() for u, x in zip(up, out)).backward()

    bvh = grtx.build(grtx.SceneTensors.from_scene(sc, "cuda"))
    cu = lambda x: x.detach().float().contiguous().cuda()
    lists = torch.full((rays, cap), -1, dtype=torch.int32)
    lists[:, :most] = ids
    fwd = dict(rgb=cu(out[0]), depth=cu(out[1]), opacity=cu(out[2]), hit_ids=lists.cuda(), hit_counts=counts.cuda())
    grads, cut = grtx.trace_backward(bvh, o.cuda(), d.cuda(), fwd, *(u.cuda() for u in up))
    assert int(cut.item()) == 0
    for k in NAMES:
        want = p64[k].grad.numpy().reshape(-1)
        got = grads[k].double().cpu().numpy().reshape(-1)
        bad = np.abs(got - want) > 5e-4 * (np.abs(want) + np.sqrt((want ** 2).mean())) + 2e-7
        assert not bad.any(), (k, int(bad.sum()), np.abs(got - want)[bad][:4], want[bad][:4])
