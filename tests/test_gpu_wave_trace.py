"""The wave-per-ray forward against the plain tracer (every record tested) and
against itself: many rounds per ray, every lane count of a launch, the channel
counts around the lanes' own, packed launches of more items than lanes, and a
tree too deep for the wave's stack.  Bit for bit: both sides composite the same
hits in the same order with the same operations."""
import numpy as np
import pytest
import torch

from gpu_util import make_scene
from paper_2412_15867_amd import TraceConfig, synth, trace, trace_packed
from paper_2412_15867_amd.tracer import alloc_result

pytestmark = pytest.mark.gpu


def same(a, b, rays=slice(None)):
    for name in ("opacity", "feat", "depth", "T", "n_hits"):
        x, y = getattr(a, name)[rays], getattr(b, name)[rays]
        assert torch.equal(x, y), name
    if a.hit_ids is not None:
        for i in range(a.n_hits[rays].numel()):
            n = min(int(a.n_hits[rays][i]), a.hit_ids.shape[1])
            assert torch.equal(a.hit_ids[rays][i, :n], b.hit_ids[rays][i, :n])
            assert torch.equal(a.hit_T[rays][i, :n], b.hit_T[rays][i, :n])


def layers(n, F, alpha, seed=5):
    """n wide, faint surfels stacked along z, seen by rays down the stack."""
    g = np.random.Generator(np.random.PCG64(seed))
    mu = np.zeros((n, 3), np.float32)
    mu[:, 2] = g.permutation(n).astype(np.float32) * 0.01
    quat = np.tile(np.array([1, 0, 0, 0], np.float32), (n, 1))
    scale = np.full((n, 2), 0.5, np.float32)
    opac = np.full(n, alpha, np.float32)
    feat = g.uniform(0, 1, (n, F)).astype(np.float32)
    s = make_scene(synth.Surfels(mu, quat, scale, opac, feat))
    xy = g.uniform(-0.4, 0.4, (37, 2))
    ro = np.concatenate([xy, np.full((37, 1), -1.0)], 1).astype(np.float32)
    rd = np.tile(np.array([0, 0, 1], np.float32), (37, 1))
    return s, torch.from_numpy(ro).cuda(), torch.from_numpy(rd).cuda()


@pytest.mark.parametrize("n", [1, 3, 63, 64, 65, 128, 129, 300])
@pytest.mark.parametrize("alpha", [0.02, 0.3])
def test_rounds(n, alpha):
    s, ro, rd = layers(n, 3, alpha)
    got = trace(s, ro, rd, TraceConfig(k=16), hit_cap=100)
    same(got, trace(s, ro, rd, TraceConfig(k=16, brute_force=True), hit_cap=100))
    assert int(got.n_hits.max()) >= min(n, 20)


@pytest.mark.parametrize("F", [1, 5, 8, 9, 15, 16, 17, 29, 61, 62, 63, 64])
def test_channels(F):
    s, ro, rd = layers(150, F, 0.05)
    same(trace(s, ro, rd, TraceConfig(k=32)), trace(s, ro, rd, TraceConfig(k=32, brute_force=True)))


@pytest.mark.parametrize("R", [1, 2, 63, 65, 8191, 8192, 8193, 20_001])
@pytest.mark.parametrize("sort_rays", [False, True])
def test_ray_counts(R, sort_rays):
    s = make_scene(synth.surface_scene(3000, F=8, seed=3))
    ro, rd = synth.mc_rays(R, 1, seed=R)
    ro, rd = torch.from_numpy(ro).cuda(), torch.from_numpy(rd).cuda()
    got = trace(s, ro, rd, TraceConfig(k=16, sort_rays=sort_rays))
    same(got, trace(s, ro, rd, TraceConfig(k=16, brute_force=True)))


@pytest.mark.parametrize("items", [1, 63, 64, 65, 150])
def test_packed_items(items):
    scenes = [make_scene(synth.surface_scene(n, F=4, seed=n)) for n in (700, 2500)]
    cfg = TraceConfig(k=32)
    reqs = []
    for i in range(items):
        ro, rd = synth.mc_rays(1 + i % 7, 9, seed=100 + i)
        ro, rd = torch.from_numpy(ro).cuda(), torch.from_numpy(rd).cuda()
        reqs.append((i % 2, ro, rd, alloc_result(ro.shape[0], 4, ro.device)))
    trace_packed(scenes, reqs, cfg)
    for s, ro, rd, res in reqs:
        same(res, trace(scenes[s], ro, rd, cfg))


@pytest.mark.parametrize("n,ratio", [(600, 1.05), (200, 1.1)])
def test_chain_of_growing_surfels(n, ratio):
    """Each surfel dwarfs the ones before it: a chain-like tree (with 600 deeper
    than the wave's stack takes, with 200 close to it)."""
    g = np.random.Generator(np.random.PCG64(9))
    size = (ratio ** np.arange(n)).astype(np.float64)
    mu = np.stack([size, size * 0.5, size * 0.25], 1).astype(np.float32)
    q = g.standard_normal((n, 4)).astype(np.float32)
    scale = np.stack([size * 0.2, size * 0.1], 1).astype(np.float32)
    sc = synth.Surfels(mu, q, scale, g.uniform(0.1, 0.9, n).astype(np.float32), g.uniform(0, 1, (n, 3)).astype(np.float32))
    s = make_scene(sc)
    idx = g.integers(0, n, 400)
    d = g.standard_normal((400, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    ro = torch.from_numpy((mu[idx] - d * size[idx, None] * 2).astype(np.float32)).cuda()
    rd = torch.from_numpy(d.astype(np.float32)).cuda()
    got = trace(s, ro, rd, TraceConfig(k=16))
    same(got, trace(s, ro, rd, TraceConfig(k=16, brute_force=True)))
    assert int(got.n_hits.sum()) > 100


@pytest.mark.parametrize("size", [0.02, 1.0, 300.0])
@pytest.mark.parametrize("offset", [0.0, 40.0])
@pytest.mark.parametrize("flip", [False, True])
def test_slabs_lose_no_hit(size, offset, flip):
    """Rays that skim their own surface and Monte Carlo rays, on scenes of
    different size and distance from the origin, with the surfels' normals as
    generated or turned to random sides: the slabs of the tree's children cull
    nothing that the plain tracer hits."""
    sc = synth.surface_scene(4000, F=3, seed=21)
    g = np.random.Generator(np.random.PCG64(4))
    quat = sc.quat.copy()
    if flip:  # half a turn about t_u: the same disc, its normal on the other side
        w, x, y, z = quat.T
        half = np.stack([-x, w, z, -y], 1)
        quat = np.where(g.random((4000, 1)) < 0.5, half, quat).astype(np.float32)
    shift = np.float32(offset * size)
    s = make_scene(synth.Surfels(sc.mu * np.float32(size) + shift, quat, sc.scale * np.float32(4 * size), sc.opac, sc.feat))
    ro, rd = (np.concatenate(p) for p in zip(synth.grazing_rays(6000), synth.mc_rays(100, 61, seed=8)))
    ro = torch.from_numpy(ro * np.float32(size) + shift).cuda()
    rd = torch.from_numpy(rd).cuda()
    got = trace(s, ro, rd, TraceConfig(k=32))
    same(got, trace(s, ro, rd, TraceConfig(k=32, brute_force=True)))
    assert float(got.n_hits.float().mean()) > 5
    s.refit()
    same(trace(s, ro, rd, TraceConfig(k=32)), got)


@pytest.mark.parametrize("R", [32_767, 32_768, 32_769, 70_001, 600_000])
def test_sorted_launch_sizes(R):
    """Ray sorts whose tile counters fill one, just over one and many spans of
    the counters' scan (4,096 counters = 16 tiles of 2,048 rays)."""
    s = make_scene(synth.surface_scene(3000, F=3, seed=3))
    g = torch.Generator(device="cuda").manual_seed(R)
    ro = torch.rand(R, 3, generator=g, device="cuda") * 4 - 2
    rd = -ro / ro.norm(dim=1, keepdim=True)
    same(trace(s, ro, rd, TraceConfig(k=16, sort_rays=True)), trace(s, ro, rd, TraceConfig(k=16)))


@pytest.mark.parametrize("items", [1000, 4096, 4097])
def test_packed_many_items(items):
    """As many items as take one, two and three looks of 64 to find a ray's own,
    some of them without rays."""
    scenes = [make_scene(synth.surface_scene(n, F=4, seed=n)) for n in (700, 2500)]
    cfg = TraceConfig(k=16)
    ro, rd = (torch.from_numpy(a).cuda() for a in synth.mc_rays(6000, 3, seed=items))
    g = np.random.Generator(np.random.PCG64(items))
    count = g.integers(0, 4, items)
    end = np.cumsum(count)
    reqs = [(i % 2, ro[e - c:e], rd[e - c:e], alloc_result(int(c), 4, ro.device))
            for i, (c, e) in enumerate(zip(count, end))]
    trace_packed(scenes, reqs, cfg)
    for s in range(2):
        ref = trace(scenes[s], ro, rd, cfg)
        rays = torch.from_numpy(np.concatenate([np.arange(e - c, e) for c, e in zip(count[s::2], end[s::2])])).cuda()
        for name in ("opacity", "feat", "depth", "T", "n_hits"):
            got = torch.cat([getattr(r[3], name) for r in reqs[s::2]])
            assert torch.equal(got, getattr(ref, name)[rays]), name
