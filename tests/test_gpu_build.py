"""The clustering build around the sizes where its last iterations move into one
block, and with every cost the same: a tree that lost, repeated or misplaced a
surfel would answer unlike the plain tracer, which looks at every surfel.  Bit
for bit: both composite the same hits in the same order."""
import numpy as np
import pytest
import torch

from gpu_util import make_scene
from paper_2412_15867_amd import TraceConfig, synth, trace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 3, 17, 1023, 1024, 1025, 2049, 20_001])
@pytest.mark.parametrize("coincident", [False, True])
def test_sizes(n, coincident):
    g = np.random.Generator(np.random.PCG64(n))
    mu = (g.uniform(-1, 1, (n, 3)) * (not coincident)).astype(np.float32)
    q = g.normal(size=(1 if coincident else n, 4))
    q = np.broadcast_to(q / np.linalg.norm(q, axis=1, keepdims=True), (n, 4)).astype(np.float32)
    s = make_scene(synth.Surfels(mu, q, np.full((n, 2), 0.05, np.float32), np.full(n, 0.3, np.float32),
                                 g.uniform(0, 1, (n, 3)).astype(np.float32)))
    ro = torch.from_numpy(g.uniform(-1, 1, (257, 3)).astype(np.float32)).cuda()
    rd = torch.nn.functional.normalize(-ro + 0.02 * torch.randn(257, 3, generator=torch.Generator().manual_seed(1)).cuda(), dim=1)
    for _ in range(2):  # the second time over the buffers of the first
        got = trace(s, ro, rd, TraceConfig())
        want = trace(s, ro, rd, TraceConfig(brute_force=True))
        for name in ("opacity", "feat", "depth", "T", "n_hits"):
            assert torch.equal(getattr(got, name), getattr(want, name)), name
        s.build()
    assert int(got.n_hits.sum()) > 0


@pytest.mark.parametrize("n,ratio", [(1, 1.0), (2, 1.0), (600, 1.0), (600, 1.05), (2049, 1.0), (9000, 1.0)])
def test_refit_levels(n, ratio):
    """Boxes and slabs level by level: levels below, at and above one block's
    size, and (growing surfels) more levels than one run holds."""
    g = np.random.Generator(np.random.PCG64(n))
    grow = (ratio ** np.arange(n)).astype(np.float32)[:, None]
    mu = (g.uniform(-1, 1, (n, 3)) * grow).astype(np.float32)
    q = g.normal(size=(n, 4))
    q = (q / np.linalg.norm(q, axis=1, keepdims=True)).astype(np.float32)
    scale = np.full((n, 2), 0.05, np.float32) * grow
    s = make_scene(synth.Surfels(mu, q, scale.astype(np.float32), np.full(n, 0.3, np.float32),
                                 g.uniform(0, 1, (n, 3)).astype(np.float32)))
    moved = torch.from_numpy((mu + 0.3 * g.uniform(-1, 1, (n, 3)) * grow).astype(np.float32)).cuda()
    s.set_params(moved, s.quat, s.scale, s.opacity, s.feat)
    s.refit()
    aim = moved[torch.arange(257, device="cuda") % n]
    ro = 2.0 * torch.from_numpy(g.uniform(-1, 1, (257, 3)).astype(np.float32)).cuda()
    rd = torch.nn.functional.normalize(aim - ro, dim=1)
    got = trace(s, ro, rd, TraceConfig())
    want = trace(s, ro, rd, TraceConfig(brute_force=True))
    for name in ("opacity", "feat", "depth", "T", "n_hits"):
        assert torch.equal(getattr(got, name), getattr(want, name)), name
    assert int(got.n_hits.sum()) > 0
