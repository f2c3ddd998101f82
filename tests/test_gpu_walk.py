"""The backward's walk over hit lists at the sizes where it can go wrong: rays
around its groups and chunks, feature counts around its instances, lists cut at
their capacity (traced again by a wave) and hits past the wave's own list
(re-marched by a lane).  Reference: FP64 autograd over the GPU's own hit lists."""
import dataclasses

import numpy as np
import pytest
import torch

from gpu_util import dev, make_scene
from oracle import grad as ograd
from paper_2412_15867_amd import TraceConfig, synth, trace, trace_backward

pytestmark = pytest.mark.gpu
KEYS = (("mu", "mu"), ("quat", "quat"), ("scale", "scale"), ("opacity", "opac"), ("feat", "feat"))


def stack(n, F, alpha, R, seed=5):
    """n tilted, faint surfels along z and R rays near the axis."""
    g = np.random.Generator(np.random.PCG64(seed))
    mu = np.concatenate([g.uniform(-0.1, 0.1, (n, 2)), (g.permutation(n) * 0.01)[:, None]], 1)
    quat = np.concatenate([np.ones((n, 1)), g.uniform(-0.05, 0.05, (n, 3))], 1)
    sc = synth.Surfels(mu.astype(np.float32), quat.astype(np.float32),
                       g.uniform(0.4, 0.7, (n, 2)).astype(np.float32), np.full(n, alpha, np.float32),
                       g.uniform(0, 1, (n, F)).astype(np.float32))
    ro = np.concatenate([g.uniform(-0.3, 0.3, (R, 2)), np.full((R, 1), -1.0)], 1).astype(np.float32)
    d = np.concatenate([g.uniform(-0.02, 0.02, (R, 2)), np.ones((R, 1))], 1)
    rd = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    return sc, ro, rd


def check(sc, ro, rd, cfg, cap, mask=None, full=256):
    s = make_scene(sc)
    R = ro.shape[0]
    gO, gF, gD, _ = synth.upstream(R, sc.F, seed=3)
    if mask is not None:
        gO[~mask], gF[~mask], gD[~mask] = 0, 0, 0
    whole = trace(s, dev(ro), dev(rd), cfg, hit_cap=full)
    res = trace(s, dev(ro), dev(rd), cfg, hit_cap=cap)
    got = trace_backward(s, dev(ro), dev(rd), res, dev(gO), dev(gF), dev(gD), cfg=cfg)
    n = whole.n_hits.cpu().numpy()
    assert n.max() <= full
    ids = np.where(np.arange(full)[None] < n[:, None], whole.hit_ids.cpu().numpy(), -1)[:, :max(int(n.max()), 1)]
    want = ograd.grad_given_hits(sc.astuple(), ro, rd, ids, gO, gF, gD)
    for a, b in KEYS:
        g, w = got[a].cpu().numpy().reshape(want[b].shape), want[b]
        assert np.all(np.abs(g - w) <= 1e-3 * (np.abs(w) + np.abs(w).mean() + 1e-12)), a
    return n


@pytest.mark.parametrize("R", [1, 15, 17, 191, 193, 3001])
@pytest.mark.parametrize("F", [3, 9])
def test_ray_counts(R, F):
    sc, ro, rd = stack(40, F, 0.2, R)
    check(sc, ro, rd, TraceConfig(k=16), 64)


@pytest.mark.parametrize("F", [1, 8, 16, 17, 20, 21, 54, 55, 64])
def test_feature_counts(F):
    sc, ro, rd = stack(70, F, 0.1, 50)
    check(sc, ro, rd, TraceConfig(k=16), 256)


def test_rays_in_landing_order():
    """Enough rays to be taken in the order of where they land, many of them
    without hits or without an upstream gradient."""
    sc, ro, rd = stack(30, 4, 0.3, 16_500)
    rd[::5] *= -1
    check(sc, ro, rd, TraceConfig(k=16), 64, mask=np.arange(16_500) % 3 != 0)


@pytest.mark.parametrize("cap", [1, 40, 63, 64, 65, 200])
@pytest.mark.parametrize("F", [3, 12])
def test_cut_lists_are_traced_again(cap, F):
    sc, ro, rd = stack(230, F, 0.03, 130)
    n = check(sc, ro, rd, TraceConfig(k=16, T_min=0.0), cap)
    assert n.max() > cap


def test_hits_past_the_wave_list():
    sc, ro, rd = stack(2600, 3, 0.006, 5)
    n = check(sc, ro, rd, TraceConfig(k=16, T_min=0.0), 256, full=2600)
    assert n.max() > 2048


MODES = {"plain3": dict(F=3), "plain12": dict(F=12), "plain20": dict(F=20), "sh": dict(F=48, sh=True),
         "normals": dict(F=5, normals=True)}


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("R", [13_000, 20_000])
@pytest.mark.parametrize("mode", list(MODES))
def test_a_bad_upstream_stays_with_its_ray(mode, R, bad):
    """A few rays with a non-finite upstream gradient among many (two or three
    rays share a group, in the caller's order and in the landing order): every
    surfel that none of them hits has the gradients of a run in which they have
    no upstream at all.  Both runs add the same terms with FP32 atomics in
    different orders, a few dozen per surfel."""
    kw = dict(MODES[mode])
    F = kw.pop("F")
    sc = synth.surface_scene(20_000, F=F, seed=11)
    if mode == "sh":
        sc.feat[:] = synth.sh_coefficients(sc.n, 3)
    ro, rd = (a[:R] for a in synth.mc_rays(-(-R // 16), 16, seed=12))
    FO = 3 if mode == "sh" else F + 3 if mode == "normals" else F
    gO, gF, gD, _ = synth.upstream(R, FO, seed=13)
    s = make_scene(sc)
    cfg = TraceConfig(k=16, **kw)
    res = trace(s, dev(ro), dev(rd), cfg, hit_cap=256)
    n = res.n_hits.cpu().numpy()
    assert n.max() <= 256
    who = np.flatnonzero(n > 4)[::400]
    spoilt = np.unique(np.concatenate([res.hit_ids[int(r), :n[r]].cpu().numpy() for r in who]))
    clean = np.setdiff1d(np.arange(sc.n), spoilt)
    grads = []
    for value in (0.0, bad):
        for g in (gO, gF, gD):
            g[who] = 0.0
        for i, r in enumerate(who):
            if i % 3 == 0:
                gO[r] = value
            elif i % 3 == 1:
                gF[r, -1] = value
            else:
                gD[r] = value
        got = trace_backward(s, dev(ro), dev(rd), res, dev(gO), dev(gF), dev(gD), cfg=cfg)
        grads.append({a: got[a].cpu().numpy().reshape(sc.n, -1) for a, _ in KEYS})
    s.close()
    want, got = grads
    assert not np.all(np.isfinite(got["mu"][spoilt]))
    for a, _ in KEYS:
        w, g = want[a][clean], got[a][clean]
        assert np.all(np.isfinite(g)), (a, np.flatnonzero(~np.isfinite(g).all(1)).size)
        np.testing.assert_allclose(g, w, rtol=1e-4, atol=1e-5 * np.abs(want[a]).max(), err_msg=a)


def scene_of(sc, mode, **kw):
    """`sc` with the features of a mode, its config and what the oracle takes."""
    F = MODES[mode]["F"]
    g = np.random.Generator(np.random.PCG64(21))
    feat = synth.sh_coefficients(sc.n, 3) if mode == "sh" else g.uniform(0, 1, (sc.n, F)).astype(np.float32)
    sc = synth.Surfels(sc.mu, sc.quat, sc.scale, sc.opac, feat)
    cfg = TraceConfig(k=16, T_min=0.0, **{k: v for k, v in MODES[mode].items() if k != "F"})
    oracle = dict(sh_deg=3) if mode == "sh" else dict(with_normal=True) if mode == "normals" else {}
    return sc, make_scene(sc, **kw), cfg, oracle


def check_cut(sc, s, ro, rd, cfg, oracle, busy, cap, full):
    """Gradients with lists cut at `cap` against the oracle over the whole lists
    of the first `busy` rays, the only ones with an upstream."""
    R, FO = ro.shape[0], cfg.out_channels(sc.F)
    gO, gF, gD, _ = synth.upstream(R, FO, seed=3)
    gO[busy:], gF[busy:], gD[busy:] = 0, 0, 0
    whole = trace(s, dev(ro[:busy]), dev(rd[:busy]), cfg, hit_cap=full)
    res = trace(s, dev(ro), dev(rd), cfg, hit_cap=cap)
    got = trace_backward(s, dev(ro), dev(rd), res, dev(gO), dev(gF), dev(gD), cfg=cfg)
    n = whole.n_hits.cpu().numpy()
    assert cap < n.max() <= full
    ids = np.where(np.arange(full)[None] < n[:, None], whole.hit_ids.cpu().numpy(), -1)[:, :int(n.max())]
    want = ograd.grad_given_hits(sc.astuple(), ro[:busy], rd[:busy], ids, gO[:busy], gF[:busy], gD[:busy], **oracle)
    for a, b in KEYS:
        g, w = got[a].cpu().numpy().reshape(want[b].shape), want[b]
        assert np.all(np.abs(g - w) <= 1e-3 * (np.abs(w) + np.abs(w).mean() + 1e-12)), a
    return n


@pytest.mark.parametrize("R", [30, 33_000])
@pytest.mark.parametrize("n", [1000, 1500, 2600])
@pytest.mark.parametrize("mode", list(MODES))
def test_cut_lists_of_every_length(mode, n, R):
    """Hits around the list lengths of the wave re-marches (1,024 and 2,048) and
    past them, in a launch that takes the longer lists at once and in one that
    takes the shorter first; plain, SH and normal channels."""
    base, ro, rd = stack(n, 1, 0.006, R)
    rd[30:] *= -1  # away from the stack
    sc, s, cfg, oracle = scene_of(base, mode)
    hits = check_cut(sc, s, ro, rd, cfg, oracle, 30, 64, n)
    s.close()
    assert hits.max() > 0.8 * n


@pytest.mark.parametrize("R", [60, 20_000])
@pytest.mark.parametrize("n", [480, 512, 513, 700])
@pytest.mark.parametrize("mode", list(MODES))
def test_cut_lists_in_a_tree_too_deep_for_a_wave(mode, n, R):
    """Coincident surfels cluster into a chain (at most three binary levels per
    wide one, the last 12 surfels in a leaf: more than 150 wide levels, the wave
    form takes 132): forward and re-march run one lane per ray, its list holding
    512 hits.  The support is capped at half a scale, so that the boxes are the
    same whatever the opacity."""
    g = np.random.Generator(np.random.PCG64(17))
    base = synth.Surfels(np.zeros((n, 3), np.float32), np.tile(np.float32([1, 0.02, 0.03, 0.01]), (n, 1)),
                         np.full((n, 2), 0.5, np.float32), g.uniform(0.005, 0.012, n).astype(np.float32),
                         np.zeros((n, 1), np.float32))
    d = np.concatenate([g.uniform(-0.05, 0.05, (R, 2)), np.ones((R, 1))], 1)
    rd = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    ro = (g.uniform(-0.05, 0.05, (R, 3)) - rd).astype(np.float32)
    rd[30:] *= -1  # away from the surfels
    sc, s, cfg, oracle = scene_of(base, mode, support_sigma=0.5)
    assert s.info()["max_depth"] == n - 1
    got, want = (trace(s, dev(ro[:60]), dev(rd[:60]), dataclasses.replace(cfg, brute_force=b)) for b in (False, True))
    for name in ("opacity", "feat", "depth", "T", "n_hits"):
        assert torch.equal(getattr(got, name), getattr(want, name)), name
    hits = check_cut(sc, s, ro, rd, cfg, oracle, 30, 8, n)
    s.close()
    assert hits.min() > 400


@pytest.mark.parametrize("F,sh", [(8, False), (16, False), (64, False), (48, True)])
def test_more_surfels_than_the_table_takes(F, sh):
    """Faint surfels all over a cube: the 64 rays of a block meet about 1,500
    different ones, twice what its table of sums holds (843 of 1,350 slots at
    F <= 8, 218 of 350 with 64 features) before it is written out, and a
    step's 768 hits bring more new ones than the slots then left, so that some
    are added to memory directly."""
    g = np.random.Generator(np.random.PCG64(23))
    n, R = 8000, 16_384
    q = g.normal(size=(n, 4))
    sc = synth.Surfels(g.uniform(-1, 1, (n, 3)).astype(np.float32), q.astype(np.float32),
                       g.uniform(0.05, 0.08, (n, 2)).astype(np.float32), g.uniform(0.03, 0.06, n).astype(np.float32),
                       synth.sh_coefficients(n, 3) if sh else g.uniform(0, 1, (n, F)).astype(np.float32))
    ro = g.uniform(-1, 1, (R, 3)).astype(np.float32)
    d = g.uniform(-1, 1, (R, 3)) - ro
    rd = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    cfg = TraceConfig(k=16, sh=sh)
    gO, gF, gD, _ = synth.upstream(R, cfg.out_channels(F), seed=3)
    s = make_scene(sc)
    res = trace(s, dev(ro), dev(rd), cfg, hit_cap=256)
    got = trace_backward(s, dev(ro), dev(rd), res, dev(gO), dev(gF), dev(gD), cfg=cfg)
    got = {a: got[a].cpu().numpy().astype(np.float64) for a, _ in KEYS}
    hits, ids = res.n_hits.cpu().numpy(), res.hit_ids.cpu().numpy()
    s.close()
    assert hits.mean() > 30 and hits.max() <= 256
    want = None
    for b in range(0, R, 2048):  # the oracle's memory
        e = slice(b, b + 2048)
        lists = np.where(np.arange(256)[None] < hits[e, None], ids[e], -1)[:, :int(hits[e].max())]
        part = ograd.grad_given_hits(sc.astuple(), ro[e], rd[e], lists, gO[e], gF[e], gD[e], sh_deg=3 if sh else -1)
        want = part if want is None else {k: want[k] + part[k] for k in part}
    for a, b in KEYS:
        x, w = got[a].reshape(want[b].shape), want[b]
        assert np.all(np.abs(x - w) <= 1e-3 * (np.abs(w) + np.abs(w).mean())), a
