"""The Splatter with an MLP over tiles of four neighbouring rays, forward and backward: tiles that end early, rays of another
scene inside of one, points past the rays' ends, contract coordinates, windows that are split, steps that fit none, values that are
not finite."""
import dataclasses

import numpy as np
import pytest

from lp_inputs import TRIPLANE, VOXEL

from parity import WIDTH_CAP_SPLAT_BORDER, check_case_splat
from test_gpu_splat_patches import _image
from tile_rules import cells, splat_mlp_routes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oracle():
    import oracle as o
    return o


CONFIGS = [(16, 5, (64,), -1), (32, 32, (64, 64), 1)]
# an image, how its steps are pushed into voxels and into triplanes, and how the prior's gradient is scattered (voxels of 16 and 32 channels, triplanes alike)
FEW, SPLIT = {("tile", 1)}, {("tile", 1), ("tile", 2)}
IMAGES = [(dict(width=64, height=72, samples=9, res=(20, 23, 17), cut=1), FEW, FEW, (FEW,) * 4),
          (dict(width=66, height=70, samples=8, res=(40, 33, 37), per_scene=7), {("tile", 2), ("ray", "walk")}, {("tile", 2), ("ray", "walk")}, (SPLIT,) * 4),
          (dict(width=64, height=72, samples=10, res=(48, 40, 44)), SPLIT, SPLIT, (FEW,) * 4),
          (dict(width=64, height=72, samples=10, res=(90, 64, 70)), SPLIT | {("tile", 4)}, SPLIT | {("tile", 4)}, (FEW,) * 4),
          (dict(width=64, height=72, samples=9, res=(24, 22, 26), contract=1.0, far=9.0), SPLIT | {("tile", 4)}, SPLIT | {("tile", 4)}, (SPLIT | {("tile", 4)},) * 2 + (SPLIT,) * 2),
          # one long axis: consecutive points of a ray are further apart along it than a window is long
          (dict(width=256, height=16, samples=9, res=(300, 16, 14), prior_res=(310, 15, 17)), SPLIT | {("tile", 4), ("tile", "walk")},
           SPLIT | {("tile", 4), ("tile", "walk")}, ({("ray", "walk")}, SPLIT | {("tile", 4), ("tile", "walk")}, {("ray", "walk"), ("ray", 1)}, SPLIT | {("tile", 4), ("tile", "walk")}))]


def _problem(kind, channels, n_in, hidden, n_freq, image):
    image = dict(dict(prior_res=(19, 16, 15)), **image)
    return _image(kind, channels, **image, n_in=n_in, hidden=hidden, n_freq=n_freq, prior_channels=channels, bias_std=0.1)


@pytest.mark.parametrize("kind", [VOXEL, TRIPLANE])
@pytest.mark.parametrize("channels,n_in,hidden,n_freq", CONFIGS)
@pytest.mark.parametrize("image,push,push_flat,prior", IMAGES)
def test_splatter_with_mlp_in_tiles(lp, oracle, kind, channels, n_in, hidden, n_freq, image, push, push_flat, prior):
    sp = _problem(kind, channels, n_in, hidden, n_freq, image)
    pushed, pulled = splat_mlp_routes(sp)
    assert set(pushed) == (push_flat if kind == TRIPLANE else push)
    assert set(pulled) == (prior[2 * (kind == TRIPLANE) + (channels == 32)])
    target, _, splat = lp.splat_to_device(sp)
    assert lp.lp_splat_has_fast_path(target, splat)
    print(check_case_splat(lp, oracle, sp, label=f"mlp tiles kind={kind} C={channels} {image}", width_cap=WIDTH_CAP_SPLAT_BORDER,
                           max_strict_fail=0.06, sparse=max(sp.res) >= 90), flush=True)


def _corners(sp, res, rays, points=None):
    """Which texels of a structure of `res` the points of `rays` reach (`points`: [rays][samples], those that count)."""
    c = cells(dataclasses.replace(sp, res=res))[rays]
    c = c.reshape(-1, 3) if points is None else c[points]
    axes = [(0, 1), (1, 2), (2, 0)] if sp.kind == TRIPLANE else [(0, 1, 2)]
    out = []
    for ax in axes:
        hit = np.zeros([res[a] for a in ax], bool)
        for d in np.ndindex(*(2,) * len(ax)):
            hit[tuple((c[:, ax] + d).T)] = True
        out.append(hit)
    return out


def _reads(sp, res, hit):
    """[rays][samples]: the points that have one of the texels `hit` among their corners."""
    c = cells(dataclasses.replace(sp, res=res))
    axes = [(0, 1), (1, 2), (2, 0)] if sp.kind == TRIPLANE else [(0, 1, 2)]
    out = np.zeros(c.shape[:2], bool)
    for ax, h in zip(axes, hit):
        for d in np.ndindex(*(2,) * len(ax)):
            out |= h[tuple(np.moveaxis(c[..., ax] + d, -1, 0))]
    return out


def _within(got, where):
    """Whether some value is infinite or undefined; none outside of `where` (texels) is."""
    import torch
    bad = [(~torch.isfinite(g)).any(-1).cpu().numpy().reshape(w.shape) for g, w in zip(got, where)]
    assert not any((b & ~w).any() for b, w in zip(bad, where))
    return any(b.any() for b in bad)


@pytest.mark.parametrize("kind", [VOXEL, TRIPLANE])
@pytest.mark.parametrize("channels,n_in,hidden,n_freq", CONFIGS)
@pytest.mark.parametrize("image", [IMAGES[0][0], IMAGES[-1][0], dict(width=24, height=16, samples=40, res=(20, 23, 17))])   # windows, walks; single rays
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_what_is_undefined_stays_with_its_points(lp, kind, channels, n_in, hidden, n_freq, image, value):
    """An infinite or undefined pixel, prior or gradient reaches what its own points reach, and no other point of its step.
    (A rectifier takes what is undefined to zero, so that a pixel or a prior need not reach anything.)"""
    import torch
    sp = _problem(kind, channels, n_in, hidden, n_freq, image)
    pushed, pulled = splat_mlp_routes(sp)
    assert {how for how, _ in pushed} == ({"ray"} if sp.n_rays < 1000 else {"tile"})
    res, prior_res, one = tuple(sp.res), tuple(sp.prior_res), sp.n_rays // 2 + 1
    gen = torch.Generator(device="cuda").manual_seed(3)
    draw = lambda theta: [torch.randn(t.shape, generator=gen, device="cuda") for t in theta]
    rays_of = lambda d_feats: (~torch.isfinite(d_feats)).any(-1).cpu().numpy()

    target, rays, splat = lp.splat_to_device(sp)
    clean, weights = lp.splat_fwd(target, rays, splat)
    assert all(torch.isfinite(t).all() for t in clean)
    # a pixel
    splat.feats[one, 1] = value
    theta, theta_w = lp.splat_fwd(target, rays, splat)
    d_feats, d_prior, _, _ = lp.splat_bwd(target, rays, splat, theta_w, draw(theta))
    _within(theta, _corners(sp, res, [one]))
    assert all(torch.isfinite(t).all() for t in theta_w)
    alone = np.arange(sp.n_rays) == one
    assert not (rays_of(d_feats) & ~alone).any()
    _within(d_prior, _corners(sp, prior_res, [one]))
    splat.feats[one, 1] = 0.5
    # a texel of the target's gradient
    d_theta = draw(theta)
    hit = [np.zeros(h.shape, bool) for h in _corners(sp, res, [one])]
    texel = tuple(cells(sp)[one, sp.samples // 2][list((0, 1) if kind == TRIPLANE else (0, 1, 2))])
    hit[0][texel] = True
    d_theta[0][(0,) + tuple(int(t) for t in texel)] = value
    read = _reads(sp, res, hit)
    d_feats, d_prior, _, _ = lp.splat_bwd(target, rays, splat, weights, d_theta)
    bad = rays_of(d_feats)
    assert bad.any() and not (bad & ~read.any(1)).any()
    assert _within(d_prior, _corners(sp, prior_res, np.arange(sp.n_rays), read))
    # a texel of the prior
    hit = [np.zeros(h.shape, bool) for h in _corners(sp, prior_res, [one])]
    texel = tuple(cells(dataclasses.replace(sp, res=prior_res))[one, sp.samples // 2][list((0, 1) if kind == TRIPLANE else (0, 1, 2))])
    hit[0][texel] = True
    splat.prior.data[0][(0,) + tuple(int(t) for t in texel)] = value
    theta, theta_w = lp.splat_fwd(target, rays, splat)
    _within(theta, _corners(sp, res, np.arange(sp.n_rays), _reads(sp, prior_res, hit)))
    assert all(torch.isfinite(t).all() for t in theta_w)
