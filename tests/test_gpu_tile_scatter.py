"""Steps of four neighbouring rays scattered as matrix products (lp_tile_scatter.h) where they have edges: what the
Splatter pushes, and the Renderer's gradient of hash tables.  Sample counts around the step widths, partial tiles, scenes
that change between tiles and inside of them, windows that are split and steps that take the walk."""
import dataclasses

import numpy as np
import pytest

import lp_inputs
from lp_inputs import HASH, TRIPLANE, VOXEL

from parity import WIDTH_CAP_SPLAT_BORDER, check_case, check_case_splat, summary

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oracle():
    import oracle as o
    return o


def _camera(n_rays, image, per_scene, n_scenes):
    rot, pos = lp_inputs.camera_pose(33.0, 17.0, 2.5)
    o, d = lp_inputs.pinhole_rays(image, rot, pos)
    idx = ((image // 2) * image + np.arange(n_rays)) % (image * image)
    full = lambda v: np.full(n_rays, v, dtype=np.float32)
    scene = None if n_scenes == 1 else (np.arange(n_rays) // per_scene % n_scenes).astype(np.int32)
    return dict(origins=np.ascontiguousarray(o[idx]), dirs=np.ascontiguousarray(d[idx]), near=full(1.0), far=full(4.0), scene=scene)


SPLATS = [(VOXEL, 16), (VOXEL, 32), (TRIPLANE, 16), (TRIPLANE, 32), (HASH, 16), (HASH, 32)]


def _splat(kind, channels, n_rays, samples, res, per_scene=None, image=128, **kw):
    n_scenes = 2 if per_scene else 1
    if kind == HASH:
        kw = dict(kw, hash_size=4096, **(dict(prior_hash_size=512) if kw.get("prior_channels") else {}))
    sp = lp_inputs.make_splat_small(kind, channels=channels, res=res, n_rays=n_rays, samples=samples, seed=301 + samples,
                                    n_scenes=n_scenes, aabb_min=(-2.75,) * 3, aabb_max=(2.75,) * 3, **kw)
    return dataclasses.replace(sp, **_camera(n_rays, image, per_scene, n_scenes))


@pytest.mark.parametrize("kind,channels", SPLATS)
@pytest.mark.parametrize("n_rays,samples,per_scene", [(5, 1, None), (203, 8, 7), (8191, 9, 4), (8190, 33, None)])
def test_pushed_features(lp, oracle, kind, channels, n_rays, samples, per_scene):
    sp = _splat(kind, channels, n_rays, samples, (40, 33, 37), per_scene)
    print(check_case_splat(lp, oracle, sp, label=f"tiles kind={kind} C={channels} M={n_rays} S={samples}"), flush=True)


@pytest.mark.parametrize("kind,channels", SPLATS)
@pytest.mark.parametrize("res,contract", [((150, 64, 90), 0.0), ((400, 64, 90), 0.0), ((64, 64, 64), 1.0)])
def test_pushed_features_split_windows(lp, oracle, kind, channels, res, contract):
    sp = dataclasses.replace(_splat(kind, channels, 8192, 24, res), contract_a=contract)
    if contract:
        sp = dataclasses.replace(sp, aabb_min=(-1.0,) * 3, aabb_max=(1.0,) * 3, far=np.full(8192, 12.0, dtype=np.float32))
    print(check_case_splat(lp, oracle, sp, label=f"windows kind={kind} C={channels} res={res}"), flush=True)


@pytest.mark.parametrize("kind,channels", SPLATS[:4])
def test_undefined_pixel_stays_on_its_ray(lp, kind, channels):
    """A pixel feature that is not a number reaches the cells of its own ray and no others: as ray by ray."""
    import torch
    sp = _splat(kind, channels, 8192, 24, (40, 33, 37))
    sp.feats[4001] = np.nan
    target, rays, splat = lp.splat_to_device(sp)
    got = lp.splat_fwd(target, rays, splat)[0]
    alone = dataclasses.replace(sp, **{n: getattr(sp, n)[4001:4002] for n in ("origins", "dirs", "near", "far", "feats")})
    want = lp.splat_fwd(*lp.splat_to_device(alone))[0]
    for a, b in zip(got, want):
        assert torch.isnan(b).any() and torch.equal(torch.isnan(a), torch.isnan(b))


@pytest.mark.parametrize("kind,channels", SPLATS)
@pytest.mark.parametrize("n_rays,samples", [(8190, 24), (8192, 29), (37, 29)])
def test_infinite_pixel_stays_infinite(lp, kind, channels, n_rays, samples):
    """The last pixel's feature is infinite: the cells of its ray are infinite and none is undefined, whether its tile
    (n_rays % 4 = 2) or its last step has places left over, whose points must not meet the infinity with weight zero."""
    import torch
    sp = _splat(kind, channels, n_rays, samples, (40, 33, 37))
    sp.feats[-1] = np.inf
    target, rays, splat = lp.splat_to_device(sp)
    got = lp.splat_fwd(target, rays, splat)[0]
    alone = dataclasses.replace(sp, **{n: getattr(sp, n)[-1:] for n in ("origins", "dirs", "near", "far", "feats")})
    reached = lp.splat_fwd(*lp.splat_to_device(alone))[1]
    for a, w in zip(got, reached):
        assert (w > 0).any() and not torch.isnan(a).any()
        assert torch.equal(torch.isposinf(a), (w > 0)[..., None].expand_as(a))


HASHES = [(16, (16, 64, 64, 4), 1 << 15), (16, (16, 32, 4), 64), (32, (32, 64, 4), 4096), (32, (32, 32, 32, 4), 1)]


@pytest.mark.parametrize("channels,dims,hash_size", HASHES)
@pytest.mark.parametrize("n_rays,samples,per_scene", [(203, 7, 7), (8190, 33, None)])
def test_hash_table_gradient(lp, oracle, channels, dims, hash_size, n_rays, samples, per_scene):
    inp = lp_inputs.make_small(HASH, channels=channels, res=(40, 33, 37), mlp_dims=dims, n_rays=n_rays, samples=samples, seed=311,
                               n_scenes=2 if per_scene else 1, grid_std=0.3, hash_size=hash_size, aabb_min=(-2.75,) * 3,
                               aabb_max=(2.75,) * 3)
    inp = dataclasses.replace(inp, **_camera(n_rays, 128, per_scene, inp.n_scenes))
    # (a table of a few entries collects the kink decisions of every sample in each of them)
    print(summary(check_case(lp, oracle, inp, lp.LP_MATH_BF16X3, label=f"hash tiles {dims} T={hash_size} S={samples}",
                             max_strict_fail=0.25 if hash_size < 100 else 0.02)), flush=True)
