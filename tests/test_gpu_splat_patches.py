"""The naive Splatter over patches of an image (lp_splat_patch.h) where it has edges: rows that are no multiple of a patch, lines
and images that end inside one, several scenes, steps that reach more texels than there are slots, features and gradients
that are not finite; and lists of rays that are no image."""
import dataclasses

import numpy as np
import pytest

import lp_inputs
from lp_inputs import HASH, TRIPLANE, VOXEL

from parity import check_case_splat
from tile_rules import gradient_in_patches, image_row, patch_routes, push_segment

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oracle():
    import oracle as o
    return o


def _image(kind, channels, width, height, samples, res, views=1, cut=0, per_scene=None, contract=0.0, far=4.0, **mlp):
    """`views` images of width x height pixels, the last `cut` rays left out; `per_scene`: rays of a scene in turn."""
    f = (max(width, height) / 2.0) / np.tan(np.radians(30.0))
    u, v = (np.arange(width) + 0.5 - width / 2.0) / f, (np.arange(height) + 0.5 - height / 2.0) / f
    vv, uu = np.meshgrid(v, u, indexing="ij")
    cam = np.stack([uu, -vv, -np.ones_like(uu)], axis=-1).reshape(-1, 3)
    cam /= np.linalg.norm(cam, axis=1, keepdims=True)
    o, d = [], []
    for k in range(views):
        rot, pos = lp_inputs.camera_pose(33.0 + 90.0 * k, 17.0, 2.5)
        d.append(cam @ np.asarray(rot, dtype=np.float64).T)
        o.append(np.broadcast_to(np.asarray(pos, dtype=np.float64), cam.shape))
    o, d = np.concatenate(o), np.concatenate(d)
    n = len(o) - cut
    o, d = np.ascontiguousarray(o[:n].astype(np.float32)), np.ascontiguousarray(d[:n].astype(np.float32))
    full = lambda x: np.full(n, x, dtype=np.float32)
    kw = dict(hash_size=4096) if kind == HASH else {}
    box = 1.0 if contract else 2.75
    sp = lp_inputs.make_splat_small(kind, channels=channels, res=res, n_rays=n, samples=samples, seed=401 + samples + width,
                                    n_scenes=2 if per_scene else 1, aabb_min=(-box,) * 3, aabb_max=(box,) * 3, **kw, **mlp)
    scene = (np.arange(n) // per_scene % 2).astype(np.int32) if per_scene else None
    return dataclasses.replace(sp, origins=o, dirs=d, near=full(1.0), far=full(far), scene=scene, contract_a=contract)


def _finds(sp, row, pixel=None, step=1e30):
    assert image_row(sp, pixel or (1.5 if sp.kind == TRIPLANE else 0.9), step) == row
    return sp


STRUCTURES = [(VOXEL, 16), (VOXEL, 32), (TRIPLANE, 16), (TRIPLANE, 32), (HASH, 16), (HASH, 32)]
IMAGES = [dict(width=64, height=32, samples=8, res=(20, 33, 17)),                     # whole patches, one step
          dict(width=61, height=43, samples=1, res=(20, 23, 17), cut=3),              # a patch of five pixels, a line that ends early
          dict(width=67, height=33, samples=19, res=(20, 23, 17), views=2),           # a patch across two views; a step of three points
          dict(width=66, height=40, samples=9, res=(20, 23, 17), per_scene=8),        # scenes that change from patch to patch
          dict(width=64, height=40, samples=9, res=(20, 23, 17), per_scene=5)]        # and inside of a patch


@pytest.mark.parametrize("kind,channels", STRUCTURES)
@pytest.mark.parametrize("image", IMAGES)
def test_pushed_images(lp, oracle, kind, channels, image):
    sp = _finds(_image(kind, channels, **image), image["width"])
    print(check_case_splat(lp, oracle, sp, label=f"patches kind={kind} C={channels} {image}"), flush=True)


def _push_routes(sp, row):
    return {k for k, n in patch_routes(sp, row, 32, push_segment(sp.n_rays, sp.samples)).items() if n}


@pytest.mark.parametrize("kind,channels", [(VOXEL, 32), (TRIPLANE, 16), (HASH, 16)])
@pytest.mark.parametrize("samples,res,contract,routes,flat", [(4, (64, 64, 64), 0.0, {8, 1}, {8}), (16, (45, 48, 50), 0.0, {8}, {8}),
                                                              (24, (64, 40, 90), 1.0, {8, 4, 1}, {8, 4})])
def test_pushed_images_that_reach_many_texels(lp, oracle, kind, channels, samples, res, contract, routes, flat):
    """Points far apart along their rays and contract coordinates: steps of eight points, of four and of one (`routes`; triplanes:
    `flat`)."""
    sp = _finds(_image(kind, channels, 96, 32, samples, res, contract=contract, far=12.0 if contract else 4.0), 96)
    assert _push_routes(sp, 96) == (flat if kind == TRIPLANE else routes)
    print(check_case_splat(lp, oracle, sp, label=f"patches many texels kind={kind} S={samples} {res}"), flush=True)


@pytest.mark.parametrize("kind,channels", [(VOXEL, 16), (TRIPLANE, 32), (HASH, 32)])
def test_pushed_images_one_point_of_one_ray_at_a_time(lp, oracle, kind, channels):
    """Where a single point of a patch's rays reaches more texels than there are slots."""
    sp = _finds(_image(kind, channels, 96, 32, 24, (120, 100, 90), contract=1.0, far=12.0), 96)
    assert _push_routes(sp, 96) == {8, 4, 1} | (set() if kind == TRIPLANE else {"ray"})
    print(check_case_splat(lp, oracle, sp, label=f"patches ray by ray kind={kind}"), flush=True)


@pytest.mark.parametrize("kind,channels", STRUCTURES)
def test_lists_of_rays_in_tiles(lp, oracle, kind, channels):
    """Four neighbouring rays here, four there: no image, and the tiles take them."""
    sp = _image(kind, channels, 128, 64, 24, (40, 33, 37))
    order = np.random.default_rng(5).permutation(sp.n_rays // 4)[:, None] * 4 + np.arange(4)
    sp = dataclasses.replace(sp, **{n: np.ascontiguousarray(getattr(sp, n)[order.reshape(-1)]) for n in ("origins", "dirs", "near", "far", "feats")})
    print(check_case_splat(lp, oracle, _finds(sp, 0), label=f"tiles of a list kind={kind} C={channels}"), flush=True)


@pytest.mark.parametrize("kind,channels", STRUCTURES)
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_undefined_pixels_stay_on_their_rays(lp, kind, channels, value):
    """What one pixel's infinite or undefined feature reaches is what its ray alone reaches."""
    import torch
    sp = _finds(_image(kind, channels, 64, 33, 11, (20, 23, 17)), 64)
    sp.feats[1000] = value
    got = lp.splat_fwd(*lp.splat_to_device(sp))[0]
    alone = dataclasses.replace(sp, **{n: getattr(sp, n)[1000:1001] for n in ("origins", "dirs", "near", "far", "feats")})
    for a, w in zip(got, lp.splat_fwd(*lp.splat_to_device(alone))[1]):
        reached = (w > 0)[..., None].expand_as(a)
        assert reached.any() and torch.equal(~torch.isfinite(a), reached)
        assert torch.equal(torch.isnan(a), reached if np.isnan(value) else torch.zeros_like(reached))


def _gradients(lp, sp, infinite=0.0):
    """(through the patches, through the generic kernel, sums of magnitudes) of the pixel features' gradient."""
    import torch
    target, rays, splat = lp.splat_to_device(sp)
    theta, theta_w = lp.splat_fwd(target, rays, splat)
    gen = torch.Generator(device="cuda").manual_seed(3)
    d_theta = [torch.randn(t.shape, generator=gen, device="cuda") for t in theta]
    for t in d_theta:
        t[torch.rand(t.shape, generator=gen, device="cuda") < infinite] = float("inf")

    def odd(t):   # 4 bytes past a 16-byte boundary: the generic kernel
        buf = torch.empty(t.numel() + 4, dtype=t.dtype, device=t.device)
        out = buf[1:1 + t.numel()].view(t.shape)
        out.copy_(t)
        return out

    ws = torch.empty(lp.lp_splat_bwd_workspace_bytes(target, rays, splat), dtype=torch.uint8, device="cuda")
    out = [torch.full_like(splat.feats, v) for v in (7.0, -7.0, 5.0)]
    for o, d in zip(out, (d_theta, [odd(t) for t in d_theta], [odd(t.abs()) for t in d_theta])):
        lp.lp_splat_bwd(target, rays, splat, theta_w, d, o, [], [], [], ws)
    return out


@pytest.mark.parametrize("kind,channels", [(VOXEL, 16), (VOXEL, 32), (HASH, 16), (HASH, 32)])
@pytest.mark.parametrize("width,height,samples,views,cut,per_scene", [(256, 256, 64, 1, 0, None), (131, 251, 67, 2, 5, None), (260, 253, 61, 1, 0, 4)])
def test_gradients_of_images(lp, kind, channels, width, height, samples, views, cut, per_scene):
    """Against the generic kernel; the bound as in test_gpu_splat_naive_backward."""
    sp = _finds(_image(kind, channels, width, height, samples, (40, 33, 37), views, cut, per_scene), width, 0.9, 2.0)
    assert gradient_in_patches(sp, width)
    got, want, total = _gradients(lp, sp)
    assert ((got - want).abs() <= 2 * (8 * samples + 3) * 2.0 ** -24 * total).all()


@pytest.mark.parametrize("kind,channels", [(VOXEL, 16), (VOXEL, 32), (HASH, 16), (HASH, 32)])
def test_gradients_of_images_in_contract_coordinates(lp, kind, channels):
    """Steps of eight points, of four and of one; the bound as above."""
    sp = _finds(_image(kind, channels, 364, 364, 64, (128, 128, 128), contract=1.0, far=12.0), 364, 0.9, 2.0)
    assert gradient_in_patches(sp, 364)
    assert {k for k, n in patch_routes(sp, 364, 16, every=61).items() if n} == {8, 4, 1}
    got, want, total = _gradients(lp, sp)
    assert ((got - want).abs() <= 2 * (8 * sp.samples + 3) * 2.0 ** -24 * total).all()


@pytest.mark.parametrize("kind,channels", [(VOXEL, 32), (HASH, 16)])
def test_infinite_gradients_of_images(lp, kind, channels):
    import torch
    sp = _finds(_image(kind, channels, 256, 256, 64, (40, 33, 37)), 256, 0.9, 2.0)
    got, want, _ = _gradients(lp, sp, infinite=2e-4)
    assert torch.isposinf(want).any() and torch.isfinite(want).any()
    assert torch.equal(torch.isposinf(got), torch.isposinf(want))
    assert torch.equal(torch.isnan(got), torch.isnan(want))


@pytest.mark.parametrize("channels,samples,width", [(16, 64, 256), (16, 160, 256), (32, 24, 416), (32, 160, 256)])
def test_gradients_of_images_are_no_further_from_64_bits(lp, channels, samples, width):
    """The 2-norm of the error of a patch's gradients against that of the same rays as a list, which go ray by ray."""
    import torch
    res = (60, 55, 64)
    sp = _finds(_image(VOXEL, channels, width, width, samples, res), width, 0.9, 2.0)
    assert gradient_in_patches(sp, width)
    target, rays, splat = lp.splat_to_device(sp)
    theta, theta_w = lp.splat_fwd(target, rays, splat)
    d_theta = torch.randn(theta[0].shape, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    order = np.random.default_rng(5).permutation(sp.n_rays)
    listed = _finds(dataclasses.replace(sp, **{n: np.ascontiguousarray(getattr(sp, n)[order]) for n in ("origins", "dirs", "near", "far", "feats")}), 0, 0.9, 2.0)
    patches = lp.splat_bwd(target, rays, splat, theta_w, [d_theta])[0]
    alone = torch.empty_like(patches)
    alone[torch.from_numpy(order).cuda()] = lp.splat_bwd(*lp.splat_to_device(listed), theta_w, [d_theta])[0]

    o, d, near, far = (t.double() for t in (rays.origins, rays.dirs, rays.near, rays.far))
    vec = lambda v: torch.tensor(np.asarray(v, dtype=np.float32), device="cuda").double()
    lo, hi, n = vec(sp.aabb_min), vec(sp.aabb_max), vec(res)
    weights, grad = theta_w[0].reshape(-1).double(), d_theta.reshape(-1, channels).double()
    want = torch.zeros_like(patches, dtype=torch.float64)
    for j in range(samples):
        t = near + (j + 0.5) * ((far - near) / samples)
        u = torch.minimum(((o + t[:, None] * d - lo) * ((n - 1) / (hi - lo))).clamp(min=0), n - 1)
        cell = torch.minimum(u.long(), n.long() - 2)
        for corner in np.ndindex(2, 2, 2):
            b = torch.tensor(corner, device="cuda")
            w = torch.where(b == 1, u - cell, 1 - (u - cell)).prod(1)
            k = cell + b
            k = (k[:, 0] * res[1] + k[:, 1]) * res[2] + k[:, 2]
            want += torch.where(weights[k] > 0, w / weights[k], 0.0)[:, None] * grad[k]
    error = lambda x: float((x.double() - want).norm() / want.norm())
    assert error(patches) <= error(alone), (error(patches), error(alone))
