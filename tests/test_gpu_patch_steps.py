"""The Renderer's backward over patches of an image (lp_mfma_bwd_tile.h) beyond one step of one window: steps that take one, two and
four windows and the walk, gradients that are not finite, grids in 16 bits, several whole rounds of patches and a partial one, patches that fall
apart into tiles and single rays, pixels on both sides of the distance up to which a list is taken in patches, and a captured graph."""
import dataclasses

import numpy as np
import pytest

import lp_inputs
from lp_inputs import HASH, TRIPLANE, VOXEL

from parity import check_case, summary
from test_gpu_captured import _replays
from test_gpu_splat_patches import _image
from tile_rules import backward_in_patches, image_row, step_routes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oracle():
    import oracle as o
    return o


def _inputs(kind, channels, dims, image, res, contract=0.0, near=1.0, far=4.0):
    rays = _image(VOXEL, 16, res=(20, 33, 17), contract=contract, far=far, **image)
    box = 1.0 if contract else 2.75
    inp = lp_inputs.make_small(kind, channels=channels, res=res, mlp_dims=dims, n_rays=8, samples=image["samples"], seed=281,
                               grid_std=0.3, aabb_min=(-box,) * 3, aabb_max=(box,) * 3, hash_size=4096 if kind == HASH else None)
    target = np.random.default_rng(5).random((rays.n_rays, 3), dtype=np.float32)
    return dataclasses.replace(inp, target=target, contract_a=contract, origins=rays.origins, dirs=rays.dirs, far=rays.far,
                               near=np.full_like(rays.near, near))


@pytest.mark.parametrize("kind,channels,dims", [(TRIPLANE, 16, (16, 32, 4)), (TRIPLANE, 32, (32, 64, 64, 4)), (HASH, 32, (32, 64, 4))])
def test_windows_and_walk(lp, oracle, kind, channels, dims):
    """Contract coordinates: pixels far apart in the middle of their rays and near at both ends."""
    inp = _inputs(kind, channels, dims, dict(width=64, height=64, samples=12, views=4), (150,) * 3, 1.0, 0.5, 12.0)
    routes = step_routes(inp)
    assert {("patch", 1), ("patch", 2), ("patch", 4), ("patch", "walk"), ("tile", 4), ("ray", "walk")} <= set(routes), routes
    print(summary(check_case(lp, oracle, inp, lp.LP_MATH_BF16X3, label=f"windows and walk {kind} {dims}")), flush=True)


@pytest.mark.parametrize("kind,channels,dims", [(VOXEL, 16, (16, 32, 32, 4)), (VOXEL, 32, (32, 64, 64, 4)), (TRIPLANE, 32, (32, 64, 64, 4)),
                                                (TRIPLANE, 16, (16, 64, 4))])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_undefined_gradient_stays_on_its_ray(lp, kind, channels, dims, value):
    import torch
    inp = _inputs(kind, channels, dims, dict(width=128, height=130, samples=9), (40, 33, 37))
    assert {how for how, _ in step_routes(inp)} == {"patch"}
    grid, mlp, rays, bg = lp.to_device(inp, "cuda:0")
    _, _, _, cache = lp.render_fwd(grid, mlp, rays, bg, lp.LP_MATH_BF16X3)
    d_rgb = torch.ones((inp.n_rays, 3), device="cuda")
    d_rgb[4001] = value
    bad = [~torch.isfinite(lp.render_bwd(grid, mlp, rays, bg, d_rgb, cache, None, None, mode)[0][0])
           for mode in (lp.LP_MATH_BF16X3, lp.LP_MATH_GENERIC)]
    assert bad[1].any() and torch.equal(bad[0], bad[1])


@pytest.mark.parametrize("kind,channels,dims", [(VOXEL, 16, (16, 64, 64, 4)), (VOXEL, 32, (32, 32, 32, 4)), (TRIPLANE, 32, (32, 64, 64, 4)),
                                                (HASH, 16, (16, 32, 4))])
@pytest.mark.parametrize("dtype", ["bfloat16", "float16"])
@pytest.mark.parametrize("contract", [0.0, 1.3])
def test_grids_in_16_bits(lp, oracle, kind, channels, dims, dtype, contract):
    import torch
    inp = _inputs(kind, channels, dims, dict(width=128, height=130, samples=4), (40, 33, 37), contract)
    assert {how for how, _ in step_routes(inp)} == {"patch"}
    tdt = getattr(torch, dtype)
    inp = dataclasses.replace(inp, grid=[torch.from_numpy(g).to(tdt).float().numpy() for g in inp.grid])
    print(summary(check_case(lp, oracle, inp, lp.LP_MATH_BF16X3, label=f"stored {kind} {dims} {dtype} a={contract}", grid_dtype=tdt)), flush=True)


@pytest.mark.parametrize("width,height", [(240, 230), (251, 262)])   # 3.4 and 4.03 patches to a wave
def test_rounds_of_patches(lp, oracle, width, height):
    inp = _inputs(VOXEL, 16, (16, 32, 4), dict(width=width, height=height, samples=4), (40, 33, 37))
    assert {how for how, _ in step_routes(inp)} == {"patch"}
    print(summary(check_case(lp, oracle, inp, lp.LP_MATH_BF16X3, label=f"rounds of patches {width} x {height}")), flush=True)


@pytest.mark.parametrize("kind,channels,dims", [(TRIPLANE, 16, (16, 64, 64, 4))])
@pytest.mark.parametrize("res,apart", [(200, 0.05), (350, 0.95)])
def test_patches_that_fall_apart(lp, oracle, kind, channels, dims, res, apart):
    """All items are patches; at 1.4 texels from pixel to pixel hardly any holds together."""
    inp = _inputs(kind, channels, dims, dict(width=128, height=128, samples=32), (res,) * 3)
    assert backward_in_patches(inp.n_rays, inp.samples, image_row(inp, 1.5, 1e30))
    routes = step_routes(inp)
    assert {how for how, _ in routes} == {"patch", "tile", "ray"}
    assert sum(n for (how, _), n in routes.items() if how == "ray") >= apart * sum(routes.values())
    print(summary(check_case(lp, oracle, inp, lp.LP_MATH_BF16X3, label=f"falling apart {kind} {dims} {res}")), flush=True)


@pytest.mark.parametrize("res,patches", [(55, True), (64, False)])   # 1.2 and 1.4 texels from pixel to pixel
def test_distance_of_pixels(lp, oracle, res, patches):
    inp = _inputs(VOXEL, 16, (16, 32, 32, 4), dict(width=24, height=24, samples=4, views=29), (res,) * 3)
    assert image_row(inp, 1.5, 1e30) == 24 and (image_row(inp, 1.3, 1e30) == 24) == patches
    print(summary(check_case(lp, oracle, inp, lp.LP_MATH_BF16X3, label=f"distance of pixels {res}")), flush=True)


@pytest.mark.parametrize("kind,channels,dims", [(VOXEL, 16, (16, 64, 64, 4)), (TRIPLANE, 32, (32, 64, 64, 4))])
def test_captured(lp, kind, channels, dims):
    import torch
    inp = _inputs(kind, channels, dims, dict(width=128, height=130, samples=9), (40, 33, 37))
    grid, mlp, rays, bg = lp.to_device(inp, "cuda:0")
    cache = lp.render_fwd(grid, mlp, rays, bg)[3]
    d_rgb = torch.ones((inp.n_rays, 3), device="cuda")
    d_grid, dW, db = lp.render_bwd(grid, mlp, rays, bg, d_rgb, cache)
    ws = torch.empty(lp.lp_bwd_workspace_bytes(grid, mlp, rays), dtype=torch.uint8, device="cuda")

    def step():
        for t in (*d_grid, *dW, *db):
            t.zero_()
        lp.lp_render_bwd(grid, mlp, rays, bg, d_rgb, None, None, cache, d_grid, dW, db, ws)

    _replays(step, [*d_grid, *dW, *db], [d_rgb])
