"""The Renderer's backward over patches of an image (lp_mfma_bwd_tile.h) where they have edges: rows that are no multiple of four
pixels, an odd number of lines, an image that ends inside a line, two views in one patch, scenes that change inside of one, ragged
last steps.  Every case is checked against the CPU oracle at the bounds of `parity.check_case`."""
import dataclasses

import numpy as np
import pytest

import lp_inputs
from lp_inputs import HASH, TRIPLANE, VOXEL

from parity import check_case, summary
from test_gpu_splat_patches import _image
from tile_rules import step_routes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oracle():
    import oracle as o
    return o


SHAPES = [(VOXEL, 16, (16, 64, 64, 4)), (VOXEL, 32, (32, 64, 4)), (TRIPLANE, 32, (32, 64, 64, 4)), (TRIPLANE, 16, (16, 32, 4)),
          (HASH, 16, (16, 32, 32, 4)), (VOXEL, 32, (32, 64, 64, 4))]
# (image, its marches).  Some 16 000 rays each: of 8 700 samples in all one hidden unit that takes the other side of its kink was
# 0.5 % of a hash table's gradient (inside the envelope, whose width was 2.9 %, but over the 0.4 % that check_case allows the whole
# tensor); its share falls as the samples grow.
IMAGES = [(dict(width=128, height=130, samples=4), {"patch"}),                        # whole patches, one step
          (dict(width=125, height=131, samples=3, cut=3), {"patch"}),                 # a patch of one pixel a line, of one line, a line that ends early
          (dict(width=131, height=65, samples=4, views=2), {"patch", "tile"}),        # a patch across two views: its lines are tiles
          (dict(width=130, height=128, samples=4, per_scene=5), {"patch", "ray"}),           # scenes that change inside of lines
          (dict(width=128, height=127, samples=4, cut=5), {"patch"}),                 # a patch without rays, among whole rounds of the waves
          (dict(width=128, height=128, samples=9), {"patch"})]                        # several steps, the last one of one sample


def _inputs(kind, channels, dims, image, contract=0.0):
    rays = _image(VOXEL, 16, res=(20, 33, 17), contract=contract, **image)
    box = 1.0 if contract else 2.75
    inp = lp_inputs.make_small(kind, channels=channels, res=(40, 33, 37), mlp_dims=dims, n_rays=8, samples=image["samples"], seed=271,
                               n_scenes=2 if rays.scene is not None else 1, grid_std=0.3, aabb_min=(-box,) * 3, aabb_max=(box,) * 3,
                               hash_size=4096 if kind == HASH else None)
    target = np.random.default_rng(5).random((rays.n_rays, 3), dtype=np.float32)
    return dataclasses.replace(inp, target=target, contract_a=contract, **{n: getattr(rays, n) for n in ("origins", "dirs", "near", "far", "scene")})


@pytest.mark.parametrize("kind,channels,dims", SHAPES)
@pytest.mark.parametrize("image,marches", IMAGES)
def test_patches(lp, oracle, kind, channels, dims, image, marches):
    inp = _inputs(kind, channels, dims, image)
    routes = step_routes(inp)
    assert {how for how, _ in routes} == marches, routes
    print(summary(check_case(lp, oracle, inp, lp.LP_MATH_BF16X3, label=f"patches {kind} {dims} {image}")), flush=True)


@pytest.mark.parametrize("kind,channels,dims", SHAPES[-1:])
def test_patches_in_contract_coordinates(lp, oracle, kind, channels, dims):
    inp = _inputs(kind, channels, dims, dict(width=128, height=130, samples=4), contract=1.3)
    assert {how for how, _ in step_routes(inp)} == {"patch"}
    print(summary(check_case(lp, oracle, inp, lp.LP_MATH_BF16X3, label=f"patches contract {kind} {dims}")), flush=True)
