"""The Renderer's backward over patches of an image (lp_mfma_bwd_tile.h): pixels on both sides of the distance up to which a list is taken in patches."""
import dataclasses

import numpy as np
import pytest

import lp_inputs
from lp_inputs import HASH, VOXEL

from parity import check_case, summary
from test_gpu_splat_patches import _image
from tile_rules import image_row

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


@pytest.mark.parametrize("res,patches", [(55, True), (64, False)])   # 1.2 and 1.4 texels from pixel to pixel
def test_distance_of_pixels(lp, oracle, res, patches):
    inp = _inputs(VOXEL, 16, (16, 32, 32, 4), dict(width=24, height=24, samples=4, views=29), (res,) * 3)
    assert image_row(inp, 1.5, 1e30) == 24 and (image_row(inp, 1.3, 1e30) == 24) == patches
    print(summary(check_case(lp, oracle, inp, lp.LP_MATH_BF16X3, label=f"distance of pixels {res}")), flush=True)
