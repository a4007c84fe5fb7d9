"""Which way the Splatter's patches of an image are taken, by the rules of the kernels replayed on the CPU (tile_rules.py)."""
import pytest

from lp_inputs import HASH, TRIPLANE, VOXEL

from test_gpu_splat_patches import _image
from tile_rules import image_row, patch_routes, patches


@pytest.mark.parametrize("n_rays", [32, 16])
@pytest.mark.parametrize("kind", [VOXEL, TRIPLANE, HASH])
@pytest.mark.parametrize("height,views,res", [(33, 2, (20, 23, 17)), (33, 4, (24, 24, 24)), (30, 3, (42, 31, 34)), (35, 2, (64, 64, 64))])
def test_patches_across_two_views_go_in_parts(kind, n_rays, height, views, res):
    """However small the structure is: marched together, their steps would be taken one point of one ray at a time."""
    sp = _image(kind, 16, 64, height, 8, res, views)
    assert image_row(sp, 1.5 if kind == TRIPLANE else 0.9, 1e30) == 64
    across = sum(len({r // (64 * height) for r in p[p >= 0]}) > 1 for p in patches(sp, 64, n_rays))
    routes = patch_routes(sp, 64, n_rays)
    assert across > 0 and routes["part"] == across and routes["lines"] == routes["ray"] == 0 and routes[8] + routes[4] + routes[1] > 0
