"""The Splatter with an MLP over tiles of four neighbouring rays, forward and backward: tiles that end early, rays of another
scene inside of one, points past the rays' ends, contract coordinates, windows that are split."""
import pytest

from lp_inputs import TRIPLANE, VOXEL

from parity import WIDTH_CAP_SPLAT_BORDER, check_case_splat
from test_gpu_splat_patches import _image

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oracle():
    import oracle as o
    return o


def _in_tiles(n_rays, samples, waves, up_to):
    """The launch rule of lp_tile_scatter.h push_order."""
    rounds = lambda items: -(-items // waves)
    return rounds(-(-n_rays // 4)) * -(-samples // 8) <= up_to * rounds(n_rays) * -(-samples // 32)


@pytest.mark.parametrize("kind", [VOXEL, TRIPLANE])
@pytest.mark.parametrize("channels,n_in,hidden,n_freq", [(16, 5, (64,), -1), (32, 32, (64, 64), 1)])
@pytest.mark.parametrize("image", [dict(width=64, height=72, samples=9, res=(20, 23, 17), cut=1),
                                   dict(width=66, height=70, samples=8, res=(40, 33, 37), per_scene=7),
                                   dict(width=64, height=72, samples=10, res=(48, 40, 44)),
                                   dict(width=64, height=72, samples=9, res=(24, 22, 26), contract=1.0, far=9.0)])
def test_splatter_with_mlp_in_tiles(lp, oracle, kind, channels, n_in, hidden, n_freq, image):
    sp = _image(kind, channels, **image, n_in=n_in, hidden=hidden, n_freq=n_freq, prior_channels=channels, prior_res=(19, 16, 15), bias_std=0.1)
    assert _in_tiles(sp.n_rays, sp.samples, 2048, 2.0) and _in_tiles(sp.n_rays, sp.samples, 1024, 1.05)
    target, _, splat = lp.splat_to_device(sp)
    assert lp.lp_splat_has_fast_path(target, splat)
    print(check_case_splat(lp, oracle, sp, label=f"mlp tiles kind={kind} C={channels} {image}", width_cap=WIDTH_CAP_SPLAT_BORDER,
                           max_strict_fail=0.06), flush=True)
