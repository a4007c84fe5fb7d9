"""The matrix-core forward with rays in pairs, 32 samples of each per step, against the generic kernels: a last ray without a
partner, sample counts around 32 and 64, the two rays of a pair in different scenes; and launches of single rays beside it."""
import pytest
import torch

import lp_inputs
from lp_inputs import HASH, TRIPLANE, VOXEL

from parity import FWD_RTOL, close
from tile_rules import forward_in_pairs, forward_workgroups

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,channels,dims,dtype", [(VOXEL, 16, (16, 64, 64, 4), torch.float32), (VOXEL, 32, (32, 32, 4), torch.bfloat16),
                                                      (TRIPLANE, 32, (32, 64, 64, 4), torch.float32), (TRIPLANE, 16, (16, 32, 32, 4), torch.float16),
                                                      (HASH, 16, (16, 64, 4), torch.float32)])
@pytest.mark.parametrize("n_rays,samples,pairs", [(1, 1, True), (6143, 31, True), (6143, 33, True), (6143, 95, True), (77, 65, False), (9001, 161, False), (4093, 49, False), (4095, 49, True),
                                                  (4690, 252, False), (50003, 129, True), (101001, 49, False)])   # (the last two: more workgroups than fit at once)
def test_equals_the_generic_kernels(lp, kind, channels, dims, dtype, n_rays, samples, pairs):
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert forward_in_pairs(n_rays, samples) == pairs
        assert (forward_workgroups(n_rays, samples) > 768) == (n_rays > 50000)
    kw = dict(hash_size=4096) if kind == HASH else {}
    inp = lp_inputs.make_small(kind, channels=channels, res=(24, 21, 26), mlp_dims=dims, n_rays=n_rays, samples=samples, seed=71 + samples,
                               n_scenes=3, grid_std=0.3, **kw)
    grid, mlp, rays, bg = lp.to_device(inp, "cuda:0")
    rays.scene = torch.randint(0, 3, (n_rays,), dtype=torch.int32, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(5))
    grid.data = [t.to(dtype) for t in grid.data]
    got = lp.render_fwd(grid, mlp, rays, bg, lp.LP_MATH_BF16X3)
    want = lp.render_fwd(grid, mlp, rays, bg, lp.LP_MATH_GENERIC)
    for name, a, b in zip(("rgb", "alpha", "depth", "cache"), got, want):
        close(a.cpu().numpy(), b.double().cpu().numpy(), FWD_RTOL, f"{name} M={n_rays} S={samples}")


@pytest.mark.parametrize("channels,dims", [(16, (16, 32, 4)), (32, (32, 64, 64, 4))])
def test_optical_depth_of_a_long_ray(lp, channels, dims):
    """Pairs add up the optical depth over twice as many steps as single rays; it comes out within one rounding of the sum
    over all samples and one of the last, partial step.  The density is 20 everywhere (softplus(20) = 20 in fp32), so that the
    sums of whole steps are exact: 32 times one value."""
    n_rays, samples = 8192, 999
    assert forward_in_pairs(n_rays, samples)
    inp = lp_inputs.make_small(VOXEL, channels=channels, res=(8, 9, 7), mlp_dims=dims, n_rays=n_rays, samples=samples, seed=5)
    grid, mlp, rays, bg = lp.to_device(inp, "cuda:0")
    for w in mlp.weights:
        w.zero_()
    for b in mlp.biases:
        b.zero_()
    mlp.biases[-1][0] = 20.0
    rays.far = rays.near + torch.rand(n_rays, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(6)) + 0.5
    cache = lp.render_fwd(grid, mlp, rays, bg, lp.LP_MATH_BF16X3)[3].double()
    one = (20.0 * ((rays.far.double() - rays.near.double()) / samples).float()).double()   # density x length, rounded once
    want = samples * one
    assert ((cache - want).abs() <= 2.0 ** -24 * (want + samples % 32 * one) * (1 + 2.0 ** -10)).all(), float(((cache - want).abs() / want).max() * 2 ** 24)
