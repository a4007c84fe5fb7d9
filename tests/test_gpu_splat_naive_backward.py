"""The naive Splatter's backward with a lane per texel piece against the generic kernel (a lane per ray)."""
import pytest
import torch

import lp_inputs
from lp_inputs import HASH, TRIPLANE, VOXEL

pytestmark = pytest.mark.gpu


def _on_odd_address(t):
    """A copy of t that starts 4 bytes past a 16-byte boundary."""
    buf = torch.empty(t.numel() + 4, dtype=t.dtype, device=t.device)
    out = buf[1:1 + t.numel()].view(t.shape)
    out.copy_(t)
    assert out.data_ptr() % 16 == 4
    return out


@pytest.mark.parametrize("kind", [VOXEL, TRIPLANE, HASH])
@pytest.mark.parametrize("channels", [16, 32])
@pytest.mark.parametrize("n_rays,samples", [(1, 1), (203, 31), (64, 33), (130, 64), (37, 161)])
def test_equals_the_generic_kernel(lp, kind, channels, n_rays, samples):
    """Point counts around the 32-point unit and the 64-point records; two scenes; points beyond the box.  Gradients that
    are not 16-byte aligned take the generic kernel, which is the reference here."""
    kw = dict(hash_size=256) if kind == HASH else {}
    sp = lp_inputs.make_splat_small(kind, channels=channels, res=(9, 8, 10), n_rays=n_rays, samples=samples, seed=7 + samples,
                                    n_scenes=2, far=(2.2, 6.0), **kw)
    target, rays, splat = lp.splat_to_device(sp)
    theta, theta_w = lp.splat_fwd(target, rays, splat)
    gen = torch.Generator(device="cuda").manual_seed(3)
    d_theta = [torch.randn(t.shape, generator=gen, device="cuda") for t in theta]
    ws = torch.empty(lp.lp_splat_bwd_workspace_bytes(target, rays, splat), dtype=torch.uint8, device="cuda")
    got, want, total = (torch.full_like(splat.feats, v) for v in (7.0, -7.0, 5.0))
    lp.lp_splat_bwd(target, rays, splat, theta_w, d_theta, got, [], [], [], ws)
    lp.lp_splat_bwd(target, rays, splat, theta_w, [_on_odd_address(t) for t in d_theta], want, [], [], [], ws)
    lp.lp_splat_bwd(target, rays, splat, theta_w, [_on_odd_address(t.abs()) for t in d_theta], total, [], [], [], ws)
    # sums of n fp32 terms in two orders: each within (n + 3) 2^-24 of the sum of the terms' magnitudes (3: the weight's
    # products and quotient)
    n = samples * (12 if kind == TRIPLANE else 8)
    assert ((got - want).abs() <= 2 * (n + 3) * 2.0 ** -24 * total).all()


@pytest.mark.parametrize("kind", [VOXEL, TRIPLANE, HASH])
@pytest.mark.parametrize("samples", [1, 33, 90])
def test_infinite_gradients_stay_infinite(lp, kind, samples):
    """An infinite gradient makes the same pixels infinite or undefined as on the generic kernel: a ray is read in units
    of 32 points, and what is read past its end must not meet the infinity."""
    kw = dict(hash_size=256) if kind == HASH else {}
    sp = lp_inputs.make_splat_small(kind, channels=32, res=(9, 8, 10), n_rays=130, samples=samples, seed=11, n_scenes=2,
                                    far=(2.2, 6.0), **kw)
    target, rays, splat = lp.splat_to_device(sp)
    theta, theta_w = lp.splat_fwd(target, rays, splat)
    gen = torch.Generator(device="cuda").manual_seed(4)
    d_theta = [torch.randn(t.shape, generator=gen, device="cuda") for t in theta]
    for t in d_theta:
        t[torch.rand(t.shape, generator=gen, device="cuda") < 0.02] = float("inf")
    ws = torch.empty(lp.lp_splat_bwd_workspace_bytes(target, rays, splat), dtype=torch.uint8, device="cuda")
    got, want = torch.full_like(splat.feats, 7.0), torch.full_like(splat.feats, -7.0)
    lp.lp_splat_bwd(target, rays, splat, theta_w, d_theta, got, [], [], [], ws)
    lp.lp_splat_bwd(target, rays, splat, theta_w, [_on_odd_address(t) for t in d_theta], want, [], [], [], ws)
    assert torch.isposinf(want).any()
    assert torch.equal(torch.isposinf(got), torch.isposinf(want))
    assert torch.equal(torch.isnan(got), torch.isnan(want))
