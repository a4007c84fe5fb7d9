"""Calls whose kernels come in pairs, the first of which finds out from the rays whose work it is (images and lists of the Splatter),
and the forward of rays in pairs, captured into a graph: every replay, on other inputs and with other work between, equals the call."""
import pytest

import lp_inputs
from lp_inputs import TRIPLANE, VOXEL

from test_gpu_splat_patches import _image
from tile_rules import forward_in_pairs, gradient_in_patches, image_row, splat_mlp_routes

pytestmark = pytest.mark.gpu


def _replays(step, outputs, inputs):
    """`step` writes `outputs` from `inputs`, all kept in place."""
    import torch
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for seed in range(4):
        gen = torch.Generator(device="cuda").manual_seed(seed)
        for t in inputs:
            t.copy_(torch.randn(t.shape, generator=gen, device="cuda"))
        step()
        want = [t.clone() for t in outputs]
        for t in outputs:
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for k, (a, b) in enumerate(zip(outputs, want)):   # (sums of the same values in another order)
            assert torch.linalg.vector_norm(a - b) <= 1e-5 * torch.linalg.vector_norm(b) > 0, (seed, k)


@pytest.mark.parametrize("kind", [VOXEL, TRIPLANE])
@pytest.mark.parametrize("mlp", [False, True])
def test_splatter(lp, kind, mlp):
    import torch
    if mlp:
        sp = _image(kind, 32, 64, 72, 9, (20, 23, 17), n_in=32, hidden=(64, 64), n_freq=1, prior_channels=32, prior_res=(19, 16, 15))
        assert [{how for how, _ in r} for r in splat_mlp_routes(sp)] == [{"tile"}, {"tile"}]
    else:
        sp = _image(kind, 16, 256, 256, 64, (40, 33, 37))
        assert image_row(sp, 0.9, 1e30) == 256 and gradient_in_patches(sp, 256) == (kind == VOXEL)
    target, rays, splat = lp.splat_to_device(sp)
    theta, theta_w = lp.splat_fwd(target, rays, splat)
    d_theta = [torch.randn_like(t) for t in theta]
    d_feats, d_prior, dW, db = lp.splat_bwd(target, rays, splat, theta_w, d_theta)
    ws = torch.empty(lp.lp_splat_bwd_workspace_bytes(target, rays, splat), dtype=torch.uint8, device="cuda")

    def step():
        lp.lp_splat_fwd(target, rays, splat, theta, theta_w)
        for t in (*d_prior, *dW, *db):
            t.zero_()
        lp.lp_splat_bwd(target, rays, splat, theta_w, d_theta, d_feats, d_prior, dW, db, ws)

    _replays(step, [*theta, *theta_w, d_feats, *d_prior, *dW, *db], [splat.feats, *d_theta])


def test_forward_in_pairs(lp):
    import torch
    inp = lp_inputs.make_small(VOXEL, channels=16, res=(24, 21, 26), mlp_dims=(16, 64, 64, 4), n_rays=6143, samples=33, seed=3, grid_std=0.3)
    assert forward_in_pairs(inp.n_rays, inp.samples)
    grid, mlp, rays, bg = lp.to_device(inp, "cuda:0")
    out = [torch.empty(s, device="cuda") for s in ((6143, 3), (6143,), (6143,), (6143,))]
    _replays(lambda: lp.lp_render_fwd(grid, mlp, rays, bg, *out), out, [grid.data[0]])
