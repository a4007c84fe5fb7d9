"""Sampling by whole texels in the forward (32-channel structures): every storage type has another number of
lanes per texel and of passes over a step. Sample counts around the 32- and 64-sample blocks, several scenes,
against the CPU oracle on the stored values at the forward's bound (1e-4, the sum of the bf16 hi + lo products'
3 * 2^-18 over the layers being far below it)."""
import dataclasses

import pytest

import lp_inputs
from lp_inputs import HASH, TRIPLANE, VOXEL

from parity import FWD_RTOL, close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("samples", [1, 31, 33, 65])
@pytest.mark.parametrize("dtype", ["float32", "bfloat16", "float16"])
@pytest.mark.parametrize("kind", [VOXEL, TRIPLANE, HASH])
def test_forward_of_32_channel_structures(lp, kind, dtype, samples):
    import oracle
    import torch
    inp = lp_inputs.make_small(kind, channels=32, res=(9, 12, 7), mlp_dims=(32, 64, 4), n_rays=37, samples=samples, seed=301,
                               n_scenes=2, grid_std=0.3, hash_size=256 if kind == HASH else None)
    tdt = getattr(torch, dtype)
    if dtype != "float32":
        inp = dataclasses.replace(inp, grid=[torch.from_numpy(g).to(tdt).float().numpy() for g in inp.grid])
    grid, mlp, rays, bg = lp.to_device(inp)
    grid.data = [t.to(tdt) for t in grid.data]
    got = lp.render_fwd(grid, mlp, rays, bg, lp.LP_MATH_BF16X3)
    want = oracle.render_fwd(oracle.Problem(inp))
    for name, a, b in zip(("rgb", "alpha", "depth"), got, want):
        close(a.cpu().numpy(), b, FWD_RTOL, f"kind={kind} {dtype} S={samples} {name}")
