"""The tile kernels of the Renderer's backward (four neighbouring rays per wavefront, eight samples of each per
step) where their layout has edges: sample counts around the step widths, a ray count that leaves a partial
tile, scenes that change inside a tile, neighbouring rays that take the windowed scatter and rays apart
from each other that are marched one at a time and take windows or the walk; grids in every storage type.  Every case is
checked against the CPU oracle at the bounds of `parity.check_case`."""
import dataclasses

import numpy as np
import pytest

import lp_inputs
from lp_inputs import HASH, TRIPLANE, VOXEL

from parity import check_case, summary
from tile_rules import backward_in_tiles, plane_lists, step_routes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oracle():
    import oracle as o
    return o


def _with_camera_rays(inp, n_rays, image, rows):
    """`inp` with the rays of a `rows` x image strip of a pinhole view (neighbouring rays in order)."""
    rot, pos = lp_inputs.camera_pose(33.0, 17.0, 2.5)
    o, d = lp_inputs.pinhole_rays(image, rot, pos)
    first = (image // 2) * image
    idx = (first + np.arange(n_rays)) % (image * image)
    assert n_rays <= rows * image
    full = lambda v: np.full(n_rays, v, dtype=np.float32)
    scene = None if inp.n_scenes == 1 else (np.arange(n_rays) // 7 % inp.n_scenes).astype(np.int32)
    target = np.random.default_rng(3).random((n_rays, 3), dtype=np.float32)
    return dataclasses.replace(inp, origins=np.ascontiguousarray(o[idx]), dirs=np.ascontiguousarray(d[idx]), near=full(1.0),
                               far=full(4.0), scene=scene, target=target)


SHAPES = [(VOXEL, 16, (16, 64, 64, 4)), (VOXEL, 32, (32, 64, 4)), (TRIPLANE, 32, (32, 64, 64, 4)), (TRIPLANE, 16, (16, 32, 4)),
          (VOXEL, 16, (16, 32, 32, 4)), (TRIPLANE, 32, (32, 32, 4))]


@pytest.mark.parametrize("kind,channels,dims", SHAPES)
@pytest.mark.parametrize("samples", [1, 7, 8])
def test_single_step_tiles(lp, oracle, kind, channels, dims, samples):
    """At most eight samples per ray: tiles of four rays in one step; 203 rays leave a partial tile, the scene
    changes inside tiles (those rays are marched one at a time)."""
    inp = lp_inputs.make_small(kind, channels=channels, res=(21, 17, 19), mlp_dims=dims, n_rays=8, samples=samples, seed=211,
                               n_scenes=2, grid_std=0.3, aabb_min=(-2.75,) * 3, aabb_max=(2.75,) * 3)
    inp = _with_camera_rays(inp, 203, 64, 4)
    print(summary(check_case(lp, oracle, inp, lp.LP_MATH_BF16X3, label=f"single step {kind} {dims} S={samples}")), flush=True)


@pytest.mark.parametrize("kind,channels,dims", SHAPES)
@pytest.mark.parametrize("samples", [33, 63])
def test_tiles_of_several_steps(lp, oracle, kind, channels, dims, samples):
    """More rays than wavefronts, neighbours in order: several tiles per wavefront, ragged last step."""
    inp = lp_inputs.make_small(kind, channels=channels, res=(40, 33, 37), mlp_dims=dims, n_rays=8, samples=samples, seed=223,
                               grid_std=0.3, aabb_min=(-2.75,) * 3, aabb_max=(2.75,) * 3)
    inp = _with_camera_rays(inp, 8190, 128, 64)
    print(summary(check_case(lp, oracle, inp, lp.LP_MATH_BF16X3, label=f"tiles {kind} {dims} S={samples}")), flush=True)


STORED = [(VOXEL, 16, (16, 64, 64, 4)), (VOXEL, 32, (32, 32, 32, 4)), (TRIPLANE, 16, (16, 64, 4)), (TRIPLANE, 32, (32, 64, 64, 4)),
          (HASH, 16, (16, 64, 64, 4)), (HASH, 32, (32, 64, 4))]


@pytest.mark.parametrize("kind,channels,dims", STORED)
@pytest.mark.parametrize("dtype", ["bfloat16", "float16"])
@pytest.mark.parametrize("contract", [0.0, 1.3])
def test_tiles_of_grids_in_16_bits(lp, oracle, kind, channels, dims, dtype, contract):
    """The storage types' own instantiations (the contraction is a branch of theirs) with side-by-side tiles."""
    import torch
    inp = lp_inputs.make_small(kind, channels=channels, res=(40, 33, 37), mlp_dims=dims, n_rays=8, samples=33, seed=251,
                               grid_std=0.3, aabb_min=(-2.75,) * 3, aabb_max=(2.75,) * 3, hash_size=4096 if kind == HASH else None)
    inp = _with_camera_rays(inp, 8190, 128, 64)
    tdt = getattr(torch, dtype)
    inp = dataclasses.replace(inp, grid=[torch.from_numpy(g).to(tdt).float().numpy() for g in inp.grid], contract_a=contract)
    if contract:   # (the box holds all of space)
        inp = dataclasses.replace(inp, aabb_min=(-1.0,) * 3, aabb_max=(1.0,) * 3)
    routes = step_routes(inp)
    assert sum(n for (how, _), n in routes.items() if how in ("tile", "patch")) >= 0.9 * sum(routes.values()), routes
    print(summary(check_case(lp, oracle, inp, lp.LP_MATH_BF16X3, label=f"stored {kind} {dims} {dtype} a={contract}", grid_dtype=tdt)), flush=True)


@pytest.mark.parametrize("kind,channels,dims", SHAPES[:4])
@pytest.mark.parametrize("samples,res,box,scatter", [(40, (40, 33, 37), 2.75, "windows"), (32, (72, 64, 68), 1.0, "walk")])
def test_rays_apart_in_tile_order(lp, oracle, kind, channels, dims, samples, res, box, scatter):
    """Enough rays for tiles, but in random order: every item is marched ray by ray.  In cells, their steps are short (whole
    and halved windows) or long (the walk; samples outside the box keep a few of them in windows)."""
    inp = lp_inputs.make_small(kind, channels=channels, res=res, mlp_dims=dims, n_rays=8190, samples=samples, seed=227,
                               grid_std=0.3, aabb_min=(-box,) * 3, aabb_max=(box,) * 3)
    routes = step_routes(inp)
    walks = routes["ray", "walk"] / sum(routes.values())
    assert not any(how == "tile" for how, _ in routes) and (walks == 0.0 if scatter == "windows" else walks > 0.9), routes
    print(summary(check_case(lp, oracle, inp, lp.LP_MATH_BF16X3, label=f"apart {kind} {dims} {scatter}")), flush=True)


@pytest.mark.parametrize("kind,channels,dims", SHAPES[:4])
@pytest.mark.parametrize("res", [64, 150, 400])
def test_split_windows(lp, oracle, kind, channels, dims, res):
    """Steps that take one, two or four windows, and some that take the walk: the coordinate steps of a ray grow with
    the resolution.  (The short axes keep the oracle's arrays small, but no shorter: on a plane of 29 x 31 texels each
    element sums so many samples that the units at their kink reach 3.5 % of the elements, as in the parameters' gradients.)"""
    shape = (res, 64, 90) if res > 64 else (64, 64, 64)
    inp = lp_inputs.make_small(kind, channels=channels, res=shape, mlp_dims=dims, n_rays=8, samples=40, seed=229,
                               grid_std=0.3, aabb_min=(-1.5,) * 3, aabb_max=(1.5,) * 3)
    inp = _with_camera_rays(inp, 2048 * 4, 128, 64)
    print(summary(check_case(lp, oracle, inp, lp.LP_MATH_BF16X3, label=f"windows {kind} {dims} res={res}")), flush=True)


@pytest.mark.parametrize("channels,dims", [(16, (16, 32, 4)), (32, (32, 64, 64, 4))])
def test_lists_of_planes(lp, oracle, channels, dims):
    """Steps whose planes' texels share one list and steps whose windows are too large for that."""
    inp = lp_inputs.make_small(TRIPLANE, channels=channels, res=(64, 64, 64), mlp_dims=dims, n_rays=8, samples=40, seed=263,
                               grid_std=0.3, aabb_min=(-1.5,) * 3, aabb_max=(1.5,) * 3)
    inp = _with_camera_rays(inp, 2048 * 4, 128, 64)
    lists = plane_lists(inp)
    assert min(lists["together"], lists["apart"]) > 500, lists
    print(summary(check_case(lp, oracle, inp, lp.LP_MATH_BF16X3, label=f"lists of planes {dims}")), flush=True)


@pytest.mark.parametrize("n_rays,samples,tiles", [(2049, 64, False), (2600, 64, False), (4103, 64, False), (8197, 8, True), (9300, 8, True)])
def test_last_partial_round(lp, oracle, n_rays, samples, tiles):
    """Items beyond whole rounds of the 2048 wavefronts, which are spread over all workgroups: one, two or three to a
    workgroup, single rays and tiles, the last tile a partial one."""
    assert backward_in_tiles(n_rays, samples) == tiles
    inp = lp_inputs.make_small(VOXEL, channels=16, res=(21, 17, 19), mlp_dims=(16, 32, 4), n_rays=8, samples=samples, seed=257,
                               grid_std=0.3, aabb_min=(-2.75,) * 3, aabb_max=(2.75,) * 3)
    inp = _with_camera_rays(inp, n_rays, 128, 128)
    print(summary(check_case(lp, oracle, inp, lp.LP_MATH_BF16X3, label=f"last round M={n_rays} S={samples}")), flush=True)


@pytest.mark.parametrize("kind,channels,dims", SHAPES[:4])
def test_undefined_gradient_stays_on_its_ray(lp, kind, channels, dims):
    """A pixel whose loss is not a number spoils the cells of its own ray and no others: as in the scalar kernels."""
    import torch

    inp = lp_inputs.make_small(kind, channels=channels, res=(40, 33, 37), mlp_dims=dims, n_rays=8, samples=40, seed=233,
                               grid_std=0.3, aabb_min=(-2.75,) * 3, aabb_max=(2.75,) * 3)
    inp = _with_camera_rays(inp, 2048 * 4, 128, 64)
    grid, mlp, rays, bg = lp.to_device(inp, "cuda:0")
    _, _, _, cache = lp.render_fwd(grid, mlp, rays, bg, lp.LP_MATH_BF16X3)
    d_rgb = torch.ones((inp.n_rays, 3), device="cuda")
    d_rgb[4001] = float("nan")
    bad = [torch.isnan(lp.render_bwd(grid, mlp, rays, bg, d_rgb, cache, None, None, mode)[0][0])
           for mode in (lp.LP_MATH_BF16X3, lp.LP_MATH_GENERIC)]
    assert bad[1].any() and torch.equal(bad[0], bad[1])


def test_optical_depth_of_opaque_rays(lp):
    """The backward walks a ray's optical depth back from its end, step by step.  Constant density (sigma Delta = 2 per
    sample, 1027 in all) makes every rounding of that walk fall to the same side: held in fp32 it ends 9.8e-4 off at
    the front after 64 steps of eight samples, where all the weight is.  What remains is the depth the forward kept: at most half
    an ulp (6.1e-5) for each of its eight steps and for the value kept."""
    import torch

    samples, n_rays, delta = 512, 8192, 0.10033512115478516
    inp = lp_inputs.make_small(VOXEL, channels=16, res=(5, 4, 6), mlp_dims=(16, 64, 64, 4), n_rays=1, samples=samples, seed=239)
    rows = lambda a: np.repeat(a, n_rays, axis=0)
    full = lambda v: np.full(n_rays, v, dtype=np.float32)
    biases = [np.zeros_like(b) for b in inp.biases]
    biases[-1][:] = (20.0, 0.3, -0.2, 0.1)   # density 20, a constant colour: the weights are zero
    inp = dataclasses.replace(inp, origins=rows(inp.origins), dirs=rows(inp.dirs), near=full(0.0), far=full(samples * delta),
                              target=rows(inp.target), weights=[np.zeros_like(w) for w in inp.weights], biases=biases)
    grid, mlp, rays, bg = lp.to_device(inp, "cuda:0")
    _, _, _, cache = lp.render_fwd(grid, mlp, rays, bg, lp.LP_MATH_BF16X3)
    d_rgb = torch.ones((n_rays, 3), device="cuda")
    db = lp.render_bwd(grid, mlp, rays, bg, d_rgb, cache, None, None, lp.LP_MATH_BF16X3)[2][-1].double().cpu().numpy()
    for k in (1, 2, 3):   # d(colour) = sum of the weights (1) x slope of the sigmoid, over the rays
        c = 1.0 / (1.0 + np.exp(-float(inp.biases[-1][k])))
        want = n_rays * c * (1.0 - c)
        assert abs(db[k] - want) <= (9 * 6.1e-5 + 1e-5) * want, (k, db[k] / want - 1.0)
