"""The launch and scatter rules of the tile kernels (lp_mfma_bwd_tile.h, lp_tile_scatter.h) on the CPU: which way the steps
of a problem take, so that a test can tell whether it reaches the branch it is meant for."""
from collections import Counter

import numpy as np

from lp_inputs import TRIPLANE

TILE_RAYS, TILE_SAMPLES = 4, 8
EXTENT, TEXELS, PLANE_TEXELS = 12, 512, 128   # of a window


def backward_in_tiles(n_rays, samples, n_cu=256):
    """Whether the Renderer's backward hands out tiles of four rays (else single rays)."""
    waves = (n_cu + 7) // 8 * 8 * 8
    rounds = lambda items: -(-items // waves)
    tile_steps = rounds(-(-n_rays // TILE_RAYS)) * -(-samples // TILE_SAMPLES)
    return 20 * tile_steps <= 21 * (rounds(n_rays) * -(-samples // 32))


def cells(inp):
    """[rays][samples][3] cell indices."""
    delta = (inp.far.astype(np.float64) - inp.near) / inp.samples
    t = inp.near[:, None] + (np.arange(inp.samples) + 0.5) * delta[:, None]
    x = inp.origins[:, None, :].astype(np.float64) + t[..., None] * inp.dirs[:, None, :]
    if inp.contract_a:
        a, m = inp.contract_a, np.maximum(np.abs(x), 1.0)
        x = np.where(m > 1.0, 0.5 * np.sign(x) * ((2.0 - a) * (1.0 - 1.0 / m) + a), 0.5 * a * x)
    lo, hi, n = (np.asarray(a, dtype=np.float64) for a in (inp.aabb_min, inp.aabb_max, inp.res))
    return np.minimum(np.clip((x - lo) * (n - 1) / (hi - lo), 0, n - 1).astype(int), n.astype(int) - 2)


def step_routes(inp):
    """Counter of (how the rays are marched, how the step is scattered): ("tile" | "ray", 1 | 2 | 4 windows | "walk")."""
    c = cells(inp)
    ray_scene = inp.scene if inp.scene is not None else np.zeros(inp.n_rays, int)
    in_tiles = backward_in_tiles(inp.n_rays, inp.samples)

    def fits(run):   # [rays][samples][3]
        e = run.reshape(-1, 3).max(0) - run.reshape(-1, 3).min(0) + 2
        if e.max() > EXTENT:
            return False
        return max(e[0] * e[1], e[1] * e[2], e[2] * e[0]) <= PLANE_TEXELS if inp.kind == TRIPLANE else e.prod() <= TEXELS

    def march(rays, how, width):
        for j0 in range(0, inp.samples, width):
            j = np.minimum(np.arange(j0, j0 + width), inp.samples - 1)
            for parts in (1, 2, 4):
                if all(fits(run) for run in np.split(c[rays][:, j], parts, axis=1)):
                    routes[how, parts] += 1
                    break
            else:
                routes[how, "walk"] += 1

    routes = Counter()
    for first in range(0, inp.n_rays, TILE_RAYS):
        rays = np.arange(first, first + TILE_RAYS)
        there = np.minimum(rays, inp.n_rays - 1)
        ends = c[there][:, [0, -1]]
        if in_tiles and (ray_scene[there] == ray_scene[first]).all() and np.abs(ends - ends[0]).max() <= 3:
            march(there, "tile", TILE_SAMPLES)
        else:
            for r in rays[rays < inp.n_rays]:
                march([r], "ray", 32)
    return routes
