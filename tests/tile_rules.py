"""The launch and scatter rules of the kernels (lp_mfma_bwd_tile.h, lp_tile_scatter.h, lp_mfma_fwd.hip) on the CPU: which way the steps
of a problem take, so that a test can tell whether it reaches the branch it is meant for."""
import dataclasses
from collections import Counter

import numpy as np

from lp_inputs import TRIPLANE, VOXEL

TILE_RAYS, TILE_SAMPLES = 4, 8
EXTENT, TEXELS, PLANE_TEXELS = 12, 512, 128   # of a window


def backward_in_tiles(n_rays, samples, n_cu=256):
    """Whether the Renderer's backward hands out tiles of four rays (else single rays)."""
    waves = (n_cu + 7) // 8 * 8 * 8
    rounds = lambda items: -(-items // waves)
    tile_steps = rounds(-(-n_rays // TILE_RAYS)) * -(-samples // TILE_SAMPLES)
    return 20 * tile_steps <= 21 * (rounds(n_rays) * -(-samples // 32))


def backward_in_patches(n_rays, samples, row, n_cu=256):
    """Whether it hands out patches of an image whose rows are `row` long: 4 x 2 pixels, four samples of each ray per step."""
    waves = (n_cu + 7) // 8 * 8 * 8
    steps = lambda items, step: -(-items // waves) * -(-samples // step)
    tiles = 21 * steps(-(-n_rays // TILE_RAYS), TILE_SAMPLES)
    lines = -(-n_rays // row) if row else 0
    return bool(row) and backward_in_tiles(n_rays, samples, n_cu) and 20 * steps(-(-n_rays // 8), 4) <= tiles and \
        20 * steps(-(-row // 4) * -(-lines // 2), 4) <= tiles


def forward_in_pairs(n_rays, samples, n_cu=256):
    """Whether the Renderer's forward takes rays in pairs (lp_mfma_fwd.hip launch_fwd)."""
    simds, items = 4 * n_cu, (n_rays + 1) // 2
    share = lambda n: -(-n // simds)
    return share(items) * -(-samples // 32) <= share(n_rays) * -(-samples // 64) and (samples <= 32 or items >= 2 * simds)


def forward_workgroups(n_rays, samples, n_cu=256):
    """Workgroups of the Renderer's forward (lp_mfma_fwd.hip launch_items)."""
    pairs = forward_in_pairs(n_rays, samples, n_cu)
    items, steps = ((n_rays + 1) // 2, -(-samples // 32)) if pairs else (n_rays, -(-samples // 64))
    blocks = max((3 * n_cu + 7) // 8 * 8, min(items * steps // 128 // 8 * 8, 1 << 20))
    return min(blocks, (-(-items // 4) + 7) // 8 * 8)


def image_row(inp, pixel, step):
    """Length of an image's row that the Splatter's patch kernels find in a list of rays (lp_image_rows.h find_row), 0: none."""
    end = (inp.origins + inp.far[:, None] * inp.dirs).astype(np.float32)
    d2 = lambda a, b: ((a - b) ** 2).sum(-1)
    along, ahead = d2(end[0], end[1]), end[1] - end[0]
    if not d2(end[1] + ahead, end[2]) < 0.25 * along:
        return 0
    def texel(r, t):
        x = inp.origins[r].astype(np.float64) + t * inp.dirs[r]
        if inp.contract_a:
            a, m = inp.contract_a, np.maximum(np.abs(x), 1.0)
            x = np.where(np.abs(x) <= 1.0, 0.5 * a * x, 0.5 * np.sign(x) * ((2.0 - a) * (1.0 - 1.0 / m) + a))
        lo, hi, n = (np.asarray(v, dtype=np.float64) for v in (inp.aabb_min, inp.aabb_max, inp.res))
        return np.clip((x - lo) * (n - 1) / (hi - lo), 0, n - 1)

    apart = lambda a, b: np.sqrt(((a - b) ** 2).sum())
    at = (inp.n_rays - 1) // 2
    t = 0.5 * (float(inp.near[at]) + float(inp.far[at]))
    if not inp.contract_a and min(apart(texel(at + i, t), texel(min(at + i + 1, inp.n_rays - 1), t)) for i in (0, 1)) > pixel:
        return 0
    k = np.arange(8, min(4096, (inp.n_rays - 1) // 2) + 1)
    back = d2(end[k], end[0])
    k = k[(back < 16 * along) & (back < 0.25 * d2(end[k - 1], end[0])) & (d2(end[k + 1], end[k] + ahead) < 0.25 * along) &
          (d2(end[2 * k], end[k] + (end[k] - end[0])) < 0.25 * back)]
    if not len(k):
        return 0
    row = int(k[0])
    down = end[row] - end[0]
    if not d2(end[row + row // 2], end[row // 2] + down) < 0.25 * d2(down, 0):
        return 0
    at = min(inp.n_rays // row - 1, row // 2) * row + row // 2

    near, far = float(inp.near[at]), float(inp.far[at])
    t = 0.5 * (near + far)
    close = apart(texel(at, t), texel(at + 1, t)) <= pixel and apart(texel(at, t), texel(at, t + (far - near) / inp.samples)) <= step
    return row if close else 0


def gradient_in_patches(sp, row):
    """Whether the naive Splatter's gradient takes an image `row` wide in patches (lp_splat_naive_bwd.hip)."""
    longest = 2.0 if sp.n_rays >= 131072 else 0.75 if sp.channels == 16 else 1.25
    return sp.kind != TRIPLANE and sp.n_rays >= 65536 and sp.n_rays * sp.samples >= 4000000 and sp.samples * sp.channels >= 768 and \
        image_row(sp, 0.9, longest) == row


SLOTS = {32: 224, 16: 160}   # texels of a step of a patch, by its rays
PATCH_TEXELS, PATCH_POINTS = 1024, 8


def patches(inp, row, n_rays=32):
    """The patches of an image whose rows are `row` long, as lists of rays (-1: none there)."""
    w = n_rays // 4
    lines = -(-inp.n_rays // row)
    for y0 in range(0, lines, 4):
        for x0 in range(0, row, w):
            at = (y0 + np.arange(4))[:, None] * row + x0 + np.arange(w)
            yield np.where((x0 + np.arange(w) < row) & (at < inp.n_rays), at, -1)


def push_segment(n_rays, samples, n_cu=256):
    """Points of an item of the Splatter's patch push."""
    waves = (n_cu + 7) // 8 * 8 * 4
    points = (n_rays // 32 + 1) * samples // (8 * waves)
    return min(max(points // PATCH_POINTS * PATCH_POINTS, PATCH_POINTS), samples)


def patch_routes(inp, row, n_rays=32, seg=None, every=1):
    """Of every `every`-th patch: Counter of how the points of an image's patches are taken (lp_splat_patch.h): "part": a patch that falls into parts, "lines": a
    part whose rays go line by line (its gradient: ray by ray), 8 | 4 | 1: points of a step of all rays, "ray": one point of one ray."""
    c = cells(inp)
    scene = inp.scene if inp.scene is not None else np.zeros(inp.n_rays, int)
    planes = [(0, 1), (1, 2), (2, 0)] if inp.kind == TRIPLANE else [(0, 1, 2)]
    corners = {n: np.stack(np.meshgrid(*[(0, 1)] * n, indexing="ij"), -1).reshape(-1, n) for n in (2, 3)}
    routes = Counter()

    def fits(at):   # [points][axes]
        if np.prod(at.max(0) - at.min(0) + 2) > PATCH_TEXELS:
            return False
        return len(np.unique((at[:, None] + corners[at.shape[1]]).reshape(-1, at.shape[1]), axis=0)) <= SLOTS[n_rays]

    def march(rays):
        for first in range(0, inp.samples, seg or inp.samples):
            end = min(first + (seg or inp.samples), inp.samples)
            for j0 in range(first, end, PATCH_POINTS):
                for axes in planes:
                    at, n = 0, PATCH_POINTS
                    while at < PATCH_POINTS:
                        points = c[rays][:, j0 + at:min(j0 + at + n, end)][..., axes].reshape(-1, len(axes))
                        if len(points) == 0 or fits(points):
                            routes[n] += len(points) > 0
                        elif n > 1:
                            n = 4 if n > 4 else 1
                            continue
                        else:
                            routes["ray"] += 1
                        at += n
                        if at % 4 == 0:
                            n = 4

    for k, patch in enumerate(patches(inp, row, n_rays)):
        if k % every:
            continue
        there = patch >= 0
        ends = c[patch][:, :, [0, -1]]
        other = lambda axis: (np.abs(np.diff(ends, axis=axis)).max((2, 3)) > 5) | (np.diff(scene[patch], axis=axis) != 0)
        bad = (there[:, 1:] & there[:, :-1] & other(1)).any(1)
        starts = [0] + [y for y in range(1, 4) if (there[y] & there[y - 1] & other(0)[y - 1]).any()] + [4]
        routes["part"] += sum(there[y0:y1].any() for y0, y1 in zip(starts, starts[1:])) > 1
        for y0, y1 in zip(starts, starts[1:]):
            rays = patch[y0:y1][there[y0:y1]]
            if len(rays) and bad[y0:y1].any():
                routes["lines"] += 1
            elif len(rays):
                march(rays)
    return routes


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
    """Counter of (how the rays are marched, how the step is scattered): ("patch" | "tile" | "ray", 1 | 2 | 4 windows | "walk")."""
    c = cells(inp)
    ray_scene = inp.scene if inp.scene is not None else np.zeros(inp.n_rays, int)
    in_tiles = backward_in_tiles(inp.n_rays, inp.samples)
    row = image_row(inp, 1.3 if inp.kind == VOXEL else 1.5, 1e30)

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

    def together(rays):
        ends = c[rays][:, [0, -1]]
        return (ray_scene[rays] == ray_scene[rays[0]]).all() and np.abs(ends - ends[0]).max() <= 3

    def line(rays):   # at most four
        there = np.concatenate([rays, np.full(TILE_RAYS - len(rays), rays[-1])])
        if in_tiles and together(there):
            march(there, "tile", TILE_SAMPLES)
        else:
            for r in rays:
                march([r], "ray", 32)

    routes = Counter()
    if backward_in_patches(inp.n_rays, inp.samples, row):
        for y in range(0, -(-inp.n_rays // row), 2):
            for x in range(0, row, TILE_RAYS):
                lines = [np.arange(l * row + x, min(l * row + min(x + TILE_RAYS, row), inp.n_rays)) for l in (y, y + 1)]
                lines = [l for l in lines if len(l)]
                if not lines:
                    continue
                rays = np.concatenate(lines)
                if together(rays):
                    march(rays, "patch", 4)
                else:
                    for l in lines:
                        line(l)
        return routes
    for first in range(0, inp.n_rays, TILE_RAYS):
        line(np.arange(first, min(first + TILE_RAYS, inp.n_rays)))
    return routes


def plane_lists(inp):
    """Of the tiles' steps whose samples fit one window of each plane of a triplane: how many list the texels of all planes together,
    how many one plane after the other (lp_tile_scatter.h)."""
    c, lists = cells(inp), Counter()
    for first in range(0, inp.n_rays - TILE_RAYS + 1, TILE_RAYS):
        for j0 in range(0, inp.samples, TILE_SAMPLES):
            run = c[first:first + TILE_RAYS, j0:j0 + TILE_SAMPLES].reshape(-1, 3)
            e = run.max(0) - run.min(0) + 2
            planes = (e[0] * e[1], e[1] * e[2], e[2] * e[0])
            if e.max() <= EXTENT and max(planes) <= PLANE_TEXELS:
                lists["together" if sum(planes) <= 240 else "apart"] += 1
    return lists


def splat_in_tiles(n_rays, samples, waves, up_to):
    """The Splatter's launch rule (lp_tile_scatter.h push_order)."""
    rounds = lambda items: -(-items // waves)
    return rounds(-(-n_rays // TILE_RAYS)) * -(-samples // TILE_SAMPLES) <= up_to * rounds(n_rays) * -(-samples // 32)


def splat_mlp_routes(sp, n_cu=256):
    """(push, gradient of the prior) of the Splatter with an MLP (lp_splat_mfma.hip, lp_splat_mfma_bwd.h): a Counter each of
    ("tile" | "ray", 1 | 2 | 4 windows | "walk"); a single ray has one window or the walk."""
    scene = sp.scene if sp.scene is not None else np.zeros(sp.n_rays, int)
    near_by = 6 if sp.kind != TRIPLANE and sp.channels == 16 else 9
    step = 1e30 if sp.channels == 32 else 18 if sp.kind != TRIPLANE else 36

    def fits(run):
        e = run.reshape(-1, 3).max(0) - run.reshape(-1, 3).min(0) + 2
        if e.max() > EXTENT:
            return False
        return max(e[0] * e[1], e[1] * e[2], e[2] * e[0]) <= PLANE_TEXELS if sp.kind == TRIPLANE else e.prod() <= TEXELS

    def march(routes, c, rays, how, parts_of_a_step, width):
        for j0 in range(0, sp.samples, width):
            j = np.minimum(np.arange(j0, j0 + width), sp.samples - 1)
            for parts in parts_of_a_step:
                if all(fits(run) for run in np.split(c[rays][:, j], parts, axis=1)):
                    routes[how, parts] += 1
                    break
            else:
                routes[how, "walk"] += 1

    def tiles(c):
        for first in range(0, sp.n_rays, TILE_RAYS):
            rays = np.arange(first, min(first + TILE_RAYS, sp.n_rays))
            there = np.minimum(np.arange(first, first + TILE_RAYS), sp.n_rays - 1)
            ends = c[rays][:, [0, -1]]
            yield rays, there, (scene[rays] == scene[first]).all(), np.abs(ends - ends[0]).max()

    def together(c, near_by, step):   # of 64 tiles
        all_tiles = list(tiles(c))
        middle = np.abs(c[:, min(sp.samples // 2 + TILE_SAMPLES, sp.samples - 1)] - c[:, sp.samples // 2]).max(1)   # (the kernel: to a fraction of a texel)
        return 4 * sum(apart <= near_by and middle[rays[0]] <= step for rays, _, _, apart in (all_tiles[i * len(all_tiles) // 64] for i in range(64))) >= 3 * 64

    push, c = Counter(), cells(sp)
    in_tiles = splat_in_tiles(sp.n_rays, sp.samples, 8 * n_cu, 2.0) and together(c, 9, 1e30)
    for rays, there, one_scene, apart in tiles(c):
        if in_tiles and one_scene and apart <= 9:
            march(push, c, there, "tile", (1, 2, 4), TILE_SAMPLES)
        else:
            for r in rays:
                ends = c[r, [0, -1]]
                windows = not in_tiles and (np.abs(ends[1] - ends[0]) * min(32, sp.samples) <= EXTENT * sp.samples).all()
                march(push, c, [r], "ray", (1,) if windows else (), 32)

    back, c = Counter(), cells(dataclasses.replace(sp, res=sp.prior_res))
    in_tiles = splat_in_tiles(sp.n_rays, sp.samples, 4 * n_cu, 1.05) and together(c, near_by, step)
    for rays, there, one_scene, _ in tiles(c):
        if in_tiles and one_scene:
            march(back, c, there, "tile", (1, 2, 4), TILE_SAMPLES)
        elif in_tiles:
            for r in rays:
                march(back, c, [r] * TILE_RAYS, "tile", (1, 2, 4), TILE_SAMPLES)
        else:
            for r in rays:
                march(back, c, [r], "ray", (1,) if sp.kind == TRIPLANE else (), 32)
    return push, back
