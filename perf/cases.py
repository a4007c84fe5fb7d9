"""The work a user of the library has it do, as cases that can be timed and compared.

A case is a dict of plain values that names sizes and options; `prepare` makes what a program holds
before the call (structure, decoder, rays, kept buffers) on the GPU from a seed, `run` is one pass
through the public entry points, `work` the bytes and operations that pass cannot do without.

Three kinds of pass:
  train   forward, gradient of a mean squared colour error, zeroed gradient buffers, backward: one
          training step without the optimiser (all gradients are returned)
  render  forward alone: showing images from a structure that is already fitted
  splat   Splatter forward and backward for a given gradient of the structure
The structures and decoders are those of the benchmark's workloads (`lp_inputs.WORKLOADS`,
`SPLAT_WORKLOADS`); cameras stand on a sphere around the object at angles drawn from the seed.
"""
import math

import torch

import paper_2404_19760_amd as lp
from paper_2404_19760_amd import autograd as lp_autograd

_KINDS = {"voxel": lp.LP_GRID_VOXEL, "triplane": lp.LP_GRID_TRIPLANE, "hash": lp.LP_GRID_HASH}
_DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}

_DEFAULTS = dict(
    path="train", kind="voxel", scenes=1, channels=16, nx=64, ny=64, nz=64, std=0.1, hidden=64, layers=2,
    views=1, width=64, height=64, pick=0, samples=128, near=1.0, far=4.0, box=2.75, contract=0.0, dtype="f32",
    hash_size=0, decoder="mlp", freq=2, alpha_depth=False, calls="entry")


def _case(**kw):
    unknown = set(kw) - set(_DEFAULTS) - {"name"}
    assert not unknown, unknown
    return {**({"name": kw["name"]} if "name" in kw else {}), **_DEFAULTS, **{k: v for k, v in kw.items() if k != "name"}}


def listed():
    return [
        # the smallest call: a 32 x 32 preview of a small triplane while it is fitted; launches and host work count
        _case(name="tiny_train", kind="triplane", nx=32, ny=32, nz=32, hidden=32, layers=1, width=32, height=32, samples=64),
        # a batch of pixels drawn at random from several views (how scenes are fitted from photographs), odd sizes
        # throughout, structure kept in bf16, losses on alpha and depth too, through torch.autograd
        _case(name="random_rays_train", nx=97, ny=128, nz=75, views=6, width=251, height=187, pick=5003, samples=193,
              dtype="bf16", alpha_depth=True, calls="autograd"),
        # one view of one scene in a triplane with the paper's decoder width
        _case(name="triplane_train", kind="triplane", channels=32, nx=128, ny=128, nz=128, width=128, height=128, samples=128),
        # four views of a coarse voxel grid, one hidden layer
        _case(name="voxel_train", channels=32, layers=1, views=4, width=256, height=256, samples=256),
        # a batch of scenes (a feed-forward reconstruction model in training): the largest pass
        _case(name="scenes_train", kind="triplane", scenes=8, channels=32, nx=256, ny=256, nz=256, views=4, width=256,
              height=256, samples=192),
        # a full image of a fine voxel grid: the headline workload
        _case(name="image_train", nx=256, ny=256, nz=256, std=0.05, width=800, height=800, samples=512),
        # showing a fitted scene: forward only, structure in bf16, an image size and sample count that are no multiples
        _case(name="image_render", path="render", nx=256, ny=256, nz=256, std=0.05, width=1001, height=563, samples=330,
              dtype="bf16"),
        # the Renderer of the paper's experiments: contract coordinates (an unbounded scene)
        _case(name="unbounded_train", channels=32, nx=160, ny=160, nz=160, width=256, height=256, samples=384,
              near=0.5, far=12.0, box=1.0, contract=1.0),
        # the same with the paper's view-dependent decoder (two MLPs)
        _case(name="two_mlp_train", channels=32, nx=160, ny=160, nz=160, width=256, height=256, samples=384,
              near=0.5, far=12.0, box=1.0, contract=1.0, decoder="two"),
        # a hash table
        _case(name="hash_train", kind="hash", nx=128, ny=128, nz=128, hash_size=1 << 19, width=128, height=128, samples=128),
        # images lifted into a structure: pixel features pushed as they are
        _case(name="splat_features", path="splat", channels=32, nx=160, ny=160, nz=160, views=4, width=128, height=128,
              samples=160, decoder="none"),
        # the same with the MLP that sees a prior structure and the view direction
        _case(name="splat_mlp", path="splat", channels=32, nx=160, ny=160, nz=160, views=4, width=64, height=64,
              samples=160, decoder="mlp", freq=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["voxel", "voxel", "triplane", "triplane", "unbounded", "render", "two", "hash", "splat", "splat_mlp"])
    width = _log_int(rng, 24, 420)
    height = max(16, int(width * rng.uniform(0.6, 1.2)))
    kw = dict(width=width, height=height, samples=rng.randint(24, 512), channels=rng.choice([16, 32]),
              hidden=rng.choice([32, 64, 64]), layers=rng.choice([1, 2, 2]), views=rng.choice([1, 1, 2, 4]),
              alpha_depth=rng.random() < 0.3)
    while kw["views"] * width * height * kw["samples"] > 8e7:   # no draw costs more than the largest listed case
        kw["views"] = max(1, kw["views"] // 2)
        kw["samples"] = max(24, int(kw["samples"] * rng.uniform(0.5, 0.9)))
    res = _log_int(rng, 24, 200)
    kw.update(nx=res, ny=max(8, int(res * rng.uniform(0.7, 1.3))), nz=max(8, int(res * rng.uniform(0.7, 1.3))))
    if what in ("voxel", "triplane", "render") and rng.random() < 0.25:
        kw["pick"] = max(1, int(kw["views"] * width * height * rng.uniform(0.05, 0.6)))
    if what in ("voxel", "triplane", "render"):
        kw["kind"] = rng.choice(["voxel", "triplane"]) if what == "render" else what
        kw["dtype"] = rng.choice(["f32", "f32", "bf16", "f16"])
        if what == "render":
            kw["path"] = "render"
        if kw["kind"] == "triplane":
            kw["scenes"] = rng.choice([1, 1, 2, 3])
    elif what in ("unbounded", "two"):
        kw.update(near=0.5, far=rng.uniform(6.0, 16.0), box=1.0, contract=rng.choice([0.8, 1.0, 1.2]))
        if what == "two":
            kw.update(decoder="two", hidden=64, layers=2, freq=rng.choice([0, 2, 4]))
    elif what == "hash":
        kw.update(kind="hash", hash_size=1 << rng.randint(15, 20))
    else:
        kw.update(path="splat", kind=rng.choice(["voxel", "voxel", "triplane"]), hidden=64, alpha_depth=False,
                  decoder="mlp" if what == "splat_mlp" else "none", freq=0)
    return _case(**kw)


# ---- sizes ----

def _rays(c):
    return c["scenes"] * (c["pick"] or c["views"] * c["width"] * c["height"])


def _shapes(c, channels):
    b, x, y, z = c["scenes"], c["nx"], c["ny"], c["nz"]
    ch = () if channels is None else (channels,)
    if c["kind"] == "voxel":
        return [(b, x, y, z) + ch]
    if c["kind"] == "hash":
        return [(b, c["hash_size"]) + ch]
    return [(b, x, y) + ch, (b, y, z) + ch, (b, z, x) + ch]


def _mlps(c):
    """Layer widths of the decoder's MLPs."""
    h = [c["hidden"]] * c["layers"]
    if c["decoder"] == "none":
        return []
    if c["path"] == "splat":
        return [[2 * c["channels"] + 3 + 6 * c["freq"], *h, c["channels"]]]
    if c["decoder"] == "two":
        return [[c["channels"], *h, 1], [c["channels"] + 3 + 6 * c["freq"], *h, 3]]
    return [[c["channels"], *h, 4]]


def work(case):
    c = {**_DEFAULTS, **case}
    m, corners = _rays(c), 12 if c["kind"] == "triplane" else 8
    points = m * c["samples"]
    elem = 4 if c["dtype"] == "f32" or c["path"] == "splat" else 2
    cells = sum(math.prod(s) for s in _shapes(c, None))
    touched = min(cells, points * corners) * c["channels"]     # values of the structure that a pass can reach
    mlp = sum(2 * a * b for d in _mlps(c) for a, b in zip(d, d[1:]))
    params = sum(a * b + b for d in _mlps(c) for a, b in zip(d, d[1:]))
    interp = 2 * corners * c["channels"]
    ray_bytes = m * 32
    if c["path"] == "render":
        return {"bytes": touched * elem + ray_bytes + 24 * m + 4 * params, "flops": points * (mlp + interp)}
    if c["path"] == "train":
        # forward, then input and weight gradients and the scatter; the structure read, its gradient written
        return {"bytes": touched * elem + cells * c["channels"] * 4 + 2 * ray_bytes + 60 * m + 8 * params,
                "flops": points * (3 * mlp + 2 * interp)}
    feats = m * c["channels"] * 4
    out = cells * (c["channels"] + 1) * 4
    if c["decoder"] == "none":
        return {"bytes": 2 * feats + 2 * out + 2 * ray_bytes, "flops": 2 * points * interp}
    return {"bytes": 2 * feats + 2 * out + 2 * touched * 4 + 2 * ray_bytes + 8 * params, "flops": points * (3 * mlp + 4 * interp)}


def tolerance(case):
    # About four times the largest difference seen per output between the matrix-core kernels and the scalar
    # fp32 kernels (another order of all sums, no operand splitting) on these cases at reduced ray counts:
    #   rendered colour, alpha, depth: relative 2-norm 1.5e-6, largest 6e-6 of the root mean square
    #   gradients: relative 2-norm 2.1e-3 and single elements beyond the root mean square, because a ReLU
    #   pre-activation within rounding distance of zero takes either side and a structure entry that few
    #   samples reach then changes by a whole contribution; parameter gradients 6e-4
    #   splatted features: 2e-7 and 2e-6 (sums in another order)
    c = {**_DEFAULTS, **case}
    if c["path"] == "render":
        return {"rel": 6e-6, "max": 4e-5}
    if c["path"] == "splat" and c["decoder"] == "none":
        return {"rel": 1e-6, "max": 2e-5}
    return {"rel": 8e-3, "max": 0.99}


# ---- a program's state ----

def _cameras(c, rng):
    """(origin, rotation) of every view: on a sphere of radius 2.5, looking at the origin."""
    first = rng.uniform(0.0, 360.0)
    out = []
    for k in range(c["views"]):
        az = math.radians(first + 360.0 * k / c["views"] + rng.uniform(-8.0, 8.0))
        el = math.radians(rng.uniform(-30.0, 30.0))
        pos = torch.tensor([math.cos(el) * math.sin(az), math.sin(el), math.cos(el) * math.cos(az)], dtype=torch.float64)
        right = torch.linalg.cross(torch.tensor([0.0, 1.0, 0.0], dtype=torch.float64), pos)
        right = right / right.norm()
        up = torch.linalg.cross(pos, right)
        out.append((2.5 * pos, torch.stack([right, up, pos], dim=1)))
    return out


def _make_rays(c, gen, rng, dev):
    w, h = c["width"], c["height"]
    f = (max(w, h) / 2.0) / math.tan(math.radians(30.0))
    u = (torch.arange(w, dtype=torch.float64, device=dev) + 0.5 - w / 2.0) / f
    v = (torch.arange(h, dtype=torch.float64, device=dev) + 0.5 - h / 2.0) / f
    vv, uu = torch.meshgrid(v, u, indexing="ij")
    cam = torch.stack([uu, -vv, -torch.ones_like(uu)], dim=-1).reshape(-1, 3)
    origins, dirs = [], []
    for pos, rot in _cameras(c, rng):
        d = cam @ rot.to(dev).T
        d = (d / d.norm(dim=1, keepdim=True)).float()
        d = d / d.double().norm(dim=1, keepdim=True).float()
        origins.append(pos.float().to(dev).expand_as(d))
        dirs.append(d)
    origins, dirs = torch.cat(origins), torch.cat(dirs)
    if c["pick"]:
        idx = torch.randint(origins.shape[0], (c["pick"],), generator=gen, device=dev)
        origins, dirs = origins[idx], dirs[idx]
    per_scene = origins.shape[0]
    origins, dirs = origins.repeat(c["scenes"], 1).contiguous(), dirs.repeat(c["scenes"], 1).contiguous()
    m = origins.shape[0]
    scene = None
    if c["scenes"] > 1:
        scene = torch.arange(c["scenes"], dtype=torch.int32, device=dev).repeat_interleave(per_scene)
    full = lambda x: torch.full((m,), float(x), dtype=torch.float32, device=dev)
    return lp.Rays(origins, dirs, full(c["near"]), full(c["far"]), c["samples"], scene)


def _make_mlp(dims, gen, dev):
    ws = [torch.randn((o, i), generator=gen, device=dev) * math.sqrt(2.0 / i) for i, o in zip(dims, dims[1:])]
    bs = [0.05 * torch.randn((o,), generator=gen, device=dev) for o in dims[1:]]
    return lp.Mlp(ws, bs)


def prepare(case, seed):
    import random
    c = {**_DEFAULTS, **case}
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    rays = _make_rays(c, gen, random.Random(int(seed)), dev)
    m = rays.n_rays
    kind, res = _KINDS[c["kind"]], (c["nx"], c["ny"], c["nz"])
    lo, hi = (-c["box"],) * 3, (c["box"],) * 3
    structure = [torch.randn(s, generator=gen, device=dev).mul_(c["std"]).to(_DTYPES[c["dtype"]])
                 for s in _shapes(c, c["channels"])] if c["path"] != "splat" or c["decoder"] != "none" else None
    s = {"case": c, "rays": rays, "bg": (1.0, 1.0, 1.0)}
    empty = lambda *shape: torch.empty(shape, dtype=torch.float32, device=dev)

    if c["path"] == "splat":
        s["target"] = lp.target_struct(kind, c["scenes"], c["channels"], res, lo, hi, c["contract"])
        prior = lp.Grid(kind, structure, res, lo, hi, c["contract"]) if structure is not None else None
        mlp = _make_mlp(_mlps(c)[0], gen, dev) if _mlps(c) else None
        s["splat"] = lp.Splat(torch.randn((m, c["channels"]), generator=gen, device=dev), prior, mlp,
                              c["freq"] if mlp is not None else -1)
        s["theta"] = [empty(*x) for x in _shapes(c, c["channels"])]
        s["theta_w"] = [empty(*x) for x in _shapes(c, None)]
        s["d_theta"] = [torch.randn(x, generator=gen, device=dev) for x in _shapes(c, c["channels"])]
        s["d_feats"] = torch.empty_like(s["splat"].feats)
        s["d_prior"] = [torch.empty_like(t) for t in structure] if structure is not None else []
        s["dW"] = [torch.empty_like(t) for t in mlp.weights] if mlp is not None else []
        s["db"] = [torch.empty_like(t) for t in mlp.biases] if mlp is not None else []
        s["ws"] = torch.empty(lp.lp_splat_bwd_workspace_bytes(s["target"], rays, s["splat"]), dtype=torch.uint8, device=dev)
        return s

    s["grid"] = grid = lp.Grid(kind, structure, res, lo, hi, c["contract"])
    s["rgb"], s["alpha"], s["depth"], s["cache"] = empty(m, 3), empty(m), empty(m), empty(m)
    s["target"] = torch.rand((m, 3), generator=gen, device=dev)
    s["p_alpha"] = torch.randn((m,), generator=gen, device=dev) / m if c["alpha_depth"] else None
    s["p_depth"] = torch.randn((m,), generator=gen, device=dev) / m if c["alpha_depth"] else None
    mlps = [_make_mlp(d, gen, dev) for d in _mlps(c)]
    if c["decoder"] == "two":
        s["dec"] = lp.Decoder(mlps[0], mlps[1], c["freq"], 3)
        fwd, bwd = lp.lp_dec_workspace_bytes(grid, s["dec"], rays)
        s["ws_fwd"] = torch.empty(fwd, dtype=torch.uint8, device=dev)
    else:
        s["mlp"] = mlps[0]
        bwd = lp.lp_bwd_workspace_bytes(grid, s["mlp"], rays)
    if c["path"] == "train" and c["calls"] == "entry":
        s["ws"] = torch.empty(bwd, dtype=torch.uint8, device=dev)
        s["d_grid"] = [torch.empty(t.shape, dtype=torch.float32, device=dev) for t in structure]
        s["d_params"] = [[torch.empty_like(t) for t in lst] for x in mlps for lst in (x.weights, x.biases)]
    if c["calls"] == "autograd":
        for t in structure + [t for x in mlps for t in x.weights + x.biases]:
            t.requires_grad_(True)
    return s


def run(s):
    c = s["case"]
    if c["path"] == "splat":
        lp.lp_splat_fwd(s["target"], s["rays"], s["splat"], s["theta"], s["theta_w"])
        for t in s["d_prior"] + s["dW"] + s["db"]:
            t.zero_()
        lp.lp_splat_bwd(s["target"], s["rays"], s["splat"], s["theta_w"], s["d_theta"], s["d_feats"], s["d_prior"],
                        s["dW"], s["db"], s["ws"])
        return {"theta": s["theta"], "theta_w": s["theta_w"], "d_feats": s["d_feats"], "d_prior": s["d_prior"],
                "dW": s["dW"], "db": s["db"]}

    grid, rays, bg = s["grid"], s["rays"], s["bg"]
    if c["calls"] == "autograd":
        params = grid.data + s["mlp"].weights + s["mlp"].biases
        rgb, alpha, depth = lp_autograd.render(grid, s["mlp"], rays, bg)
        loss = torch.nn.functional.mse_loss(rgb, s["target"])
        if c["alpha_depth"]:
            loss = loss + (alpha * s["p_alpha"]).sum() + (depth * s["p_depth"]).sum()
        return {"rgb": rgb.detach(), "alpha": alpha.detach(), "depth": depth.detach(),
                "gradients": list(torch.autograd.grad(loss, params))}

    out = {"rgb": s["rgb"], "alpha": s["alpha"], "depth": s["depth"]}
    two = c["decoder"] == "two"
    if two:
        lp.lp_render_dec_fwd(grid, s["dec"], rays, bg, s["rgb"], s["alpha"], s["depth"], s["cache"], s["ws_fwd"])
    else:
        lp.lp_render_fwd(grid, s["mlp"], rays, bg, s["rgb"], s["alpha"], s["depth"], s["cache"])
    if c["path"] == "render":
        return out
    d_rgb = (s["rgb"] - s["target"]) * (2.0 / s["rgb"].numel())      # mean squared error
    for t in s["d_grid"] + [t for lst in s["d_params"] for t in lst]:
        t.zero_()
    if two:
        lp.lp_render_dec_bwd(grid, s["dec"], rays, bg, d_rgb, s["p_alpha"], s["p_depth"], s["cache"], s["d_grid"],
                             *s["d_params"], s["ws"])
    else:
        lp.lp_render_bwd(grid, s["mlp"], rays, bg, d_rgb, s["p_alpha"], s["p_depth"], s["cache"], s["d_grid"],
                         *s["d_params"], s["ws"])
    return {**out, "d_grid": s["d_grid"], "d_params": s["d_params"]}
