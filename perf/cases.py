"""Performance cases: what a user of the library has it do, over the range of sizes, types and options it is used with.

`listed()` names the standing cases, `draw(rng)` gives further ones of the same ranges.  `prepare(case, seed)` builds
what a program holds before a pass (seeded inputs on the GPU, runners, contexts, packed weights, captured graphs),
`run(state)` is one pass through the public entry points, `work(case)` the bytes and operations a pass cannot do
without, `tolerance(case)` how far two correct implementations may be apart.

Kinds of case:
  stack   one pass of a workload configuration (voxelization, kernel maps, convolutions of every branch; the
          point-to-image gather where the configuration has a camera), call by call or as a replayed HIP graph
  routed  scene-routed batch: dispatcher, grouping by expert, every expert's stack on its group
  bridge  one scale of the multimodal bridge: voxelize, pool the image features by depth, fuse
  decode  up-path of the backbone: inverse kernel maps and transposed convolutions over two levels, BEV flattening
  quant   quantised layers (int8 or E4M3) on a frame's own kernel maps, the quantiser included
  ingest  many frames at once through the voxelizer and the first submanifold map
"""
from __future__ import annotations

import dataclasses
import functools
import math

import numpy as np
import torch

from paper_2507_04123_amd import binding as B
from paper_2507_04123_amd import gen
from paper_2507_04123_amd.configs import (BF16, EPI_AFFINE_RELU, F16, F32, STRIDED, VoxelSpec, expert_branches, get_config,
                                          out_grid)
from paper_2507_04123_amd.pipeline import ConfigRunner, RoutedRunner, cells_of

_DT = {"f32": F32, "f16": F16, "bf16": BF16}
_RECIPE = {1: "uniform_tiny", 2: "front", 3: "front", 4: "surround", 5: "front"}
_DIST, _CONF = 23.5, 0.5       # dispatcher thresholds: distance in metres, confidence


def listed():
    return [
        # one small cloud, fp32, a single convolution: a dozen launches, so latency and host issue are everything
        {"name": "tiny_f32", "kind": "stack", "config": 1, "points": 2000, "frames": 1, "dtype": "f32", "replay": False},
        # a sparse sensor (16 beams) through the full backbone, issued call by call: short kernels, many launches
        {"name": "sparse_front_f16", "kind": "stack", "config": 2, "points": 17003, "frames": 1, "dtype": "f16", "replay": False},
        # the ordinary 64-beam frame through the full backbone, as a captured graph: the serving loop of one camera-side car
        {"name": "front64_f16_graph", "kind": "stack", "config": 2, "points": 120000, "frames": 1, "dtype": "f16", "replay": True},
        # three voxel scales of one frame and the point-to-image gather, as a captured graph
        {"name": "three_scales_f16_graph", "kind": "stack", "config": 3, "points": 120000, "frames": 1, "dtype": "f16", "replay": True},
        # 360-degree multi-sweep frame, bf16, channels up to 128, issued call by call
        {"name": "surround_bf16", "kind": "stack", "config": 4, "points": 300000, "frames": 1, "dtype": "bf16", "replay": False},
        # eight frames in one pass, points routed by range to a near and a far stack: the headline workload
        {"name": "routed8_f16_graph", "kind": "stack", "config": 5, "points": 120000, "frames": 8, "dtype": "f16", "replay": True},
        # scene-level routing, an odd batch: dispatcher, grouping and three expert stacks, issued call by call
        {"name": "scenes5_f16", "kind": "routed", "scenes": 5, "points": 90001, "replay": False},
        # image features lifted by depth, pooled at the finest cells and fused with the frame's voxels
        {"name": "bridge_fine_mean", "kind": "bridge", "points": 120000, "height": 375, "width": 1242, "channels": 64, "scale": 1, "max": False},
        # decoder side of the 64-beam frame: two inverse maps, two transposed convolutions, the bird's-eye-view tensor
        {"name": "decode_front64_f16", "kind": "decode", "points": 120000, "dtype": "f16"},
        # int8 layers on the 64-beam frame's maps: quantise, two submanifold layers, one stride-2, one submanifold
        {"name": "quant_int8", "kind": "quant", "points": 120000, "e4m3": False},
        # the same in 8-bit floating point on a smaller, ragged frame
        {"name": "quant_e4m3_ragged", "kind": "quant", "points": 61237, "e4m3": True},
        # offline ingest: 64 frames per call through voxelization and the full-resolution kernel map
        {"name": "ingest64", "kind": "ingest", "points": 120000, "frames": 64},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["stack", "stack", "stack", "stack", "routed", "bridge", "decode", "quant", "ingest"])
    if kind == "stack":
        config = rng.choice([1, 2, 3, 4, 5])
        if config == 1:
            return {"kind": kind, "config": 1, "points": _log_int(rng, 500, 20000), "frames": 1, "dtype": "f32",
                    "replay": rng.random() < 0.5}
        frames = {2: rng.randint(1, 3), 3: 1, 4: 1, 5: rng.randint(1, 8)}[config]
        return {"kind": kind, "config": config, "points": _log_int(rng, 5000, 300000 if config == 4 else 120000), "frames": frames,
                "dtype": rng.choice(["f16", "f16", "bf16"]), "replay": rng.random() < 0.5}
    if kind == "routed":
        return {"kind": kind, "scenes": rng.randint(1, 6), "points": _log_int(rng, 10000, 80000), "replay": rng.random() < 0.5}
    if kind == "bridge":
        return {"kind": kind, "points": _log_int(rng, 10000, 120000), "height": rng.randint(240, 400), "width": rng.randint(300, 1300),
                "channels": rng.choice([32, 64, 64]), "scale": rng.choice([1, 2, 4]), "max": rng.random() < 0.5}
    if kind == "decode":
        return {"kind": kind, "points": _log_int(rng, 10000, 120000), "dtype": rng.choice(["f16", "bf16"])}
    if kind == "quant":
        return {"kind": kind, "points": _log_int(rng, 10000, 120000), "e4m3": rng.random() < 0.5}
    return {"kind": kind, "points": _log_int(rng, 20000, 120000), "frames": rng.randint(1, 48)}


# --------------------------------------------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------------------------------------------

def _clouds(recipe, n, frames, seed, device):
    """points[frames * n][4] f32 and batch[frames * n] i32 by the density laws of gen.make_cloud, drawn on `device`."""
    g = torch.Generator(device=device)
    g.manual_seed(seed)

    def u(lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(shape, generator=g, device=device)

    if recipe == "uniform_tiny":
        xyz = torch.stack([u(0.0, 20.0, frames, n), u(-10.0, 10.0, frames, n), u(-3.0, 1.0, frames, n)], dim=2)
    else:
        boxes, r_lo, r_hi, az, xb, yb, z_g, cx, cy, z_f = {
            "front": (20, 2.0, 70.4, math.pi / 2, (0.0, 70.4), (-40.0, 40.0), (-1.65, -1.55), (5.0, 65.4), (-35.0, 35.0), -1.6),
            "surround": (60, 1.0, 76.4, math.pi, (-54.0, 54.0), (-54.0, 54.0), (-1.85, -1.75), (-50.0, 50.0), (-50.0, 50.0), -1.8),
        }[recipe]
        per = (n * 3 // 10) // boxes
        n_ground = n - per * boxes
        # ground: range uniform, azimuth uniform (areal density ~ 1/r), restricted to the field of view
        m = 3 * frames * n_ground + 4096
        r, a = u(r_lo, r_hi, m), u(-az, az, m)
        x, y = r * torch.cos(a), r * torch.sin(a)
        keep = (x >= xb[0]) & (x < xb[1]) & (y >= yb[0]) & (y < yb[1])
        x, y = x[keep][: frames * n_ground], y[keep][: frames * n_ground]
        ground = torch.stack([x, y, u(*z_g, frames * n_ground)], dim=1).view(frames, n_ground, 3)
        # objects: points uniform in 4 x 1.8 x 1.6 m boxes with random centre and yaw
        shape = (frames, boxes, per)
        lx, ly, lz = u(-2.0, 2.0, *shape), u(-0.9, 0.9, *shape), u(0.0, 1.6, *shape)
        yaw = u(-math.pi, math.pi, frames, boxes, 1)
        bx, by = u(*cx, frames, boxes, 1), u(*cy, frames, boxes, 1)
        c, s = torch.cos(yaw), torch.sin(yaw)
        box = torch.stack([bx + c * lx - s * ly, by + s * lx + c * ly, z_f + lz], dim=3).view(frames, boxes * per, 3)
        xyz = torch.cat([ground, box], dim=1)
    order = torch.argsort(u(0.0, 1.0, frames, n), dim=1)
    xyz = torch.gather(xyz, 1, order.unsqueeze(2).expand(-1, -1, 3))
    pts = torch.cat([xyz, u(0.0, 1.0, frames, n, 1)], dim=2).view(frames * n, 4).contiguous()
    batch = torch.arange(frames, dtype=torch.int32, device=device).repeat_interleave(n).contiguous()
    return pts, batch


def _config(case):
    cfg = get_config(case["config"])
    branches = tuple(dataclasses.replace(b, spec=dataclasses.replace(b.spec, n_batch=case["frames"])) for b in cfg.branches)
    return dataclasses.replace(cfg, n_points=case["points"], n_frames=case["frames"], dtype=_DT[case["dtype"]], branches=branches)


def _randn(seed, shape, dtype):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda").to(dtype)


def _front_stack(points, dtype, seed):
    """The 64-beam backbone after one pass over a seeded frame: levels, kernel maps and features of its encoder."""
    case = {"config": 2, "points": points, "frames": 1, "dtype": dtype}
    cr = ConfigRunner(_config(case), points)
    pts, _ = _clouds("front", points, 1, seed, "cuda")
    cr.run(pts, None)
    cr.status_sync()
    return cr, cr.branches[0][0], cr.branches[0][1]


# --------------------------------------------------------------------------------------------------------------
# prepare / run
# --------------------------------------------------------------------------------------------------------------

def prepare(case, seed):
    return {"kind": case["kind"], **_PREPARE[case["kind"]](case, seed)}


def run(state):
    return _RUN[state["kind"]](state)


def _bounds(case, branch):
    """Rows shown of a branch's first and last level: those that its scenes fill, with room for other seeds, the same
    for every seed.  What a pass does not write of them stays zero."""
    vox = _frame_work(_RECIPE[case.get("config", 2)], case["points"], dataclasses.replace(branch.spec, n_batch=1), branch.layers)[0]
    return [case.get("frames", case.get("scenes", 1)) * (v * 5 // 4 + 256) for v in vox]


def _branch_views(case, runner):
    """What one branch leaves behind, as views of the runner's own buffers: features and sites of its last level, sites,
    means and counts of its first, the counts of all."""
    bound = _bounds(case, runner.branch)
    n0, n1 = min(bound[0], runner.levels[0].cap), min(bound[-1], runner.levels[-1].cap)
    return [runner.acts[-1][:n1], runner.levels[-1].coords[:n1], runner.levels[0].coords[:n0], runner.feats32[:n0],
            runner.counts[:n0]] + [lv.n for lv in runner.levels]


def _zeroed(out):
    for v in out:
        v.zero_()
    return out


def _prepare_stack(case, seed):
    cfg = _config(case)
    n = case["points"] * case["frames"]
    pts, batch = _clouds(_RECIPE[case["config"]], case["points"], case["frames"], seed, "cuda")
    batch = batch if case["frames"] > 1 else None
    cr = ConfigRunner(cfg, n)
    if cr.camera is not None:
        cr.camera["img"] = _randn(seed + 1, tuple(cr.camera["img"].shape), torch.float16)
    out = [v for _, r in cr.branches for v in _branch_views(case, r)]
    if cr.camera is not None:
        out += [cr.camera["out"], cr.camera["valid"]]
    _zeroed(out)
    cr.run(pts, batch)
    if case["replay"]:
        cr.capture(pts, batch, overlapped=False)
    cr.status_sync()
    return {"cr": cr, "points": pts, "batch": batch, "replay": case["replay"], "out": out}


def _run_stack(s):
    if s["replay"]:
        s["cr"].replay()
    else:
        s["cr"].run(s["points"], s["batch"])
    return s["out"]


def _prepare_routed(case, seed):
    n_sc = case["scenes"]
    pts, scene = _clouds("front", case["points"], n_sc, seed, "cuda")
    # redraw until some scene has a proposal: an empty set is not what a dispatcher is called with
    k, props = 0, np.zeros((0, 4), np.float32)
    while len(props) == 0:
        props, prop_scene = gen.make_proposals(n_sc, seed + 7919 * k, _DIST, _CONF)
        k += 1
    props, prop_scene = torch.from_numpy(props).cuda(), torch.from_numpy(prop_scene).cuda()
    rr = RoutedRunner(expert_branches(n_sc), F16, len(pts), n_sc, seed=7)
    args = (pts, scene, props, prop_scene, _DIST, _CONF)
    out = _zeroed([v for _, r in rr.runners for v in _branch_views(case, r)]) + [rr.expert, rr.counts, rr.order]
    rr.run(*args)
    if case["replay"]:
        rr.capture(*args)
    rr.status_sync()
    return {"rr": rr, "args": args, "replay": case["replay"], "out": out}


def _run_routed(s):
    if s["replay"]:
        s["rr"].replay()
    else:
        s["rr"].run(*s["args"])
    return s["out"]


def _prepare_bridge(case, seed):
    h, w, c, n = case["height"], case["width"], case["channels"], case["points"]
    spec = get_config(3).branches[(1, 2, 4).index(case["scale"])].spec
    pts, _ = _clouds("front", n, 1, seed, "cuda")
    cap = h * w + n
    ctx = B.Context(max(h * w, n), cap, cells_of(spec.grid, 1), n_slots=3)
    i32 = dict(dtype=torch.int32, device="cuda")
    s = {"ctx": ctx, "points": pts, "spec": spec, "cap": cap, "n_pts": n, "mode": B.POOL_MAX if case["max"] else B.POOL_MEAN,
         "img": _randn(seed + 1, (h, w, c), torch.float16),
         "depth": torch.from_numpy(gen.make_depth(h, w, seed)).cuda(), "q": gen.make_unprojection(gen.make_camera(seed)).tolist(),
         # LiDAR side: voxels of the frame with the 32 features a branch gives them
         "lc": torch.zeros((n, 4), **i32), "lm": torch.zeros((n, 4), device="cuda"), "lcnt": torch.zeros((n,), **i32),
         "ln": torch.zeros(1, **i32), "lf": _randn(seed + 2, (n, 32), torch.float16),
         "ic": torch.zeros((h * w, 4), **i32), "if": torch.zeros((h * w, c), dtype=torch.float16, device="cuda"),
         "icnt": torch.zeros((h * w,), **i32), "in": torch.zeros(1, **i32),
         "fc": torch.zeros((cap, 4), **i32), "ff": torch.zeros((cap, 32 + c), dtype=torch.float16, device="cuda"),
         "fn": torch.zeros(1, **i32)}
    _bridge_pass(s)
    ctx.status_sync()
    # there are several pixels to an image cell: fewer cells than half of the pixels
    ni, nf = h * w // 2, n + h * w // 2
    s["out"] = [s["lc"], s["lm"], s["lcnt"], s["ic"][:ni], s["if"][:ni], s["icnt"][:ni], s["fc"][:nf], s["ff"][:nf],
                s["ln"], s["in"], s["fn"]]
    return s


def _bridge_pass(s):
    ctx, sp = s["ctx"], s["spec"]
    ctx.voxelize(s["points"], None, sp, s["n_pts"], s["lc"], s["lm"], s["lcnt"], s["ln"], index_slot=0)
    ctx.pool_image(s["img"], s["depth"], s["q"], sp, s["mode"], s["ic"].shape[0], s["ic"], s["if"], s["icnt"], s["in"], index_slot=1)
    ctx.fuse(F16, s["lc"], s["lf"], s["ln"], s["n_pts"], s["ic"], s["if"], s["in"], s["ic"].shape[0], sp.grid, 1, s["cap"],
             s["fc"], s["ff"], s["fn"], out_slot=2)


def _run_bridge(s):
    _bridge_pass(s)
    return s["out"]


def _prepare_decode(case, seed):
    cr, ctx, r = _front_stack(case["points"], case["dtype"], seed)
    td = torch.float16 if case["dtype"] == "f16" else torch.bfloat16
    dt = _DT[case["dtype"]]
    l1, l2, l3 = r.levels[1:4]
    steps, x = [], r.acts[-1]
    for k, (fine, coarse, cin, cout) in enumerate(((l2, l3, 64, 64), (l1, l2, 64, 32))):
        w = _randn(seed + 10 + k, (27, cin, cout), torch.float32).mul_(0.1).to(td)
        wp = torch.empty_like(w)
        ctx.pack_weights(dt, w, wp)
        steps.append({"fine": fine, "coarse": coarse, "w": wp, "x": x,
                      "scale": torch.full((cout,), 10.0 / math.sqrt(3.0 * cin), device="cuda"), "shift": torch.zeros(cout, device="cuda"),
                      "nbr": torch.empty((27, fine.cap), dtype=torch.int32, device="cuda"),
                      "y": torch.empty((fine.cap, cout), dtype=td, device="cuda")})
        x = steps[-1]["y"]
    gx, gy, gz = l3.grid
    s = {"cr": cr, "ctx": ctx, "dt": dt, "steps": steps, "l3": l3, "enc": r.acts[-1],
         "bev": torch.empty((1, gy, gx, gz * 64), dtype=td, device="cuda")}
    s["out"] = [s["bev"]]
    bound = _bounds(case, r.branch)
    for st, nf in zip(steps, (bound[2], bound[1])):
        s["out"] += _zeroed([st["nbr"][:, :nf], st["y"][:nf]])
    return s


def _run_decode(s):
    ctx, dt = s["ctx"], s["dt"]
    for st in s["steps"]:
        f, c = st["fine"], st["coarse"]
        ctx.build_inverse_kmap(f.coords, f.n, f.cap, c.grid, 1, c.slot, c.n, st["nbr"])
        ctx.spconv(dt, st["x"], st["w"], st["scale"], st["shift"], EPI_AFFINE_RELU, st["nbr"], f.n, f.cap, st["y"], w_layout=B.W_PACKED)
    l3 = s["l3"]
    ctx.bev_flatten(dt, l3.coords, s["enc"], l3.n, l3.cap, l3.grid, 1, s["bev"])
    return s["out"]


def _prepare_quant(case, seed):
    cr, ctx, r = _front_stack(case["points"], "f16", seed)
    l2, l3 = r.levels[2:4]
    n2, n3 = int(l2.n.item()), int(l3.n.item())
    e4 = case["e4m3"]
    code = torch.uint8 if e4 else torch.int8
    layers, bound = [], _bounds(case, r.branch)
    # (map, output level): two submanifold layers, down to the next level, one submanifold layer there
    for k, (nbr, lv, n_in) in enumerate(((l2.subm_nbr, l2, n2), (l2.subm_nbr, l2, n2), (l3.down_nbr, l3, n2), (l3.subm_nbr, l3, n3))):
        packed = torch.empty((27 * 64 * 64,), dtype=torch.int8, device="cuda")
        if e4:
            w = torch.empty((27, 64, 64), dtype=torch.uint8, device="cuda")
            ctx.quantize_e4m3(_randn(seed + 20 + k, (27, 64, 64), torch.float32).mul_(0.1), 8.0, w)
            ctx.pack_weights_i8(w.view(torch.int8), packed)
            mul = 1.0 / (8.0 * 0.1 * math.sqrt(12.0 * 64.0))
        else:
            w = _randn(seed + 20 + k, (27, 64, 64), torch.float32).mul_(20.0).round_().clamp_(-127, 127).to(torch.int8)
            ctx.pack_weights_i8(w, packed)
            mul = 1.0 / (20.0 * 30.0 * math.sqrt(12.0 * 64.0))      # int8 features carry a scale of 1/30
        last = k == 3
        out = torch.empty((lv.cap, 64), dtype=torch.float16 if (e4 or last) else torch.int8, device="cuda")
        layers.append({"nbr": nbr, "lv": lv, "n_in": n_in, "w": packed, "y": out,
                       "mul": torch.full((64,), mul, device="cuda"), "add": torch.zeros(64, device="cuda"),
                       "q": torch.empty((n_in, 64), dtype=code, device="cuda") if (k == 0 or e4) else None,
                       "show": _zeroed([out[: bound[2] if lv is l2 else bound[3]]])[0]})
    s = {"cr": cr, "ctx": ctx, "e4m3": e4, "layers": layers, "x": _randn(seed + 19, (n2, 64), torch.float16).clamp_(min=0.0)}
    s["out"] = [ly["show"] for ly in layers]
    return s


def _run_quant(s):
    ctx, x = s["ctx"], s["x"]
    for ly in s["layers"]:
        lv = ly["lv"]
        if s["e4m3"]:
            ctx.quantize_e4m3(x[: ly["n_in"]], 1.0, ly["q"])
            ctx.spconv_e4m3(ly["q"], ly["w"], 64, 64, ly["mul"], ly["add"], True, ly["nbr"], lv.n, lv.cap, ly["y"])
        else:
            if ly["q"] is not None:
                ctx.quantize_i8(x, 30.0, ly["q"])
                x = ly["q"]
            ctx.spconv_i8(x, ly["w"], 64, 64, ly["mul"], ly["add"], True, ly["nbr"], lv.n, lv.cap, ly["y"], inv_out_scale=30.0,
                          n_in_rows=ly["n_in"])
        x = ly["y"]
    return s["out"]


def _prepare_ingest(case, seed):
    frames, cap = case["frames"], case["points"] * case["frames"]
    base = get_config(2).branches[0].spec
    spec = VoxelSpec(base.lo, base.vs, base.grid, n_batch=frames)
    pts, batch = _clouds("front", case["points"], frames, seed, "cuda")
    i32 = dict(dtype=torch.int32, device="cuda")
    s = {"ctx": B.Context(cap, cap, cells_of(spec.grid, frames), n_slots=1), "spec": spec, "points": pts, "batch": batch, "cap": cap,
         "coords": torch.zeros((cap, 4), **i32), "feats": torch.zeros((cap, 4), device="cuda"), "counts": torch.zeros((cap,), **i32),
         "lp": torch.zeros((cap, 4), dtype=torch.float16, device="cuda"), "n": torch.zeros(1, **i32),
         "nbr": torch.zeros((27, cap), **i32)}
    _ingest_pass(s)
    s["ctx"].status_sync()
    s["out"] = [s["coords"], s["feats"], s["counts"], s["lp"], s["n"], s["nbr"]]
    return s


def _ingest_pass(s):
    ctx, sp, cap = s["ctx"], s["spec"], s["cap"]
    ctx.voxelize(s["points"], s["batch"], sp, cap, s["coords"], s["feats"], s["counts"], s["n"], feats_lp=s["lp"], index_slot=0)
    ctx.build_kmap(B.SUBM, s["coords"], s["n"], cap, sp.grid, sp.n_batch, cap, s["nbr"], s["n"], in_slot=0)


def _run_ingest(s):
    _ingest_pass(s)
    return s["out"]


_PREPARE = {"stack": _prepare_stack, "routed": _prepare_routed, "bridge": _prepare_bridge, "decode": _prepare_decode,
            "quant": _prepare_quant, "ingest": _prepare_ingest}
_RUN = {"stack": _run_stack, "routed": _run_routed, "bridge": _run_bridge, "decode": _run_decode, "quant": _run_quant,
        "ingest": _run_ingest}


# --------------------------------------------------------------------------------------------------------------
# work and tolerance
# --------------------------------------------------------------------------------------------------------------

@functools.lru_cache(maxsize=64)
def _frame_work(recipe, n, spec, layers):
    """One frame of a branch, counted on the host: voxels per level, and per layer the (input row, tap, output row)
    pairs (submanifold layers from a sample of 4096 rows)."""
    pts = _clouds(recipe, n, 1, 1, "cpu")[0].numpy()
    cell = np.floor((pts[:, :3] - np.float32(spec.lo)) / np.float32(spec.vs)).astype(np.int64)
    r2 = pts[:, 0] ** 2 + pts[:, 1] ** 2
    grid = np.array(spec.grid, np.int64)
    ok = ((cell >= 0) & (cell < grid)).all(1) & (r2 >= spec.r2_min) & (r2 < spec.r2_max)
    cell = cell[ok]

    def key(c, g):
        return (c[:, 2] * g[1] + c[:, 1]) * g[0] + c[:, 0]

    def unkey(k, g):
        return np.stack([k % g[0], k // g[0] % g[1], k // (g[0] * g[1])], axis=1)

    keys = np.unique(key(cell, grid))
    voxels, pairs = [len(keys)], []
    for layer in layers:
        if layer.kind == STRIDED:
            c, g2 = unkey(keys, grid), np.array(out_grid(tuple(int(v) for v in grid)), np.int64)
            parts = []
            for dz in (0, 1):
                for dy in (0, 1):
                    for dx in (0, 1):
                        d = np.array([dx, dy, dz])
                        o = c // 2 + d
                        take = ((d == 0) | (c % 2 == 1)).all(1) & (o < g2).all(1)
                        parts.append(key(o[take], g2))
            every = np.concatenate(parts)
            pairs.append(len(every))
            keys, grid = np.unique(every), g2
            voxels.append(len(keys))
        else:
            at = np.random.RandomState(3).choice(len(keys), min(4096, len(keys)), replace=False)
            c, hits = unkey(keys[at], grid), 0
            for k in range(27):
                o = c + np.array([k % 3 - 1, k // 3 % 3 - 1, k // 9 - 1])
                o = o[((o >= 0) & (o < grid)).all(1)]
                ko = key(o, grid)
                pos = np.minimum(np.searchsorted(keys, ko), len(keys) - 1)
                hits += int((keys[pos] == ko).sum())
            pairs.append(hits * len(keys) // max(1, len(at)))
    return tuple(voxels), tuple(pairs)


def _branch_work(recipe, n, frames, branch, dtype, batched):
    spec = dataclasses.replace(branch.spec, n_batch=1)
    vox, pairs = _frame_work(recipe, n, spec, branch.layers)
    esz = 4 if dtype == F32 else 2
    flops = sum(2.0 * p * ly.cin * ly.cout for p, ly in zip(pairs, branch.layers)) * frames
    weights = sum(27.0 * ly.cin * ly.cout * esz for ly in branch.layers)
    written = frames * (vox[0] * 36.0 + vox[-1] * (16.0 + branch.layers[-1].cout * esz))
    return frames * n * (20.0 if batched else 16.0) + weights + written, flops, [v * frames for v in vox], [p * frames for p in pairs]


def work(case):
    """Bytes: every input of the pass read once, every output written once (features between layers and kernel maps
    that only later layers read are neither).  Operations: two per channel pair of every pair of rows a map names."""
    kind = case["kind"]
    if kind == "stack":
        cfg = _config(case)
        got = [_branch_work(_RECIPE[case["config"]], case["points"], case["frames"], b, cfg.dtype, case["frames"] > 1)
               for b in cfg.branches]
        nbytes, flops = sum(g[0] for g in got), sum(g[1] for g in got)
        if cfg.camera is not None:      # an image, read once at the most, and a row of features and a flag per point
            cam = cfg.camera
            nbytes += min(cam.height * cam.width, 4 * case["points"]) * cam.channels * 2.0 + case["points"] * (cam.channels * 2.0 + 1.0)
            flops += case["points"] * cam.channels * 8.0
        return {"bytes": nbytes, "flops": flops}
    if kind == "routed":                # on average a third of the scenes goes to each expert
        got = [_branch_work("front", case["points"], case["scenes"], b, F16, True) for b in expert_branches(case["scenes"])]
        return {"bytes": sum(g[0] for g in got) / 3.0, "flops": sum(g[1] for g in got) / 3.0}
    if kind == "bridge":
        branch = get_config(3).branches[(1, 2, 4).index(case["scale"])]
        vox = _branch_work("front", case["points"], 1, branch, F16, False)[2][0]
        pix, c = case["height"] * case["width"], case["channels"]
        pooled = case["width"] * (case["height"] - 203)      # rows of a road scene that carry a depth
        cells = pooled // (3 * case["scale"])
        nbytes = (case["points"] * 16.0 + vox * 36.0 + pix * 4.0 + pooled * c * 2.0 + cells * (20.0 + c * 2.0)
                  + vox * 64.0 + (vox + cells) * (16.0 + (32 + c) * 2.0))
        return {"bytes": nbytes, "flops": float(pooled * c)}
    front = get_config(2).branches[0]
    if kind == "decode":
        _, _, vox, pairs = _branch_work("front", case["points"], 1, front, F16, False)
        down = [p for p, ly in zip(pairs, front.layers) if ly.kind == STRIDED]
        gx, gy, gz = out_grid(out_grid(out_grid(front.spec.grid)))
        nbytes = (vox[3] * (64 * 2.0 + 16.0) + gx * gy * gz * 64 * 2.0
                  + vox[2] * (16.0 + 108.0 + 64 * 2.0) + vox[1] * (16.0 + 108.0 + 32 * 2.0) + 27 * 2.0 * (64 * 64 + 64 * 32))
        return {"bytes": nbytes, "flops": 2.0 * (down[2] * 64 * 64 + down[1] * 64 * 32)}
    if kind == "quant":
        _, _, vox, pairs = _branch_work("front", case["points"], 1, front, F16, False)
        esz = 2.0 if case["e4m3"] else 1.0
        # layers 4..6 of the backbone are stride-2 and submanifold at level 2, 7..9 at level 3
        nbytes = (vox[2] * 64 * 3.0 + 2 * vox[2] * 64 * esz + vox[3] * 64 * (esz + 2.0) + vox[2] * 108.0 + 2 * vox[3] * 108.0
                  + 4 * 27 * 64 * 64)
        return {"bytes": nbytes, "flops": 2.0 * 64 * 64 * (2 * pairs[5] + pairs[7] + pairs[8])}
    vox = _frame_work("front", case["points"], front.spec, front.layers[:1])[0][0] * case["frames"]
    n = case["points"] * case["frames"]
    return {"bytes": n * 20.0 + vox * (44.0 + 108.0), "flops": 4.0 * n}


def tolerance(case):
    """Coordinates, counts, maps and routing are whole numbers and agree exactly.  Features: sums of fp32 products in
    any order; 16-bit stacks round every layer's activations once (2^-11 fp16, 2^-9 bf16), up to twelve layers deep, and a
    different order of a sum can move single values by a few such steps.  int8 layers are exact."""
    kind = case["kind"]
    if kind == "quant":
        return {"rel": 2e-3, "max": 0.05} if case["e4m3"] else "exact"
    if kind == "ingest":                # means fp32; their fp16 copy may round the other way
        return {"rel": 1e-4, "max": 2e-3}
    if kind == "bridge":
        return {"rel": 1e-3, "max": 1e-2}
    dtype = case.get("dtype", "f16")
    return {"f32": {"rel": 1e-5}, "f16": {"rel": 2e-3, "max": 0.08}, "bf16": {"rel": 1e-2, "max": 0.3}}[dtype]
