"""What is timed: one pass of the library's paths at the sizes a planner uses.

A planner in a room with people builds the room's distance field once (and
again when the map changes), then for every new prediction of the people's
motion either builds one composite field per predicted time slice and samples
them at the robot's collision spheres, or samples the composites without
building them; a learner of the surrogate trains on the library's own labels.
The listed cases are those calls on the rooms this repository uses throughout
(64^3 at 5 cm, 256x256x128 at 2 cm, 512x512x256 at 1 cm, a room of odd sizes,
and a batch of uneven rooms); `draw` gives others of the same ranges.

Inputs are made from the seed alone: rooms of axis-aligned boxes of 0.1 to
0.8 m, cylinders of human size on constant-velocity or piecewise-linear
paths, spheres uniform over the room.  `exact` computes the same results in
64 bits by an exhaustive separable minimum, without the library.
"""
import math
import os

import numpy as np
import torch

import paper_2201_05058_amd as pc
from paper_2201_05058_amd import surrogate

RADIUS, HEIGHT = 0.25, 1.8  # a standing person
WEIGHTS = os.path.join(os.path.dirname(os.path.abspath(pc.__file__)),
                       "weights", "surrogate_room256.npz")
HID = 128


def listed():
    room = {"nx": 256, "ny": 256, "nz": 128, "h": 0.02, "boxes": 40}
    hall = {"nx": 512, "ny": 512, "nz": 256, "h": 0.01, "boxes": 200}
    return [
        # the room's own field: when the robot enters it, and at each change
        # of its map
        {"name": "static_room", "kind": "static", **room},
        {"name": "static_hall", "kind": "static", **hall},
        # one update of a coarse reactive controller: the smallest composite
        {"name": "composite_cube", "kind": "composite", "nx": 64, "ny": 64,
         "nz": 64, "h": 0.05, "boxes": 12, "n": 1, "k": 1, "motion": "cv",
         "outputs": "sdf"},
        # one update of the planner: 2 s of predictions of three people
        {"name": "composite_room", "kind": "composite", **room, "n": 20,
         "k": 3, "motion": "cv", "outputs": "both"},
        # the same in a room cut to odd sizes (no row or layer is a multiple
        # of a vector)
        {"name": "composite_ragged", "kind": "composite", "nx": 255,
         "ny": 241, "nz": 127, "h": 0.02, "boxes": 40, "n": 20, "k": 3,
         "motion": "cv", "outputs": "both"},
        # the largest update: a 1 cm map, eight people, 50 slices
        {"name": "composite_hall", "kind": "composite", **hall, "n": 50,
         "k": 8, "motion": "paths", "outputs": "both"},
        # a planner that reads 10k spheres per update and builds no field
        {"name": "direct_room", "kind": "direct", **room, "n": 20, "k": 3,
         "motion": "cv", "q": 10_000},
        # a sampling planner's sweep over the built fields of the hall
        {"name": "query_hall", "kind": "query", **hall, "n": 50, "k": 8,
         "motion": "paths", "q": 5_000_000},
        # the obstacle factors of one optimiser iteration: 100 support
        # states of a robot of 64 spheres
        {"name": "factors_room", "kind": "factors", **room, "n": 20, "k": 3,
         "motion": "cv", "states": 100, "spheres": 64},
        # 1M spheres answered by the trained surrogate with exact fallback
        {"name": "surrogate_room", "kind": "surrogate", **room, "n": 20,
         "k": 3, "motion": "cv", "q": 1_000_000},
        # forward and backward of one training batch of the surrogate
        {"name": "train_batch", "kind": "train", "rows": 65_536},
        # a fleet: uneven rooms updated together by one captured graph
        {"name": "batch_rooms", "kind": "batch", "scenes": 16,
         "shapes": 3},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["static", "static", "composite", "composite",
                       "composite", "direct", "query", "factors",
                       "surrogate", "train", "batch"])
    if kind == "train":
        return {"kind": kind, "rows": _logint(rng, 2_000, 131_072)}
    if kind == "batch":
        return {"kind": kind, "scenes": rng.randint(4, 24),
                "shapes": rng.randint(10, 10_000)}
    if kind == "surrogate":  # the trained network is one of 2 cm voxels
        return {"kind": kind, "nx": rng.randint(128, 320),
                "ny": rng.randint(128, 320), "nz": rng.randint(96, 160),
                "h": 0.02, "boxes": rng.randint(20, 60),
                "n": rng.randint(5, 30), "k": rng.randint(1, 4),
                "motion": "cv", "q": _logint(rng, 10_000, 1_000_000)}
    nx, ny = _logint(rng, 48, 512), _logint(rng, 48, 512)
    nz = _logint(rng, 24, 256)
    h = max(math.exp(rng.uniform(math.log(0.01), math.log(0.05))),
            0.8 / min(nx, ny))
    vol = nx * ny * nz * h ** 3
    c = {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "h": h,
         "boxes": min(200, max(4, round(40 * vol / 67.1)))}
    if kind == "static":
        return c
    n = min(_logint(rng, 1, 50), max(1, 1_500_000_000 // (nx * ny * nz)))
    c |= {"n": n, "k": rng.randint(1, 8),
          "motion": rng.choice(["cv", "paths"])}
    if kind == "composite":
        c["outputs"] = rng.choice(["both", "both", "sdf"])
    elif kind == "direct":
        c["q"] = _logint(rng, 1_000, 1_000_000)
    elif kind == "query":
        c["q"] = _logint(rng, 1_000, 5_000_000)
    else:
        c |= {"states": _logint(rng, 10, 400), "spheres": rng.randint(8, 128)}
    return c


# ------------------------------------------------------------------ inputs

def _dev():
    return torch.device("cuda", torch.cuda.current_device())


def _occupancy(c, r):
    """uint8 [nz, ny, nx] of axis-aligned boxes, made on the GPU."""
    n = np.array([c["nx"], c["ny"], c["nz"]])
    L = n * c["h"]
    occ = torch.zeros((c["nz"], c["ny"], c["nx"]), dtype=torch.uint8,
                      device=_dev())
    for _ in range(c["boxes"]):
        s = np.minimum(r.uniform(0.1, 0.8, size=3), L)
        lo = r.uniform(0.0, 1.0, size=3) * (L - s)
        a = np.maximum(np.ceil(lo / c["h"] - 0.5).astype(int), 0)
        b = np.minimum(np.floor((lo + s) / c["h"] - 0.5).astype(int), n - 1)
        occ[a[2]:b[2] + 1, a[1]:b[1] + 1, a[0]:b[0] + 1] = 1
    return occ


def _people(c, r):
    """Predicted positions [n, k, 2] in metres, slices 0.1 s apart ("cv") or
    0.05 s apart on four-waypoint paths held at their end ("paths")."""
    n, k = c["n"], c["k"]
    lx, ly = c["nx"] * c["h"], c["ny"] * c["h"]
    xy = np.empty((n, k, 2))
    for p in range(k):
        if c["motion"] == "paths":
            w = np.stack([r.uniform(RADIUS, lx - RADIUS, size=4),
                          r.uniform(RADIUS, ly - RADIUS, size=4)], axis=1)
            leg = np.hypot(*np.diff(w, axis=0).T) / r.uniform(0.5, 1.5, 3)
            at = np.concatenate([[0.0], np.cumsum(leg)])
            t = np.arange(n) * 0.05
            xy[:, p, 0] = np.interp(t, at, w[:, 0])
            xy[:, p, 1] = np.interp(t, at, w[:, 1])
        else:
            x0 = np.array([r.uniform(RADIUS, lx - RADIUS),
                           r.uniform(RADIUS, ly - RADIUS)])
            a, v = r.uniform(0.0, 2 * np.pi), r.uniform(0.5, 1.5)
            xy[:, p] = x0 + np.arange(n)[:, None] * 0.1 * v * np.array(
                [np.cos(a), np.sin(a)])
    return xy


def _spheres(c, q, seed):
    """Centres [q, 3] inside the span of voxel centres, radii [q], slices."""
    g = torch.Generator(device=_dev()).manual_seed(seed)
    n = torch.tensor([c["nx"], c["ny"], c["nz"]], dtype=torch.float64,
                     device=_dev())
    u = torch.rand((q, 3), generator=g, dtype=torch.float64, device=_dev())
    centre = ((0.51 + u * (n - 1.02)) * c["h"]).float()
    rad = 0.05 + 0.1 * torch.rand(q, generator=g, device=_dev())
    sl = (torch.arange(q, device=_dev()) % c["n"]).int()
    return centre, rad, sl


def _scene(c, seed):
    r = np.random.default_rng(seed)
    occ = _occupancy(c, r)
    return occ, _people(c, r) if "n" in c else None


def _grid(c):
    return pc.Grid.make(c["nx"], c["ny"], c["nz"], c["h"])


def _batch_scenes(c):
    """The rooms of a batch: sizes from the case, contents from the seed."""
    r = np.random.default_rng(c["shapes"])
    out = []
    for _ in range(c["scenes"]):
        d = {"nx": int(r.integers(64, 257)), "ny": int(r.integers(64, 257)),
             "nz": int(r.integers(64, 129)), "h": float(r.uniform(.02, .05))}
        vol = d["nx"] * d["ny"] * d["nz"] * d["h"] ** 3
        d |= {"boxes": max(4, round(40 * vol / 67.1)),
              "n": int(r.integers(5, 31)), "k": int(r.integers(1, 5)),
              "motion": "cv", "outputs": "both"}
        out.append(d)
    return out


def _rows(c, seed):
    """A training batch: rows of the surrogate's 16 features around a person
    in a 256x256x128 room of 2 cm voxels, residual targets in voxels, and
    the network's parameters and normalisation (host)."""
    n, dev = c["rows"], _dev()
    g = torch.Generator(device=dev).manual_seed(seed)

    def u(*shape):
        return torch.rand(shape, generator=g, dtype=torch.float64, device=dev)

    x = torch.empty((n, 16), dtype=torch.float64, device=dev)
    ang, rv, kt = 2 * math.pi * u(n), RADIUS / 0.02, 89.0
    rho = 75 * u(n).sqrt() + 1e-3
    a, w = rho - rv, 127 * u(n) - kt
    d = torch.hypot(a.clamp(min=0), w.clamp(min=0))
    x[:, 0], x[:, 1] = torch.cos(ang), torch.sin(ang)
    x[:, 2], x[:, 3], x[:, 4], x[:, 5] = a, w, d, 1 / (1 + d)
    ph = 2 * math.pi * u(n, 5)
    x[:, 6::2], x[:, 7::2] = torch.sin(ph), torch.cos(ph)
    x = x.float().contiguous()
    t = (0.45 + 0.2 * torch.sin(3 * ang) * torch.cos(ph[:, 0])
         + 0.1 * torch.sin(ph[:, 2]) + 0.1 * u(n)).float()
    r = np.random.default_rng(seed)
    fan = [(16, 128), (128, 128), (128, 128), (128, 128), (128, 1)]
    params = np.concatenate([
        r.uniform(-1, 1, size=i * o + o) / math.sqrt(i)
        for i, o in fan]).astype(np.float32)
    off = x.mean(0).cpu().numpy()
    scale = (1.0 / x.std(0).clamp(min=1e-3)).cpu().numpy()
    return x, t, params, off, scale


# -------------------------------------------------------- prepare and run

def _fields(c, seed):
    """A built room: its static field and the people's positions."""
    occ, xy = _scene(c, seed)
    ssq, sdf = pc.build_static_sdf(_grid(c), occ)
    return ssq, sdf, xy


def _buffers(c):
    shape = (c["nz"], c["ny"], c["nx"])
    return pc.composite_outputs(c["n"], shape, _dev(),
                                want_ssq=c["outputs"] == "both")


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"case": c}
    if kind == "train":
        x, t, params, off, scale = _rows(c, seed)
        net = surrogate.Mlp(n_in=16)
        net.set_params(params, off, scale, 1.0)
        return s | {"net": net, "x": x, "t": t,
                    "loss": torch.zeros(1, device=_dev())}
    if kind == "batch":
        scenes, xys = [], []
        for q, d in enumerate(_batch_scenes(c)):
            ssq, _, xy = _fields(d, seed * 1000 + q)
            oc, of = _buffers(d)
            scenes.append({"grid": _grid(d), "static_ssq": ssq,
                           "human_xy": xy, "radius": RADIUS,
                           "height": HEIGHT, "out_ssq": oc, "out_sdf": of})
            xys.append(xy)
        return s | {"graph": pc.BatchGraph(scenes), "scenes": scenes,
                    "xy": xys}
    s["grid"] = _grid(c)
    if kind == "static":
        occ, _ = _scene(c, seed)
        return s | {"occ": occ,
                    "ssq": torch.empty(occ.shape, dtype=torch.int32,
                                       device=_dev()),
                    "sdf": torch.empty(occ.shape, device=_dev())}
    ssq, sdf, xy = _fields(c, seed)
    s |= {"ssq": ssq, "sdf": sdf, "xy": xy}
    if kind == "composite":
        s["out"] = _buffers(c)
    elif kind in ("query", "factors"):
        _, s["fields"] = pc.predicted_composite_sdf(
            s["grid"], ssq, xy, RADIUS, HEIGHT, want_ssq=False)
    if kind == "factors":
        m, j = c["states"], c["spheres"]
        centre, rad, _ = _spheres(c, m * j, seed)
        s |= {"centre": centre.view(m, j, 3), "rad": rad[:j].contiguous(),
              "slice": (torch.arange(m, device=_dev()) * c["n"] // m).int()}
    elif kind != "composite":
        s["centre"], s["rad"], s["slice"] = _spheres(c, c["q"], seed)
    if kind == "surrogate":
        w = np.load(WEIGHTS)
        s["net"] = surrogate.Mlp(n_in=16)
        s["net"].set_params(w["params"], w["in_offset"], w["in_scale"],
                            float(w["out_scale"]))
    return s


EPS, SIGMA = 0.2, 0.05  # the hinge's distance (m), the factors' weight


def run(state):
    s = state
    c, kind = s["case"], s["case"]["kind"]
    if kind == "static":
        return pc.build_static_sdf(s["grid"], s["occ"], s["ssq"], s["sdf"])
    if kind == "composite":
        oc, of = s["out"]
        return pc.predicted_composite_sdf(
            s["grid"], s["ssq"], s["xy"], RADIUS, HEIGHT, out_ssq=oc,
            out_sdf=of, want_ssq=oc is not None)
    if kind == "direct":
        return pc.query_spheres_direct(
            s["grid"], s["ssq"], s["xy"], RADIUS, HEIGHT, s["centre"],
            s["rad"], s["slice"], hinge_eps=EPS, want_cost=True)
    if kind == "query":
        return pc.query_spheres(s["grid"], s["fields"], s["centre"],
                                s["rad"], s["slice"], hinge_eps=EPS,
                                want_cost=True)
    if kind == "factors":
        return pc.obstacle_factors(s["grid"], s["fields"], s["centre"],
                                   s["rad"], s["slice"], EPS, SIGMA)
    if kind == "surrogate":
        o = surrogate.query_spheres_surrogate(
            s["net"], s["grid"], s["ssq"], s["sdf"], s["xy"], RADIUS, HEIGHT,
            s["centre"], s["rad"], s["slice"], hinge_eps=EPS, want_cost=True)
        return (o["dist"], o["grad"], o["status"], o["cost"],
                o["used_fallback"])
    if kind == "train":
        return s["net"].loss_gradients(s["x"], s["t"], s["loss"]), s["loss"]
    for q, xy in enumerate(s["xy"]):
        s["graph"].set_positions(q, xy)
    s["graph"].launch()
    return s["graph"].outputs


# -------------------------------------------------------------------- work

def work(case):
    c, kind = case, case["kind"]
    if kind == "train":
        macs = 16 * HID + 3 * HID * HID + HID
        return {"bytes": c["rows"] * 17 * 4 + 2 * 4 * 51_841,
                "flops": 6.0 * macs * c["rows"]}
    if kind == "batch":
        return {"bytes": sum(work(d | {"kind": "composite"})["bytes"]
                             for d in _batch_scenes(c)), "flops": 0}
    v = c["nx"] * c["ny"] * c["nz"]
    if kind == "static":  # the map read, the two fields written
        return {"bytes": 9 * v, "flops": 0}
    if kind == "composite":  # the static field read, the fields written
        per = 8 if c["outputs"] == "both" else 4
        return {"bytes": 4 * v + per * c["n"] * v, "flops": 0}
    if kind == "factors":  # centre, eight corners; error, Jacobian
        return {"bytes": c["states"] * (c["spheres"] * (12 + 32 + 16) + 12),
                "flops": 0}
    # centre, radius, slice, eight corners; distance, gradient, status, cost
    return {"bytes": c["q"] * (20 + 32 + 21), "flops": 0}


# ---------------------------------------------------- the same in 64 bits

def _edt2(sites, axes):
    """Squared distance (fp64, inf without sites) to the True elements, by
    an exhaustive minimum along each axis in turn."""
    f = torch.where(sites, 0.0, math.inf).to(torch.float64)
    for ax in axes:
        n = f.shape[ax]
        at = torch.arange(n, device=f.device, dtype=torch.float64)
        at = at.view([n if d == ax else 1 for d in range(f.dim())])
        out = torch.full_like(f, math.inf)
        for p in range(n):
            torch.minimum(out, f.select(ax, p).unsqueeze(ax) + (at - p) ** 2,
                          out=out)
        f = out
    return f


def _signed2(sites, axes):
    return torch.where(sites, -_edt2(~sites, axes), _edt2(sites, axes))


def _metres(ssq, h):
    return torch.sign(ssq) * h * ssq.abs().sqrt()


def _people_planes(c, xy):
    """Per slice the planar squared distance to the people's discs, to their
    complement, and the discs (bool), [n, ny, nx]; and the top layer."""
    f = 65536.0
    ctr = torch.from_numpy(np.rint(xy / c["h"] * f).astype(np.int64))
    ctr = ctr.to(_dev())
    r2 = int(np.rint(RADIUS / c["h"] * f)) ** 2
    i = 32768 * (2 * torch.arange(c["nx"], device=_dev()) + 1)
    j = 32768 * (2 * torch.arange(c["ny"], device=_dev()) + 1)
    disc = torch.zeros((c["n"], c["ny"], c["nx"]), dtype=torch.bool,
                       device=_dev())
    for p in range(c["k"]):
        dx = i[None, None, :] - ctr[:, p, 0, None, None]
        dy = j[None, :, None] - ctr[:, p, 1, None, None]
        disc |= dx * dx + dy * dy <= r2
    hq = int(np.rint(HEIGHT / c["h"] * f))
    top = min((hq - 32768) // 65536, c["nz"] - 1)
    return _edt2(disc, (2, 1)), _edt2(~disc, (2, 1)), disc, top


def _people_value(c, out, ins, disc, top, k):
    """The people's signed squared distance at layer k (broadcast)."""
    up = (k - top).clamp(min=0).double()
    cap = (top + 1 - k).double() ** 2 if top + 1 < c["nz"] \
        else torch.full_like(up, math.inf)
    return torch.where(disc & (k <= top), -torch.minimum(ins, cap),
                       out + up ** 2)


def _exact_composite(c, seed):
    occ, xy = _scene(c, seed)
    env = _signed2(occ > 0, (2, 1, 0))
    out, ins, disc, top = _people_planes(c, xy)
    k = torch.arange(c["nz"], device=_dev())[:, None, None]
    f = torch.empty((c["n"],) + tuple(env.shape), dtype=torch.float64,
                    device=_dev())
    for s in range(c["n"]):
        f[s] = _metres(torch.minimum(env, _people_value(
            c, out[s], ins[s], disc[s], top, k)), c["h"])
    return f


def _exact_samples(c, seed, centre, sl):
    """Distance and gradient of the trilinear composite at centres [q, 3]."""
    occ, xy = _scene(c, seed)
    env = _signed2(occ > 0, (2, 1, 0))
    out, ins, disc, top = _people_planes(c, xy)
    n = torch.tensor([c["nx"], c["ny"], c["nz"]], device=_dev())
    g = (centre.double() / c["h"] - 0.5).clamp(min=0).minimum(n - 1)
    i = g.floor().long().minimum(n - 2)
    u, sl = g - i, sl.long()
    d = torch.zeros(len(g), dtype=torch.float64, device=_dev())
    grad = torch.zeros_like(g)
    for b in range(8):
        o = [(b >> a) & 1 for a in range(3)]
        x, y, z = (i[:, a] + o[a] for a in range(3))
        f = _metres(torch.minimum(env[z, y, x], _people_value(
            c, out[sl, y, x], ins[sl, y, x], disc[sl, y, x], top, z)),
            c["h"])
        w = [u[:, a] if o[a] else 1 - u[:, a] for a in range(3)]
        d += f * w[0] * w[1] * w[2]
        for a in range(3):
            e = w[(a + 1) % 3] * w[(a + 2) % 3] / c["h"]
            grad[:, a] += f * e * (1 if o[a] else -1)
    return d, grad


def _exact_train(c, seed):
    x, t, params, off, scale = _rows(c, seed)
    p = torch.from_numpy(params).to(_dev()).double()
    dims, layers, at = [16, HID, HID, HID, HID, 1], [], 0
    for a, b in zip(dims, dims[1:]):
        layers.append((p[at:at + a * b].view(b, a),
                       p[at + a * b:at + a * b + b]))
        at += a * b + b
    acts = [(x.double() - torch.from_numpy(off).to(_dev()).double())
            * torch.from_numpy(scale).to(_dev()).double()]
    pre = []
    for l, (w, b) in enumerate(layers):
        z = acts[-1] @ w.T + b
        pre.append(z)
        acts.append(z * torch.sigmoid(z) if l < 4 else z)
    r = acts[-1][:, 0] - t.double()
    dz, got = (2 * r / len(r))[:, None], []
    for l in range(4, -1, -1):
        got = [(dz.T @ acts[l]).reshape(-1), dz.sum(0)] + got
        if l:
            s = torch.sigmoid(pre[l - 1])
            dz = (dz @ layers[l][0]) * s * (1 + pre[l - 1] * (1 - s))
    return torch.cat(got), (r * r).mean().view(1)


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "train":
        return _exact_train(c, seed)
    if kind == "static":
        return None, _metres(_signed2(_scene(c, seed)[0] > 0, (2, 1, 0)),
                             c["h"])
    if kind == "composite":
        return None, _exact_composite(c, seed)
    if kind == "batch":
        return [(None, _exact_composite(d, seed * 1000 + q))
                for q, d in enumerate(_batch_scenes(c))]
    if kind == "factors":
        m, j = c["states"], c["spheres"]
        centre, rad, _ = _spheres(c, m * j, seed)
        sl = torch.arange(m, device=_dev()) * c["n"] // m
        d, g = _exact_samples(c, seed, centre, sl.repeat_interleave(j))
        e = (EPS - (d.view(m, j) - rad[:j].double())).clamp(min=0)
        jac = torch.where((e > 0)[:, :, None], -g.view(m, j, 3), 0.0)
        return e, jac, (0.5 * (e / SIGMA) ** 2).sum(1)
    centre, rad, sl = _spheres(c, c["q"], seed)
    d, g = _exact_samples(c, seed, centre, sl)
    d = d - rad.double()
    got = (d, g, None, (EPS - d).clamp(min=0))
    return got + (None,) if kind == "surrogate" else got
