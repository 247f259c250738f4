"""The workloads this library's performance is judged on.

A user of this library has a voxelised point cloud that it has not seen before, weights that it has, and
runs layers on it: kernel map first, then convolutions, and in training the two gradients.  A pass
is therefore always a whole one, from the coordinates on: the kernel maps are built in it.  Three kinds:

  layer  `layers` 3x3x3 (or 5x5x5) submanifold convolutions with ReLU in between that share one kernel
         map, forward only or with input and weight gradients (one stage of a network)
  pair   a stride-2 convolution C -> 2C and the transposed convolution 2C -> C that pairs with it
  net    an encoder (or encoder-decoder) of residual blocks with stride-2 stages, after the network
         that the library's tests run, built from the public calls

In training a ReLU takes the gradient's way by the sign of a rounded sum: after a dozen 16-bit layers two
correct programs differ in 1 of 1,000 such decisions, and by several per cent in the gradients behind
them.  Nets in training therefore gate their activations with masks drawn beforehand (dropout of one
half, the same call), and layers in training have at most one ReLU, right behind the inputs.

Clouds are synthetic, drawn on the device from the seed: LiDAR-like scans (ground plane and vertical
objects, density falling as 1/r^2), rooms (dense surfaces) and uniform clouds; rows in random order.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2311_12862_amd as sp

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
C_FEAT = 8              # channels of a network's input points
SCAN_MAX = 110_000      # voxels that one scan yields at most


def listed():
    return [
        # the smallest call: 2,000 points, one fp32 layer; launches and host time are all of it
        _layer("tiny_infer_f32", "uniform", 2_000, "f32", 16, 16),
        # one deep, wide stage of a segmentation network on a coarse grid: few rows, long reductions
        _layer("deep_infer_f16_256", "lidar", 9_001, "f16", 256, 256, layers=4),
        # one training step of the layer the headline benchmark is quoted on (build not waited for)
        _layer("lidar_train_f16_64", "lidar", 100_049, "f16", 64, 64, train=True, asynchronous=True),
        # fp32 training of a mid-size stage
        _layer("lidar_train_f32_64", "lidar", 30_011, "f32", 64, 64, layers=2, train=True),
        # the 5x5x5 stem of a segmentation network
        _layer("stem_infer_f16_k5", "lidar", 60_013, "f16", 8, 32, K=5),
        # a dense indoor cloud, bf16 training, at the three widths the library is tested on; the widest
        # on the bitmask-sorted map, as its tuner picks there
        _layer("room_train_bf16_32", "room", 300_000, "bf16", 32, 32, train=True),
        _layer("room_train_bf16_96", "room", 300_000, "bf16", 96, 96, train=True),
        _layer("room_train_bf16_256", "room", 300_000, "bf16", 256, 256, train=True, n_split=1),
        # down- and up-sampling of two scans, inference
        _pair("pair_infer_f16_64", 200_003, 2, "f16", 64),
        # the backbone of a detector on anisotropic voxels: 16/16/32/64 channels, one scan
        _net("detector_infer_f16", "detection", 79_000, 1, "f16", 16, 3, decoder=False),
        # segmentation of one scan, and one training step on four
        _net("unet_infer_f16", "lidar", 100_003, 1, "f16", 32, 4),
        _net("unet_train_f16", "lidar", 400_000, 4, "f16", 32, 4, train=True),
    ]


def _layer(name, scene, voxels, dtype, c_in, c_out, K=3, layers=1, train=False, n_split=0, asynchronous=False):
    return {"name": name, "kind": "layer", "scene": scene, "voxels": voxels, "scans": -(-voxels // SCAN_MAX), "dtype": dtype,
            "c_in": c_in, "c_out": c_out, "K": K, "layers": layers, "train": train, "n_split": n_split,
            "asynchronous": asynchronous}


def _pair(name, voxels, scans, dtype, c, K=3, train=False):
    return {"name": name, "kind": "pair", "scene": "lidar", "voxels": voxels, "scans": scans, "dtype": dtype, "c_in": c,
            "c_out": 2 * c, "K": K, "train": train}


def _net(name, scene, voxels, scans, dtype, base, levels, decoder=True, train=False):
    return {"name": name, "kind": "net", "scene": scene, "voxels": voxels, "scans": scans, "dtype": dtype, "base": base,
            "levels": levels, "decoder": decoder, "train": train}


def draw(rng: random.Random):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def channels(lo, hi, q=8):
        return max(q, size(lo, hi) // q * q)

    kind = rng.choices(["layer", "pair", "net"], [5, 2, 2])[0]
    if kind == "layer":
        dtype = rng.choices(["f16", "bf16", "f32"], [5, 4, 2])[0]
        scene = rng.choices(["lidar", "room", "uniform"], [5, 3, 1])[0]
        lo, hi = {"lidar": (4_000, 220_000), "room": (20_000, 300_000), "uniform": (500, 8_000)}[scene]
        K = 5 if dtype != "f32" and scene != "room" and rng.random() < 0.15 else 3
        c_hi = 96 if dtype == "f32" else 64 if K == 5 else 256
        c_in = channels(8 if K == 5 else 16, c_hi, 4 if dtype == "f32" else 8)
        c_out = c_in if rng.random() < 0.5 else channels(16, c_hi, 4 if dtype == "f32" else 8)
        train = rng.random() < 0.5
        layers = rng.randint(1, 2 if train else 4)
        # no more work than the largest listed case has
        most = (4e9 if dtype == "f32" else 5e10) / (c_in * c_out + (layers - 1) * c_out * c_out) / (3 if train else 1)
        voxels = max(500, min(size(lo, hi), int(most), 120_000 if K == 5 else hi))
        case = _layer("", scene, voxels, dtype, c_in, c_out, K, layers, train,
                      1 if dtype != "f32" and rng.random() < 0.35 else 0, K == 3 and rng.random() < 0.4)
    elif kind == "pair":
        voxels = size(20_000, 220_000)
        case = _pair("", voxels, rng.randint(-(-voxels // SCAN_MAX), 4), rng.choice(["f16", "bf16"]), channels(16, 128),
                     rng.choice([3, 3, 2]), rng.random() < 0.4)
    else:
        voxels = size(20_000, 220_000)
        decoder = rng.random() < 0.7
        case = _net("", "lidar", voxels, rng.randint(-(-voxels // SCAN_MAX), 4), "f16", rng.choice([16, 24, 32]),
                    rng.randint(2, 4), decoder, decoder and rng.random() < 0.5)
    del case["name"]
    return case


# ---- clouds ------------------------------------------------------------------------------------

def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _generator(seed):
    g = torch.Generator(device=_device())
    g.manual_seed(seed)
    return g


def _rand(g, n):
    return torch.rand(n, generator=g, device=g.device)


def _cells(points, cell):
    """floor(p / cell), shifted to start at 0, and one integer per occupied cell for each point."""
    q = torch.floor(points / torch.tensor(cell, device=points.device)).to(torch.int64)
    q -= q.amin(0)
    span = q.amax(0) + 1
    return q, (q[:, 0] * span[1] + q[:, 1]) * span[2] + q[:, 2], span


def _split_cells(flat, span):
    yz = span[1] * span[2]
    return torch.stack([flat // yz, flat % yz // span[2], flat % span[2]], 1)


def _scan(g, seed, cell, limit):
    """One LiDAR-like scan: the first `limit` cells that its points fall into, in that order."""
    rng = random.Random(seed)
    n_ground, n_object, dev = 45_000, 375_000, g.device
    r = torch.exp(math.log(2.0) + _rand(g, n_ground) * math.log(25.0))
    th = _rand(g, n_ground) * (2 * math.pi)
    z = torch.randn(n_ground, generator=g, device=dev) * 0.01
    ground = torch.stack([r * th.cos(), r * th.sin(), z], 1)
    # 40 vertical cylinders and boxes inside the 50 m disc, points in proportion to side area / r^2
    rows = []
    for _ in range(40):
        rad, ang, h = math.sqrt(rng.uniform(9.0, 2500.0)), rng.uniform(0, 2 * math.pi), rng.uniform(1.0, 4.0)
        cr, a, b, box = rng.uniform(0.2, 1.0), rng.uniform(1.0, 5.0), rng.uniform(1.0, 5.0), rng.random() < 0.5
        area = 2 * (a + b) * h if box else 2 * math.pi * cr * h
        rows.append([rad * math.cos(ang), rad * math.sin(ang), h, cr, a, b, float(box), area / rad ** 2])
    t = torch.tensor(rows, device=dev)
    o = t[torch.multinomial(t[:, 7], n_object, replacement=True, generator=g)]
    a, b, u = o[:, 4], o[:, 5], _rand(g, n_object)
    s = u * 2 * (a + b)
    px = torch.where(s < a, s - a / 2, torch.where(s < a + b, a / 2, torch.where(s < 2 * a + b, a * 1.5 + b - s, -a / 2)))
    py = torch.where(s < a, -b / 2, torch.where(s < a + b, s - a - b / 2, torch.where(s < 2 * a + b, b / 2, 2 * a + 1.5 * b - s)))
    box = o[:, 6] > 0.5
    px = torch.where(box, px, o[:, 3] * (u * 2 * math.pi).cos())
    py = torch.where(box, py, o[:, 3] * (u * 2 * math.pi).sin())
    things = torch.stack([o[:, 0] + px, o[:, 1] + py, _rand(g, n_object) * o[:, 2]], 1)
    p = torch.cat([ground, things])
    p = p[torch.randperm(p.shape[0], generator=g, device=dev)]
    _, flat, span = _cells(p, cell)
    u, inv = torch.unique(flat, return_inverse=True)
    first = torch.full((u.shape[0],), p.shape[0], dtype=torch.int64, device=dev)
    first.scatter_reduce_(0, inv, torch.arange(p.shape[0], device=dev), "amin")
    return _split_cells(u[torch.argsort(first)[:limit]], span)


def _room(g, seed, limit):
    """Surfaces of a 10 x 10 x 3 m room with 30 boxes, 2 cm cells, as far as `limit` cells from its middle."""
    rng = random.Random(seed)
    solids = [([0.0, 0.0, 0.0], [10.0, 10.0, 3.0])]
    for _ in range(30):
        size = [rng.uniform(0.3, 2.0) for _ in range(3)]
        solids.append(([rng.uniform(0, 10 - size[0]), rng.uniform(0, 10 - size[1]), 0.0], size))
    faces = []
    for lo, d in solids:
        for ax in range(3):
            a1, a2 = (ax + 1) % 3, (ax + 2) % 3
            u, v = [0.0] * 3, [0.0] * 3
            u[a1], v[a2] = d[a1], d[a2]
            for side in (0.0, d[ax]):
                at = list(lo)
                at[ax] += side
                faces.append(at + u + v + [d[a1] * d[a2]])
    f = torch.tensor(faces, device=g.device)
    n = 6_000_000
    counts = (f[:, 9] / f[:, 9].sum() * n).long()
    pick = torch.repeat_interleave(torch.arange(f.shape[0], device=g.device), counts)
    e = f[pick]
    n = pick.shape[0]
    p = e[:, 0:3] + _rand(g, n)[:, None] * e[:, 3:6] + _rand(g, n)[:, None] * e[:, 6:9]
    _, flat, span = _cells(p, [0.02] * 3)
    q = _split_cells(torch.unique(flat), span)
    r = (((q + 0.5) * 0.02 - torch.tensor([5.0, 5.0, 1.5], device=g.device)) ** 2).sum(1)
    q = q[torch.argsort(r)[:limit]]
    return (q - q.amin(0))[torch.randperm(q.shape[0], generator=g, device=g.device)]


def _cloud(case, seed):
    """int32 [N, 4] rows (batch, x, y, z)."""
    g = _generator(seed)
    n, scene, scans = case["voxels"], case["scene"], case["scans"]
    if scene == "uniform":  # as sparse as 2,000 points in a 64^3 grid
        side = int(round((n * 64 ** 3 / 2000) ** (1 / 3)))
        flat = torch.randperm(side ** 3, generator=g, device=g.device)[:n]
        parts = [_split_cells(flat, torch.tensor([side] * 3, device=g.device))]
    elif scene == "room":
        parts = [_room(g, seed, n)]
    else:
        # 5 cm cells give about 100k voxels a scan; smaller clouds are coarser grids, as the deep
        # levels of a network see them
        cell = [0.1, 0.1, 0.15] if scene == "detection" else [0.05 * math.sqrt(max(1.0, 100_000 * scans / n))] * 3
        parts = [_scan(g, seed * 131 + b, cell, n * (b + 1) // scans - n * b // scans) for b in range(scans)]
    rows = torch.cat([torch.cat([torch.full_like(q[:, :1], b), q], 1) for b, q in enumerate(parts)])
    rows = rows[torch.randperm(rows.shape[0], generator=g, device=g.device)]
    return rows.to(torch.int32).contiguous()


# ---- passes ------------------------------------------------------------------------------------

def _net_layers(case):
    """name -> (K, c_in, c_out) of a net, in the order it runs them."""
    b, depth = case["base"], case["levels"]
    enc = [b] + [b << i for i in range(depth)]
    shapes = {"stem": (3, C_FEAT, enc[0])}

    def block(name, c, d, proj):
        shapes[name + ".c1"], shapes[name + ".c2"] = (3, c, d), (3, d, d)
        if proj:
            shapes[name + ".proj"] = (1, c, d)
    for i in range(1, depth + 1):
        shapes["down%d" % i] = (3, enc[i - 1], enc[i])
        block("e%db1" % i, enc[i], enc[i], False)
        block("e%db2" % i, enc[i], enc[i], False)
    h = enc[depth]
    for l in reversed(range(depth if case["decoder"] else 0)):
        shapes["up%d" % l] = (3, h, enc[l])
        block("d%db1" % l, 2 * enc[l], enc[l], True)
        block("d%db2" % l, enc[l], enc[l], False)
        h = enc[l]
    return shapes


def _level_of(name):
    """Level of a net's layer: that of its outputs."""
    return 0 if name == "stem" else int(name[4:]) if name.startswith("down") else int(name[2:]) if name[0] == "u" else int(name[1])


def _layer_shapes(case):
    if case["kind"] == "net":
        return _net_layers(case)
    K, a, b = case["K"], case["c_in"], case["c_out"]
    if case["kind"] == "pair":
        return {"down": (K, a, b), "up": (K, b, a)}
    return {"conv%d" % i: (K, a if i == 0 else b, b) for i in range(case["layers"])}


def prepare(case, seed):
    g, dt = _generator(seed + 1), DTYPES[case["dtype"]]
    coords = _cloud(case, seed)

    def normal(*shape):
        return torch.randn(*shape, generator=g, device=g.device)
    w = {}
    for name, (K, a, b) in _layer_shapes(case).items():
        # variance-preserving for the handful of neighbours that a voxel has
        fan = {1: a, 2: 2 * a, 3: 8 * a, 5: 12 * a}[K]
        w[name] = (normal(K ** 3, a, b) / math.sqrt(fan)).to(dt)
    c_in = C_FEAT if case["kind"] == "net" else case["c_in"]
    state = {"case": case, "coords": coords, "w": w, "x": normal(coords.shape[0], c_in).to(dt), "built": None}
    if case["train"]:  # the gradient that reaches the output from the loss
        c_out = {"layer": case.get("c_out"), "pair": case.get("c_in"), "net": case.get("base")}[case["kind"]]
        state["g"] = normal(coords.shape[0], c_out).to(dt)
    if case["train"] and case["kind"] == "net":
        n, rows = [], coords
        for _ in range(case["levels"] + 1):
            n.append(rows.shape[0])
            rows = _coarse(rows)
        state["gate"] = {name: normal(n[_level_of(name)], c).to(dt) for name, (_, _, c) in _net_layers(case).items()
                         if not name.endswith((".c2", ".proj"))}
    if case.get("n_split"):
        state["cfg"] = sp.Config(n_split=case["n_split"])
    return state


def run(state):
    return {"layer": _run_layer, "pair": _run_pair, "net": _run_net}[state["case"]["kind"]](state)


def _run_layer(state):
    case, w, cfg = state["case"], state["w"], state.get("cfg")
    if state["built"] is not None:  # an unwaited build: its verdict is read one pass later
        state["built"].status()
    km = sp.build_kmap(state["coords"], case["K"], 1, asynchronous=case["asynchronous"])
    state["built"] = km if case["asynchronous"] else None
    n = case["layers"]
    acts = [state["x"]]
    for i in range(n):
        y = sp.fwd(acts[-1], w["conv%d" % i], km, cfg)
        acts.append(sp.ew(sp.EW_RELU, y) if i + 1 < n else y)
    out = {"y": acts[-1]}
    if case["train"]:
        g = state["g"]
        for i in reversed(range(n)):
            if i + 1 < n:
                g = sp.ew(sp.EW_RELU_BWD, g, acts[i + 1])
            out["dw%d" % i] = sp.wgrad(acts[i], g, km)
            g = sp.dgrad(g, w["conv%d" % i], km, cfg)
        out["dx"] = g
    return out


def _run_pair(state):
    case, w = state["case"], state["w"]
    down = sp.build_kmap(state["coords"], case["K"], 2)
    up = down.transpose()
    pre = sp.fwd(state["x"], w["down"], down)
    h = sp.ew(sp.EW_RELU, pre)
    y = sp.fwd(h, w["up"], up)
    out = {"y": y}
    if case["train"]:
        g = state["g"]
        out["dw_up"] = sp.wgrad(h, g, up)
        g = sp.ew(sp.EW_RELU_BWD, sp.dgrad(g, w["up"], up), h)
        out["dw_down"] = sp.wgrad(state["x"], g, down)
        out["dx"] = sp.dgrad(g, w["down"], down)
    return out


def _concat(a, b):
    out = torch.empty((a.shape[0], a.shape[1] + b.shape[1]), dtype=a.dtype, device=a.device)
    sp.copy_cols(a, 0, out, 0, a.shape[1])
    sp.copy_cols(b, 0, out, a.shape[1], b.shape[1])
    return out


def _parts(d, ca):
    a = torch.empty((d.shape[0], ca), dtype=d.dtype, device=d.device)
    b = torch.empty((d.shape[0], d.shape[1] - ca), dtype=d.dtype, device=d.device)
    sp.copy_cols(d, 0, a, 0, ca)
    sp.copy_cols(d, ca, b, 0, d.shape[1] - ca)
    return a, b


def _run_net(state):
    case, w, gate = state["case"], state["w"], state.get("gate")
    depth, decoder = case["levels"], case["decoder"]
    sub, one, down, up, rows = [], [], [], [], state["coords"]
    for l in range(depth + 1):
        sub.append(sp.build_kmap(rows, 3, 1))
        if l < depth:
            down.append(sp.build_kmap(rows, 3, 2))
            rows = down[l].out_coords()
            if decoder:
                one.append(sub[l].pointwise())
                up.append(down[l].transpose())
    tape = []

    def act(y, name):
        return sp.ew(sp.EW_RELU_BWD, y, gate[name]) if gate else sp.ew(sp.EW_RELU, y)

    def conv_act(name, km, x):
        y = act(sp.fwd(x, w[name], km), name)
        tape.append(("conv", name, km, x))
        return y

    def block(name, km, km1, x):
        h = act(sp.fwd(x, w[name + ".c1"], km), name + ".c1")
        z = sp.fwd(h, w[name + ".c2"], km)
        y = sp.ew(sp.EW_ADD if gate else sp.EW_ADD_RELU, z, sp.fwd(x, w[name + ".proj"], km1) if km1 else x)
        tape.append(("block", name, km, km1, x, h))
        return y

    h = conv_act("stem", sub[0], state["x"])
    enc = [h]
    for i in range(1, depth + 1):
        h = conv_act("down%d" % i, down[i - 1], h)
        h = block("e%db2" % i, sub[i], None, block("e%db1" % i, sub[i], None, h))
        enc.append(h)
    for l in reversed(range(depth if decoder else 0)):
        u = conv_act("up%d" % l, up[l], h)
        tape.append(("concat", l, u.shape[1]))
        h = block("d%db1" % l, sub[l], one[l], _concat(u, enc[l]))
        h = block("d%db2" % l, sub[l], None, h)
    if not case["train"]:
        if not decoder:  # a head takes the coarse level padded to a fixed number of rows
            y = h.new_zeros((case["voxels"], h.shape[1]))
            y[:h.shape[0]] = h
            return {"y": y}
        return {"y": h}

    out, g, skip = {"y": h}, state["g"], {}
    for step in reversed(tape):
        if step[0] == "concat":
            g, skip[step[1]] = _parts(g, step[2])
        elif step[0] == "block":
            _, name, km, km1, x, hid = step
            if name[0] == "e" and name.endswith("b2") and int(name[1]) in skip:
                g = sp.ew(sp.EW_ADD, g, skip.pop(int(name[1])))
            out[name + ".c2"] = sp.wgrad(hid, g, km)
            dh = act(sp.dgrad(g, w[name + ".c2"], km), name + ".c1")
            out[name + ".c1"] = sp.wgrad(x, dh, km)
            dx = sp.dgrad(dh, w[name + ".c1"], km)
            if km1:
                out[name + ".proj"] = sp.wgrad(x, g, km1)
                g = sp.ew(sp.EW_ADD, dx, sp.dgrad(g, w[name + ".proj"], km1))
            else:
                g = sp.ew(sp.EW_ADD, dx, g)
        else:
            _, name, km, x = step
            if name == "stem" and 0 in skip:
                g = sp.ew(sp.EW_ADD, g, skip.pop(0))
            g = act(g, name)
            out[name] = sp.wgrad(x, g, km)
            g = sp.dgrad(g, w[name], km)
    out["dx"] = g
    return out


# ---- what a pass cannot do without -------------------------------------------------------------

def _keys(rows):
    r = rows.to(torch.int64)
    return ((r[:, 0] << 48) | ((r[:, 1] + 4096) << 32) | ((r[:, 2] + 4096) << 16) | (r[:, 3] + 4096))


def _pairs_of(rows, out_rows, K, stride):
    """Present (output, input) pairs of a K^3 convolution with this stride."""
    table = torch.sort(_keys(rows))[0]
    lo = -(K // 2) if K % 2 else 0
    total = 0
    for dx in range(lo, lo + K):
        for dy in range(lo, lo + K):
            for dz in range(lo, lo + K):
                at = out_rows * torch.tensor([1, stride, stride, stride], device=rows.device) + \
                    torch.tensor([0, dx, dy, dz], device=rows.device)
                k = _keys(at)
                i = torch.searchsorted(table, k).clamp_(max=table.shape[0] - 1)
                total += int((table[i] == k).sum())
    return total


def _coarse(rows):
    half = torch.cat([rows[:, :1], torch.div(rows[:, 1:], 2, rounding_mode="floor")], 1)
    return torch.unique(half, dim=0)


def work(case):
    """Coordinates in, and of every layer's calls the features, gradients and weights in and out, once
    each; two operations for each present pair, input and output channel."""
    rows = _cloud(case, 0)
    e = 4 if case["dtype"] == "f32" else 2
    levels, pairs = [rows], {}
    for _ in range({"layer": 0, "pair": 1}.get(case["kind"], case.get("levels"))):
        levels.append(_coarse(levels[-1]))
    n = [r.shape[0] for r in levels]

    def layer(name):  # (rows in, rows out, key of the pair count)
        if case["kind"] == "layer":
            return n[0], n[0], ("sub", 0)
        if case["kind"] == "pair":
            return (n[0], n[1], ("down", 0)) if name == "down" else (n[1], n[0], ("down", 0))
        if name == "stem":
            return n[0], n[0], ("sub", 0)
        if name.startswith("down"):
            l = int(name[4:])
            return n[l - 1], n[l], ("down", l - 1)
        if name.startswith("up"):
            l = int(name[2:])
            return n[l + 1], n[l], ("down", l)
        l = int(name[1])
        return n[l], n[l], ("one" if name.endswith("proj") else "sub", l)

    nbytes, flops = 16.0 * n[0], 0.0
    for name, (K, a, b) in _layer_shapes(case).items():
        n_in, n_out, key = layer(name)
        if key not in pairs:
            what, l = key
            pairs[key] = n[l] if what == "one" else _pairs_of(levels[l], levels[l + 1 if what == "down" else l], K,
                                                              2 if what == "down" else 1)
        io, wb = (n_in * a + n_out * b) * e, K ** 3 * a * b
        nbytes += io + wb * e
        flops += 2.0 * pairs[key] * a * b
        if case["train"]:
            nbytes += 2 * io + wb * e + wb * 4
            flops += 4.0 * pairs[key] * a * b
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """fp32: sums in another order.  16-bit types: roundings of the activations (2^-12, 2^-9 of their
    value each) that fall differently after such sums, through up to 40 layers."""
    return {"rel": {"f32": 1e-5, "f16": 4e-3, "bf16": 1e-2}[case["dtype"]]}
