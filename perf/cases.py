"""The work a user of this library has it do, as cases that can be timed: set partition + DSVT blocks over a frame (or
a batch of frames), attention-style 3D pooling, points to voxel rows, voxel rows to a bird's-eye-view map.

Every case goes through the public entry points the way a serving program calls them: coordinates and features
already on the GPU, weights packed once, maps and output buffers allocated once per frame size, everything enqueued on
the current stream.  Inputs are synthetic frames of the shapes the configurations in `synth` and `bench.py` describe.
"""
import math

import numpy as np
import torch

import paper_2301_06051_amd as dsvt

# channels, heads, MLP width of the supported layer shapes, with the feature type each runs in
SHAPES = {"c64f32": (64, 4, 128, "f32"), "c64": (64, 4, 128, "bf16"), "c128": (128, 8, 256, "bf16"), "c192": (192, 8, 384, "bf16")}


def _stack(name, x, y, z, win, win2, shift2, tau, n, batch, shape, blocks, dist):
    """win2 / shift2 (per axis x and y): what every other block uses; shift2 = -1: every block takes `win` unshifted."""
    return {"name": name, "kind": "stack", "gx": x, "gy": y, "gz": z, "win": win[0], "win_z": win[1], "win2": win2,
            "shift2": shift2, "tau": tau, "n": n, "batch": batch, "shape": shape, "blocks": blocks, "dist": dist}


def listed():
    return [
        # one block of a small fp32 model on a small grid: the smallest call, launches and host time count
        _stack("tiny_f32", 48, 48, 1, (12, 1), 12, -1, 36, 2000, 1, "c64f32", 1, "uniform"),
        # a sparse sweep (a short-range or night frame) through the whole pillar backbone
        _stack("pillar_sparse", 468, 468, 1, (12, 1), 12, 6, 36, 3001, 1, "c192", 4, "radial"),
        # the ordinary pillar frame: 30,000 pillars, four blocks, the benchmark's own size
        _stack("pillar_frame", 468, 468, 1, (12, 1), 12, 6, 36, 30000, 1, "c192", 4, "radial"),
        # a dense sweep with window sizes alternating between blocks
        _stack("pillar_hybrid", 468, 468, 1, (12, 1), 24, 12, 36, 41237, 1, "c192", 4, "radial"),
        # four pillar frames served in one call
        _stack("pillar_batch4", 468, 468, 1, (12, 1), 12, 6, 36, 26999, 4, "c192", 4, "radial"),
        # the wide-window pillar model: 30 x 30 windows, sets of 90, 128 channels
        _stack("pillar_wide", 360, 360, 1, (30, 1), 30, 15, 90, 20000, 1, "c128", 4, "radial"),
        # the 3D voxel frame
        _stack("voxel_frame", 468, 468, 32, (12, 8), 12, 6, 48, 120000, 1, "c192", 2, "radial"),
        # the largest: four frames whose voxels crowd into few tall windows
        _stack("skewed_batch", 468, 468, 32, (12, 32), 12, 6, 36, 200000, 4, "c192", 4, "skewed"),
        # pooling between the voxel backbone's stages
        {"name": "pool_voxel", "kind": "pool", "gx": 468, "gy": 468, "gz": 32, "px": 1, "py": 1, "pz": 4, "n": 120000, "batch": 1,
         "shape": "c192", "mask_empty": 1},
        # pooling of a small frame, empty cells kept as keys
        {"name": "pool_small", "kind": "pool", "gx": 360, "gy": 360, "gz": 8, "px": 2, "py": 2, "pz": 2, "n": 9973, "batch": 1,
         "shape": "c128", "mask_empty": 0},
        # the backbone's output laid out for the 2D network
        {"name": "bev_pillar", "kind": "bev", "gx": 468, "gy": 468, "n": 30000, "batch": 1, "shape": "c192"},
        # a LiDAR sweep turned into pillar rows
        {"name": "vfe_pillar", "kind": "vfe", "gx": 468, "gy": 468, "gz": 1, "n": 180000, "f_in": 5, "batch": 1, "shape": "c192"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["stack"] * 6 + ["pool", "pool", "bev", "vfe"])
    if kind == "stack":
        form = rng.choice(["pillar", "pillar", "pillar", "wide", "voxel", "small"])
        batch = rng.choice([1, 1, 2, 4])
        if form == "small":
            g, w = rng.randint(40, 120), rng.randint(8, 16)
            return _stack_drawn(g, g + rng.randint(0, 9), 1, (w, 1), w, rng.choice([-1, w // 2]), rng.choice([24, 36, 48]),
                                _log(rng, 300, 3000 if g > 80 else 700), 1, rng.choice(sorted(SHAPES)), 1, "uniform")
        if form == "voxel":
            wz = rng.choice([8, 32])
            return _stack_drawn(468, 468, 32, (12, wz), 12, 6, rng.choice([36, 48]), _log(rng, 20000, 200000 if batch < 4 else 100000),
                                batch, "c192", rng.choice([1, 2, 4]), rng.choice(["radial", "radial", "skewed"]))
        n = _log(rng, 1500, 50000)
        if form == "wide":
            return _stack_drawn(360, 360, 1, (30, 1), 30, 15, rng.choice([60, 90]), min(n, 30000), batch, "c128", rng.choice([2, 4]), "radial")
        win2 = rng.choice([12, 12, 24])
        return _stack_drawn(468, 468, 1, (12, 1), win2, win2 // 2, rng.choice([36, 36, 48]), n, batch, rng.choice(["c192", "c192", "c128"]),
                            rng.choice([2, 4]), "radial")
    if kind == "pool":
        px, py, pz = rng.choice([(1, 1, 4), (1, 1, 4), (1, 1, 2), (2, 2, 2), (2, 2, 1)])
        return {"kind": "pool", "gx": 468, "gy": 468, "gz": rng.choice([8, 32]), "px": px, "py": py, "pz": pz, "n": _log(rng, 3000, 150000),
                "batch": rng.choice([1, 1, 2]), "shape": rng.choice(["c192", "c192", "c128", "c64f32"]), "mask_empty": rng.choice([0, 1])}
    if kind == "bev":
        return {"kind": "bev", "gx": rng.choice([360, 468]), "gy": rng.choice([360, 468]), "n": _log(rng, 2000, 50000),
                "batch": rng.choice([1, 2, 4]), "shape": rng.choice(["c192", "c192", "c128", "c64f32"])}
    return {"kind": "vfe", "gx": 468, "gy": 468, "gz": rng.choice([1, 1, 32]), "n": _log(rng, 20000, 400000), "f_in": rng.choice([4, 5, 5]),
            "batch": rng.choice([1, 1, 2]), "shape": rng.choice(["c192", "c192", "c128", "c64f32"])}


def _stack_drawn(*args):
    c = _stack("", *args)
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _cells(g, m, grid, dist, hot, win):
    """m candidate cells: `uniform` over the grid; `radial`: 80 % with an area density ~ 1/r around the sensor, 20 %
    clutter, heights near the ground; `skewed`: 70 % in the `hot` windows, the rest uniform."""
    X, Y, Z = grid
    u = lambda: torch.rand(m, generator=g, device="cuda", dtype=torch.float64)
    x, y, z = (u() * X).long(), (u() * Y).long(), (u() * Z).long()
    if dist == "radial":
        r, th, near = 2.0 + u() * (min(X, Y) / 2.0 - 2.0), u() * (2.0 * math.pi), u() < 0.8
        x = torch.where(near, torch.floor(X / 2.0 + r * torch.cos(th)).long(), x)
        y = torch.where(near, torch.floor(Y / 2.0 + r * torch.sin(th)).long(), y)
        zg = torch.round(5.0 + 3.0 * torch.randn(m, generator=g, device="cuda", dtype=torch.float64)).clamp(0, min(12, Z) - 1).long()
        z = torch.where(u() < 0.9, zg, z)
    elif dist == "skewed":
        nwy = -(-Y // win[0])
        nwz = -(-Z // win[1])
        w = hot[(u() * len(hot)).long()]
        pick = u() < 0.7
        x = torch.where(pick, torch.div(w, nwy * nwz, rounding_mode="floor") * win[0] + (u() * win[0]).long(), x)
        y = torch.where(pick, torch.div(w, nwz, rounding_mode="floor") % nwy * win[0] + (u() * win[0]).long(), y)
        z = torch.where(pick, w % nwz * win[1] + (u() * win[1]).long(), z)
    ok = (x >= 0) & (x < X) & (y >= 0) & (y < Y) & (z >= 0) & (z < Z)
    return ((x * Y + y) * Z + z)[ok]


def _frames(g, n, batch, grid, dist="radial", win=(12, 1)):
    """int32 [batch * n, 4] rows (b, x, y, z), unique per frame, in random order inside a frame."""
    X, Y, Z = grid
    assert n <= 0.9 * X * Y * Z
    out = []
    for b in range(batch):
        nw = -(-X // win[0]) * -(-Y // win[0]) * -(-Z // win[1])
        hot = torch.randperm(nw, generator=g, device="cuda")[: max(1, nw // 20)]
        seen = torch.empty(0, dtype=torch.int64, device="cuda")
        while len(seen) < n:
            seen = torch.unique(torch.cat([seen, _cells(g, 2 * n, grid, dist, hot, win)]))
        lin = seen[torch.randperm(len(seen), generator=g, device="cuda")[:n]]
        out.append(torch.stack([torch.full_like(lin, b), torch.div(lin, Y * Z, rounding_mode="floor"),
                                torch.div(lin, Z, rounding_mode="floor") % Y, lin % Z], 1))
    return torch.cat(out).to(torch.int32).contiguous()


def _features(g, n, C, dtype):
    return torch.randn((n, C), generator=g, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)


def _matrix(rng, o, i):
    a = math.sqrt(6.0 / (i + o))
    return ((2.0 * a) * rng.random((o, i), dtype=np.float32) - np.float32(a)).astype(np.float32)


def _vector(rng, n, centre=0.0):
    return (centre + 0.2 * rng.random(n, dtype=np.float32) - 0.1).astype(np.float32)


def _layer(rng, shape, win):
    C, heads, hid, dtype = SHAPES[shape]
    w = dict(C=C, heads=heads, hidden=hid, dtype=dtype, win=win, ln_eps=1e-5)
    for k, o, i in (("qkv", 3 * C, C), ("o", C, C), ("1", hid, C), ("2", C, hid)):
        w["w_" + k], w["b_" + k] = _matrix(rng, o, i), _vector(rng, o)
    for k in ("ln1", "ln2"):
        w[k + "_g"], w[k + "_b"] = _vector(rng, C, 1.0), _vector(rng, C)
    size = (2 * win[0] - 1) * (2 * win[1] - 1) * (2 * win[2] - 1)
    w["rel_bias"] = np.float32(0.02) * rng.standard_normal((heads, size), dtype=np.float32)
    return dsvt.LayerWeights(w)


def prepare(case, seed):
    g, rng = _generator(seed), np.random.Generator(np.random.Philox(seed))
    return {"stack": _prepare_stack, "pool": _prepare_pool, "bev": _prepare_bev, "vfe": _prepare_vfe}[case["kind"]](case, g, rng)


def _prepare_stack(c, g, rng):
    C, _, _, dtype = SHAPES[c["shape"]]
    grid = (c["gx"], c["gy"], c["gz"])
    coords = _frames(g, c["n"], c["batch"], grid, c["dist"], (c["win"], c["win_z"]))
    kinds = [((c["win"], c["win"], c["win_z"]), (0, 0, 0))]
    if c["shift2"] >= 0:
        kinds.append(((c["win2"], c["win2"], c["win_z"]), (c["shift2"], c["shift2"], 0)))
    cfgs = [dsvt.part_cfg(grid, w, s, c["tau"], c["batch"], 0) for w, s in kinds]
    layers = [[_layer(rng, c["shape"], kinds[b % len(kinds)][0]) for _ in (0, 1)] for b in range(c["blocks"])]
    x = _features(g, len(coords), C, dtype)
    ws = torch.empty(max(1, dsvt.dsvt_block_workspace_size(layers[0][0], len(coords))), dtype=torch.uint8, device="cuda")
    return dict(kind="stack", cfgs=cfgs, coords=coords, x=x, out=torch.empty_like(x), layers=layers, ws=ws,
                maps=[dsvt.SetMapsXY(p, len(coords)) for p in cfgs])


def _prepare_pool(c, g, rng):
    C, heads, _, dtype = SHAPES[c["shape"]]
    grid = (c["gx"], c["gy"], c["gz"])
    coords = _frames(g, c["n"], c["batch"], grid)
    w = dict(C=C, heads=heads, dtype=dtype, ln_eps=1e-5, ln_g=_vector(rng, C, 1.0), ln_b=_vector(rng, C))
    for k in "qkvo":
        w["w_" + k], w["b_" + k] = _matrix(rng, C, C), _vector(rng, C)
    pool = dsvt.PoolWeights(w, grid, (c["px"], c["py"], c["pz"]), c["batch"], c["mask_empty"])
    x = _features(g, len(coords), C, dtype)
    one = lambda: torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(max(1, dsvt.dsvt_attn_pool_workspace_size(pool, len(coords))), dtype=torch.uint8, device="cuda")
    return dict(kind="pool", pool=pool, coords=coords, x=x, out=(torch.zeros_like(coords), torch.zeros_like(x), one(), one()), ws=ws)


def _prepare_bev(c, g, rng):
    C, _, _, dtype = SHAPES[c["shape"]]
    grid = (c["gx"], c["gy"], 1)
    coords = _frames(g, c["n"], c["batch"], grid)
    x = _features(g, len(coords), C, dtype)
    return dict(kind="bev", coords=coords, x=x, batch=c["batch"], grid=grid,
                out=torch.empty((c["batch"], *grid, C), dtype=x.dtype, device="cuda"))


def _prepare_vfe(c, g, rng):
    """Points in 600 blobs (objects, ground patches) at uniform range plus a thin 1/r background reaching a little
    beyond the grid, x, y, z in metres and attributes in [0, 1)."""
    C, _, _, dtype = SHAPES[c["shape"]]
    n, R = c["n"], 74.88
    u = lambda *s: torch.rand(*s, generator=g, device="cuda")
    cr, ca, pick, blob = u(600) * R, u(600) * (2.0 * math.pi), (u(n) * 600).long().clamp(max=599), u(n) < 0.95
    r, a = u(n) * (1.07 * R), u(n) * (2.0 * math.pi)
    jit = 0.45 * torch.randn((2, n), generator=g, device="cuda")
    pts = u(n, c["f_in"])
    pts[:, 0] = torch.where(blob, (cr * torch.cos(ca))[pick] + jit[0], r * torch.cos(a))
    pts[:, 1] = torch.where(blob, (cr * torch.sin(ca))[pick] + jit[1], r * torch.sin(a))
    pts[:, 2] = -2.0 + 6.0 * (0.25 + 0.2 * torch.randn(n, generator=g, device="cuda")).abs()
    frame = torch.randint(0, c["batch"], (n,), generator=g, device="cuda", dtype=torch.int32) if c["batch"] > 1 else None
    w = torch.as_tensor(_matrix(rng, C, c["f_in"])).cuda()
    b = torch.as_tensor(_vector(rng, C)).cuda()
    vfe = dsvt.Vfe((c["gx"], c["gy"], c["gz"]), c["batch"], (-R, -R, -2.0), (2 * R / c["gx"], 2 * R / c["gy"], 6.0 / c["gz"]), c["f_in"], C, dtype,
                   n, n, w, b, True)
    vfe.x.zero_()                                    # the rows past the voxels found are not written
    vfe.coords.zero_()
    return dict(kind="vfe", vfe=vfe, points=pts, frame=frame)


# ------------------------------------------------------------------------------------------------ one pass
def run(s):
    if s["kind"] == "stack":
        dsvt.dsvt_partition_xy_multi(s["cfgs"], s["coords"], s["maps"])
        src = s["x"]
        for b, pair in enumerate(s["layers"]):
            src = dsvt.dsvt_block(pair, s["maps"][b % len(s["maps"])], s["coords"], src, x_out=s["out"], ws=s["ws"])
        return {"x": src, "maps": [[(m.set_inds, m.voxel_slot) for m in pair] + [pair.x.n_sets, pair.x.set_win, pair.x.status]
                                   for pair in s["maps"]]}
    if s["kind"] == "pool":
        return dsvt.dsvt_attn_pool(s["pool"], s["coords"], s["x"], out=s["out"], ws=s["ws"])
    if s["kind"] == "bev":
        return dsvt.dsvt_bev_scatter(s["coords"], s["x"], s["batch"], s["grid"], out=s["out"])
    v = dsvt.dsvt_vfe(s["vfe"], s["points"], s["frame"])
    return v.coords, v.x, v.n_voxels, v.status


def work(c):
    C, heads, hid, dtype = SHAPES[c["shape"]]
    es = 2 if dtype == "bf16" else 4
    N = c["n"] * c["batch"]
    if c["kind"] == "stack":
        # the frame's coordinates and rows in, rows and maps (about two slots per voxel in sets, one slot per voxel) out,
        # every layer's weights once; a layer's four projections and the products of every query with the keys of its
        # set (sets are about half full of distinct voxels)
        kinds, layers = (2 if c["shift2"] >= 0 else 1), 2 * c["blocks"]
        weights = (4 * C * C + 2 * C * hid) * es
        return {"bytes": N * (16 + 2 * C * es + kinds * 2 * 12) + layers * weights,
                "flops": layers * N * (2 * (4 * C * C + 2 * C * hid) + 4 * C * c["tau"] // 2)}
    if c["kind"] == "pool":
        # about two occupied cells in a region of several
        M = N / max(1.0, min(2.0, c["px"] * c["py"] * c["pz"] / 2.0))
        return {"bytes": (N + M) * (16 + C * es) + 4 * C * C * es, "flops": 2 * C * C * (2 * N + 2 * M)}
    if c["kind"] == "bev":
        return {"bytes": c["batch"] * c["gx"] * c["gy"] * C * es + N * (16 + C * es), "flops": 0}
    N = c["n"]
    V = 0.2 * N                                      # about five points in a voxel that holds any
    return {"bytes": N * c["f_in"] * 4 + V * (16 + C * es), "flops": 2 * N * c["f_in"] * C}


def tolerance(c):
    dtype = SHAPES[c["shape"]][3]
    if c["kind"] == "bev":
        return "exact"                               # rows are moved, not computed
    if dtype == "f32":
        return {"rel": 1e-5}                         # 32-bit sums, nothing stored in fewer bits on the way
    # bf16 rows (half a unit in the last place is 2^-9) through up to eight layers, each rounding its rows, its
    # queries, keys, values, probabilities and hidden values; integers (maps, coordinates, counts) are the same
    return {"rel": 1e-2, "max": 0.1}
