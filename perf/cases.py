"""Performance cases of the sparse-convolution path: the layers that a point-cloud network runs, from
the first layer on a couple of thousand voxels to a 10^6-voxel, 128-channel one.

A case is a dict of plain values:

  op       "layer"  one layer: location table, kernel map, convolution (strided layers need no table)
           "stage"  two submanifold layers that share one table and one map, then the strided layer
                    that leads to the next resolution
           "up"     an up-sampling layer over the map that the encoder's strided layer left behind
  table    "hash"   hash table, built anew for every pass (a layer); "dense": dense array and kernel
           map; "fused": dense array, look-ups inside the convolution; "none": strided layers;
           "transposed" / "direct": the two forms of an up-sampling layer
  weights  "packed" once beforehand, as inference does, or "raw", as where they change between calls
  scene    voxel sets shaped like the package's own synthetic ones: "lidar" (surfaces seen by a
           rotating sensor, 5 cm cells), "indoor" (dense surfaces, 2 cm cells), "uniform" (random cells)
  n        voxels: scenes are generated one after the other (batch index 0, 1, ...) until there are n

Inputs are made on the GPU from the seed alone, features ~ N(0, 1), weights ~ N(0, 1/sqrt(K^3 C_in)).
"""
from __future__ import annotations

import functools
import math

import torch

from paper_2402_07710_amd import binding as sc
from paper_2402_07710_amd import synth

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
DEVICE = "cuda:0"
LIDAR_BOX, INDOOR_BOX = (1408, 1600, 41), (512, 512, 512)


def _layer(name, scene, n, K, stride, c_in, c_out, dtype, *, sweeps=1, table="hash", weights="packed", out=None):
    return {"name": name, "op": "layer", "scene": scene, "sweeps": sweeps, "n": n, "K": K, "stride": stride, "c_in": c_in,
            "c_out": c_out, "dtype": dtype, "out": out or dtype, "table": table, "weights": weights}


def listed():
    return [
        # a small cloud in single precision: launches and latency are all there is
        _layer("small f32 16-16", "uniform", 2000, 3, 1, 16, 16, "f32"),
        # the standard early layer of an outdoor network, one sensor revolution per frame
        _layer("sweep f16 32-32", "lidar", 53373, 3, 1, 32, 32, "f16"),
        # the same layer over the dense location table, no kernel map (a single layer per resolution)
        _layer("sweep f16 32-32 fused", "lidar", 53373, 3, 1, 32, 32, "f16", table="fused", weights="raw"),
        # the down-sampling layer of most encoders: 3x3x3, stride 2
        _layer("down k3s2 f16 32-64", "lidar", 53373, 3, 2, 32, 64, "f16", table="none"),
        # an encoder stage as a network runs it: two layers on one map, then 2x2x2 down-sampling
        {"name": "stage f16 32-32-64", "op": "stage", "scene": "lidar", "sweeps": 1, "n": 53373, "K": 2, "stride": 2,
         "c_in": 32, "c_out": 64, "dtype": "f16", "out": "f16", "table": "hash", "weights": "packed"},
        # the decoder's layer back to the fine voxels: transpose the encoder's map, convolve
        {"name": "up k2s2 f16 64-32", "op": "up", "scene": "lidar", "sweeps": 1, "n": 53373, "K": 2, "stride": 2,
         "c_in": 64, "c_out": 32, "dtype": "f16", "out": "f16", "table": "transposed", "weights": "raw"},
        # several accumulated sweeps, the middle of the network
        _layer("sweeps f16 64-64", "lidar", 110545, 3, 1, 64, 64, "f16", sweeps=3),
        # four scenes in one batch
        _layer("batch4 bf16 64-64", "lidar", 261574, 3, 1, 64, 64, "bf16"),
        # dense indoor surfaces, the largest layer
        _layer("indoor f16 128-128", "indoor", 1000000, 3, 1, 128, 128, "f16"),
        # the same middle layer for who needs single precision throughout
        _layer("sweep f32 64-64", "lidar", 53373, 3, 1, 64, 64, "f32", weights="raw"),
        # deep in the network: few voxels left, many channels
        _layer("deep f16 256-256", "lidar", 14001, 3, 1, 256, 256, "f16"),
        # a larger receptive field: 5x5x5
        _layer("sweep k5 bf16 32-32", "lidar", 53373, 5, 1, 32, 32, "bf16"),
    ]


def _between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: a family of layers, then sizes spread over the logarithm of its range."""
    kind = rng.choice(["small", "early", "early", "middle", "middle", "large", "single", "deep", "k5", "down", "down", "stage", "up"])
    half = rng.choice(["f16", "bf16"])
    weights = rng.choice(["packed", "raw"])
    if kind == "small":
        c = rng.choice([(4, 16), (16, 16), (16, 32), (32, 32)])
        return _unnamed(_layer("", "uniform", _between(rng, 300, 8000), 3, 1, *c, "f32", weights=weights))
    if kind == "early":
        table = rng.choice(["hash", "hash", "dense", "fused"])
        c = rng.choice([(32, 32), (32, 64)])
        return _unnamed(_layer("", "lidar", _between(rng, 2000, 200000), 3, 1, *c, half, table=table,
                               weights="raw" if table == "fused" else weights, out=rng.choice([half, half, "f32"])))
    if kind == "middle":
        table = rng.choice(["hash", "hash", "dense", "fused"])
        c = rng.choice([(64, 64), (64, 64), (64, 128), (128, 128)])
        return _unnamed(_layer("", "lidar", _between(rng, 2000, 260000), 3, 1, *c, half, sweeps=rng.choice([1, 3]), table=table,
                               weights="raw" if table == "fused" else weights))
    if kind == "large":
        c = rng.choice([(64, 64), (128, 128)])
        return _unnamed(_layer("", "indoor", _between(rng, 200000, 1000000), 3, 1, *c, half, weights=weights))
    if kind == "single":
        c = rng.choice([(4, 32), (16, 32), (32, 32), (32, 64), (64, 64)])
        return _unnamed(_layer("", "lidar", _between(rng, 3000, 80000), 3, 1, *c, "f32", weights=weights))
    if kind == "deep":
        c = rng.choice([(128, 256), (256, 256), (256, 128)])
        return _unnamed(_layer("", "lidar", _between(rng, 500, 16000), 3, 1, *c, half, weights=weights))
    if kind == "k5":
        c = rng.choice([(32, 32), (32, 64), (64, 64)])
        return _unnamed(_layer("", "lidar", _between(rng, 2000, 60000), 5, 1, *c, half, weights=weights))
    if kind == "down":
        K, stride = rng.choice([(3, 2), (3, 2), (2, 2)])
        c = rng.choice([(32, 32), (32, 64), (64, 64), (64, 128)])
        return _unnamed(_layer("", "lidar", _between(rng, 2000, 200000), K, stride, *c, half, table="none", weights=weights))
    if kind == "stage":
        c_in, c_out = rng.choice([(32, 64), (64, 128)])
        return {"op": "stage", "scene": "lidar", "sweeps": 1, "n": _between(rng, 2000, 130000), "K": 2, "stride": 2, "c_in": c_in,
                "c_out": c_out, "dtype": half, "out": half, "table": "hash", "weights": weights}
    table = rng.choice(["transposed", "direct"])
    c_in, c_out = rng.choice([(64, 32), (64, 64), (128, 64)])
    return {"op": "up", "scene": "lidar", "sweeps": 1, "n": _between(rng, 2000, 260000), "K": 2, "stride": 2, "c_in": c_in,
            "c_out": c_out, "dtype": half, "out": half, "table": table, "weights": "raw"}


def _unnamed(case):
    del case["name"]
    return case


# ---- voxel sets (the recipes of the package's synth module, on the GPU) ---------------------------
def _first_occurrences(cells, box):
    """Distinct rows of integer cells [m, 3] inside the box, in the order of their first occurrence."""
    limit = torch.tensor(box, device=cells.device)
    cells = cells[((cells >= 0) & (cells < limit)).all(dim=1)]
    key = (cells[:, 0] * box[1] + cells[:, 1]) * box[2] + cells[:, 2]
    key, order = torch.sort(key, stable=True)
    first = torch.ones_like(key, dtype=torch.bool)
    first[1:] = key[1:] != key[:-1]
    return cells[torch.sort(order[first]).values]


def _lidar(gen, sweeps):
    """Ground plane and boxes seen by a 64 x 2048 ray sweep (sensor moved 1 m per further sweep)."""
    dev = gen.device
    u = lambda lo, hi, *size: lo + (hi - lo) * torch.rand(size, generator=gen, device=dev, dtype=torch.float64)  # noqa: E731
    nb = synth.LIDAR_BOXES
    r, ang = u(5.0, 60.0, nb), u(0.0, 2 * math.pi, nb)
    cx, cy, sx, sy, h = r * torch.cos(ang), r * torch.sin(ang), u(1.5, 6.0, nb), u(1.5, 6.0, nb), u(1.0, 3.0, nb)
    floor = torch.full_like(cx, -synth.LIDAR_HEIGHT)
    lo = torch.stack([cx - sx / 2, cy - sy / 2, floor], dim=1)
    hi = torch.stack([cx + sx / 2, cy + sy / 2, floor + h], dim=1)
    elev = torch.deg2rad(torch.linspace(*synth.LIDAR_ELEV_DEG, synth.LIDAR_RINGS, device=dev, dtype=torch.float64))[:, None]
    azim = (torch.arange(synth.LIDAR_AZIMUTHS, device=dev, dtype=torch.float64) * (2 * math.pi / synth.LIDAR_AZIMUTHS))[None, :]
    d = torch.stack([torch.cos(elev) * torch.cos(azim), torch.cos(elev) * torch.sin(azim), torch.sin(elev).expand(-1, azim.shape[1])],
                    dim=-1).reshape(-1, 3)
    points = []
    for s in range(sweeps):
        o = torch.tensor([1.0 * s, 0.0, 0.0], device=dev, dtype=torch.float64)
        inf = torch.full((len(d),), math.inf, device=dev, dtype=torch.float64)
        t = torch.where(d[:, 2] < -1e-9, -synth.LIDAR_HEIGHT / d[:, 2], inf)
        t0, t1 = (lo[None] - o) / d[:, None], (hi[None] - o) / d[:, None]
        near, far = torch.minimum(t0, t1).amax(dim=2), torch.maximum(t0, t1).amin(dim=2)
        t = torch.minimum(t, torch.where((near <= far) & (near > 0), near, inf[:, None]).amin(dim=1))
        t_noisy = t + synth.LIDAR_NOISE * torch.randn(len(t), generator=gen, device=dev, dtype=torch.float64)
        keep = (t >= synth.LIDAR_RANGE[0]) & (t <= synth.LIDAR_RANGE[1])
        points.append(o + d[keep] * t_noisy[keep, None])
    origin = torch.tensor([-LIDAR_BOX[0] * synth.LIDAR_VOXEL / 2, -LIDAR_BOX[1] * synth.LIDAR_VOXEL / 2, synth.LIDAR_Z0],
                          device=dev, dtype=torch.float64)
    return _first_occurrences(torch.floor((torch.cat(points) - origin) / synth.LIDAR_VOXEL).long(), LIDAR_BOX)


def _indoor(gen):
    """Random right triangles and spheres, sampled on a 1 cm lattice, surface by surface."""
    dev = gen.device
    u = lambda lo, hi, *size: lo + (hi - lo) * torch.rand(size, generator=gen, device=dev, dtype=torch.float64)  # noqa: E731
    ext, step = synth.INDOOR_GRID * synth.INDOOR_VOXEL, synth.INDOOR_SAMPLE
    nt, ns = synth.INDOOR_TRIANGLES, synth.INDOOR_SPHERES
    p0 = u(0.0, ext, nt, 3)
    a, b = (torch.randn((nt, 3), generator=gen, device=dev, dtype=torch.float64) for _ in range(2))
    a = a / a.norm(dim=1, keepdim=True)
    b = torch.linalg.cross(a, b)
    b = b / b.norm(dim=1, keepdim=True)
    na, nb = (torch.floor(u(*synth.INDOOR_TRI_LEG, nt) / step) + 1 for _ in range(2))
    i = torch.arange(int(synth.INDOOR_TRI_LEG[1] / step) + 1, device=dev, dtype=torch.float64)
    inside = i[None, :, None] / (na - 1)[:, None, None] + i[None, None, :] / (nb - 1)[:, None, None] <= 1.0
    t, v, w = inside.nonzero(as_tuple=True)
    triangles = p0[t] + (v * step)[:, None] * a[t] + (w * step)[:, None] * b[t]
    c, r = u(0.0, ext, ns, 3), u(*synth.INDOOR_SPHERE_R, ns)
    n_lat = torch.floor(math.pi * r / step) + 1
    lat = torch.arange(int(math.pi * synth.INDOOR_SPHERE_R[1] / step) + 1, device=dev, dtype=torch.float64)
    theta = lat[None, :] * math.pi / (n_lat - 1)[:, None]
    n_lon = torch.where(lat[None, :] < n_lat[:, None], torch.clamp(torch.floor(2 * math.pi * r[:, None] * torch.sin(theta) / step), min=1.0), 0.0)
    lon = torch.arange(int(2 * math.pi * synth.INDOOR_SPHERE_R[1] / step) + 1, device=dev, dtype=torch.float64)
    s, j, m = (lon[None, None, :] < n_lon[:, :, None]).nonzero(as_tuple=True)
    th, ph = theta[s, j], m * (2 * math.pi) / n_lon[s, j]
    spheres = c[s] + r[s, None] * torch.stack([torch.sin(th) * torch.cos(ph), torch.sin(th) * torch.sin(ph), torch.cos(th)], dim=1)
    return _first_occurrences(torch.floor(torch.cat([triangles, spheres]) / synth.INDOOR_VOXEL).long(), INDOOR_BOX)


def _uniform(gen, n):
    """n distinct random cells of a cube, as dense as 2,000 in 64^3, in random order."""
    side = max(4, round(64 * (n / 2000) ** (1 / 3)))
    lin = torch.randperm(side ** 3, generator=gen, device=gen.device)[:n]
    return torch.stack([lin // (side * side), lin // side % side, lin % side], dim=1)


def _coords(case, seed, device):
    gen = torch.Generator(device=device)
    gen.manual_seed(seed)
    n, scenes, have = case["n"], [], 0
    while have < n:
        xyz = {"lidar": lambda: _lidar(gen, case["sweeps"]), "indoor": lambda: _indoor(gen),
               "uniform": lambda: _uniform(gen, n)}[case["scene"]]()[: n - have]
        scenes.append(torch.cat([torch.full_like(xyz[:, :1], len(scenes)), xyz], dim=1))
        have += len(xyz)
    return torch.cat(scenes).to(torch.int32).contiguous(), len(scenes)


def _features(n, c, dtype, seed, device):
    gen = torch.Generator(device=device)
    gen.manual_seed(seed + 1_000_003)
    return torch.randn((n, c), generator=gen, device=device).to(DTYPES[dtype])


def _weights(k3, c_in, c_out, dtype, seed, device):
    gen = torch.Generator(device=device)
    gen.manual_seed(seed + 2_000_003)
    return (torch.randn((k3, c_in, c_out), generator=gen, device=device) / math.sqrt(k3 * c_in)).to(DTYPES[dtype])


# ---- what a program holds before the call, and the call ---------------------------------------------
def _buffers(n, K, stride, mode, c_in, c_out, dtype, out, dims=None):
    """A layer's buffers.  Rows past the last output row are never written: they are zero here."""
    buf = sc.LayerBuffers(n, K, stride, mode, c_in, c_out, dtype, out, device=DEVICE, grid_dims=dims)
    buf.feat_out.zero_()
    if buf.out_coords is not None:
        buf.out_coords.zero_()
    return buf


def prepare(case, seed):
    coords, scenes = _coords(case, seed, DEVICE)
    n, K, stride, c_in, c_out, dtype = case["n"], case["K"], case["stride"], case["c_in"], case["c_out"], case["dtype"]
    state = {"case": case, "coords": coords}
    if case["op"] == "up":
        # the encoder's strided map; its coarse rows carry the features that go up
        down = _buffers(n, K, stride, "strided", 32, 32, dtype, dtype)
        down.kmap_build(coords, standalone=True)
        coarse = int(down.read_counts().n_out)
        state.update(down=down, feat=_features(coarse, c_in, dtype, seed, DEVICE), w=_weights(K ** 3, c_in, c_out, dtype, seed, DEVICE),
                     out=torch.zeros((n, c_out), dtype=DTYPES[case["out"]], device=DEVICE))
        if case["table"] == "transposed":
            state["kmap_inv"] = torch.empty(sc.sc_kmap_bytes(n, K, stride, "inverse"), dtype=torch.uint8, device=DEVICE)
            state["workspace"] = torch.empty(max(sc.sc_conv_workspace_bytes(K, c_in, c_out, dtype), 16), dtype=torch.uint8, device=DEVICE)
        return state
    state["feat"] = _features(n, c_in, dtype, seed, DEVICE)
    if case["op"] == "stage":
        state["subm"] = _buffers(n, 3, 1, "subm", c_in, c_in, dtype, dtype)
        state["down"] = _buffers(n, K, stride, "strided", c_in, c_out, dtype, case["out"])
        state["mid"] = torch.empty((n, c_in), dtype=DTYPES[dtype], device=DEVICE)
        ws = [_weights(27, c_in, c_in, dtype, seed, DEVICE), _weights(27, c_in, c_in, dtype, seed + 1, DEVICE),
              _weights(K ** 3, c_in, c_out, dtype, seed + 2, DEVICE)]
        state["w"] = [sc.sc_conv_weight_pack(w, k) for w, k in zip(ws, (3, 3, K))] if case["weights"] == "packed" else ws
        state["counts"] = _head(state["down"])
        return state
    mode = "subm" if stride == 1 else "strided"
    dims = None
    if case["table"] in ("dense", "fused"):
        dims = (scenes,) + (INDOOR_BOX if case["scene"] == "indoor" else LIDAR_BOX)
    state["buf"] = buf = _buffers(n, K, stride, mode, c_in, c_out, dtype, case["out"], dims)
    w = _weights(K ** 3, c_in, c_out, dtype, seed, DEVICE)
    state["w"] = sc.sc_conv_weight_pack(w, K) if case["weights"] == "packed" else w
    state["counts"] = _head(buf)
    return state


def _head(buf):
    """n_in and n_out of a layer's counts block, as numbers on the device."""
    return buf.counts[:16].view(torch.int64)


def run(state):
    case, coords, feat, w = state["case"], state["coords"], state["feat"], state["w"]
    packed = case["weights"] == "packed"
    if case["op"] == "up":
        K, stride, down, out = case["K"], case["stride"], state["down"], state["out"]
        if case["table"] == "direct":
            sc.sc_conv_up_fwd(feat, case["n"], w, out, down.kmap, down.counts, K)
        else:
            sc.sc_kmap_transpose(down.kmap, case["n"], K, stride, down.counts, state["kmap_inv"])
            sc.sc_conv_fwd(feat, w, out, state["kmap_inv"], down.counts, K, stride, "inverse", state["workspace"], n_map=case["n"])
        return out
    if case["op"] == "stage":
        subm, down, mid = state["subm"], state["down"], state["mid"]
        subm.hash_build(coords)
        subm.kmap_build(coords)
        if packed:
            subm.conv_fwd_packed(feat, w[0])
            sc.sc_conv_fwd_packed(subm.feat_out, w[1], case["c_in"], mid, subm.kmap, subm.counts, 3, 1, "subm")
        else:
            subm.conv_fwd(feat, w[0])
            sc.sc_conv_fwd(subm.feat_out, w[1], mid, subm.kmap, subm.counts, 3, 1, "subm", subm.workspace)
        down.kmap_build(coords, standalone=True)
        (down.conv_fwd_packed if packed else down.conv_fwd)(mid, w[2])
        return {"first": subm.feat_out, "second": mid, "down": down.feat_out, "coords": down.out_coords, "counts": state["counts"]}
    buf = state["buf"]
    if case["table"] == "fused":
        buf.layer_fused(coords, feat, w)
        return buf.feat_out
    if case["table"] == "none":
        buf.kmap_build(coords, standalone=True)
    else:
        buf.hash_build(coords)
        buf.kmap_build(coords)
    (buf.conv_fwd_packed if packed else buf.conv_fwd)(feat, w)
    if case["table"] == "none":
        return {"feat": buf.feat_out, "coords": buf.out_coords, "counts": state["counts"]}
    return {"feat": buf.feat_out, "counts": state["counts"]}


# ---- what a pass cannot do without -------------------------------------------------------------------
@functools.lru_cache(maxsize=None)
def _pairs(scene, sweeps, n, K, stride):
    """(pairs, output rows) of the layer's map, counted on one voxel set of the case."""
    device = DEVICE if torch.cuda.is_available() else "cpu"
    c = _coords({"scene": scene, "sweeps": sweeps, "n": n}, 0, device)[0].long()
    key = lambda b, x, y, z: ((b * 2048 + x + 8) * 2048 + y + 8) * 2048 + z + 8  # noqa: E731
    offsets = [(dx, dy, dz) for dx in range(K) for dy in range(K) for dz in range(K)]
    if stride == 1:
        keys = torch.sort(key(*c.T)).values
        pad, total = (K - 1) // 2, 0
        for dx, dy, dz in offsets:
            probe = key(c[:, 0], c[:, 1] + dx - pad, c[:, 2] + dy - pad, c[:, 3] + dz - pad)
            at = torch.searchsorted(keys, probe).clamp(max=len(keys) - 1)
            total += int((keys[at] == probe).sum())
        return total, n
    cells = []
    for d in offsets:
        p = c[:, 1:] - torch.tensor(d, device=c.device)
        ok = ((p >= 0) & (p % stride == 0)).all(dim=1)
        cells.append(key(c[ok, 0], *(p[ok] // stride).T))
    cells = torch.cat(cells)
    return len(cells), len(torch.unique(cells))


def work(case):
    n, K, stride, c_in, c_out = case["n"], case["K"], case["stride"], case["c_in"], case["c_out"]
    e_in, e_out = (4 if case[k] == "f32" else 2 for k in ("dtype", "out"))
    P, n_out = _pairs(case["scene"], case["sweeps"], n, K, stride)
    w = K ** 3 * c_in * c_out * e_in
    if case["op"] == "up":
        # coarse rows in, fine rows out, the strided map's pairs (8 bytes each)
        return {"bytes": n_out * c_in * e_in + n * c_out * e_out + w + 8 * P, "flops": 2 * P * c_in * c_out}
    strided = 16 * n + n * c_in * e_in + n_out * (c_out * e_out + 16) + w
    if case["op"] == "stage":
        P3, _ = _pairs(case["scene"], case["sweeps"], n, 3, 1)
        layer = 2 * n * c_in * e_in + 27 * c_in * c_in * e_in
        return {"bytes": 16 * n + 2 * layer + strided, "flops": 4 * P3 * c_in * c_in + 2 * P * c_in * c_out}
    if stride > 1:
        return {"bytes": strided, "flops": 2 * P * c_in * c_out}
    return {"bytes": 16 * n + n * c_in * e_in + n * c_out * e_out + w, "flops": 2 * P * c_in * c_out}


def tolerance(case):
    """32-bit sums in another order; one rounding to 11 bits (f16) or 8 bits (bf16) at the end of a
    layer, which another order of summation moves by one step now and then."""
    if case["dtype"] == "f32" or case["out"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 1e-3} if case["dtype"] == "f16" else {"rel": 8e-3}
