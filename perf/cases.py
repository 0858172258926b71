"""The work that the layer library is timed on: sparse-convolution layers, blocks, maps
and one whole network, through the package's public entry points.

A case is a dict of plain values.  Its ``kind`` says what one pass runs:

  layer     a whole layer on a new cloud: kernel map and forward (``binding.conv``)
  cached    one layer on a kernel map that the program keeps (as inside a network,
            where several layers share a map)
  resblock  a basic residual block on a kept map: two convolutions with ReLU, the second
            with the residual added
  decblock  a decoder block on kept maps: concatenation with the skip features, a K = 3
            convolution, a K = 1 projection, a K = 3 convolution with the residual
  downup    a downsampling layer on a new cloud and the transposed layer back
  map       the kernel map of a new cloud, with its pair lists
  unet      the UNet-style network on a new cloud, its maps included

Scenes are drawn like the package's workloads (LiDAR-like frames, an indoor-like room,
uniform cells); a cloud has exactly ``n`` voxels at its finest
level, and ``level`` > 0 takes the coordinates of that downsampling level.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2401_06145_amd import binding as B
from paper_2401_06145_amd import net, scenes

DEV = "cuda"
DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
FIELD = 1 << 15  # room of a coordinate field in the packed keys used below


def listed():
    return [
        # the smallest workload of the package: 2k uniform cells, float32; ten short
        # kernels in a row, where launches and latency count
        _layer("layer_uniform2k_f32_c16", "uniform", 2000, 3, 16, 16, "f32"),
        # the LiDAR layer of the benchmark's extras: one 120k-voxel frame, float16
        _layer("layer_lidar120k_f16_c64", "lidar", 120_357, 3, 64, 64, "f16"),
        # the benchmark's headline layer: a 300k-voxel room, 256 channels, float16
        _layer("layer_indoor300k_f16_c256", "indoor", 300_231, 3, 256, 256, "f16"),
        # a network's first layer with the large kernel: few input features, K = 5
        _layer("stem_k5_lidar60k_f16_c8_32", "lidar", 60_013, 5, 8, 32, "f16"),
        # a downsampling layer and its transposed counterpart on one large frame
        {"name": "downup_lidar200k_f16_c32_64", "kind": "downup", "scene": "lidar", "n": 198_858, "K": 2, "stride": 2,
         "c_in": 32, "c_out": 64, "dtype": "f16"},
        # the odd-kernel strided layer of the ResNet-style encoder, map kept, bfloat16
        {"name": "cached_k3s2_lidar120k_bf16_c32_64", "kind": "cached", "scene": "lidar", "n": 120_357, "level": 0,
         "K": 3, "mode": "down", "stride": 2, "c_in": 32, "c_out": 64, "dtype": "bf16"},
        # a float32 layer on a kept map
        {"name": "cached_lidar120k_f32_c64", "kind": "cached", "scene": "lidar", "n": 120_357, "level": 0, "K": 3,
         "mode": "subm", "stride": 1, "c_in": 64, "c_out": 64, "dtype": "f32"},
        # a residual block of the encoders, bfloat16, on the room
        {"name": "resblock_indoor300k_bf16_c128", "kind": "resblock", "scene": "indoor", "n": 300_231, "level": 0,
         "c_in": 128, "c_out": 128, "dtype": "bf16"},
        # the same at a coarse level of two frames: fewer, denser rows, many channels
        {"name": "resblock_level3_f16_c256", "kind": "resblock", "scene": "lidar", "n": 241_686, "level": 3,
         "c_in": 256, "c_out": 256, "dtype": "f16"},
        # a decoder block of the UNet at level 1 (128 channels with the skip features -> 96)
        {"name": "decblock_level1_f16_c96", "kind": "decblock", "scene": "lidar", "n": 241_686, "level": 1,
         "c_in": 96, "c_skip": 32, "c_out": 96, "dtype": "f16"},
        # the kernel map of a large batch of frames, as in the scaling study
        {"name": "map_lidar4M", "kind": "map", "scene": "lidar", "n": 4_070_000, "K": 3, "mode": "subm", "stride": 1},
        # one whole forward of the UNet-style network on two frames, maps included
        {"name": "unet_lidar240k_f16", "kind": "unet", "scene": "lidar", "n": 241_686, "dtype": "f16"},
    ]


def _layer(name, scene, n, K, c_in, c_out, dtype):
    return {"name": name, "kind": "layer", "scene": scene, "n": n, "K": K, "c_in": c_in, "c_out": c_out, "dtype": dtype}


def draw(rng):
    def between(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b))))) | 1

    kind = rng.choice(["layer", "layer", "cached", "cached", "resblock", "decblock", "downup", "map"])
    scene = rng.choice(["lidar", "lidar", "indoor", "uniform"])
    dtype = rng.choice(["f16", "f16", "bf16", "f32"])
    if kind == "map":
        K = rng.choice([2, 3, 3, 5])
        return {"kind": "map", "scene": scene, "n": between(2000, 600_000 if K == 5 else 2_500_000), "K": K,
                "mode": "subm", "stride": 1}
    if kind in ("resblock", "decblock"):
        dtype = rng.choice(["f16", "bf16"])
        c = rng.choice([32, 64, 96, 128, 192, 256])
        d = {"kind": kind, "scene": rng.choice(["lidar", "indoor"]), "n": between(4000, 240_000),
             "level": rng.choice([0, 1, 2, 3]), "c_in": c, "c_out": c, "dtype": dtype}
        if kind == "decblock":
            d["c_skip"] = rng.choice([32, 64, 128])
        return d
    widths = [16, 32, 48, 64, 96, 128] + ([192, 256] if dtype != "f32" else [])
    c_in, c_out = rng.choice([8] + widths), rng.choice(widths)
    if kind == "downup":
        return {"kind": kind, "scene": scene, "n": between(2000, 250_000), "K": rng.choice([2, 3]), "stride": 2,
                "c_in": c_in, "c_out": c_out, "dtype": dtype}
    K = rng.choice([1, 2, 3, 3, 3, 5])
    n = between(2000, 60_000 if K == 5 else 120_000 if dtype == "f32" else 300_000)
    if kind == "layer":
        return {"kind": kind, "scene": scene, "n": n, "K": K, "c_in": c_in, "c_out": c_out, "dtype": dtype}
    mode = rng.choice(["subm", "subm", "down"])
    return {"kind": "cached", "scene": scene, "n": n, "level": rng.choice([0, 1, 2]), "K": 2 if mode == "down" and K == 1
            else K, "mode": mode, "stride": 2 if mode == "down" else 1, "c_in": c_in, "c_out": c_out, "dtype": dtype}


# ----------------------------------------------------------------------------
# Inputs
# ----------------------------------------------------------------------------

def _pack(c):
    """Rows (b, x, y, z) as one integer in their order; fields are centred in their room."""
    c = c.to(torch.int64)
    k = c[:, 0]
    for f in range(1, 4):
        k = k * FIELD + (c[:, f] + FIELD // 2)
    return k


def _unpack(k):
    out = []
    for _ in range(3):
        out.append(k % FIELD - FIELD // 2)
        k = torch.div(k, FIELD, rounding_mode="floor")
    return torch.stack([k] + out[::-1], 1).to(torch.int32)


def _voxels(points, size, batch):
    q = np.floor(points / size).astype(np.int32)
    q = torch.from_numpy(np.concatenate([np.full((len(q), 1), batch, np.int32), q], 1)).to(DEV)
    return torch.unique(_pack(q))


def _geometry(case):
    """Exactly n unique voxels (packed, sorted), the same for every seed.  Frames are
    cropped to the voxels nearest to one of them, so that a small cloud keeps a frame's
    density."""
    n, scene = case["n"], case["scene"]
    g = torch.Generator(DEV).manual_seed(7_000_003)
    if scene == "uniform":
        # the density of 2000 cells in 64^3
        side = max(8, round(64 * (n / 2000) ** (1 / 3)))
        cells = torch.unique(torch.randint(0, side ** 3, (int(n * 1.2) + 1024,), device=DEV, generator=g))
        cells = cells[torch.randperm(len(cells), device=DEV, generator=g)[:n]]
        return _pack(torch.stack([torch.zeros_like(cells), cells // (side * side), (cells // side) % side, cells % side], 1))
    # frames of about this many voxels
    per = 300_000 if scene == "indoor" else 200_000 if n <= 200_000 else 120_843
    frames = -(-n // per)
    if abs(n - per * frames) > abs(n - per * (frames - 1)) and frames > 1 and n < per * (frames - 1) * 1.02:
        frames -= 1
    target = -(-n // frames)
    geo = []
    for f in range(min(frames, 4)):  # later frames repeat a geometry under their own batch index
        if scene == "lidar":
            k = _voxels(scenes.lidar_points(1000 + 100 * f, max(298_000, int(2.9 * target))), 0.05, 0)
        else:
            k = _voxels(scenes.indoor_points(1003 + 100 * f, scenes.INDOOR_BUDGET_300K + 2000), 0.02, 0)
        if len(k) > target:
            c = _unpack(k).to(torch.float32)
            at = c[torch.randint(0, len(c), (1,), device=DEV, generator=g)]
            d = ((c[:, 1:] - at[:, 1:]) ** 2).sum(1)
            k = k[torch.sort(d, stable=True).indices[:target]]
        geo.append(k)
    parts = [geo[f % len(geo)] + f * FIELD ** 3 for f in range(frames)]
    while sum(len(p) for p in parts) < n:  # frames that came out short: one more
        parts.append(geo[len(parts) % len(geo)] + len(parts) * FIELD ** 3)
    return torch.cat(parts)[:n]


def _cloud(case, seed):
    """The case's voxels, int32 [n][4]: moved by whole cells of the coarsest level,
    perhaps with x and y exchanged, and in random order, so that every seed gives other
    coordinates but as many cells and pairs."""
    g = torch.Generator(DEV).manual_seed(7_000_003 + seed)
    c = _unpack(_geometry(case))
    move = 96 * torch.randint(-30, 31, (3,), device=DEV, generator=g)
    if int(torch.randint(0, 2, (1,), device=DEV, generator=g)):
        c = c[:, [0, 2, 1, 3]]
    c[:, 1:] += move.to(torch.int32)
    return c[torch.randperm(len(c), device=DEV, generator=g)].contiguous()


def _coarse(c, cell):
    """Sorted unique floor(c / cell) cell: the coordinates of a downsampling layer."""
    k = c.to(torch.int64)
    k = torch.cat([k[:, :1], torch.div(k[:, 1:], cell, rounding_mode="floor") * cell], 1)
    return _unpack(torch.unique(_pack(k))).contiguous()


def _normal(shape, dtype, seed, scale=1.0):
    g = torch.Generator(DEV).manual_seed(seed)
    return (torch.randn(shape, device=DEV, generator=g) * scale).to(DT[dtype])


def _weight(K, c_in, c_out, dtype, seed):
    return _normal((K ** 3, c_in, c_out), dtype, seed, 1.0 / math.sqrt(K ** 3 * c_in))


def _inputs(case, seed):
    """Everything a pass reads, as tensors, from the seed alone."""
    kind, s = case["kind"], 10_000 * seed
    d = {"coords": _cloud(case, seed)}
    if kind == "map":
        return d
    dt = case["dtype"]
    if kind == "unet":
        d["x"] = _normal((case["n"], net.STEM_C), dt, s + 1)
        d["w"] = {op.out: _weight(op.K, op.c_in, op.c_out, dt, s + 100 + i)
                  for i, op in enumerate(net.unet_ops()) if op.kind == "conv"}
        return d
    if case.get("level"):
        d["coords"] = _coarse(d["coords"], 1 << case["level"])
    n, ci, co = len(d["coords"]), case["c_in"], case["c_out"]
    d["x"] = _normal((n, ci), dt, s + 1)
    if kind in ("layer", "cached"):
        d["w"] = _weight(case["K"], ci, co, dt, s + 2)
    elif kind == "downup":
        d["w"] = _weight(case["K"], ci, co, dt, s + 2)
        d["w_up"] = _weight(case["K"], co, ci if ci % 16 == 0 else 16, dt, s + 3)
    elif kind == "resblock":
        d["w"], d["w2"] = _weight(3, ci, co, dt, s + 2), _weight(3, co, co, dt, s + 3)
    elif kind == "decblock":
        cc = ci + case["c_skip"]
        d["skip"] = _normal((n, case["c_skip"]), dt, s + 4)
        d["w"], d["wp"], d["w2"] = (_weight(3, cc, co, dt, s + 2), _weight(1, cc, co, dt, s + 3),
                                    _weight(3, co, co, dt, s + 5))
    return d


def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case)
    kind = case["kind"]
    if kind in ("cached", "resblock", "decblock"):
        t = 1 << case["level"]
        # a deeper level's coordinates come out of the previous layer's map sorted
        opt = B.Options.make(presorted=1) if case["level"] else None
        c, dt = s["coords"], DT[case["dtype"]]
        K, mode, stride = case.get("K", 3), case.get("mode", "subm"), case.get("stride", 1)
        km = s["map"] = B.KernelMap.build(c, K, stride, t, mode, opt=opt)
        if kind == "cached":
            s["f"] = B.Forward(km, case["c_in"], case["c_out"], dt)
        elif kind == "resblock":
            s["f"], s["f2"] = B.Forward(km, case["c_in"], case["c_out"], dt), B.Forward(km, case["c_out"], case["c_out"], dt)
        else:
            k1 = s["map1"] = B.KernelMap.build(c, 1, 1, t, "subm", opt=opt)
            cc = case["c_in"] + case["c_skip"]
            s["f"], s["fp"] = B.Forward(km, cc, case["c_out"], dt), B.Forward(k1, cc, case["c_out"], dt)
            s["f2"] = B.Forward(km, case["c_out"], case["c_out"], dt)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "layer":
        return B.conv(s["coords"], s["x"], s["w"], case["K"])[1]
    if kind == "cached":
        return s["f"](s["x"], s["w"])
    if kind == "resblock":
        h = s["f"](s["x"], s["w"], relu=True)
        return s["f2"](h, s["w2"], residual=s["x"], relu=True)
    if kind == "decblock":
        cat = B.spconv_concat_rows(s["x"], s["skip"])
        h = s["f"](cat, s["w"], relu=True)
        p = s["fp"](cat, s["wp"])
        return s["f2"](h, s["w2"], residual=p, relu=True)
    if kind == "downup":
        km, y = B.conv(s["coords"], s["x"], s["w"], case["K"], case["stride"], 1, "down")
        kt = km.transpose()
        up = B.Forward(kt, case["c_out"], s["w_up"].shape[2], DT[case["dtype"]])(y, s["w_up"])
        return {"coords": km.out_coords(), "down": y, "up": up}
    if kind == "map":
        km = B.KernelMap.build(s["coords"], case["K"], case["stride"], 1, case["mode"])
        pin, pout, counts = km.all_pairs()
        return {"pin": pin, "pout": pout, "pairs": sum(counts)}
    if kind == "unet":
        model = net.Network(s["coords"], DT[case["dtype"]], weights=s["w"])
        return model.forward(s["x"])["out"]
    raise ValueError(kind)


# ----------------------------------------------------------------------------
# The same in 64 bits: neighbours by a search over packed keys, one dense product per
# kernel offset
# ----------------------------------------------------------------------------

def _offsets(K, t):
    c = (K - 1) // 2 if K % 2 else 0
    return [(t * (i - c), t * (j - c), t * (k - c)) for i in range(K) for j in range(K) for k in range(K)]


class _Finder:
    """Rows of a cloud by coordinate."""

    def __init__(self, coords):
        self.keys, self.rows = torch.sort(_pack(coords))

    def __call__(self, k):
        at = torch.searchsorted(self.keys, k).clamp(max=len(self.keys) - 1)
        hit = torch.nonzero(self.keys[at] == k).squeeze(1)
        return hit, self.rows[at[hit]]


def _pairs_of(src, q, K, t):
    """(query rows, source rows) of each offset: source = query + offset."""
    find, k = _Finder(src), _pack(q)
    for dx, dy, dz in _offsets(K, t):
        yield find(k + (dx * FIELD + dy) * FIELD + dz)


def _conv64(pairs, x, w, n_out, up=False):
    x, w = x.double(), w.double()
    y = torch.zeros((n_out, w.shape[2]), dtype=torch.float64, device=DEV)
    for k, (q, p) in enumerate(pairs):
        i, o = (q, p) if up else (p, q)
        if len(i):
            y.index_add_(0, o, x[i] @ w[k])
    return y


def exact(case, seed):
    kind = case["kind"]
    if kind == "map":
        return None
    d = _inputs(case, seed)
    c, t = d["coords"], 1 << case.get("level", 0)
    if kind == "unet":
        return _unet64(d)
    if kind == "layer" or (kind == "cached" and case["mode"] == "subm"):
        return _conv64(_pairs_of(c, c, case["K"], t), d["x"], d["w"], len(c))
    if kind == "cached":
        q = _coarse(c, t * case["stride"])
        return _conv64(_pairs_of(c, q, case["K"], t), d["x"], d["w"], len(q))
    if kind == "downup":
        q = _coarse(c, case["stride"])
        pairs = list(_pairs_of(c, q, case["K"], 1))
        y = _conv64(pairs, d["x"], d["w"], len(q))
        return {"coords": None, "down": y, "up": _conv64(pairs, y, d["w_up"], len(c), up=True)}
    pairs = list(_pairs_of(c, c, 3, t))
    if kind == "resblock":
        h = _conv64(pairs, d["x"], d["w"], len(c)).relu()
        return (_conv64(pairs, h, d["w2"], len(c)) + d["x"].double()).relu()
    cat = torch.cat([d["x"], d["skip"]], 1).double()
    h = _conv64(pairs, cat, d["w"], len(c)).relu()
    return (_conv64(pairs, h, d["w2"], len(c)) + cat @ d["wp"][0].double()).relu()


def _unet64(d):
    coords, maps, t = {0: d["coords"]}, {}, {"x0": d["x"].double()}

    def pairs(level, K, mode):
        if (level, K, mode) not in maps:
            c = coords[level]
            if mode == "down":
                coords[level + 1] = _coarse(c, 2 << level)
            maps[level, K, mode] = list(_pairs_of(c, coords[level + 1] if mode == "down" else c, K, 1 << level))
        return maps[level, K, mode]

    for op in net.unet_ops():
        if op.kind == "alias":
            t[op.out] = t[op.inp]
        elif op.kind == "concat":
            t[op.out] = torch.cat([t[op.inp], t[op.other]], 1)
        else:
            up = op.mode == "up"
            p = pairs(op.level - 1, op.K, "down") if up else pairs(op.level, op.K, op.mode)
            n = len(coords[op.level + {"up": -1, "down": 1, "subm": 0}[op.mode]])
            y = _conv64(p, t[op.inp], d["w"][op.out], n, up)
            if op.residual:
                y = y + t[op.residual]
            t[op.out] = y.relu() if op.relu else y
    return t[net.unet_ops()[-1].out]


# ----------------------------------------------------------------------------
# What a pass cannot do without
# ----------------------------------------------------------------------------

@functools.lru_cache(maxsize=64)
def _count(scene, n, level, K, stride):
    """(rows, output rows, pairs) of a layer of this kind, on one cloud of it."""
    c, t = _cloud({"scene": scene, "n": n}, 1), 1 << level
    if level:
        c = _coarse(c, t)
    q = _coarse(c, t * stride) if stride > 1 else c
    return len(c), len(q), sum(len(a) for a, _ in _pairs_of(c, q, K, t))


def work(case):
    kind, n = case["kind"], case["n"]
    e = 4 if case.get("dtype") == "f32" else 2
    if kind == "unet":
        byts, flops, seen = 16.0 * n, 0.0, set()
        for op in net.unet_ops():
            if op.kind != "conv":
                continue
            down = op.mode != "subm"
            lvl = op.level - 1 if op.mode == "up" else op.level
            rows, outs, pairs = _count(case["scene"], n, lvl, op.K, 2 if down else 1)
            flops += 2.0 * pairs * op.c_in * op.c_out
            byts += e * (op.K ** 3 * op.c_in * op.c_out)
            if (lvl, op.K, down) not in seen:
                seen.add((lvl, op.K, down))
                byts += 8.0 * pairs  # the map's pair lists
        return {"bytes": byts + e * n * (net.STEM_C + net.DEC_C[-1]), "flops": flops}
    rows, outs, pairs = _count(case["scene"], n, case.get("level", 0), case.get("K", 3), case.get("stride", 1))
    if kind == "map":
        return {"bytes": 16.0 * rows + 8.0 * pairs, "flops": 0}
    ci, co, k3 = case["c_in"], case["c_out"], case.get("K", 3) ** 3
    layer = e * (rows * ci + outs * co + k3 * ci * co)
    if kind == "layer":
        return {"bytes": 16.0 * rows + 8.0 * pairs + layer, "flops": 2.0 * pairs * ci * co}
    if kind == "cached":
        return {"bytes": float(layer + 8 * pairs), "flops": 2.0 * pairs * ci * co}
    if kind == "resblock":
        return {"bytes": float(e * (rows * (ci + co) + k3 * (ci + co) * co) + 8 * pairs),
                "flops": 2.0 * pairs * (ci + co) * co}
    if kind == "decblock":
        cc = ci + case["c_skip"]
        return {"bytes": float(e * (rows * (cc + co) + k3 * (cc + co) * co + cc * co) + 8 * pairs),
                "flops": 2.0 * pairs * (cc + co) * co + 2.0 * rows * cc * co}
    cu = ci if ci % 16 == 0 else 16
    return {"bytes": float(16 * (rows + outs) + 8 * pairs + layer + e * (rows * cu + k3 * co * cu)),
            "flops": 2.0 * pairs * co * (ci + cu)}


def tolerance(case):
    """About four times what two correct orders of the sums differ by (the centre offset's
    product rounded to the partial type or kept in float32, float32 partials or not),
    measured on the listed cases."""
    kind = case["kind"]
    if kind == "map":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 2e-5}
    if kind == "unet":
        return {"rel": 2.5e-3, "max": 5e-2}
    bf = case["dtype"] == "bf16"
    return {"rel": 1e-2 if bf else 1.5e-3, "max": 8e-2 if bf else 1.6e-2}
