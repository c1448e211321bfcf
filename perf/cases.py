"""Measured cases of the sparse-convolution (SpC) layer library: what a program that runs this library on
voxel clouds has it do, from a 2 k-voxel layer to a 3 M-voxel one and a 25-layer network.

A pass of a "layer" case is one layer on one new cloud: pack + sort the coordinates, build the kernel map with
the sort permutation folded in, compute the features, release the map.  A pass of a "unet" case is the 25-layer
UNet-style stack on one cloud, either call by call ("unet_eager") or replayed from the graph that the program
recorded for clouds of this size ("unet_graph").  Clouds are drawn on the GPU from the seed alone and stand for
LiDAR sweeps, indoor scans and the uniformly random volumes of the paper's size sweep.
"""
from __future__ import annotations

import functools
import math

import torch

from paper_2511_20834_amd import binding as B
from paper_2511_20834_amd import synth
from paper_2511_20834_amd.network import SpcNetwork

_DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}


def _layer(name, cloud, n, K, stride, cin, cout, dtype, dataflow="os", batch=1, key_bits=0):
    return {"name": name, "path": "layer", "cloud": cloud, "n": n, "batch": batch, "K": K, "stride": stride,
            "cin": cin, "cout": cout, "dtype": dtype, "dataflow": dataflow, "key_bits": key_bits}


def listed():
    return [
        # the smallest call: a few thousand voxels in fp32 (an object crop, or a unit test of a user's model)
        _layer("tiny_f32", "surface", 2118, 3, 1, 16, 16, "f32"),
        # a coarse, wide level of a network in bf16, with a ragged voxel count
        _layer("coarse_bf16", "lidar", 6011, 3, 1, 128, 128, "bf16"),
        # the headline layer: one LiDAR cloud, 3x3x3, 64 channels
        _layer("lidar_k3", "lidar", 120_000, 3, 1, 64, 64, "f16"),
        # downsampling layer of an encoder: the output voxels are found on the way and their number is waited for
        _layer("lidar_stride2", "lidar", 120_000, 3, 2, 64, 128, "f16"),
        # the weight-stationary dataflow on the headline layer
        _layer("lidar_k3_ws", "lidar", 120_000, 3, 1, 64, 64, "f16", dataflow="ws"),
        # the fp32 mode on an ordinary level
        _layer("lidar_f32", "lidar", 50_021, 3, 1, 32, 32, "f32"),
        # four indoor scans as one batch, large kernel
        _layer("indoor_k5", "indoor", 240_000, 5, 1, 32, 32, "f16", batch=4),
        # the same in bf16 with the hybrid dual dataflow (dense offsets output-, sparse ones weight-stationary)
        _layer("indoor_k5_hybrid", "indoor", 240_000, 5, 1, 32, 32, "bf16", dataflow="hybrid3", batch=4),
        # channel counts that are no multiple of the matrix tiles, 64-bit keys, odd voxel count
        _layer("ragged_24_40", "random", 70_001, 3, 1, 24, 40, "f16", key_bits=64),
        # a large scene of the size sweep (1.25 % of the volume is occupied)
        _layer("random_3m", "random", 3_000_000, 3, 1, 64, 64, "f16"),
        # whole network, call by call: maps of all layers, then 25 feature layers, host work included
        {"name": "unet_eager", "path": "unet_eager", "cloud": "lidar", "n": 120_000},
        # whole network in a serving loop: the recorded step, replayed on the cloud in its input buffers
        {"name": "unet_graph", "path": "unet_graph", "cloud": "lidar", "n": 120_000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = [work(c) for c in listed()]
    most = {k: max(w[k] for w in most) for k in ("bytes", "flops")}
    while True:
        kind = rng.random()
        if kind < 0.2:  # networks: one sweep at several resolutions
            return {"path": rng.choice(["unet_eager", "unet_graph"]), "cloud": "lidar", "n": _log_int(rng, 15_000, 120_000)}
        c = {"path": "layer", "cloud": rng.choice(["surface", "lidar", "lidar", "indoor", "random", "random"])}
        c["batch"] = rng.randint(1, 4) if c["cloud"] == "indoor" else 1
        lo, hi = {"surface": (1000, 4000), "lidar": (4000, 200_000), "indoor": (15_000 * c["batch"], 80_000 * c["batch"]),
                  "random": (4000, 3_000_000)}[c["cloud"]]
        c["n"] = _log_int(rng, lo, hi)
        c["n"] -= c["n"] % c["batch"]
        c["K"], c["stride"] = rng.choice([(3, 1), (3, 1), (3, 1), (3, 2), (2, 2), (5, 1)])
        c["dtype"] = rng.choice(["f16", "f16", "bf16", "bf16", "f32"])
        c["dataflow"] = rng.choice(["os", "os", "os", "os", "ws", "hybrid2"])
        c["key_bits"] = rng.choice([0, 0, 0, 64])
        if c["dtype"] == "f32":
            c["cin"], c["cout"] = rng.choice([(16, 16), (6, 10), (32, 32), (32, 64), (64, 64)])
        else:
            c["cin"], c["cout"] = rng.choice([(4, 32), (16, 32), (24, 40), (32, 32), (32, 64), (64, 32), (64, 64), (64, 96),
                                              (64, 128), (128, 128), (128, 256), (256, 256)])
        w = work(c)
        if w["bytes"] <= most["bytes"] and w["flops"] <= most["flops"]:
            return c


# ---------------------------------------------------------------- clouds
def _take(keys, n, gen):
    """n of the distinct values, in random order (rows of a cloud arrive unsorted)."""
    if keys.numel() < n:
        raise RuntimeError("the scene holds %d voxels, %d are wanted" % (keys.numel(), n))
    return keys[torch.randperm(keys.numel(), generator=gen, device=keys.device)[:n]]


def _rows(lin, dims, b=0):
    z = lin % dims[2]
    y = (lin // dims[2]) % dims[1]
    x = lin // (dims[1] * dims[2])
    return torch.stack([torch.full_like(x, b), x, y, z], dim=1).to(torch.int32)


def _distinct(points, dims):
    """Distinct voxels of integer points inside [0, dims), as sorted linear indices."""
    ok = ((points >= 0) & (points < torch.tensor(dims, device=points.device))).all(dim=1)
    p = points[ok]
    return torch.unique((p[:, 0] * dims[1] + p[:, 1]) * dims[2] + p[:, 2])


def _surface(n, gen, dev):
    """A ground plane and three spheres in a 64^3 grid."""
    r = functools.partial(torch.rand, generator=gen, device=dev)
    m = 2 * n
    plane = torch.cat([r(m, 2) * 64, torch.full((m, 1), 4.5, device=dev)], dim=1)
    d = torch.randn(m, 3, generator=gen, device=dev)
    d = d / d.norm(dim=1, keepdim=True)
    which = torch.arange(m, device=dev) % 3
    ball = (16 + 32 * r(3, 3))[which] + (8 + 7 * r(3, 1))[which] * d
    p = torch.cat([plane, ball]).floor().long()
    lin = _distinct(p, (64, 64, 64))
    return _rows(_take(lin, n, gen), (64, 64, 64))


def _lidar(n, gen, dev):
    """A 64-beam sensor at 1.8 m over the ground among 40 boxes and cylinders, accumulated over sweeps 0.7 m apart
    until n voxels are hit.  0.1 m voxels from 120 k voxels on; fewer voxels come from coarser ones, as the levels
    of a network do."""
    r = functools.partial(torch.rand, generator=gen, device=dev)
    voxel = 0.1 * max(1.0, 120_000 / n) ** 0.7
    dims = (int(102.4 / voxel) + 1, int(102.4 / voxel) + 1, int(8.0 / voxel) + 1)
    low = torch.tensor([-51.2, -51.2, -3.0], device=dev)
    ang, dist = 2 * math.pi * r(40), 4 + 41 * r(40)
    cx, cy = dist * ang.cos(), dist * ang.sin()
    size = 1 + 4 * r(20, 3)
    blo = torch.stack([cx[:20] - size[:, 0] / 2, cy[:20] - size[:, 1] / 2, torch.zeros(20, device=dev)], dim=1)
    bhi = torch.stack([cx[:20] + size[:, 0] / 2, cy[:20] + size[:, 1] / 2, size[:, 2]], dim=1)
    rad, height = 0.2 + 0.8 * r(20), 1 + 4 * r(20)
    elev = torch.deg2rad(torch.linspace(-25.0, 3.0, 64, device=dev))
    inf = torch.tensor(float("inf"), device=dev)
    lin = torch.empty(0, dtype=torch.long, device=dev)
    for sweep in range(40):
        az = (torch.arange(2048, device=dev) + r(1)) * (2 * math.pi / 2048)
        e = (elev + 2e-4 * torch.randn(64, generator=gen, device=dev))[:, None].expand(64, 2048).reshape(-1)
        a = az[None, :].expand(64, 2048).reshape(-1)
        d = torch.stack([e.cos() * a.cos(), e.cos() * a.sin(), e.sin()], dim=1)
        o = torch.tensor([0.7 * sweep, 0.0, 1.8], device=dev) + 0.05 * torch.randn(3, generator=gen, device=dev)
        t = torch.where(d[:, 2] < 0, -o[2] / d[:, 2], inf)
        inv = (1.0 / d)[:, None, :]
        t0, t1 = (blo - o)[None] * inv, (bhi - o)[None] * inv
        tn, tx = torch.minimum(t0, t1).amax(2), torch.maximum(t0, t1).amin(2)
        t = torch.minimum(t, torch.where((tx >= tn) & (tn > 0), tn, inf).amin(1))
        ox, oy = o[0] - cx[20:], o[1] - cy[20:]
        qa = (d[:, 0] ** 2 + d[:, 1] ** 2)[:, None]
        qb = 2 * (ox * d[:, 0:1] + oy * d[:, 1:2])
        disc = qb * qb - 4 * qa * (ox * ox + oy * oy - rad * rad)
        tc = (-qb - disc.clamp(min=0).sqrt()) / (2 * qa)
        zc = o[2] + tc * d[:, 2:3]
        t = torch.minimum(t, torch.where((disc > 0) & (tc > 0) & (zc >= 0) & (zc <= height), tc, inf).amin(1))
        hit = torch.isfinite(t)
        p = o + t[hit][:, None] * d[hit]
        p[:, 2] = p[:, 2].clamp(min=0.0) + 1e-4
        lin = torch.unique(torch.cat([lin, _distinct(((p - low) / voxel).floor().long(), dims)]))
        if lin.numel() >= n:
            break
    return _rows(_take(lin, n, gen), dims)


def _indoor(n, batch, gen, dev):
    """Rooms of 10 m x 10 m x 3 m at 2 cm voxels: floor, ceiling, walls and 30 boxes, sampled at random."""
    dims, out = (500, 500, 150), []
    size = torch.tensor(dims, device=dev, dtype=torch.float32)
    for b in range(batch):
        s = 15 + (85 * torch.rand(30, 3, generator=gen, device=dev)).floor()
        x0 = 1 + ((size - s - 2) * torch.rand(30, 3, generator=gen, device=dev)).floor()
        x0[:, 2] = 0
        lo = torch.cat([torch.zeros(1, 3, device=dev), x0])
        hi = torch.cat([(size - 1)[None], x0 + s])
        ext = (hi - lo + 1).repeat_interleave(6, 0)
        lo, hi = lo.repeat_interleave(6, 0), hi.repeat_interleave(6, 0)
        axis = (torch.arange(len(lo), device=dev) % 6) // 2
        side = torch.arange(len(lo), device=dev) % 2
        at = torch.where((side == 1)[:, None], hi, lo)
        area = ext.prod(1) / ext.gather(1, axis[:, None])[:, 0]
        m = 2 * (n // batch)
        f = torch.multinomial(area, m, replacement=True, generator=gen)
        p = lo[f] + (ext[f] * torch.rand(m, 3, generator=gen, device=dev)).floor()
        p.scatter_(1, axis[f][:, None], at[f].gather(1, axis[f][:, None]))
        out.append(_rows(_take(_distinct(p.long(), dims), n // batch, gen), dims, b))
    rows = torch.cat(out)
    return rows[torch.randperm(len(rows), generator=gen, device=dev)]


def _random(n, gen, dev):
    """Uniformly random voxels in [m, m, 200] at 1.25 % density."""
    m = max(8, int(round(math.sqrt(n / (0.0125 * 200.0)))))
    lin = torch.unique(torch.randint(0, m * m * 200, (int(1.05 * n) + 64,), generator=gen, device=dev))
    return _rows(_take(lin, n, gen), (m, m, 200))


def _cloud(case, gen, dev):
    if case["cloud"] == "surface":
        return _surface(case["n"], gen, dev)
    if case["cloud"] == "lidar":
        return _lidar(case["n"], gen, dev)
    if case["cloud"] == "indoor":
        return _indoor(case["n"], case["batch"], gen, dev)
    return _random(case["n"], gen, dev)


# ---------------------------------------------------------------- one pass
def _weights(k_vol, cin, cout, dtype, gen, dev):
    w = torch.randn(k_vol, cin, cout, generator=gen, device=dev) * math.sqrt(2.0 / (k_vol * cin))
    return w.to(dtype)


@functools.lru_cache(maxsize=None)
def _side_streams():
    """Two streams for the map build of a network, kept for the life of the program."""
    return torch.cuda.Stream(), torch.cuda.Stream()


def prepare(case, seed):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    coords = _cloud(case, gen, dev).contiguous()
    n = coords.shape[0]
    lo, hi = coords[:, 1:].amin(0).tolist(), coords[:, 1:].amax(0).tolist()
    if case["path"] != "layer":
        layers = synth.unet_layers()
        desc = B.spc_pack_desc_fit(lo, hi, 1, 16, 16)
        feats = torch.randn(n, 4, generator=gen, device=dev).to(torch.float16)
        net = SpcNetwork(layers, [_weights(l["K"] ** 3, l["cin"], l["cout"], torch.float16, gen, dev) for l in layers])
        net.prepare_weights()
        if case["path"] == "unet_graph":
            return {"step": net.capture_step(coords, feats, desc, _side_streams(), B.NET_PIPELINED)}
        return {"net": net, "coords": coords, "desc": desc, "feats": feats, "sorted": torch.empty_like(feats),
                "ws": torch.empty(B.spc_pack_workspace_bytes(n, desc), dtype=torch.uint8, device=dev),
                "keys": torch.empty(n, dtype=torch.int32 if desc.key_bits == 32 else torch.int64, device=dev),
                "perm": torch.empty(n, dtype=torch.int32, device=dev)}
    K, cin, cout, dtype = case["K"], case["cin"], case["cout"], _DTYPES[case["dtype"]]
    desc = B.spc_pack_desc_fit(lo, hi, case["batch"], case["stride"], (K - 1) // 2 if K % 2 else K - 1, case["key_bits"])
    hybrid = int(case["dataflow"][6:]) if case["dataflow"].startswith("hybrid") else None
    dataflow = B.DATAFLOW_WS if case["dataflow"] == "ws" else B.DATAFLOW_OS
    layout = {"os": B.LAYOUT_OS, "ws": B.LAYOUT_WS}.get(case["dataflow"]) or B.LAYOUT_BOTH | B.LAYOUT_HYBRID_T(hybrid)
    feats = torch.randn(n, cin, generator=gen, device=dev).to(dtype)
    weights, flags = _weights(K ** 3, cin, cout, dtype, gen, dev), 0
    # weights are constant in inference: re-laid once where the library takes them so
    if dtype != torch.float32 and (cout % 32 == 0 if case["dataflow"] == "os" else cout in (32, 64, 128, 256)):
        weights, flags = B.spc_conv_prepare_weights(weights), B.CONV_PACKED_WEIGHTS
    return {"coords": coords, "desc": desc, "feats": feats, "weights": weights, "flags": flags, "K": K, "stride": case["stride"],
            "layout": layout, "dataflow": dataflow, "hybrid": hybrid,
            "ws": torch.empty(B.spc_pack_workspace_bytes(n, desc), dtype=torch.uint8, device=dev),
            "keys": torch.empty(n, dtype=torch.int32 if desc.key_bits == 32 else torch.int64, device=dev),
            "perm": torch.empty(n, dtype=torch.int32, device=dev),
            # room for the largest output; a strided layer fills its first rows
            "out": torch.zeros((n, cout), dtype=dtype, device=dev)}


def run(state):
    if "step" in state:
        step = state["step"]
        step.replay()
        return {"keys": step.keys, "perm": step.perm, "out": step.output}
    s = state
    B.spc_pack_coords(s["coords"], s["desc"], True, 0, None, s["ws"], s["keys"], s["perm"])
    if "net" in s:
        B.spc_permute_rows(s["feats"], s["perm"], s["sorted"])
        s["net"].build_maps(s["keys"], s["desc"], [torch.cuda.current_stream(), *_side_streams()])
        out = s["net"].forward(s["sorted"])
        s["net"].destroy_maps()
        return {"keys": s["keys"], "perm": s["perm"], "out": out}
    m = B.spc_build_kmap(s["keys"], s["desc"], s["K"], 1, s["stride"], 0, s["layout"], in_perm=s["perm"])
    n_out = m.n_out  # known for stride 1, else waited for: whoever reads the output needs it
    B.spc_conv_forward(m, s["feats"], s["weights"], s["dataflow"], s["flags"], out=s["out"][:n_out], hybrid_t=s["hybrid"])
    m.destroy()
    return {"keys": s["keys"], "perm": s["perm"], "n_out": n_out, "out": s["out"]}


# ---------------------------------------------------------------- what a pass cannot do without
def _pairs_per_input(cloud, K, stride):
    """Valid (input, output, offset) triples per input voxel, about: the occupied share of the neighbourhood is what
    these clouds show on average."""
    if K == stride:
        return 1.0  # a strided 2x2x2 layer partitions its input
    if stride == 2:  # 3x3x3: the voxel's own cell, and a neighbouring cell for 19 of 8 positions
        return 1.0 + 2.375 * {"surface": 0.35, "lidar": 0.45, "indoor": 0.15, "random": 0.1}[cloud]
    near = {"surface": 0.07, "lidar": 0.21, "indoor": 0.03, "random": 0.0125}[cloud]
    if K == 5:
        near *= {"surface": 0.7, "lidar": 0.65, "indoor": 0.35, "random": 1.0}[cloud]
    return 1.0 + near * (K ** 3 - 1)


_COARSE = {"surface": 0.45, "lidar": 0.42, "indoor": 0.75, "random": 0.92}  # output voxels of a stride-2 layer per input voxel


def work(case):
    n, cloud = case["n"], case["cloud"]
    if case["path"] == "layer":
        e = 4 if case["dtype"] == "f32" else 2
        n_out = n if case["stride"] == 1 else _COARSE[cloud] * n
        key = 8 if case["key_bits"] == 64 else 4
        k3, cin, cout = case["K"] ** 3, case["cin"], case["cout"]
        pairs = n * _pairs_per_input(cloud, case["K"], case["stride"])
        return {"bytes": n * (16 + key + 4) + (n * cin + n_out * cout + k3 * cin * cout) * e, "flops": 2 * pairs * cin * cout}
    # network: coordinates, four input and 32 output channels, the weights of 25 layers
    nbytes, flops = n * (16 + 4 + 4 + 2 * 4 + 2 * 32), 0.0
    for l in synth.unet_layers():
        fine = n * _COARSE["lidar"] ** round(math.log2(l["in_stride"]))  # voxels of the finer level of the layer
        flops += 2 * fine * _pairs_per_input("lidar", l["K"], l["layer_stride"]) * l["cin"] * l["cout"]
        nbytes += 2 * l["K"] ** 3 * l["cin"] * l["cout"]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["path"] != "layer":  # activations are rounded to fp16 after each of 25 layers
        return {"rel": 5e-3}
    # fp32 accumulation in any order; the output is rounded to its own type
    return {"rel": {"f16": 1e-3, "bf16": 8e-3, "f32": 1e-5}[case["dtype"]]}
