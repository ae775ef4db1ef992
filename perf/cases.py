"""The work that a user of this library has it do, as cases that can be timed.

Four kinds of call: one convolution layer (`nm_conv2d` / `nm_conv2d_res` on a
pruned, packed layer), a whole network (`Network.forward`), and the pruning and
packing of a layer's weights with their export (`nm_prune` and the two exports a
program uses to save them).  Layer and network shapes are those of `workloads.py`;
values follow its generators (x uniform in [0, 1), He-normal weights, N(0, 0.01)
biases).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2507_17301_amd import binding as nm
from paper_2507_17301_amd import workloads as wl
from paper_2507_17301_amd.network import Network

_CODE = {"f32": nm.NM_F32, "bf16": nm.NM_BF16, "f8": nm.NM_F8E4M3}
_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f8": torch.float8_e4m3fn}
_IN_BYTES = {"f32": 4, "bf16": 2, "f8": 1}
_OUT_BYTES = {"f32": 4, "bf16": 2, "f8": 2}
_DEV = "cuda:0"


def _conv(name, dtype, batch, h, w, cin, cout, k, stride=1, pad=0, dil=1, n=2, m=4, tile=16, relu=True,
          residual=False, tune=True):
    c = {"kind": "conv", "dtype": dtype, "batch": batch, "h": h, "w": w, "cin": cin, "cout": cout, "k": k,
         "stride": stride, "pad": pad, "dil": dil, "n": n, "m": m, "tile": tile, "relu": relu, "residual": residual,
         "tune": tune}
    return {"name": name, **c} if name else c


def _net(name, depth, dtype, batch, hw=224, n=2, m=4, tile=16):
    """depth 18 and 50: one N:M for every stage; depth 101: the mixed table (n = m = 0)."""
    c = {"kind": "net", "depth": depth, "dtype": dtype, "batch": batch, "hw": hw, "n": n, "m": m, "tile": tile}
    return {"name": name, **c} if name else c


def _prune(name, dtype, cout, k, cin, n=2, m=4, tile=16):
    c = {"kind": "prune", "dtype": dtype, "cout": cout, "k": k, "cin": cin, "n": n, "m": m, "tile": tile}
    return {"name": name, **c} if name else c


def listed():
    return [
        # one image through one early 3x3 layer: the latency of a single small call
        _conv("conv3x3_1img_f32", "f32", 1, 56, 56, 64, 64, 3, pad=1),
        # the layer of the N:M sweep, a mid-network 3x3 at a medium batch, as it runs without tuning
        _conv("conv3x3_14px_f32_untuned", "f32", 32, 14, 14, 256, 256, 3, pad=1, tune=False),
        # the adaptive setting: one group spans all input channels of a tap, half of them kept
        _conv("conv3x3_cin_groups_f32", "f32", 16, 28, 28, 128, 128, 3, pad=1, n=64, m=128),
        # odd sizes, dilation, channel counts off every tile, narrow column tiles, another ratio
        _conv("conv3x3_ragged_f32_untuned", "f32", 5, 37, 45, 48, 72, 3, stride=1, pad=2, dil=2, n=1, m=4, tile=8,
              relu=False, tune=False),
        # an ordinary 3x3 layer in bf16 at the benchmark's batch
        _conv("conv3x3_28px_bf16", "bf16", 64, 28, 28, 128, 128, 3, pad=1),
        # the dense first layer of every network here, three input channels
        _conv("conv7x7_stem_bf16", "bf16", 64, 224, 224, 3, 64, 7, stride=2, pad=3, n=1, m=1),
        # a late 1x1 layer in fp8
        _conv("conv1x1_14px_f8", "f8", 64, 14, 14, 1024, 256, 1),
        # loading a model: prune and pack one late 3x3 layer's weights, export the compressed form
        _prune("prune_512x3x3x512_f32", "f32", 512, 3, 512),
        # answering one image
        _net("resnet18_1img_f32", 18, "f32", 1),
        # the benchmark's network and batch in both tensor types
        _net("resnet50_b64_bf16", 50, "bf16", 64),
        _net("resnet50_b64_f32", 50, "f32", 64),
        # the largest configuration: mixed sparsity per stage, column tiles of 32
        _net("resnet101_b256_bf16", 101, "bf16", 256, n=0, m=0, tile=32),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_RATIOS = [(1, 4), (2, 4), (1, 8), (2, 8), (4, 8)]


def draw(rng):
    """One more case of the listed ranges: single layers most of the time."""
    what = rng.random()
    if what < 0.15:
        depth = rng.choice([18, 50])
        n, m = rng.choice(_RATIOS)
        return _net(None, depth, rng.choice(["f32", "bf16"]), _logint(rng, 1, 64), 32 * rng.randrange(5, 9), n, m,
                    rng.choice([16, 32]))
    if what < 0.25:
        n, m = rng.choice(_RATIOS)
        return _prune(None, rng.choice(["f32", "bf16"]), _logint(rng, 64, 1024), rng.choice([1, 3]),
                      8 * _logint(rng, 8, 64), n, m, rng.choice([8, 16, 32]))
    dtype = rng.choice(["f32", "f32", "bf16", "bf16", "f8"])
    k = rng.choice([1, 3, 3])
    n, m = rng.choice(_RATIOS)
    tile = rng.choice([8, 16, 16, 32])
    if dtype == "f8" or rng.random() < 0.7:      # channel counts as the networks have them
        cin, cout = 64 * _logint(rng, 1, 16), 64 * _logint(rng, 1, 16)
        tile = max(tile, 16)
    else:                                        # and off every tile
        cin, cout = 8 * _logint(rng, 1, 64), _logint(rng, 9, 500)
    if k > 1 and dtype == "f32" and rng.random() < 0.15:
        n, m = cin // 2, cin
    h, w = _logint(rng, 7, 80), _logint(rng, 7, 80)
    dil = 2 if k == 3 and rng.random() < 0.1 else 1
    stride = 2 if rng.random() < 0.15 else 1
    pad = dil * (k // 2)
    batch = _logint(rng, 1, 128)
    while batch > 1 and batch * h * w * max(cin, cout, k * k * cin * cout // 1024) > 120_000_000:
        batch //= 2
    return _conv(None, dtype, batch, h, w, cin, cout, k, stride, pad, dil, n, m, tile, rng.random() < 0.7,
                 rng.random() < 0.3, rng.random() < 0.5)


def _layer(c):
    return wl.ConvLayer("case", c["h"], c["w"], c["cin"], c["cout"], c["k"], c["k"], c["stride"], c["pad"], c["dil"],
                        c["n"], c["m"], c["tile"])


def _ops(c):
    if c["depth"] == 101:
        return wl.resnet101_graph(c["tile"])
    blocks, bottleneck = {18: ((2, 2, 2, 2), False), 50: ((3, 4, 6, 3), True)}[c["depth"]]
    return wl.resnet_graph(blocks, (64, 128, 256, 512), bottleneck, c["hw"], [(c["n"], c["m"])] * 4, c["tile"])


def _uniform(shape, dtype, seed):
    g = torch.Generator(device=_DEV)
    g.manual_seed(int(seed))
    return torch.rand(shape, generator=g, device=_DEV, dtype=torch.float32).to(dtype)


def prepare(case, seed):
    c, dt = case, _CODE[case["dtype"]]
    rng = np.random.default_rng(int(seed))
    if c["kind"] == "net":
        net = Network(_ops(c), c["batch"], c["hw"], dt, seed0=int(seed) * 1000, device=_DEV)
        net.autotune()                           # profiled once per shape and process, as a serving program does
        return {"kind": "net", "net": net, "x": _uniform(net.shapes[0], net.tdt, seed)}
    if c["kind"] == "prune":
        sigma = math.sqrt(2.0 / (c["k"] * c["k"] * c["cin"]))
        w = rng.standard_normal((c["cout"], c["k"], c["k"], c["cin"]), dtype=np.float32) * np.float32(sigma)
        return {"kind": "prune", "w": w, "n": c["n"], "m": c["m"], "tile": c["tile"], "dt": dt}
    layer = _layer(c)
    _, w, bias = wl.make_tensors(layer, c["batch"], int(seed), with_input=False)
    packed = nm.nm_prune(w, layer.n, layer.m, layer.tile, dt)
    x = _uniform((c["batch"], c["h"], c["w"], c["cin"]), _TORCH[c["dtype"]], seed)
    yt = torch.bfloat16 if c["dtype"] == "f8" else x.dtype
    y = torch.empty((c["batch"], layer.Ho, layer.Wo, c["cout"]), dtype=yt, device=_DEV)
    res = _uniform(tuple(y.shape), yt, int(seed) + 1) if c["residual"] else None
    if c["tune"]:
        nm.nm_autotune(dt, c["batch"], c["h"], c["w"], c["cin"], packed, True, layer.stride, layer.pad, layer.dil,
                       c["relu"])
    return {"kind": "conv", "packed": packed, "x": x, "y": y, "bias": torch.from_numpy(bias).to(_DEV), "res": res,
            "stride": layer.stride, "pad": layer.pad, "dil": layer.dil, "relu": c["relu"]}


def run(state):
    s = state
    if s["kind"] == "net":
        return s["net"].forward(s["x"])
    if s["kind"] == "prune":
        packed = nm.nm_prune(s["w"], s["n"], s["m"], s["tile"], s["dt"])
        out = (nm.nm_packed_indices(packed), nm.nm_packed_values(packed))
        packed.free()
        return out
    if s["res"] is not None:
        return nm.nm_conv2d_res(s["x"], s["packed"], s["res"], s["bias"], s["stride"], s["pad"], s["dil"], s["relu"],
                                y=s["y"])
    return nm.nm_conv2d(s["x"], s["packed"], s["bias"], s["stride"], s["pad"], s["dil"], s["relu"], y=s["y"])


def _layer_work(layer, batch, dtype, residual):
    ib, ob = _IN_BYTES[dtype], _OUT_BYTES[dtype]
    y = layer.P(batch) * layer.Cout * ob
    return layer.algorithmic_bytes(batch, ib, ob) + (y if residual else 0), layer.effective_flops(batch)


def work(case):
    c = case
    if c["kind"] == "conv":
        b, f = _layer_work(_layer(c), c["batch"], c["dtype"], c["residual"])
        return {"bytes": b, "flops": f}
    if c["kind"] == "prune":
        n_w = c["cout"] * c["k"] * c["k"] * c["cin"]
        kept = n_w // c["m"] * c["n"]
        return {"bytes": 4 * n_w + 4 * kept + 4 * (kept // c["tile"]), "flops": n_w}
    ops = _ops(c)
    shapes = wl.net_tensor_shapes(ops, c["batch"], c["hw"])
    es, nbytes, flops = _IN_BYTES[c["dtype"]], 0, 0
    for op in ops:
        if op.kind == "conv":
            b, f = _layer_work(op.layer, c["batch"], c["dtype"], op.residual >= 0)
            nbytes, flops = nbytes + b, flops + f
        else:
            nbytes += es * (math.prod(shapes[op.src]) + math.prod(shapes[op.dst]))
    nbytes += 2 * es * math.prod(shapes[0])      # the caller's image batch goes into the network's input tensor
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Measured: fp32 layers are 2e-7 .. 6e-7 from float64 and as far from one another under other summation
    # orders (6e-6 at the worst element), whole fp32 networks 3e-7 .. 9e-7.  One rounding to bf16 is 1.7e-3
    # (2-norm) and one unit in the last place is 7.8e-3; bf16 networks are 2.7e-3 from float64.
    c = case
    if c["kind"] == "prune":
        return "exact"
    if c["kind"] == "net":
        return {"rel": 4e-6} if c["dtype"] == "f32" else {"rel": 1e-2}
    return {"rel": 4e-6, "max": 4e-5} if c["dtype"] == "f32" else {"rel": 5e-3, "max": 2e-2}
