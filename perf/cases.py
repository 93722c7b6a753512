"""Performance cases of the banded chain library: what its users run, with the sizes and options
they run it with.

A case names a chain of local operators (`chain`), its input (`n`, `h`, `w` and the storage type,
or the rows and columns of a matrix chain), the number of row bands, the way the bands are run
(`mode`) and how the call is made:

  mode      "independent"  every band recomputes its halo rows (the default flag)
            "reuse"        bands in order on shared buffers (LOP_FLAG_REUSE)
            "batched"      one launch per operator for all bands (LOP_FLAG_BATCH_BANDS)
  fuse      False: every layer a launch of its own (LOP_FLAG_NO_FUSE)
  graph     replay from a captured graph (LOP_FLAG_GRAPH)
  copy      the result also travels to pinned host memory, as it does for a remote consumer
  call      "free"     lop_run_chain on the plan's own streams: the serving loop, chains of
                       consecutive calls overlap
            "ordered"  lop_run_chain on a stream of the caller's, between other work on it
            "static"   lop_run_chain_static: callers that may not allocate or fork streams

A program keeps one plan per chain and sends many inputs through it, so the states of one case
share a plan for as long as any of them lives; its weights belong to the plan. Inputs and output
buffers are the state's own. Building schedules (lop_loss_solve) and the two-party emulation are
offline instruments with timed waits and are no cases.
"""
import math
import weakref

import numpy as np
import torch

import workloads
from paper_2507_05829_amd import lop

_MODES = {"independent": lop.LOP_FLAG_INDEPENDENT, "reuse": lop.LOP_FLAG_REUSE, "batched": lop.LOP_FLAG_BATCH_BANDS}
_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}


def _image(name, chain, n, h, w, dtype, bands, mode, graph=True, copy=True, call="free", fuse=True):
    return {"name": name, "chain": chain, "n": n, "h": h, "w": w, "dtype": dtype, "bands": bands, "mode": mode,
            "fuse": fuse, "graph": graph, "copy": copy, "call": call}


def _matrix(name, m, k, hidden, dtype, bands, mode="independent", graph=True, copy=False, call="free"):
    return {"name": name, "chain": "mlp", "m": m, "k": k, "hidden": hidden, "dtype": dtype, "bands": bands,
            "mode": mode, "fuse": True, "graph": graph, "copy": copy, "call": call}


def listed():
    return [
        # The smallest call anybody makes: two small layers, no graph. Launches and host work only.
        _image("tiny", "tiny", 1, 32, 32, "f32", 4, "independent", graph=False),
        # One camera frame through the fp32 backbone, each band independent: the benchmark's headline.
        _image("resnet18 independent", "resnet18", 1, 224, 224, "f32", 4, "independent"),
        # The same stream of frames on one device, where nothing needs to be computed twice.
        _image("resnet18 reuse", "resnet18", 1, 224, 224, "f32", 4, "reuse"),
        # The bf16 stack with the most arithmetic per image, in both forms that recompute halos.
        _image("vgg16 independent", "vgg16", 1, 224, 224, "bf16", 8, "independent"),
        _image("vgg16 batched", "vgg16", 1, 224, 224, "bf16", 8, "batched"),
        # High-resolution frames: many bands, large first layers, a result of megabytes.
        _image("detector720p independent", "detector720p", 1, 720, 1280, "bf16", 16, "independent"),
        _image("detector720p reuse", "detector720p", 1, 720, 1280, "bf16", 16, "reuse"),
        # A batch through the memory-bound chain, with its blocks fused and layer by layer (what any
        # 1x1 or depthwise layer outside such a block costs).
        _image("mbv2", "mbv2", 8, 640, 640, "bf16", 8, "independent"),
        _image("mbv2 layers", "mbv2", 8, 640, 640, "bf16", 8, "independent", copy=False, fuse=False),
        # Crops of an odd size, a few at a time, between other work on the caller's stream.
        _image("resnet18 crops", "resnet18", 3, 173, 201, "bf16", 5, "reuse", graph=False, copy=False, call="ordered"),
        # The feed-forward block of a transformer on a long batch of tokens: the largest products.
        _matrix("mlp", 65536, 1024, 4096, "bf16", 8),
        # The same in fp32 on a ragged number of rows, from code that may not allocate.
        _matrix("mlp ragged", 3001, 512, 2048, "f32", 4, graph=False, call="static"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    chain = rng.choice(["tiny", "resnet18", "resnet18", "vgg16", "vgg16", "detector720p", "detector720p", "mbv2", "mbv2",
                        "mlp", "mlp"])
    graph, copy = rng.random() < 0.6, rng.random() < 0.6
    call = rng.choice(["free", "free", "free", "ordered"])
    if chain == "mlp":
        dtype = rng.choice(["bf16", "bf16", "f32"])
        # Matrix rows are tokens: any number. Columns are model widths: multiples of the 16-byte vector.
        m = _log(rng, 256, 65536 if dtype == "bf16" else 8192)
        k, hidden = 8 * _log(rng, 16, 128), 8 * _log(rng, 32, 512)
        c = _matrix("", m, k, hidden, dtype, rng.randint(1, 8), rng.choice(["independent", "reuse"]), graph, copy and m < 16384, call)
        if rng.random() < 0.2 and m <= 4096 and hidden <= 1024:
            c.update(call="static", graph=False, copy=False)
        del c["name"]
        return c
    mode = rng.choice(["independent", "reuse", "batched"])
    fuse, dtype = True, "bf16"
    if chain == "tiny":
        dtype = rng.choice(["f32", "bf16"])
        n, h, w, bands = 1, _log(rng, 20, 160), _log(rng, 20, 160), rng.randint(1, 6)
    elif chain == "resnet18":
        dtype = rng.choice(["f32", "bf16"])
        n, h, w, bands = rng.choice([1, 1, 2, 3]), _log(rng, 96, 320), _log(rng, 96, 320), rng.randint(1, 8)
    elif chain == "vgg16":
        n, h, w, bands = rng.choice([1, 1, 2]), _log(rng, 64, 288), _log(rng, 64, 288), rng.randint(1, 8)
    elif chain == "detector720p":
        n, h = 1, _log(rng, 180, 720)
        w, bands = min(1280, int(h * rng.uniform(1.0, 1.78))), rng.randint(2, 16)
    else:
        n, h, w, bands = rng.choice([1, 2, 4, 8]), _log(rng, 128, 640), _log(rng, 128, 640), rng.randint(1, 8)
        fuse = rng.random() < 0.6
        if mode == "batched":        # (its blocks have no launch that takes several bands)
            mode = "independent"
    c = _image("", chain, n, h, w, dtype, bands, mode, graph, copy, call, fuse)
    if chain in ("tiny", "resnet18") and mode != "batched" and n == 1 and h * w <= 224 * 224 and rng.random() < 0.2:
        c.update(call="static", graph=False, copy=False)
    del c["name"]
    return c


def _chain(case):
    if case["chain"] == "mlp":
        return workloads.mlp_chain(case["m"], case["k"], case["hidden"], case["dtype"], case["bands"])
    if case["chain"] == "tiny":
        c = workloads.tiny_chain()
        c.in_shape, c.dtype, c.n_bands = (case["n"], 16, case["h"], case["w"]), case["dtype"], case["bands"]
        return c
    return workloads.CONFIGS[case["chain"]](h=case["h"], w=case["w"], n=case["n"], n_bands=case["bands"], dtype=case["dtype"])


def _weights(chain):
    """He-normal weights and small biases, the same for every plan of a chain."""
    rng = np.random.default_rng(chain.seed)
    ws, bs = [], []
    for L in chain.layers:
        shape = (L.n, L.k) if hasattr(L, "n") else (L.c_out, L.c_in // L.groups) + tuple(L.k) if L.has_weight else None
        w = None
        if shape is not None:
            w = rng.standard_normal(shape, dtype=np.float32) * np.float32(math.sqrt(2.0 / math.prod(shape[1:])))
            w = workloads.to_bf16_values(w) if chain.dtype == "bf16" else w
        ws.append(w)
        bs.append(rng.uniform(-0.1, 0.1, shape[0]).astype(np.float32) if shape is not None else None)
    return workloads.Tensors(None, ws, bs)


class _Served:
    """A plan and what has to stay allocated for as long as it lives: every buffer passed to it."""

    def __init__(self, case):
        chain = _chain(case)
        flags = _MODES[case["mode"]] | (0 if case["fuse"] else lop.LOP_FLAG_NO_FUSE)
        flags |= (lop.LOP_FLAG_GRAPH if case["graph"] else 0) | (0 if case["copy"] else lop.LOP_FLAG_NO_D2H)
        make = lop.Plan.rowwise if case["chain"] == "mlp" else lop.Plan
        self.plan = make(chain, _weights(chain), flags=flags)
        self.stream = torch.cuda.Stream() if case["call"] == "ordered" else None
        self.buffers = []

    def __del__(self):
        # (the plan goes before the buffers and the stream that its last calls used)
        if getattr(self, "plan", None) is not None:
            self.plan.destroy()


_served = weakref.WeakValueDictionary()


def prepare(case, seed):
    key = repr(sorted((k, v) for k, v in case.items() if k != "name"))
    served = _served.get(key)
    if served is None:
        served = _served[key] = _Served(case)
    chain = _chain(case)
    n, c, h, w = chain.in_shape
    lo, hi = getattr(chain, "in_range", (-1.0, 1.0))
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = _TORCH[case["dtype"]]
    x = torch.empty((n, h, w, c), dtype=dt, device="cuda").uniform_(lo, hi, generator=gen)   # NHWC
    on, oc, oh, ow = served.plan.out_shape()
    out = torch.empty((on, oh, ow, oc), dtype=dt, device="cuda")
    host = torch.empty((on, oh, ow, oc), dtype=dt, pin_memory=True) if case["copy"] else None
    served.buffers.append((x, out, host))
    torch.cuda.synchronize()    # (the plan's own streams are not ordered behind torch's)
    return {"served": served, "call": case["call"], "x": x, "out": out, "host": host}


def run(state):
    served, x, out, host = state["served"], state["x"], state["out"], state["host"]
    if state["call"] == "static":
        served.plan.run_chain_static(x, out, torch.cuda.current_stream())
    else:
        served.plan.run_chain(x, out, host, served.stream)
    return {"device": out} if host is None else {"device": out, "host": host}


def work(case):
    """Every row of every layer once; input, weights and result (device and host) once."""
    chain = _chain(case)
    esz = 4 if case["dtype"] == "f32" else 2
    if case["chain"] == "mlp":
        m, out = case["m"], case["m"] * chain.layers[-1].n
        flops = sum(2.0 * m * L.k * L.n for L in chain.layers)
        weights = sum(L.k * L.n for L in chain.layers)
        read = m * case["k"]
    else:
        n, c, h, w = chain.in_shape
        sizes, flops, weights, read = [], 0.0, 0, n * c * h * w
        for L in chain.layers:
            ih, iw = (h, w) if L.input_from < 0 else sizes[L.input_from]
            oh, ow = ((i + 2 * p - d * (k - 1) - 1) // s + 1 for i, p, d, k, s in zip((ih, iw), L.p, L.d, L.k, L.s))
            sizes.append((oh, ow))
            if L.has_weight:
                per = L.c_in // L.groups * L.k[0] * L.k[1]
                flops += 2.0 * n * oh * ow * L.c_out * per
                weights += L.c_out * per
        out = n * sizes[-1][0] * sizes[-1][1] * chain.layers[-1].c_out
    return {"bytes": float(esz * (read + weights + out * (2 if case["copy"] else 1))), "flops": flops}


def tolerance(case):
    # fp32: sums of up to 4608 products over up to 21 layers in another order. bf16: one rounding per
    # layer, so a sum in another order moves an intermediate value by one unit in the last place
    # (2^-8) now and then.
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 1e-2}
