"""Checks of merged chains (the launches of all bands, or of several images' bands, in one) against
the stand-in HIP runtime: what a merged chain asks of its scratch and of the launchers, compared
with the same plan's bands run one by one. Run as `python merged.py <stub dir> <check>` with the
AddressSanitizer runtime preloaded (see build_stub.py). Kernels do nothing here, so tensors are
addresses only.
"""
import ctypes
import os
import sys
import types

stub_dir, check = sys.argv[1], sys.argv[2]
HERE = os.path.dirname(os.path.abspath(__file__))
sys.path[:0] = [stub_dir, os.path.dirname(os.path.dirname(HERE)), os.path.dirname(HERE)]
sys.modules["torch"] = types.ModuleType("torch")   # the binding imports it only for its runtime

import numpy as np  # noqa: E402

import workloads  # noqa: E402
import joined_chains as joined  # noqa: E402
from paper_2507_05829_amd import lop  # noqa: E402

assert lop.LIB_PATH.startswith(stub_dir), lop.LIB_PATH
stub = ctypes.CDLL(os.path.join(stub_dir, "paper_2507_05829_amd", "libhipstub.so"))
stub.hipstub_unordered.restype = ctypes.c_long
stub.hipstub_created.restype = ctypes.c_long
stub.hipstub_launched.restype = ctypes.c_char_p
stub.hipstub_launched.argtypes = [ctypes.c_long]
stub.hipstub_launched_workgroups.restype = ctypes.c_long
stub.hipstub_launched_workgroups.argtypes = [ctypes.c_long]
GRAPH_EXEC = 3
stub.hipstub_mark.argtypes = [ctypes.c_void_p]
stub.hipStreamCreateWithFlags.argtypes = [ctypes.c_void_p, ctypes.c_uint]
stub.hipStreamDestroy.argtypes = [ctypes.c_void_p]
_room = np.zeros(64, np.uint8)
TENSOR = (_room.ctypes.data + 15) & ~15


def conv_chain(dtype, shape, bands, layers):
    """layers: (c_out, k, stride, dilation), padded to keep the size at stride 1."""
    chain = workloads.Chain("merged", shape, dtype, bands)
    c = shape[1]
    for c_out, k, s, d in layers:
        chain.add(workloads.CONV, c, c_out, k, s, d * (k // 2), d, "relu")
        c = c_out
    return chain


def shrinking(dtype, shape, bands, c0, s1, s2, c1, k=5):
    """Three convolutions at growing stride and two with a large filter and few pixels behind them."""
    return conv_chain(dtype, shape, bands, [(c0, 3, 1, 1), (c0, 3, 1, 1), (128, 3, s1, 1), (c1, 3, s2, 1),
                                            (c1, k, 1, 1), (c1, k, 1, 1)])


class ZeroWeights:
    """Weights of a chain's shapes without values (one block of zeros serves every layer)."""

    def __init__(self, chain):
        shapes = [(L.c_out, L.c_in // L.groups) + tuple(L.k) for L in chain.layers]
        block = np.zeros(max(int(np.prod(s)) for s in shapes), np.float32)
        self.weights = [block[:int(np.prod(s))].reshape(s) if L.has_weight else None
                        for s, L in zip(shapes, chain.layers)]
        self.biases = [None] * len(shapes)


def make(chain, flags):
    return lop.Plan(chain, ZeroWeights(chain), None, flags | lop.LOP_FLAG_LANES(1))


def status(call):
    try:
        call()
    except lop.LopError as e:
        return e.code
    return 0


def run_both_ways(chain, flags):
    """Status of the whole chain, and of its bands run one by one."""
    plan = make(chain, flags)
    whole = status(lambda: plan.run_chain(TENSOR, TENSOR))
    bands = [status(lambda: plan.run_band(b, TENSOR, TENSOR)) for b in range(plan.n_bands)]
    plan.synchronize()
    plan.destroy()
    return whole, min(bands)


def random_chain(rng):
    dtype = str(rng.choice(["f32", "bf16"]))
    reuse = bool(rng.random() < 0.4)
    c0, c1 = int(rng.choice([12, 16, 24, 32, 40, 64])), int(rng.choice([72, 128, 192, 256]))
    n, bands = int(rng.choice([1, 2, 3, 5, 7, 8])), int(rng.integers(1, 8))
    h, w = int(rng.integers(48, 400)), int(rng.integers(48, 400))
    layers = [(c0, 3, 1, 1)]
    for _ in range(int(rng.integers(1, 5))):
        layers.append((int(rng.choice([c0, c1, 128])), int(rng.choice([1, 3, 3, 5, 7])), int(rng.choice([1, 2, 2, 4])),
                       int(rng.choice([1, 1, 2]))))
    layers.append((c1, int(rng.choice([5, 7])), 1, 1))
    return conv_chain(dtype, (n, int(rng.choice([3, 16, 24])), h, w), bands, layers), lop.LOP_FLAG_REUSE if reuse else 0


def workspace():
    """The partial sums of every launch a chain makes fit the workspace its plan holds: also those of
    a last pass over fewer images, which can be cut into more slices than the passes before it."""
    named = [("bf16", (3, 16, 240, 409), 5, 0, 32, 2, 4, 384, 5), ("f32", (8, 16, 119, 113), 5, 0, 64, 2, 4, 512, 5),
             ("f32", (5, 16, 336, 315), 5, lop.LOP_FLAG_REUSE, 16, 4, 4, 256, 7),
             ("bf16", (9, 16, 372, 406), 2, 0, 32, 2, 4, 256, 5)]
    bad = []
    for dtype, shape, bands, flags, *rest in named:
        got = run_both_ways(shrinking(dtype, shape, bands, *rest), flags)
        if got != (0, 0):
            bad.append((dtype, shape, got))
    rng = np.random.default_rng(77)
    for i in range(120):
        chain, flags = random_chain(rng)
        got = run_both_ways(chain, flags)
        if got[0] != got[1]:
            bad.append((i, chain, flags, got))
    return bad


def wide_tiles():
    """Bands that together are large enough for the widest tile, in a layer that only the tiled kernel takes
    (channel counts that are no multiple of 32, filters of 5 x 5, dilation)."""
    bad = []
    for shape, bands, layers in (((1, 24, 512, 512), 8, [(24, 3, 1, 1), (256, 3, 1, 1)]),
                                 ((1, 40, 512, 512), 4, [(40, 3, 1, 1), (192, 3, 1, 1)]),
                                 ((1, 64, 320, 320), 4, [(64, 3, 1, 1), (256, 5, 1, 1)]),
                                 ((2, 256, 224, 224), 4, [(256, 3, 1, 1), (256, 3, 1, 2)])):
        for flags in (0, lop.LOP_FLAG_GRAPH, lop.LOP_FLAG_REUSE, lop.LOP_FLAG_BATCH_BANDS):
            got = run_both_ways(conv_chain("bf16", shape, bands, layers), flags)
            if got != (0, 0):
                bad.append((shape, layers, flags, got))
    return bad


def static_scratch():
    """lop_run_chain_static takes every plan whose bands, one by one, fit the static array, and no other;
    lop_plan_stats says which. (A plan-only plan merges nothing, and these chains have no fused layers.)"""
    bad = []
    rng = np.random.default_rng(78)
    chains = [(shrinking("bf16", (2, 16, 201, 348), 3, 16, 2, 2, 256), 0)]
    for _ in range(150):
        d, n, h, w = str(rng.choice(["f32", "bf16"])), int(rng.integers(1, 9)), int(rng.integers(80, 420)), int(rng.integers(80, 420))
        chains.append((shrinking(d, (n, 16, h, w), int(rng.integers(1, 7)), int(rng.choice([16, 32, 64])), int(rng.choice([2, 4])),
                                 int(rng.choice([2, 4])), int(rng.choice([192, 256])), int(rng.choice([5, 7]))),
                       int(rng.choice([0, lop.LOP_FLAG_REUSE]))))
    taken = 0
    for chain, flags in chains:
        one_by_one = lop.Plan(chain, None, None, flags)
        fits = one_by_one.stats()[2] <= lop.LOP_STATIC_SCRATCH_BYTES
        one_by_one.destroy()
        plan = make(chain, flags)
        said = plan.stats()[2] <= lop.LOP_STATIC_SCRATCH_BYTES
        got = status(lambda: plan.run_chain_static(TENSOR, TENSOR))
        plan.destroy()
        taken += got == 0
        if got != (0 if fits else lop.LOP_ERR_TOO_LARGE) or said != fits:
            bad.append((chain, flags, fits, said, got))
    print(taken, "of", len(chains), "plans taken", flush=True)
    return bad


def new_stream():
    s = ctypes.c_void_p()
    assert stub.hipStreamCreateWithFlags(ctypes.byref(s), 1) == 0
    return s.value


def layer_by_layer(n):
    """A batch of the inverted-residual chain whose launches take one band each: its bands run one by
    one, and where `n` makes their results long, leave through the copy lane."""
    return workloads.mbv2_chain(h=192, w=192, n=n, n_bands=4)


def order_of_streams():
    """Bands that lop_run_band runs on a caller's stream use the lanes' scratch: whatever lop_run_chain
    launches next waits for that stream, with the copies on their own lane and without."""
    bad = []
    for chain, flags, copy in ((layer_by_layer(8), lop.LOP_FLAG_NO_FUSE, True), (layer_by_layer(8), lop.LOP_FLAG_NO_FUSE, False),
                               (layer_by_layer(2), lop.LOP_FLAG_NO_FUSE, True), (workloads.tiny_chain(), 0, False)):
        for graph in (0, lop.LOP_FLAG_GRAPH):
            plan = lop.Plan(chain, ZeroWeights(chain), None, flags | graph)
            on, oc, oh, ow = plan.out_shape()
            h_out = np.zeros(on * oc * oh * ow * 4 + 16, np.uint8)
            stub.hipstub_pin(ctypes.c_void_p(h_out.ctypes.data), ctypes.c_size_t(h_out.nbytes))
            host = (h_out.ctypes.data + 15) & ~15 if copy else None
            user, other = new_stream(), None
            for first in (True, False):
                for b in range(plan.n_bands):
                    plan.run_band(b, TENSOR, TENSOR, None, user)
                    if b == plan.n_bands - 4:      # (no lane's last band is earlier)
                        stub.hipstub_mark(user)
                plan.run_chain(TENSOR, TENSOR, host)
                if stub.hipstub_unordered():
                    bad.append((chain.name, chain.in_shape, flags | graph, copy, first, stub.hipstub_unordered()))
            # chains on two callers' streams in turn, and one on the plan's own (a replayed graph of a chain that
            # runs band by band uses every lane's scratch on the caller's stream; a merged chain one lane's)
            if chain.in_shape[0] == 8:
                other = new_stream()
                for mine, then in ((user, other), (other, user), (user, None)):
                    plan.run_chain(TENSOR, TENSOR, None, mine)
                    stub.hipstub_mark(mine)
                    plan.run_chain(TENSOR, TENSOR, host, then)
                    if stub.hipstub_unordered():
                        bad.append((chain.in_shape, flags | graph, copy, "chains", mine == user, then is None))
                stub.hipstub_mark(None)
            plan.synchronize()
            stub.hipstub_mark(None)
            plan.destroy()
            stub.hipstub_unpin(ctypes.c_void_p(h_out.ctypes.data))
            for s in (user, other):
                if s:
                    stub.hipStreamDestroy(s)
    return bad


def poison():
    """LOP_FLAG_POISON_SCRATCH fills the scratch before every pass of a merged chain: what a pass left
    behind is not there for the next one to read."""
    bad = []
    stub.hipstub_launches.restype = ctypes.c_long

    def launches(chain, flags):
        plan = make(chain, flags)
        before = stub.hipstub_launches()
        plan.run_chain(TENSOR, TENSOR)
        count = stub.hipstub_launches() - before
        plan.destroy()
        return count

    layers = [(64, 3, 1, 1)] * 3          # (one launch each, without partial sums)
    for shape, bands, flags, least in (((8, 64, 300, 300), 1, 0, 2), ((8, 64, 300, 300), 3, 0, 2), ((7, 64, 300, 300), 3, lop.LOP_FLAG_REUSE, 2),
                                       ((1, 64, 800, 1000), 9, 0, 2), ((1, 64, 64, 64), 2, 0, 1)):
        chain = conv_chain("bf16", shape, bands, layers)
        plain, poisoned = launches(chain, flags), launches(chain, flags | lop.LOP_FLAG_POISON_SCRATCH)
        if plain < 3 * least or plain % 3 or poisoned - plain != plain // 3:
            bad.append((shape, bands, flags, plain, poisoned))
    return bad


def grids():
    """Depthwise layers whose bands' launches fit the grid, and whose launch over all rows would not, and of more
    images than a launch takes (the stand-in ends the process on a grid that the runtime refuses). One whose single row is more
    than a launch takes is an error."""
    bad = []
    for dtype, shape, s in (("f32", (600, 4, 1030, 2), 1), ("bf16", (3000, 8, 90, 3), 2), ("f32", (1, 4, 600000, 1), 1),
                            ("bf16", (9000000, 4, 2, 1), 1), ("bf16", (17000000, 4, 1, 1), 1)):
        for flags in (0, lop.LOP_FLAG_REUSE):
            chain = workloads.Chain("depthwise", shape, dtype, min(4, shape[2]))
            for _ in range(2):
                chain.add(workloads.DWCONV, shape[1], shape[1], 3, s, 1, 1, "relu6")
            got = run_both_ways(chain, flags)
            if got != (0, 0):
                bad.append((shape, flags, got))
    for flags in (0, lop.LOP_FLAG_REUSE):
        chain = workloads.Chain("depthwise", (1, 1024, 2, 1 << 24), "bf16", 2)
        chain.add(workloads.DWCONV, 1024, 1024, 3, 1, 1, 1, "relu6")
        got = run_both_ways(chain, flags)
        if 0 in got:
            bad.append((chain.name, flags, got))
    return bad


def pinned(nbytes):
    buf = np.zeros(nbytes + 16, np.uint8)
    stub.hipstub_pin(ctypes.c_void_p(buf.ctypes.data), ctypes.c_size_t(buf.nbytes))
    return buf, (buf.ctypes.data + 15) & ~15


def copy_streams():
    """lop_synchronize also waits for the copy streams that lop_run_band was given."""
    chain = layer_by_layer(8)
    plan, probe = lop.Plan(chain, ZeroWeights(chain), None, lop.LOP_FLAG_NO_FUSE), make(workloads.tiny_chain(), 0)
    buf, host = pinned(int(np.prod(plan.out_shape())) * 4)
    compute, copies = new_stream(), new_stream()
    for b in range(plan.n_bands):
        plan.run_band(b, TENSOR, TENSOR, host, compute, copies)
    stub.hipstub_mark(copies)
    plan.synchronize()
    probe.run_chain(TENSOR, TENSOR)       # whatever comes after the wait is behind the copies
    bad = [stub.hipstub_unordered()] if stub.hipstub_unordered() else []
    stub.hipstub_mark(None)
    probe.destroy()
    plan.destroy()
    stub.hipstub_unpin(ctypes.c_void_p(buf.ctypes.data))
    for s in (compute, copies):
        stub.hipStreamDestroy(s)
    return bad


def timed_layer():
    """lop_time_layer waits for what the plan has in flight before it uses a lane's scratch."""
    chain = layer_by_layer(2)
    plan, user = lop.Plan(chain, ZeroWeights(chain)), new_stream()
    plan.run_chain(TENSOR, TENSOR, None, user)
    stub.hipstub_mark(user)
    plan.time_layer(0, plan.n_layers - 1, TENSOR, TENSOR, 2)
    bad = [stub.hipstub_unordered()] if stub.hipstub_unordered() else []
    stub.hipstub_mark(None)
    plan.destroy()
    stub.hipStreamDestroy(user)
    return bad


def matrix_rows():
    """A chain of matrix products is one launch per layer from 2048 rows on, or from 2^27 products of its largest layer on; below
    both its bands run one by one."""
    bad = []
    stub.hipstub_launches.restype = ctypes.c_long
    for m, k, hidden, bands, merged in ((2048, 128, 256, 4, True), (3001, 128, 256, 8, True), (20000, 64, 64, 4, True), (256, 1024, 1024, 4, True),
                                        (2047, 128, 256, 4, False), (257, 256, 1024, 3, False)):
        for dtype in ("bf16", "f32"):
            for flags in (0, lop.LOP_FLAG_REUSE):
                chain = workloads.RowChain("rows", m, k, dtype, bands).add(hidden, "relu").add(k, "none", residual_from=-1)
                weights = types.SimpleNamespace(weights=[np.zeros((L.n, L.k), np.float32) for L in chain.layers], biases=[None, None])
                plan = lop.Plan.rowwise(chain, weights, flags=flags)
                before = stub.hipstub_launches()
                plan.run_chain(TENSOR, TENSOR)
                count = stub.hipstub_launches() - before
                plan.destroy()
                if (count < 2 * bands) != merged:
                    bad.append((m, k, hidden, bands, dtype, flags, count))
    return bad


def kernels(plan, out=None, stream=None):
    """What a call launches, or captures: (name, workgroups along x) of each. The result lies apart from the input."""
    n, c, h, w = plan.out_shape()
    result = np.zeros(n * c * h * w * 4 + 16, np.uint8) if out is None else None
    stub.hipstub_forget()
    plan.run_chain(TENSOR, (result.ctypes.data + 15) & ~15 if out is None else out, None, stream)
    plan.synchronize()
    got = []
    while stub.hipstub_launched(len(got)) is not None:
        got.append((stub.hipstub_launched(len(got)).decode(), stub.hipstub_launched_workgroups(len(got))))
    return got


def plan_of(chain, flags):
    if not isinstance(chain, workloads.RowChain):
        return make(chain, flags)
    weights = types.SimpleNamespace(weights=[np.zeros((L.n, L.k), np.float32) for L in chain.layers], biases=[None] * len(chain.layers))
    return lop.Plan.rowwise(chain, weights, flags=flags | lop.LOP_FLAG_LANES(1))


def joined_launches():
    """The chains of joined_chains.py make the launches that their tests on the GPU are about: a pair or a first layer and the
    convolution behind it in one launch, over bands with slabs of their own where there are such, and with more tiles than workgroups
    where those are to take several."""
    bad = []

    def launches(chain, flags):
        plan = make(chain, flags)
        got = kernels(plan)
        plan.destroy()
        return got

    for dtype in ("f32", "bf16"):
        for shape, bands, flags, acts in joined.PAIRS:
            for around in joined.AROUND:
                names = [n for n, _ in launches(joined.pair(shape, dtype, bands, acts, around), flags)]
                want = {"alone": ["P"], "first": ["P", "-"], "last": ["-", "P"]}.get(around, ["-"] * 4)
                slabs = around in ("first", "last") and bands > 1 and not flags & lop.LOP_FLAG_REUSE
                if ["P" if "conv_pair_kernel" in n else "-" for n in names] != want or any("conv_pair_kernel_bands" in n for n in names) != slabs:
                    bad.append((shape, bands, flags, dtype, around, names))
    fronts = [(f, behind, flags) for *f, flags in joined.FRONTS for behind in (False, True)]
    walked = [([*f, bands], False, flags) for f in joined.WALKED_FRONTS for bands, flags in joined.WALKED_AS]
    several = set()
    for f, behind, flags in fronts + walked:
        c, s, pool, (n, _, h, w), bands = f
        got = launches(joined.front(*f, behind), flags)
        if ["F" if "conv_front_kernel" in name else "-" for name, _ in got] != ["F", "-"][:1 + behind]:
            bad.append((f, behind, flags, got))
        tiles = n * -(-h // s) * -(-w // s) / (256 if c == 32 else 128)      # (at least)
        if tiles > got[0][1] > 0 and got[0][1] <= (768 if c == 32 else 512):
            several.add((c, s, pool, "_bands" in got[0][0]))
    for c, s, pool, shape, bands, pads, bias in joined.FRONT_FORMS:
        got = launches(joined.front(c, s, pool, shape, bands, pads=pads, bias=bias), 0)
        if len(got) != 1 or "conv_front_kernel" not in got[0][0]:
            bad.append((c, s, pool, shape, bands, pads, got))
    forms = {(c, s, pool) for c, s, pool, _ in joined.WALKED_FRONTS}
    bad += [("no workgroup with several tiles", *f, b) for f in forms for b in (False, True) if (*f, b) not in several]
    for n, bands, flags, often, first in joined.PASSES:
        names = [name for name, _ in launches(joined.passes(n, bands), flags)]
        if len(names) != often * first + (6 - first) or sum("conv_igemm_kernel" in k for k in names) != often:   # (the first layer's)
            bad.append((n, bands, flags, names))
    return bad


def graphs():
    """LOP_FLAG_GRAPH captures merged chains of more than four launches, or of fewer over many bands, and enqueues the others by
    every call."""
    bad, user = [], new_stream()
    for (layers, bands), eager in joined.BY_BANDS.items():
        for stream, want in zip((None, user), eager):
            plan, before = plan_of(joined.few_layers(layers, bands), lop.LOP_FLAG_GRAPH), stub.hipstub_created(GRAPH_EXEC)
            kernels(plan, TENSOR, stream)
            if (stub.hipstub_created(GRAPH_EXEC) == before) != want:
                bad.append((layers, bands, stream is None, want))
            plan.destroy()
    stub.hipStreamDestroy(user)
    for chains, captured in ((joined.REPLAYED, 1), (joined.ENQUEUED, 0)):
        for name, build in chains.items():
            chain, flags = build()
            plan, before, counts = plan_of(chain, flags | lop.LOP_FLAG_GRAPH), stub.hipstub_created(GRAPH_EXEC), []
            for _ in range(3):
                counts.append(len(kernels(plan, TENSOR)))
            if stub.hipstub_created(GRAPH_EXEC) - before != captured or counts[0] == 0 or any((c == 0) != bool(captured) for c in counts[1:]):
                bad.append((name, captured, stub.hipstub_created(GRAPH_EXEC) - before, counts))
            plan.destroy()
    return bad


def alone():
    """Depthwise launches between a workgroup and one and a half to a compute unit: two columns a thread where chains of
    consecutive calls run beside each other, one where the chain is on a caller's stream or may not allocate. Matrix products whose last
    round of the largest tile is nearly empty: that tile beside other chains, the next smaller one on a caller's stream."""
    bad, user = [], new_stream()
    thin = []
    for m, k, n, residual in joined.THIN:
        chain = workloads.RowChain("thin", m, k, "bf16", 1).add(n, "none")
        thin.append(chain.add(n, "relu", residual_from=0, input_from=-1) if residual else chain)
    thin.append(workloads.RowChain("thin", 34816, 512, "bf16", 1).add(1024, "none").add(512, "none"))   # (too large to merge: one band, on its lane)
    for chain in thin:
        plan = plan_of(chain, 0)
        for stream, tile in ((None, "Li256ELi256E"), (user, "Li192ELi256E"), (None, "Li256ELi256E")):
            got = kernels(plan, None, stream)
            if len(got) != len(chain.layers) or any("conv_gemm_kernelIDF16b" + tile not in name for name, _ in got):
                bad.append((chain.m, tile, got))
        plan.destroy()
    for shape, s, free, own in (((1, 192, 160, 160), 1, 2, 1), ((1, 192, 224, 224), 2, 2, 1), ((1, 192, 128, 128), 1, 1, 1), ((1, 192, 192, 192), 1, 2, 2)):
        chain = workloads.Chain("depthwise", shape, "bf16", 1)
        chain.add(workloads.DWCONV, 192, 192, 3, s, 1, 1, "relu6")
        plan = make(chain, 0)
        static = lambda: (stub.hipstub_forget(), plan.run_chain_static(TENSOR, TENSOR), [(stub.hipstub_launched(0).decode(), 0)])[2]
        for got, want in ((kernels(plan), free), (kernels(plan, None, user), own), (static(), own), (kernels(plan), free)):
            if len(got) != 1 or ("column" in got[0][0]) != (want == 1):
                bad.append((shape, s, want, got))
        plan.destroy()
    stub.hipStreamDestroy(user)
    return bad


bad = {"joined_launches": joined_launches, "graphs": graphs, "alone": alone, "matrix_rows": matrix_rows, "copy_streams": copy_streams, "timed_layer": timed_layer, "grids": grids, "poison": poison, "order_of_streams": order_of_streams, "workspace": workspace, "wide_tiles": wide_tiles, "static_scratch": static_scratch}[check]()
for b in bad:
    print("FAILED", b, flush=True)
print("CHECK %s" % ("FAILED" if bad else "OK"), flush=True)
sys.exit(1 if bad else 0)
