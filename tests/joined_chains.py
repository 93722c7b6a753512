"""Chains whose layers a merged chain joins into one launch, or runs in passes up to one of them, for the tests on the GPU
(results) and for those on the stand-in runtime (which launches they make)."""
import workloads
from paper_2507_05829_amd import lop

# (N, C, H, W), bands, flags, activations of the two layers
PAIRS = [
    ((1, 16, 1, 1), 1, 0, ("relu", "relu")),                                     # one pixel: padding alone around it
    ((1, 16, 8, 8), 2, 0, ("relu", "relu")), ((1, 16, 9, 17), 3, 0, ("none", "relu6")),   # a tile, and one pixel more
    ((3, 16, 33, 31), 5, 0, ("relu6", "none")), ((1, 16, 40, 50), 16, lop.LOP_FLAG_GRAPH, ("relu", "relu")),
    ((2, 16, 37, 70), 4, lop.LOP_FLAG_REUSE, ("relu", "relu")), ((1, 16, 61, 45), 4, lop.LOP_FLAG_BATCH_BANDS, ("relu", "relu")),
    ((1, 16, 190, 204), 3, 0, ("relu", "relu")),                                 # more tiles than compute units
]
# "first": from the caller's input to a buffer, "last": from a buffer to the caller's output (with independent bands each has
# slabs of its own there). "between" two buffers the second layer's output takes the input's place, and "read twice" the
# first layer's result is needed again: two launches.
AROUND = ["alone", "first", "last", "between", "read twice"]


def pair(shape, dtype, bands, acts, around):
    chain = workloads.Chain("pair", shape, dtype, bands)
    if around in ("last", "between"):
        chain.add(workloads.CONV, 16, 16, 1, 1, 0, act="relu")
    chain.add(workloads.CONV, 16, 16, 3, 1, 1, act=acts[0])
    chain.add(workloads.CONV, 16, 16, 3, 1, 1, act=acts[1])
    if around in ("first", "between"):
        chain.add(workloads.MAXPOOL, 16, 16, 3, 1, 1)
    if around == "read twice":
        chain.add(workloads.CONV, 16, 32, 1, 1, 0, act="none")
        chain.add(workloads.CONV, 16, 32, 1, 1, 0, act="none", input_from=len(chain.layers) - 3, residual_from=len(chain.layers) - 1)
    return chain


# channels, stride of the first layer, pooled, (N, C, H, W), bands, flags
FRONTS = [
    (32, 2, False, (1, 3, 37, 41), 1, 0),                                    # fewer tiles than XCDs
    (32, 2, False, (2, 3, 180, 333), 5, 0),                                  # an odd width: rows of the image start between two words
    (32, 1, False, (1, 3, 65, 63), 4, lop.LOP_FLAG_REUSE | lop.LOP_FLAG_GRAPH),
    (32, 1, False, (1, 3, 3, 150), 3, 0),                                    # bands of one row
    (64, 1, True, (1, 3, 96, 98), 3, 0), (64, 1, True, (3, 3, 70, 75), 4, lop.LOP_FLAG_REUSE),
    (64, 1, False, (1, 3, 90, 97), 2, lop.LOP_FLAG_BATCH_BANDS), (64, 2, True, (1, 3, 200, 231), 6, 0), (64, 2, False, (2, 3, 161, 190), 3, 0),
]
# The same (bands aside) for the walking kernel's sizes, and for more tiles than workgroups are resident (768 with 32
# channels, 512 with 64), so that each does several, the last of them cut at both borders.
WALKED_FRONTS = [
    (32, 2, False, (1, 3, 451, 433)), (32, 1, False, (1, 3, 221, 226)), (64, 1, True, (1, 3, 225, 223)), (64, 1, False, (2, 3, 150, 161)),
    (64, 2, True, (1, 3, 430, 447)), (64, 2, False, (1, 3, 433, 440)),
    (32, 2, False, (1, 3, 901, 931)), (32, 1, False, (1, 3, 451, 470)), (64, 1, True, (2, 3, 290, 287)), (64, 1, False, (1, 3, 271, 263)),
    (64, 2, True, (1, 3, 541, 523)), (64, 2, False, (1, 3, 541, 523)),
]
WALKED_AS = [(1, 0), (3, 0), (4, lop.LOP_FLAG_REUSE)]   # bands, flags of each


def front(c, s, pool, shape, bands, behind=False, acts=("relu", "relu"), pads=(1, 1), bias=True):
    chain = workloads.Chain("front", shape, "bf16", bands)
    chain.add(workloads.CONV, 3, c, 3, s, pads[0], act=acts[0], has_bias=bias)
    chain.add(workloads.CONV, c, c, 3, 1, pads[1], act=acts[1], has_bias=bias)
    if pool:
        chain.add(workloads.MAXPOOL, c, c, 2, 2, 0)
    if behind:
        chain.add(workloads.CONV, c, 32, 3, 1, 1, act="relu")
    return chain


# What else such a launch takes: channels, stride, pooled, (N, C, H, W), bands, paddings of the two layers, biases
FRONT_FORMS = [
    (32, 1, False, (1, 3, 45, 39), 2, (0, 0), True), (32, 2, False, (2, 3, 50, 61), 3, (2, 2), False), (32, 1, False, (1, 3, 33, 30), 2, (3, 0), True),
    (64, 1, True, (1, 3, 101, 99), 2, (0, 2), False), (64, 2, True, (1, 3, 190, 197), 3, (3, 0), True), (64, 1, False, (1, 3, 95, 90), 3, (2, 0), True),
    (32, 1, False, (1, 3, 1, 1), 1, (1, 1), True), (32, 2, False, (1, 3, 2, 1), 1, (1, 1), True), (32, 1, False, (1, 3, 1, 300), 1, (1, 1), True),
    (32, 2, False, (1, 3, 301, 2), 3, (1, 1), True), (32, 1, False, (300, 3, 4, 5), 2, (1, 1), True), (64, 1, True, (70, 3, 5, 3), 1, (1, 1), True),
]


# images, bands, flags; how often the chain below makes the launches of its first and of its last layers, and how many are
# first ones (all: whole passes)
PASSES = [(5, 1, 0, 2, 6), (5, 4, lop.LOP_FLAG_REUSE | lop.LOP_FLAG_GRAPH, 2, 6), (5, 3, 0, 3, 3), (3, 6, lop.LOP_FLAG_GRAPH, 2, 2), (1, 7, 0, 4, 3),
          (7, 1, 0, 4, 3), (7, 4, lop.LOP_FLAG_REUSE | lop.LOP_FLAG_GRAPH, 4, 3)]


def passes(n, bands):
    chain = workloads.Chain("passes", (n, 16, 1500 if n == 1 else 400, 640 if n == 1 else 420), "bf16", bands)
    chain.add(workloads.CONV, 16, 32, 3, 1, 1, act="relu")
    chain.add(workloads.CONV, 32, 32, 3, 1, 1, act="relu")
    cut = chain.add(workloads.CONV, 32, 32, 3, 2, 1, act="relu")
    chain.add(workloads.CONV, 32, 32, 3, 1, 1, act="relu")
    chain.add(workloads.CONV, 32, 32, 3, 1, 1, act="none", residual_from=cut)
    chain.add(workloads.CONV, 32, 64, 3, 2, 1, act="relu")
    return chain


# Chains of more merged launches than are enqueued without a graph, in every way that a captured chain can run: name -> chain, flags.
def _products(name, m, k, hidden, dtype, bands, layers):
    chain = workloads.RowChain(name, m, k, dtype, bands)
    for l in range(layers):
        chain.add(k if l % 2 else hidden, "relu")
    return chain


def _behind(chain, c, layers):
    for _ in range(layers):
        chain.add(workloads.CONV, c, c, 1, 1, 0, act="relu")
    return chain


REPLAYED = {
    "few rows": lambda: (_products("rows", 1031, 1000, 136, "bf16", 8, 5), 0),
    "passes over rows": lambda: (_products("rows", 20011, 64, 1704, "bf16", 7, 4), lop.LOP_FLAG_REUSE),
    "passes over rows, fp32": lambda: (_products("rows", 12011, 64, 1704, "f32", 8, 4), 0),
    "pair": lambda: (_behind(pair((1, 16, 40, 50), "f32", 5, ("relu", "relu"), "alone"), 16, 4), 0),
    "front": lambda: (_behind(front(32, 1, False, (1, 3, 65, 63), 4), 32, 4), lop.LOP_FLAG_REUSE),
    "passes up to a layer": lambda: (passes(7, 4), lop.LOP_FLAG_REUSE),
    "passes of bands up to a layer": lambda: (passes(3, 6), 0),
    "four launches of eight bands": lambda: (few_layers(4, 8), 0),
}
# ... and of no more than that, over few bands: enqueued by every call.
ENQUEUED = {
    "few rows": lambda: (_products("rows", 1031, 1000, 136, "bf16", 8, 4), 0),
    "passes over rows": lambda: (_products("rows", 20011, 64, 1704, "bf16", 7, 2), lop.LOP_FLAG_REUSE),
    "pair": lambda: (_behind(pair((1, 16, 40, 50), "f32", 4, ("relu", "relu"), "alone"), 16, 2), 0),
    "front": lambda: (_behind(front(32, 1, False, (1, 3, 65, 63), 4), 32, 2), lop.LOP_FLAG_REUSE),
}
# Chains whose launches' bands decide: 3 x 3 layers, bands -> whether a call in flight and one on a caller's stream enqueue it.
BY_BANDS = {(4, 4): (True, True), (4, 8): (False, True), (3, 8): (True, True), (3, 16): (False, True), (4, 16): (False, False), (2, 16): (True, True)}


def few_layers(layers, bands):
    chain = workloads.Chain("few", (1, 32, 64, 64), "f32", bands)
    for _ in range(layers):
        chain.add(workloads.CONV, 32, 32, 3, 1, 1, act="relu")
    return chain


# Matrix products whose last round of 256 x 256 tiles is nearly empty: rows, elements, channels, residual
THIN = [
    (8400, 520, 2040, False),     # nine stages, the last of 8 elements; 44 x 8 tiles, those of the last row and column cut
    (8400, 520, 2040, True),      # a workgroup per tile
    (8448, 256, 2048, False),     # whole tiles, the shortest reduction
]
