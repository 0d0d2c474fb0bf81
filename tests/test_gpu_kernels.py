"""The kernels at the sizes where their tiling, remainders and dispatch rules change, against the CPU oracle."""
import sys

import numpy as np
import pytest

from oracle import ripple_oracle as O
from paper_2505_12112_amd import synth
from paper_2505_12112_amd.ripple import Ripple
from tests.harness import Pair, check_embeddings_conditioned, fp32_forward_bound, random_valid_batch

pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, file=sys.stderr, flush=True)


def _pair(rng, n, m, dims, agg, undirected=False, **kw):
    src, dst = synth.erdos_renyi(n, m, rng, undirected=undirected)
    x = rng.standard_normal((n, dims[0])).astype(np.float32)
    w = synth.model_weights(synth.ModelSpec(agg, tuple(dims), gin_eps=0.2 if agg == "gin" else 0.0), rng, bias_std=0.1)
    edge_w = synth.arc_weights(rng, src.size) if agg == "gc_wsum" else None
    return Pair(n, src, dst, x, w, undirected=undirected, edge_w=edge_w, **kw)


# Tiles of 2048 vertices up to 2^19, of 4096 beyond; by block index up to 256 tiles (2^20 vertices), then by ticket.
@pytest.mark.parametrize("n", [31, 2047, 2048, 2049, 2057, 70001, 1 << 19, (1 << 19) + 1, 1 << 20, (1 << 20) + 4099])
@pytest.mark.parametrize("mode", ["bucket", "recompute", "dense"])
def test_frontier_compaction_at_tile_edges(n, mode):
    _say("compaction", n, mode)
    rng = np.random.default_rng(n)
    p = _pair(rng, n, min(2 * n, n * (n - 1) // 4), (4, 5, 3), "sum", mode=mode)
    try:
        for bs in (min(n, 3), min(n, 400)):
            p.step(random_valid_batch(rng, p.orc, bs, 4))
        check_embeddings_conditioned(p)
    finally:
        p.close()


# Lane groups of 4 to 64 four-float lanes by row width; rows of more than 1024 in-arcs are summed by a block.
@pytest.mark.parametrize("width", [1, 3, 4, 5, 16, 17, 32, 33, 64, 65, 100, 128, 129, 256, 257, 512, 513, 1024])
@pytest.mark.parametrize("agg", ["mean", "gcn", "gc_wsum"])
def test_bootstrap_rows_of_every_width_and_length(width, agg):
    _say("bootstrap", width, agg)
    rng = np.random.default_rng(width)
    n = 3000
    keys = [np.arange(1, n, dtype=np.int64) * n]                                    # a hub of 2999 in-arcs
    for v, deg in ((1, 1024), (2, 1025), (3, 64), (4, 65), (5, 63), (6, 128), (7, 1), (8, 1500)):
        keys.append((np.sort(rng.choice(np.arange(100, n), deg, replace=False)) * n + v).astype(np.int64))
    s, t = synth.erdos_renyi(n, 9000, rng)
    rest = t > 8  # (vertices above 8 keep ordinary rows, some of them none)
    keys.append(s[rest].astype(np.int64) * n + t[rest])
    k = np.unique(np.concatenate(keys))
    src, dst = (k // n).astype(np.int32), (k % n).astype(np.int32)
    x = rng.standard_normal((n, width)).astype(np.float32)
    w = synth.model_weights(synth.ModelSpec(agg, (width, 3)), rng, bias_std=0.1)
    edge_w = synth.arc_weights(rng, src.size) if agg == "gc_wsum" else None
    p = Pair(n, src, dst, x, w, edge_w=edge_w)
    try:
        g = p.orc.graph
        c = 1.0 / np.sqrt(g.out_degree() + 1.0) if agg == "gcn" else np.ones(n)
        u, _ = g.arcs()
        a = g.in_adjacency(weights=c[u] * (g.w if agg == "gc_wsum" else 1.0))
        x64 = x.astype(np.float64)
        want, mag = a @ x64, abs(a) @ np.abs(x64)
        # summed in fp64 and rounded once: half a unit of the value, and of the fp64 sum of up to 3000 terms
        bound = 2.0 ** -24 * np.abs(want) + 4000 * 2.0 ** -53 * mag
        assert np.all(np.abs(p.lib.get_aggregates(1).astype(np.float64) - want) <= bound)
    finally:
        p.close()


def _hub_graph(rng, n):
    """Rows of 0, 1, 63, 64, 65, 128, 1024, 1025, 1500 and n - 1 in-arcs among ordinary ones."""
    keys = [np.arange(1, n, dtype=np.int64) * n]
    for v, deg in ((1, 1024), (2, 1025), (3, 64), (4, 65), (5, 63), (6, 128), (7, 1), (8, 1500)):
        keys.append((np.sort(rng.choice(np.arange(100, n), deg, replace=False)) * n + v).astype(np.int64))
    s, t = synth.erdos_renyi(n, 3 * n, rng)
    rest = (t > 8) & (s != t)
    keys.append(s[rest].astype(np.int64) * n + t[rest])
    k = np.unique(np.concatenate(keys))
    return (k // n).astype(np.int32), (k % n).astype(np.int32)


# The pulls' lane groups by message width (the first hidden width), on rows either side of the length that whole blocks
# sum; the sum and the weighted sum (coefficients per message). A message is added once per sink in fp32.
@pytest.mark.parametrize("width", [1, 16, 17, 32, 33, 47, 64, 65, 96, 97, 128, 129, 192, 193, 256, 257, 512, 513, 1024])
@pytest.mark.parametrize("mode,agg", [("pull", "sum"), ("dense", "gc_wsum"), ("recompute", "gcn"), ("dense", "mean")])
def test_pulled_messages_of_every_width_and_length(width, mode, agg):
    _say("pull", width, mode, agg)
    rng = np.random.default_rng(width)
    n = 3000
    src, dst = _hub_graph(rng, n)
    x = rng.standard_normal((n, 8)).astype(np.float32)
    w = synth.model_weights(synth.ModelSpec(agg, (8, width, 3)), rng, bias_std=0.1)
    edge_w = synth.arc_weights(rng, src.size) if agg == "gc_wsum" else None
    p = Pair(n, src, dst, x, w, edge_w=edge_w, mode=mode)
    try:
        for bs in (2, 120):
            p.step(random_valid_batch(rng, p.orc, bs, 8))
        check_embeddings_conditioned(p)
        p.check_aggregates()
    finally:
        p.close()


def _transform_reference(p, l=1):
    """Float64 pre-activation of layer l (no ReLU on a one-layer model) and the magnitude of each output's terms."""
    ref = p.orc.embeddings()[l]
    return ref, fp32_forward_bound(p.orc, p.orc.embeddings(), l)


def _check_fp32_rms(err, rss, k, more=0.0):
    """Errors of an fp32 sum of k products, given each output's root sum of squares: a running sum rounded k times is off by
    0.3 sqrt(k) units of 2^-24 of it (rms; sqrt(k / 6), times 0.72 for the mean place in a binade), and by `more` where the
    operands themselves are rounded. A sum whose weights lack their last bf16 part is off by 42 at any k (59 if both operands
    do), one of all nine part products but the three last by 0.1. Returns the errors in units."""
    e = err / (2.0 ** -24 * np.maximum(rss, 1e-30))
    rms = np.sqrt(np.mean(e * e))
    assert rms <= 0.3 * np.sqrt(k) + more, rms
    return e


def _check_transform(p, k, agg):
    """Layer 1 of a one-layer model against float64: half the forward error bound and, but for GIN's two products and rows
    shorter than a K step's half, the errors of an fp32 sum over the operand (its scales and sums are rounded: 1 unit)."""
    want, bound = _transform_reference(p)
    err = p.lib.get_embeddings(1).astype(np.float64) - want
    assert np.all(np.abs(err) <= 0.5 * bound[:, None] + 1e-30)
    if agg == "gin" or k < 16:
        return
    m, h = p.orc.model, p.orc.embeddings()[0]
    rss = O.aggregate(p.orc.graph, h, agg) ** 2 @ (m.w_neigh[0] ** 2).T + m.bias[0] ** 2
    if m.w_self[0] is not None:
        rss = rss + h ** 2 @ (m.w_self[0] ** 2).T
        k *= 2
    _check_fp32_rms(err, np.sqrt(rss), k, more=1.0)


# The transform of long row lists: column tiles of 16, 32, 48, 64 and 128, remainders of the 32-deep K steps and of the
# 128-row tiles, every operand form. 33,001 rows take the long-list kernel at every width.
@pytest.mark.parametrize("k,n_out", [(4, 16), (8, 17), (28, 32), (32, 33), (36, 47), (60, 48), (64, 49), (100, 64),
                                     (96, 65), (128, 128), (132, 130), (256, 256), (20, 3), (1, 5), (3, 47), (5, 33),
                                     (31, 70), (75, 130), (130, 131), (67, 19)])
@pytest.mark.parametrize("agg,tf", [("sum", 0), ("sum", 1), ("mean", 0), ("gcn", 0), ("gcn", 1), ("gc_sum", 0), ("gin", 0)])
def test_long_list_transform_matches_float64(k, n_out, agg, tf):
    _say("transform", k, n_out, agg, tf)
    rng = np.random.default_rng(k * 1000 + n_out)
    p = _pair(rng, 33001, 66000, (k, n_out), agg, transform_first=tf)
    try:
        _check_transform(p, k, agg)
        p.step(random_valid_batch(rng, p.orc, 50, k))
    finally:
        p.close()


# From 65536 rows on, outputs of whole pairs of 128 columns take 256-column tiles: one and a remainder of one, odd widths
# on either side, K of one step to nine, and with 1024 columns more tiles (2056) than blocks (2048).
@pytest.mark.parametrize("k,n_out,agg,tf", [(64, 129, "sum", 0), (67, 130, "gcn", 0), (128, 200, "mean", 0), (132, 256, "gc_sum", 0),
                                            (128, 385, "sum", 0), (257, 256, "gc_mean", 0), (100, 256, "gin", 0), (256, 200, "sum", 1),
                                            (75, 130, "gcn", 1), (1, 256, "sum", 0), (20, 256, "gcn", 0), (36, 1024, "gc_sum", 0)])
def test_wide_tile_transform_matches_float64(k, n_out, agg, tf):
    _say("wide tiles", k, n_out, agg, tf)
    rng = np.random.default_rng(k * 1000 + n_out)
    p = _pair(rng, 65667, 130000, (k, n_out), agg, transform_first=tf)
    try:
        _check_transform(p, k, agg)
    finally:
        p.close()


# The short-list transform on widths that are no multiple of 4 (rows at any 4-byte boundary, last chunks cut): few rows
# (eight waves a tile) and a few thousand (four).
@pytest.mark.parametrize("n", [90, 2500])
@pytest.mark.parametrize("k,n_out", [(1, 5), (2, 16), (3, 47), (5, 33), (31, 70), (75, 130), (130, 131), (67, 19), (509, 9)])
@pytest.mark.parametrize("agg,tf", [("sum", 0), ("sum", 1), ("mean", 0), ("gcn", 0), ("gcn", 1), ("gc_mean", 0), ("gin", 0)])
def test_short_list_transform_on_odd_widths(n, k, n_out, agg, tf):
    _say("short transform", n, k, n_out, agg, tf)
    rng = np.random.default_rng(k * 1000 + n_out + n)
    p = _pair(rng, n, 4 * n, (k, n_out, 3), agg, transform_first=tf)
    try:
        for l in (1, 2):
            want, bound = _transform_reference(p, l)
            err = np.abs(p.lib.get_embeddings(l).astype(np.float64) - want)
            assert np.all(err <= bound[:, None] + 1e-30)
        p.step(random_valid_batch(rng, p.orc, 20, k))
        check_embeddings_conditioned(p)
    finally:
        p.close()


# Infinities, NaNs and values past bf16's range reach exactly the outputs that fp32 arithmetic gives them.
@pytest.mark.parametrize("k,n_out", [(32, 128), (100, 47), (100, 256)])
@pytest.mark.parametrize("where", ["features", "weights"])
def test_long_list_transform_keeps_infinities_and_nans(k, n_out, where):
    _say("non-finite", k, n_out, where)
    rng = np.random.default_rng(k)
    n = 65667 if n_out == 256 else 33001  # 256-column tiles
    src, dst = synth.erdos_renyi(n, 40000, rng)
    x = rng.standard_normal((n, k)).astype(np.float32)
    w = synth.model_weights(synth.ModelSpec("gc_sum", (k, n_out)), rng, bias_std=0.1)
    if where == "features":
        x[5, 3], x[700, 0], x[12345, k - 1], x[33000, 1] = np.inf, -np.inf, np.nan, 3.4e38
        w.w_neigh[0][:, 1] *= 1e-3
    else:
        w.w_neigh[0][2, 5], w.w_neigh[0][7, 0] = np.inf, np.nan
    p = Pair(n, src, dst, x, w)
    try:
        agg = np.zeros((n, k))
        with np.errstate(invalid="ignore"):
            np.add.at(agg, dst, x[src].astype(np.float64))
            want = np.zeros((n, n_out))
            for i in range(k):  # term by term: a matrix product may reorder infinities into NaNs
                want += agg[:, i:i + 1] * w.w_neigh[0][:, i].astype(np.float64)
            want += w.bias[0]
        got = p.lib.get_embeddings(1)
        np.testing.assert_array_equal(np.isnan(got), np.isnan(want))
        inf = np.isinf(want)
        np.testing.assert_array_equal(got[inf], want[inf])
        fine = np.isfinite(want)
        mag = np.abs(np.nan_to_num(agg, nan=0, posinf=0, neginf=0)) @ np.abs(np.nan_to_num(w.w_neigh[0], nan=0, posinf=0)).T + 1
        assert np.all(np.abs(got[fine] - want[fine]) <= ((k + 16) * 2.0 ** -23 * mag)[fine])
    finally:
        p.close()


# Reads through the pinned buffer (ids and rows up to 1 MiB) and past it, and scatter-built lists sorted from either side
# of the radix sort's threshold (128 ids) and digits (2048): the same rows and sets as whole reads and the oracle give.
@pytest.mark.parametrize("count", [1, 2, 127, 4096, 15887, 15888, 15900, 40000])
def test_reads_of_every_size(count):
    _say("reads", count)
    rng = np.random.default_rng(count)
    p = _pair(rng, 50000, 100000, (12, 16, 9), "sum", mode="push")
    try:
        p.step(random_valid_batch(rng, p.orc, min(count, 900), 12))
        for layer in range(3):
            ids = rng.integers(0, 50000, count).astype(np.int32)
            whole = p.lib.get_embeddings(layer)
            np.testing.assert_array_equal(p.lib.get_embeddings(layer, ids), whole[ids])
            np.testing.assert_array_equal(p.lib.get_embeddings_static(layer, ids), whole[ids])
        np.testing.assert_array_equal(p.lib.get_aggregates(1, ids), p.lib.get_aggregates(1)[ids])
    finally:
        p.close()


class _OneLayer:
    """A one-layer GraphConv-sum model without a bias."""

    def __init__(self, w):
        self.agg, self.dims, self.w_self, self.w_neigh = "gc_sum", (w.shape[1], w.shape[0]), [None], [w]
        self.bias, self.relu, self.w_out, self.b_out, self.gin_eps = [np.zeros(w.shape[0], np.float32)], [False], [], [], 0.0


def _ring_transform(x, w):
    """The transform alone: on a ring every aggregate row is one row of x. The library's output, W times the aggregates in
    float64, and the magnitudes of each output's terms."""
    n = x.shape[0]
    v = np.arange(n, dtype=np.int32)
    lib = Ripple(n, v, (v + 1) % n)
    try:
        lib.init_embeddings(x, _OneLayer(w), transform_first=0)
        got = lib.get_embeddings(1).astype(np.float64)
    finally:
        lib.close()
    s, w64 = np.roll(x, 1, axis=0).astype(np.float64), w.astype(np.float64)
    return got, s @ w64.T, np.abs(s) @ np.abs(w64).T


# Long row lists at column tiles of 48, 128 and (from 65536 rows) 256.
LONG_LISTS = [(33001, 48), (33001, 128), (65667, 256)]


# A product inside the fp32 range whose operands' first bf16 parts, rounded up, have an infinite one.
@pytest.mark.parametrize("n,n_out", LONG_LISTS)
@pytest.mark.parametrize("k", [32, 100])
def test_long_list_transform_at_the_end_of_the_range(n, n_out, k):
    _say("range", n, k, n_out)
    rng = np.random.default_rng(k)
    x, w = (rng.standard_normal(s).astype(np.float32) for s in ((n, k), (n_out, k)))
    x[7], w[5] = 0, 0
    x[7, 3] = w[5, 3] = (2 - 2.0 ** -9) * 2.0 ** 63
    x[70], w[9] = 0, 0
    x[70, :2], w[9, :2] = 0.99 * 2.0 ** 67, 2.0 ** 60  # two products in the last binade but one
    got, want, mag = _ring_transform(x, w)
    assert 3.3e38 < want[8, 5] < 3.4e38 and 3.3e38 < want[71, 9] < 3.4e38
    assert np.all(np.abs(got - want) <= (k + 16) * 2.0 ** -24 * mag)


# Operands whose low bf16 parts would be denormals (unscaled, 2^-118 loses the last bits and 2^-128 most of them), on
# either side, against ones large enough that every result is an ordinary number. The bound is fp32's.
@pytest.mark.parametrize("n,n_out", LONG_LISTS)
@pytest.mark.parametrize("x_exp,w_exp", [(-118, 40), (-128, 60), (40, -118), (60, -128), (-146, 90), (0, 0)])
def test_long_list_transform_of_tiny_operands(n, n_out, x_exp, w_exp):
    _say("tiny", n, n_out, x_exp, w_exp)
    rng = np.random.default_rng(n_out)
    k = 64
    x = (rng.standard_normal((n, k)) * 2.0 ** x_exp).astype(np.float32)
    w = (rng.standard_normal((n_out, k)) * 2.0 ** w_exp).astype(np.float32)
    got, want, mag = _ring_transform(x, w)
    assert np.all(np.abs(got - want) <= (k + 16) * 2.0 ** -24 * mag)


# K of one step of 32, two, five and sixteen: the signs of the steps balance, or nearly, or cannot. No side is favoured: the
# mean of the row means is within six of its standard errors of zero, over all rows and over even and odd ones (an error on
# one side adds up over a sink's neighbours). Without a bias: adding one constant to every row rounds all of them alike.
@pytest.mark.parametrize("n,n_out", LONG_LISTS)
@pytest.mark.parametrize("k", [20, 64, 132, 512])
def test_long_list_transform_has_the_errors_of_an_fp32_sum(n, n_out, k):
    _say("errors", n, k, n_out)
    rng = np.random.default_rng(k)
    x, w = (rng.standard_normal(s).astype(np.float32) for s in ((n, k), (n_out, k)))
    got, want, _ = _ring_transform(x, w)
    rss = np.sqrt(np.roll(x, 1, axis=0).astype(np.float64) ** 2 @ (w.astype(np.float64) ** 2).T)
    rows = _check_fp32_rms(got - want, rss, k).mean(axis=1)
    for part in (rows, rows[0::2], rows[1::2]):
        assert abs(part.mean()) <= 6.0 * part.std() / np.sqrt(part.size), (part.mean(), part.std() / np.sqrt(part.size))


# Equal messages, whose fp32 sums are off on one side by up to half a unit of 2^-24 of the sum per addition, into sinks of
# few and of very many in-arcs. Additions in a row: a group's share of 1024 in-arcs (groups of up to 16 lanes); its share
# of 64, then 16 such sums (32 and 64 lanes); its share of 64 for rows that a block sums, in fp64 from there. Then the
# groups (at most 4 levels), the row and the rounding.
@pytest.mark.parametrize("width,lanes", [(16, 4), (32, 8), (64, 16), (96, 8), (100, 32), (160, 16), (256, 64), (512, 64)])
@pytest.mark.parametrize("mode", ["pull", "dense"])
def test_pulled_messages_of_hubs_are_summed_in_blocks(width, lanes, mode):
    _say("hub sums", width, mode)
    n, degs = 62000, np.array([60000, 1024, 1025, 500, 64])
    src = np.concatenate([np.arange(100, 100 + d, dtype=np.int32) for d in degs])
    dst = np.repeat(np.arange(degs.size, dtype=np.int32), degs)
    lib = Ripple(n, src, dst)
    try:
        lib.init_embeddings(np.zeros((n, width), np.float32), _OneLayer(np.ones((3, width), np.float32)), transform_first=0)
        lib.set_scatter_mode(mode)
        ops = np.full((60000, 4), -1, np.int32)
        ops[:, 0], ops[:, 1], ops[:, 3] = 3, np.arange(100, 60100), np.arange(60000)
        message = np.float32(1 + 0.9 * 2.0 ** -11)  # sums from 2^13 on round most of its low bits off, always down
        lib.apply_updates(ops, np.full((60000, width), message, np.float32))
        got = lib.get_aggregates(1, np.arange(degs.size, dtype=np.int32)).astype(np.float64)
    finally:
        lib.close()
    want = degs[:, None] * np.float64(message)
    groups = 64 // lanes
    chain = np.where(degs > 1024, 64 // groups, 64 // groups + 16 if lanes >= 32 else 1024 // groups)
    assert np.all(np.abs(got - want) <= (chain + 6)[:, None] * 2.0 ** -24 * want)
