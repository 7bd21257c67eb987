"""The fp32 combine, term by term: every product of an input and a weight is
held to fp32's precision whatever the size of its neighbours, so inputs whose
large entries meet small weights (and the other way round) come out as exact as
ordinary ones.  Each row against float64 within TERM_TOL, at many rows (fp16
parts on the matrix cores) and at few (fp32 matrix cores), twice with the same
bits.

TERM_TOL: a term is off by at most 2^-21 of itself (each operand's two parts
miss 2^-23 of it, the product left out is below 2^-22 of the term), 4.8e-7 of a
row's norm if all terms were off in the same direction; the fp32 sums of a few
hundred terms add about 1e-7, rounding at random.  1e-6 covers both."""
import numpy as np
import pytest

import workloads as W
from test_gpu_combine_f32 import _combine
from test_gpu_parity import G, say  # noqa: F401  (G is a fixture)

pytestmark = pytest.mark.gpu

TERM_TOL = 1e-6
# every tile shape: 32, 64 and 96 rows by 256 columns, 64 and 128 by 128; and the
# six products that narrow calls take
MANY = [(2_600, 130, 256), (10_500, 70, 200), (20_902, 66, 256), (6_000, 72, 96), (20_000, 80, 128), (11_000, 70, 40)]
FEW = [(96, 130, 256)]


def _inputs(m, d_in, d_out, seed):
    rng = np.random.default_rng(seed)
    S, A = (rng.standard_normal((m, d_in)).astype(np.float32) for _ in range(2))
    return rng, S, A, W.glorot(d_in, d_out, "f32", seed=d_out)


def _check(G, S, A, Wt, what):
    got = _combine(G, S, A, Wt, False)
    assert np.array_equal(got, _combine(G, S, A, Wt, False)), f"{what}: two runs differ"
    got = got.astype(np.float64)
    z = np.concatenate([S, A], axis=1).astype(np.float64) @ Wt.astype(np.float64)
    assert np.isfinite(got).all(), what
    err = np.linalg.norm(got - z, axis=1) / np.linalg.norm(z, axis=1)
    print(f"[rows] {what}: worst relative error {err.max():.3e} (tolerance {TERM_TOL:.0e})", flush=True)
    assert err.max() <= TERM_TOL, f"{what}: row {int(err.argmax())} off by {err.max():.3e}"


@pytest.mark.parametrize("m,d_in,d_out", MANY + FEW)
@pytest.mark.parametrize("x,w", [(1e34, 1e-26), (1e37, 1e-33), (1e-26, 1e34), (1e-30, 1e30)])
def test_scales_are_undone_without_overflow(G, m, d_in, d_out, x, w):
    """Rows and weights far apart whose products are ordinary numbers."""
    say("combine f32 scales", m, d_in, d_out, x, w)
    _, S, A, Wt = _inputs(m, d_in, d_out, m)
    _check(G, S * np.float32(x), A * np.float32(x), Wt * np.float32(w), f"rows {x:g}, weights {w:g}")


@pytest.mark.parametrize("m,d_in,d_out", MANY + FEW)
@pytest.mark.parametrize("half", ["self", "agg", "both"])
@pytest.mark.parametrize("columns", [1, 5])
@pytest.mark.parametrize("p", [-24, -21, 10, 20, 30, 40])
def test_raw_columns_with_weights_to_match(G, m, d_in, d_out, half, columns, p):
    """A few features 2^p times the others, their weights 2^-p times (2^-21 and
    2^-24: at the lower end of the fp16 parts, the low ones subnormal)."""
    say("combine f32 raw columns", m, d_in, d_out, half, columns, p)
    rng, S, A, Wt = _inputs(m, d_in, d_out, abs(p))
    for x, w, name in ((S, Wt[:d_in], "self"), (A, Wt[d_in:], "agg")):
        if half in (name, "both"):
            k = rng.choice(d_in, columns, replace=False)
            x[:, k] *= np.float32(2.0 ** p)
            w[k] *= np.float32(2.0 ** -p)
    _check(G, S, A, Wt, f"{columns} columns of {half} by 2^{p}")


@pytest.mark.parametrize("m,d_in,d_out", MANY + FEW)
@pytest.mark.parametrize("kind", ["zero_weights", "some_zero_weights", "zero_feature", "tiny_weight", "small_rest"])
def test_large_entries_that_do_not_count(G, m, d_in, d_out, kind):
    """Large entries whose partner is zero (or all but): the small rest is the result."""
    say("combine f32 large entries", m, d_in, d_out, kind)
    rng, S, A, Wt = _inputs(m, d_in, d_out, 7)
    k = d_in // 3
    if kind == "zero_weights":          # a raw column no output reads
        S[:, k] *= np.float32(2.0 ** 27)
        Wt[k] = 0
    elif kind == "some_zero_weights":   # one that half of the outputs read
        A[:, k] *= np.float32(2.0 ** 30)
        Wt[d_in + k, ::2] = 0
        Wt[d_in + k, 1::2] *= np.float32(2.0 ** -30)
    elif kind == "zero_feature":        # huge weights on a feature that is always zero
        S[:, k] = 0
        Wt[k] *= np.float32(2.0 ** 40)
    elif kind == "tiny_weight":         # the same the other way round
        S[:, k] *= np.float32(2.0 ** -40)
        Wt[k] *= np.float32(2.0 ** 40)
    elif kind == "small_rest":          # one entry of 2^40 in one row that meets a zero weight
        S[m // 2, k] = np.float32(2.0 ** 40)
        Wt[k] = 0
    _check(G, S, A, Wt, kind)


@pytest.mark.parametrize("m,d_in,d_out", MANY)
@pytest.mark.parametrize("count", [1, 32, 33, 500])
@pytest.mark.parametrize("size", ["small", "large", "both"])
def test_outliers_of_one_tile(G, m, d_in, d_out, count, size):
    """Single entries far outside the range of the rows around them, their
    column's weights scaled to match: `count` of them among 32 rows."""
    say("combine f32 outliers", m, d_in, d_out, count, size)
    rng, S, A, Wt = _inputs(m, d_in, d_out, count)
    small, large = rng.choice(d_in, 2, replace=False)
    S[:, small] = 0
    A[:, large] = 0
    Wt[small] *= np.float32(2.0 ** 45)
    Wt[d_in + large] *= np.float32(2.0 ** -45)
    rows = (m // 64) * 32 + np.resize(rng.permutation(32), count)
    if size != "large":
        S[rows[::2], small] = np.float32(1.25 * 2.0 ** -45)
    if size != "small":
        A[rows[1::2] if count > 1 else rows, large] = np.float32(-1.75 * 2.0 ** 45)
    _check(G, S, A, Wt, f"{count} {size} outliers")


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("m,d_in,d_out,ld_extra", [
    (2_601, 65, 256, 0), (2_688, 127, 250, 1), (10_496, 128, 192, 0), (10_497, 66, 256, 3), (20_929, 129, 255, 0),
    (24_576, 128, 256, 1), (5_153, 129, 500, 0), (5_120, 192, 128, 0), (5_185, 193, 127, 1), (16_384, 65, 65, 0),
    # either side of where narrow and short rows go to the six products
    (32_768, 100, 128, 0), (32_769, 100, 128, 0), (40_000, 257, 100, 1), (2_600, 64, 256, 0), (16_384, 100, 64, 0),
    (9_000, 256, 384, 0), (9_000, 257, 300, 0), (9_000, 100, 385, 3)])
def test_edges(G, m, d_in, d_out, ld_extra, relu):
    """Rows, widths and columns around a tile, a step and a column group."""
    say("combine f32 edges", m, d_in, d_out, ld_extra, relu)
    _, S, A, Wt = _inputs(m, d_in, d_out, m + d_in)
    z = np.concatenate([S, A], axis=1).astype(np.float64) @ Wt.astype(np.float64)
    scale = np.linalg.norm(z, axis=1)
    got = _combine(G, S, A, Wt, relu, ld_extra)
    err = np.linalg.norm(got - (np.maximum(z, 0) if relu else z), axis=1) / scale
    assert err.max() <= TERM_TOL, f"row {int(err.argmax())} off by {err.max():.3e}"


@pytest.mark.parametrize("n", [60_000, 20_000])
def test_rows_counted_on_the_device(G, n):
    """An asynchronous sample leaves the row count on the device, where the tile
    height is chosen by it (96 rows for some 21,000 of a bound of 26,624, 64 for
    some 14,000): the same bits as with the count on the host."""
    import torch
    from test_gpu_parity import dev, graph_case, host, padded
    say("combine f32 counted", n)
    _, u, v = graph_case(f"random-{n}-{n * 40}-3")
    g = G.Graph(n, u, v)
    rng = np.random.default_rng(n)
    x = dev(padded(rng.standard_normal((n, 70)).astype(np.float32), "f32"))
    dims = [70, 256, 41]
    ws = [dev(W.glorot(a, b, "f32", seed=a)) for a, b in zip(dims[:-1], dims[1:])]
    seeds = dev(rng.permutation(n)[:1024].astype(np.int32))
    out = []
    for call in (G.sample, G.sample_async):
        blk = G.Blocks()
        call(g, seeds, [25, 10], 7, blk)
        logits = torch.zeros((1024, 41), device="cuda")
        G.sage_forward(blk, x, ws, dims, "f32", logits)
        torch.cuda.synchronize()
        blk.sync()
        say("rows", blk.sizes()[0])
        out.append(host(logits))
    assert out[0].any() and np.array_equal(*out)
