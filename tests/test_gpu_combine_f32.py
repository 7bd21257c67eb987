"""The fp32 combine of many rows (three products of two fp16 parts per value, or
six of three bf16 parts, as the sizes say) at the edges of its tiles and of its
number range: rows, widths and columns around
one block, step and column group; NaN in the row padding; output rows that are
not 16-byte aligned, with guard words; and data whose rows, columns or halves
differ by powers of two up to 2^60, where tiles of the fp16 parts must fall back
to the bf16 split.  Against float64, 1e-5 per row as everywhere."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from parity_util import FP32_TOL, assert_rows_close
from test_gpu_parity import G, dev, host, padded, say  # noqa: F401  (G is a fixture)

pytestmark = pytest.mark.gpu

CASES = [(10_240, 1, 8, 0), (10_241, 15, 32, 1), (10_303, 16, 33, 0), (10_305, 17, 64, 0), (5_121, 63, 65, 0),
         (5_152, 64, 96, 1), (5_185, 65, 128, 0), (3_649, 127, 129, 3), (2_561, 128, 256, 0), (8_192, 129, 250, 0),
         (8_193, 192, 256, 0), (16_385, 200, 256, 1), (24_576, 33, 256, 0), (24_577, 100, 257, 0), (33_000, 300, 128, 0),
         (2_600, 602, 300, 0)]


def _combine(G, S, A, Wt, relu, ld_extra=0, pad_nan=True):
    import torch
    m, d_in = S.shape
    d_out = Wt.shape[1]
    Sp, Ap = padded(S, "f32"), padded(A, "f32")
    if pad_nan:
        Sp[:, d_in:] = Ap[:, d_in:] = np.nan
    out = torch.full((m + 1, d_out + ld_extra), -7.0, device="cuda")
    G.combine(dev(Sp), dev(Ap), m, d_in, dev(Wt), d_out, "f32", relu, False, out)
    got = host(out)
    assert (got[m] == -7.0).all() and (got[:, d_out:] == -7.0).all()
    return got[:m, :d_out]


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("m,d_in,d_out,ld_extra", CASES)
def test_combine_f32_edges(G, m, d_in, d_out, ld_extra, relu):
    say("combine f32", m, d_in, d_out, ld_extra, relu)
    assert G.combine_kernel(m, d_out, "f32") == "split"
    S, A = W.features(m, d_in, "f32", seed=m + d_in), W.features(m, d_in, "f32", seed=m + d_in + 1)
    Wt = W.glorot(d_in, d_out, "f32", seed=d_out)
    z = np.concatenate([O.to_f64(S, "f32"), O.to_f64(A, "f32")], axis=1) @ O.to_f64(Wt, "f32")
    assert_rows_close(_combine(G, S, A, Wt, relu, ld_extra), np.maximum(z, 0) if relu else z, FP32_TOL, "combine f32")


@pytest.mark.parametrize("kind", ["rows", "columns", "agg_small", "agg_large", "tiny", "huge", "weights", "zero_rows",
                                  "one_large_value"])
@pytest.mark.parametrize("m,d_in,d_out", [(2_600, 130, 256), (6_000, 40, 96), (11_000, 70, 40)])
def test_combine_f32_number_range(G, m, d_in, d_out, kind):
    say("combine f32 range", m, d_in, d_out, kind)
    rng = np.random.default_rng(m + len(kind))
    S, A = (rng.standard_normal((m, d_in)).astype(np.float32) for _ in range(2))
    Wt = W.glorot(d_in, d_out, "f32", seed=d_out)

    def powers(lo, hi, shape):
        return np.exp2(rng.integers(lo, hi, shape)).astype(np.float32)
    if kind == "rows":
        f = powers(-30, 31, (m, 1))
        S, A = S * f, A * f
    elif kind == "columns":
        f = powers(-12, 13, (1, d_in))
        S, A = S * f, A * f
    elif kind == "agg_small":
        A = A * np.float32(2.0 ** -40)
        Wt[:d_in] *= np.float32(2.0 ** -40)      # both halves weigh the same in the result
    elif kind == "agg_large":
        A = A * np.float32(2.0 ** 40)
    elif kind == "tiny":
        S, A = S * np.float32(1e-30), A * np.float32(1e-30)
    elif kind == "huge":
        S, A, Wt = S * np.float32(1e30), A * np.float32(1e30), Wt * np.float32(1e-20)
    elif kind == "weights":
        Wt = Wt * powers(-30, 31, (1, d_out))
    elif kind == "zero_rows":
        S[::3] = 0
        A[::2] = 0
    elif kind == "one_large_value":
        S[m // 3, d_in // 2] = np.float32(1e9)
    got = _combine(G, S, A, Wt, False)
    z = np.concatenate([S.astype(np.float64), A.astype(np.float64)], axis=1) @ Wt.astype(np.float64)
    if kind == "rows":                           # rows of very different norms: each against its own
        scale = np.maximum(np.linalg.norm(z, axis=1, keepdims=True), 1e-300)
        got, z = got / scale, z / scale
    if kind == "weights":                        # and columns
        scale = np.linalg.norm(z, axis=0, keepdims=True)
        got, z = got / scale, z / scale
    assert_rows_close(got, z, FP32_TOL, "combine f32 range")
    assert (got[(np.abs(S).sum(1) + np.abs(A).sum(1)) == 0] == 0).all()
