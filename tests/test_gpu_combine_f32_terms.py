"""The fp32 combine on rows and weights whose sizes lie far apart, each row
against float64 within TERM_TOL (the operands' parts miss 2^-23 of a value
each, the fp32 sums of a few hundred terms add about 1e-7), at many rows and at
few."""
import numpy as np
import pytest

import workloads as W
from test_gpu_combine_f32 import _combine
from test_gpu_parity import G, say  # noqa: F401  (G is a fixture)

pytestmark = pytest.mark.gpu

TERM_TOL = 1e-6
MANY = [(2_600, 130, 256), (6_000, 40, 96), (11_000, 70, 40)]
FEW = [(96, 130, 256)]


def _inputs(m, d_in, d_out, seed):
    rng = np.random.default_rng(seed)
    S, A = (rng.standard_normal((m, d_in)).astype(np.float32) for _ in range(2))
    return rng, S, A, W.glorot(d_in, d_out, "f32", seed=d_out)


def _check(G, S, A, Wt, what):
    got = _combine(G, S, A, Wt, False).astype(np.float64)
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
