"""The streaming bf16 combine (weights in registers, row tiles through LDS) at
the edges of its tiles and of its rule: row counts around one tile and around
one tile per compute unit, input widths around one k step and around each
register budget, output widths around one column group, bf16 and fp32 outputs
with guard words behind every row, and NaN in the row padding it must not
read into a result."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from parity_util import BF16_TOL, assert_rows_close
from test_gpu_parity import G, dev, host, padded, say  # noqa: F401  (G is a fixture)

pytestmark = pytest.mark.gpu

CASES = [(10_240, 1, 8), (10_241, 8, 16), (10_303, 15, 32), (10_304, 16, 40), (10_305, 17, 64), (5_121, 100, 72),
         (5_152, 112, 128), (3_649, 128, 136), (2_561, 127, 200), (2_561, 128, 256), (16_384, 128, 256),
         (16_385, 128, 256), (8_193, 129, 256), (8_192, 256, 256), (2_593, 250, 248), (10_272, 200, 48),
         (5_153, 256, 96), (2_600, 96, 264), (33_000, 128, 64), (16_448, 257, 64),
         # either side of where the ring takes over again
         (32_768, 130, 72), (32_769, 130, 72), (16_384, 144, 16), (16_385, 144, 16), (10_240, 200, 64), (65_536, 40, 8),
         (65_537, 40, 8), (8_192, 100, 264), (8_193, 100, 264), (4_096, 160, 512), (4_097, 160, 512)]


@pytest.mark.parametrize("out_bf16", [True, False])
@pytest.mark.parametrize("m,d_in,d_out", CASES)
def test_combine_stream_edges(G, m, d_in, d_out, out_bf16):
    import torch
    say("combine stream", m, d_in, d_out, out_bf16)
    assert G.combine_kernel(m, d_out, "bf16") == "ring"
    S = W.features(m, d_in, "bf16", seed=m + d_in)
    A = W.features(m, d_in, "bf16", seed=m + d_in + 1)
    Wt = W.glorot(d_in, d_out, "bf16", seed=d_out)
    Sp, Ap = padded(S, "bf16"), padded(A, "bf16")
    Sp[:, d_in:] = Ap[:, d_in:] = 0x7FC0            # NaN padding
    guard = 8
    dt, fill = (torch.int16, -7) if out_bf16 else (torch.float32, -7.0)
    out = torch.full((m + 1, d_out + guard), fill, dtype=dt, device="cuda")
    G.combine(dev(Sp), dev(Ap), m, d_in, dev(Wt), d_out, "bf16", out_bf16, out_bf16, out)
    got = host(out, "bf16" if out_bf16 else "f32")
    keep = np.array(fill).astype(np.int16).view(np.uint16) if out_bf16 else np.float32(fill)
    assert (got[m] == keep).all() and (got[:, d_out:] == keep).all()
    z = np.concatenate([O.to_f64(S, "bf16"), O.to_f64(A, "bf16")], axis=1) @ O.to_f64(Wt, "bf16")
    if out_bf16:
        z = O.round_bf16_array(np.maximum(z, 0))
    assert_rows_close(O.to_f64(got[:m, :d_out], "bf16" if out_bf16 else "f32"), z, BF16_TOL, "combine stream")


@pytest.mark.parametrize("dtype,m,d_in,d_out", [("bf16", 6_000, 256, 256), ("bf16", 40_000, 60, 96), ("f32", 13_720, 70, 256),
                                                ("f32", 30_000, 80, 128)])
def test_combine_on_a_share_of_the_units(G, dtype, m, d_in, d_out):
    """A stream that holds a share of the compute units gets grids of that
    share; the bits are those of the whole chip."""
    import torch
    say("combine share", dtype, m, d_in, d_out)
    S, A = W.features(m, d_in, dtype, seed=1), W.features(m, d_in, dtype, seed=2)
    ops = dev(padded(S, dtype)), dev(padded(A, dtype)), dev(W.glorot(d_in, d_out, dtype, seed=3))
    outs = []
    for share in (None, (0, 2), (1, 3)):
        out = torch.zeros((m, d_out), dtype=torch.int16 if dtype == "bf16" else torch.float32, device="cuda")
        torch.cuda.synchronize()
        st = G.stream_create(*share) if share else torch.cuda.current_stream()
        G.combine(ops[0], ops[1], m, d_in, ops[2], d_out, dtype, True, dtype == "bf16", out, stream=st)
        torch.cuda.synchronize()
        if share:
            G.stream_destroy(st)
        outs.append(host(out, dtype))
    assert outs[0].any() and all(np.array_equal(outs[0], o) for o in outs[1:])
