"""Mean aggregation over rows of every length around the neighbours in flight.

The kernel keeps eight neighbour rows in flight where a lane holds one unit of
a row and four where it holds several, and takes the last few of a row
together; widths cover one lane per row up to several units per lane.
"""
import numpy as np
import pytest
import torch

import paper_2404_09544_amd as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [3, 8, 17, 64, 100, 256, 300, 602, 1100])
def test_row_lengths_around_the_rows_in_flight(d, dtype):
    rng = np.random.default_rng(d)
    cnt = np.concatenate([np.arange(0, 20), [31, 32, 33, 63, 64, 65, 71, 130]])
    cnt = np.concatenate([cnt, rng.permutation(cnt)])
    indptr = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int32)
    n_src = 37
    indices = rng.integers(0, n_src, indptr[-1]).astype(np.int32)
    indices[::5] = n_src - 1
    ld = G.padded_ld(d, dtype)
    x = torch.zeros((n_src, ld))
    x[:, :d] = torch.from_numpy(rng.standard_normal((n_src, d)).astype(np.float32))
    if dtype == "bf16":
        x = x.to(torch.bfloat16)
    values = x.float().numpy()
    want = np.zeros((len(cnt), ld), np.float32)
    for i in range(len(cnt)):
        for p in range(indptr[i], indptr[i + 1]):   # fp32, in CSR order
            want[i] += values[indices[p]]
        want[i] *= np.float32(1.0) / np.float32(max(cnt[i], 1))
    dev = (x.view(torch.int16) if dtype == "bf16" else x).cuda()
    out = torch.full((len(cnt), ld), 7, dtype=dev.dtype, device="cuda")
    ip, ix = torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda()
    G.aggregate_mean(ip.data_ptr(), ix.data_ptr(), len(cnt), dev, d, dtype, out)
    got = (out.view(torch.bfloat16) if dtype == "bf16" else out).float().cpu().numpy()
    # the sums are the same fp32 sums; the reciprocal and the product round
    # once each (2^-24), a bf16 result once more (2^-9, or its next value)
    rtol = 2.0 ** -22 if dtype == "f32" else 2.0 ** -8
    np.testing.assert_allclose(got, want, rtol=rtol, atol=0)
