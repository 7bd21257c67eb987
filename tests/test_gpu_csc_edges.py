"""The transposed block behind the aggregation's adjoint at the sizes where its
sort changes form: edge counts around the tile sizes, around 64 tiles of each
size and around the largest that needs no scan launch; one, two and three digit
passes; long columns and repeated edges.  Rows of four edges have the exact
weight 1/4, so a column's sum in edge order has one right bit pattern."""
import numpy as np
import pytest

from test_gpu_parity import G, dev, host, say  # noqa: F401  (G is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_src", [1, 200, 256, 257, 9000, 65_537])
@pytest.mark.parametrize("n_dst", [1, 63, 64, 65, 4095, 4096, 4097, 8193, 16_385, 32_768, 32_769])
def test_columns_in_edge_order(G, n_src, n_dst):
    import torch
    say("csc", n_src, n_dst)
    rng = np.random.default_rng(n_src + n_dst)
    ix = rng.integers(0, n_src, 4 * n_dst).astype(np.int32)
    ix[rng.random(ix.size) < 0.2] = n_src // 2
    ip = (4 * np.arange(n_dst + 1)).astype(np.int32)
    dagg = rng.normal(size=(n_dst, 4)).astype(np.float32)
    out = torch.full((n_src, 4), 3.0, device="cuda")
    ipd, ixd, daggd = dev(ip), dev(ix), dev(dagg)
    want = np.zeros((n_src, 4), np.float32)
    np.add.at(want, ix, np.repeat(dagg * np.float32(0.25), 4, axis=0))
    for _ in range(2):
        G.aggregate_mean_backward(ipd.data_ptr(), ixd.data_ptr(), n_dst, n_src, daggd, 4, out)
        assert np.array_equal(host(out), want)
