"""The one-launch gather of caches whose rows are all in HBM (every vertex
cached, or a device store): request counts around a wavefront's 64 and around
one per wavefront, every lane-group width, repeated and out-of-range ids, host
and device request counts, bit-exact with the oracle, and twice in a row (its
counters must be back at zero)."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from test_gpu_parity import G, dev, graph_case, host, say  # noqa: F401  (G is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,dtype", [(3, "f32"), (8, "f32"), (16, "f32"), (33, "f32"), (64, "bf16"), (100, "f32"),
                                     (129, "f32"), (602, "f32"), (1100, "f32")])
@pytest.mark.parametrize("r,on_device", [(0.0, True), (0.4, True), (1.0, True), (1.0, False)])
def test_gather_direct(G, d, dtype, r, on_device):
    import torch
    n, u, v = graph_case("random-3000-40000-1")
    g = G.Graph(n, u, v)
    feats = W.features(n, d, dtype, seed=d)
    c = G.Cache(g, feats, dtype, r, store_on_device=on_device)
    _, slot, _ = O.rank_cache(O.build_csr(n, u, v), r)
    rng = np.random.default_rng(d)
    tdt = torch.int16 if dtype == "bf16" else torch.float32
    counts = torch.full((3,), 5, dtype=torch.int64, device="cuda")
    for m in (0, 1, 63, 64, 65, 257, 8191, 8193, 40_000):
        say("gather direct", d, dtype, r, on_device, m)
        ids = rng.integers(-1, n + 1, m).astype(np.int32)
        ids_d = dev(ids) if m else None
        rows, want = O.gather(feats, slot, ids)
        for through in ("count", "device count", "count"):
            out = torch.full((m + 1, c.ld), 7, dtype=tdt, device="cuda")
            if through == "count":
                G.gather(c, ids_d.data_ptr() if m else 0, m, out, counts)
            else:
                n_dev = dev(np.array([m], np.int32))
                big = torch.full((m + 64,), 3, dtype=torch.int32, device="cuda")
                if m:
                    big[:m] = ids_d
                room = torch.full((m + 64, c.ld), 7, dtype=tdt, device="cuda")
                G.gather_n(c, big.data_ptr(), n_dev.data_ptr(), m + 64, room, counts)
                out = room[:m + 1]
            assert np.array_equal(host(counts), want)
            got = host(out, dtype)
            assert np.array_equal(got[:m, :d].view(np.uint8), rows.view(np.uint8))
            assert (got[m] == 7).all()
    G.sync()
    c.close()
