"""The biased sampler's lane groups: fan-outs at the edges of every group width
and of the wavefront-per-row form past them, both row-pointer types, frontiers
that end inside a wavefront, and a hub whose weights pass 2^32 (the 64-bit
class steps); bit for bit against the oracle."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from test_gpu_parity import G, compare_blocks, dev, graph_case, say  # noqa: F401  (G is a fixture)

pytestmark = pytest.mark.gpu


def check(G, n, u, v, r, eta, seeds, fanouts, i64):
    csr = O.build_csr(n, u, v)
    g = G.Graph(n, u, v, offsets_i64=i64)
    c = G.Cache(g, W.features(n, 4, "f32"), "f32", r)
    _, slot, _ = O.rank_cache(csr, r)
    ref = O.sample_blocks(csr, seeds, fanouts, 99, bias_slot_map=slot, eta=eta)
    for async_ in (False, True):
        b = G.Blocks()
        seeds_d = dev(seeds)
        G.sample_biased(g, c, eta, seeds_d, fanouts, 99, b, async_=async_)
        if async_:
            b.sync()
        compare_blocks(G, b, ref)
        b.close()


@pytest.mark.parametrize("i64", [False, True])
@pytest.mark.parametrize("k", [1, 2, 7, 8, 9, 15, 16, 17, 31, 32, 33])
@pytest.mark.parametrize("m", [1, 3, 129])
def test_group_widths(G, m, k, i64):
    say("biased groups", m, k, i64)
    n, u, v = graph_case("random-3000-40000-1")
    check(G, n, u, v, 0.3, 4, W.epoch_permutation(n, 5)[:m], [k, min(k, 9)], i64)


@pytest.mark.parametrize("r", [1.0, 0.99])
def test_hub_past_32_bits(G, r):
    say("biased hub", r)
    n = 70_001
    u, v = np.zeros(n - 1, np.int32), np.arange(1, n, dtype=np.int32)
    check(G, n, u, v, r, 65536, np.array([5, 0, 9, 11], np.int32), [9, 25], False)
