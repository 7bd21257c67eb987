"""Sampler kernels at the edges of their tiles, bit-exact against the oracle:
seed lists around each size of the one-workgroup dedup (with repeats and
out-of-range ids) and slot lists around one scan tile of 2,048 slots, at
strides that divide the tile and that do not."""
import numpy as np
import pytest

import oracle as O
from test_gpu_parity import G, dev, graph_case, say  # noqa: F401  (G is a fixture)

pytestmark = pytest.mark.gpu

N, M = 30_000, 150_000
_CSR = {}


def _graph(G):
    if not _CSR:
        n, u, v = graph_case(f"random-{N}-{M}-5")
        _CSR["csr"], _CSR["g"] = O.build_csr(n, u, v), G.Graph(n, u, v)
    return _CSR["csr"], _CSR["g"]


def _check(blk, ref):
    nodes, sizes, ip, nb, ix = blk.to_host()
    assert sizes == ref.sizes and np.array_equal(nodes, ref.nodes)
    for h in range(len(ip)):
        assert np.array_equal(ip[h], ref.indptr[h])
        assert np.array_equal(nb[h], ref.nbrs[h])
        assert np.array_equal(ix[h], ref.indices[h])


@pytest.mark.parametrize("n_seeds", [1, 63, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193])
def test_seed_dedup_sizes(G, n_seeds):
    csr, g = _graph(G)
    rng = np.random.default_rng(n_seeds)
    blk = G.Blocks()
    for span in (N, max(2, n_seeds // 3)):     # few repeats; most ids repeated
        say("seed dedup", n_seeds, span)
        seeds = rng.integers(0, span, n_seeds).astype(np.int32)
        G.sample(g, dev(seeds), [3], 9, blk)
        _check(blk, O.sample_blocks(csr, seeds, [3], 9))
    bad = seeds.copy()
    bad[0] = -1
    bad[-1] = N
    with pytest.raises(G.GnnavError) as e:
        G.sample(g, dev(bad), [3], 9, blk)
    assert e.value.status == 2                  # E_RANGE
    G.sample(g, dev(seeds), [3, 2], 10, blk)    # the blocks stay usable
    _check(blk, O.sample_blocks(csr, seeds, [3, 2], 10))


@pytest.mark.parametrize("k,rows", [(1, 2047), (1, 2048), (1, 2049), (7, 292), (7, 293), (8, 256), (8, 257),
                                    (25, 82), (33, 62), (33, 63), (64, 32), (64, 33), (64, 7)])
def test_slot_list_tiles(G, k, rows):
    csr, g = _graph(G)
    say("slot list", k, rows)
    seeds = np.random.default_rng(k * 10_000 + rows).permutation(N)[:rows].astype(np.int32)
    blk = G.Blocks()
    for fan in ([k], [k, 2], [-1, k] if rows < 100 else [k, -1]):
        G.sample(g, dev(seeds), fan, 21, blk)
        _check(blk, O.sample_blocks(csr, seeds, fan, 21))
