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


def test_slot_list_up_to_int32(G):
    """The largest slot list: 33,554,431 rows of 64 slots, 64 short of 2^31, so
    that the last tile's last threads start within 8 of 2^31.  A ring whose
    vertex 0 also points at 100 others (for a maximum degree above 64)."""
    import torch
    n = 33_554_431
    say("slot list up to int32", n)
    src = np.concatenate([np.arange(n, dtype=np.int32), np.zeros(100, np.int32)])
    dst = np.concatenate([(np.arange(n, dtype=np.int64) + 1) % n, np.arange(1000, 1100)]).astype(np.int32)
    g = G.Graph(n, src, dst, symmetrize=False)
    blk = G.Blocks()
    seeds = torch.arange(n, dtype=torch.int32, device="cuda")
    G.sample(g, seeds, [64], 3, blk)
    nodes, sizes, ip, nb, ix = blk.to_host()
    assert sizes == [n, n] and np.array_equal(nodes, np.arange(n, dtype=np.int32))
    deg = np.ones(n, np.int64)
    deg[0] = 64
    assert np.array_equal(np.diff(ip[0]), deg) and ip[0][0] == 0
    assert len(nb[0]) == n + 63 and np.array_equal(nb[0], ix[0])   # every vertex is its own local id
    assert np.array_equal(nb[0][64:], (np.arange(1, n, dtype=np.int64) + 1) % n)
    assert set(nb[0][:64].tolist()) <= {1, *range(1000, 1100)} and len(set(nb[0][:64].tolist())) == 64
    blk.close()
    g.close()
