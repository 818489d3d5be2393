"""Launch shapes chosen from sizes: tiles, workgroups per class of tiles.  Whatever is chosen, the assignments are those of
the oracle and of the plain shape."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import assert_estep_parity, saber

pytestmark = pytest.mark.gpu


def corpus_of_word_counts(counts, D, seed):
    """Random documents in which word v occurs counts[v] times."""
    rng = np.random.default_rng(seed)
    words = np.repeat(np.arange(len(counts), dtype=np.int32), counts)
    rng.shuffle(words)
    cuts = np.sort(rng.integers(0, words.size + 1, D - 1))
    return np.r_[0, cuts, words.size].astype(np.int64), words


@pytest.mark.parametrize("K", [60, 1000, 2000, 9000])
def test_workgroups_sized_by_the_tile(K):
    """Light words on both sides of every class boundary (64, 128, 256, 512 tokens), enough of each for launches of their
    own, and a few frequent words cut into tiles."""
    edges = [1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513]
    counts = np.r_[np.repeat(edges, 60), [3000, 9000]]
    doc_ptr, words = corpus_of_word_counts(counts, 700, K)
    pk, V, alpha = saber(), counts.size, 50.0 / K
    g = pk.Saber(doc_ptr, words, V, K, alpha, 0.01, 11)
    o = oracle.Model(doc_ptr, words, V, K, alpha, 0.01, 11)
    assert_estep_parity(g, o)
    assert_estep_parity(g, o)
    z = g.get_z()
    ll = g.loglik()
    g.close()
    p = pk.Saber(doc_ptr, words, V, K, alpha, 0.01, 11, block_threads=256, light_block_threads=256, tile_tokens=8192)
    p.iterate(2)
    assert np.array_equal(p.get_z(), z)
    assert abs(p.loglik() - ll) <= 1e-12 * abs(ll)
    p.close()
    o.close()
