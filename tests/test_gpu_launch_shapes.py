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
    """Light words of 1 to 513 tokens and a few frequent words cut into tiles: too few tiles for classes by size, so all of a
    chunk's share one launch and one size of workgroup."""
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


def corpus_of_three_classes():
    """17,500 light words and two frequent ones.  With whole words as tiles the classes of light words are, where a wavefront is
    the least workgroup, more than 128 tokens, 65 to 128 and fewer; 200 words on every side of each line."""
    edges = [63, 64, 65, 127, 128, 129, 255, 256, 257, 400]
    counts = np.r_[np.repeat(edges, 200), 3000, 9000, np.resize([1, 2, 3, 17], 15500)]
    return counts, *corpus_of_word_counts(counts, 900, 5)


# topics -> sampling launches per chunk: at K = 1,000 a CU holds 32 workgroups of one wavefront, at K = 2,000 two wavefronts
# are the least, at K = 9,000 LDS takes four workgroups, all of 512 threads then
CLASSES = {1000: 3, 2000: 2, 9000: 1}


@pytest.mark.parametrize("K", sorted(CLASSES))
def test_classes_of_light_words(K):
    """Tiles of light words in several launches: the classes' offsets into tiles and partial sums, and the first launch, which
    takes the frequent words too."""
    counts, doc_ptr, words = corpus_of_three_classes()
    pk, V, alpha = saber(), counts.size, 50.0 / K
    tok = np.random.default_rng(K).integers(0, words.size, 50000)
    results = []
    for opts in ({"tile_tokens": 1024}, {"block_threads": 256, "light_block_threads": 256, "tile_tokens": 8192}):
        g = pk.Saber(doc_ptr, words, V, K, alpha, 0.01, 11, **opts)
        if not results:
            o = oracle.Model(doc_ptr, words, V, K, alpha, 0.01, 11)
            z_ref, _, _, _, margin = o.estep_detail(nthreads=4)
        g.iterate(1)
        if not results:
            bad = np.nonzero(g.get_z() != z_ref)[0]
            assert bad.size <= 1e-3 * words.size and np.all(margin[bad] < 1e-5)
            o.close()
        g.iterate(1)
        results.append((g.get_z(), g.loglik(), *g.token_probs(tok)))
        g.close()
    for a, b in zip(*results):
        if isinstance(a, float):                    # partial sums of other tiles, 64 bits
            assert abs(a - b) <= 1e-12 * abs(b)
        else:
            assert np.array_equal(a, b)


@pytest.mark.parametrize("K,T", [(15361, 16383), (36864, 16385), (36865, 40000), (73729, 300_001), (262144, 5000), (100, 1), (7, 65537)])
def test_topic_totals_and_word_counts_at_the_edges_of_an_lds_histogram(K, T):
    """One LDS histogram holds 36,864 topics; shares of z have at least 16,384 assignments.  The highest and the lowest
    topic of every range occur, one topic takes a third of all tokens, and one word most of them."""
    rng = np.random.default_rng(K)
    V = 5
    words = np.where(rng.random(T) < 0.9, 0, rng.integers(0, V, T)).astype(np.int32)
    z = rng.integers(0, K, T)
    edges = np.array([k for k in (0, K - 1, 36863, 36864, K // 2 - 1, K // 2, (K + 1) // 2, (K + 2) // 3) if 0 <= k < K])
    z[: min(T, edges.size)] = edges[: min(T, edges.size)]
    z[T // 2: T // 2 + T // 3] = K // 3
    doc_ptr = np.minimum(np.arange(0, T + 300, 300), T).astype(np.int64)
    g = saber().Saber(doc_ptr, words, V, K, 0.1, 0.01, 3)
    g.set_z(z.astype(np.int32), 1)
    _, _, _, cwk, ck = g.counts(want_cd=False)
    assert np.array_equal(ck, np.bincount(z, minlength=K))
    assert np.array_equal(cwk.reshape(-1), np.bincount(words.astype(np.int64) * K + z, minlength=V * K))
    g.close()


@pytest.mark.parametrize("K", [5, 1024, 1025, 4096, 4097])
def test_m_step_of_a_small_corpus(K):
    """Counts in one launch, what follows from them in another (up to 4,096 topics): documents and light words of lengths on
    both sides of what a wavefront sorts in one register and in two and counts in LDS, empty ones, one that takes a workgroup,
    frequent words' slabs, several shares of the totals.  Counts and Bhat against the oracle, twice in a row."""
    edges = np.array([0, 1, 3, 63, 64, 65, 127, 128, 129, 511, 512, 513, 700])
    lens = np.r_[np.repeat(edges, 9), 40_000, 0]
    doc_ptr = np.r_[0, np.cumsum(lens)].astype(np.int64)
    rng = np.random.default_rng(K)
    counts = np.r_[np.repeat(edges, 7), 0, 21_000]                     # (the last two have dense rows)
    counts[-2] = doc_ptr[-1] - counts.sum()
    words = np.repeat(np.arange(counts.size, dtype=np.int32), counts)
    rng.shuffle(words)
    pk, V = saber(), counts.size
    g = pk.Saber(doc_ptr, words, V, K, 0.1, 0.01, 4, light_word_tokens=1000)
    o = oracle.Model(doc_ptr, words, V, K, 0.1, 0.01, 4)
    for state in (0, 1):
        z = np.minimum((K * rng.random(words.size) ** 3).astype(np.int32), K - 1)
        g.set_z(z, 1)
        o.set_z(z, it=1)
        cd_ptr, topic, count, cwk, ck = g.counts()
        assert np.array_equal(cd_ptr, o.cd[0]) and np.array_equal(topic, o.cd[1]) and np.array_equal(count, o.cd[2])
        assert np.array_equal(cwk, o.cwk) and np.array_equal(ck, o.ck)
        phi, prefix = g.get_phi(np.arange(V, dtype=np.int32))
        assert np.array_equal(phi, o.phi)
        assert np.mean(prefix != o.c32) < 1e-5 and np.allclose(prefix, o.c32, rtol=1.2e-7, atol=0)
        st = g.get_stats()
        assert st["nnz_cd"] == topic.size and st["next_row_entries"] == int((np.diff(cd_ptr) * np.diff(doc_ptr)).sum())
        assert st["next_light_entries"] == np.count_nonzero(cwk[counts < 1000])
    assert_estep_parity(g, o)
    g.close()
    o.close()


@pytest.mark.parametrize("K", [37_889, 65_536, 65_537, 70_000, 262_144])
def test_light_words_where_lds_cannot_hold_a_row(K):
    """Light words are read from the base vector and marks in LDS: none, one, all 32 topics of a mark and neighbours across its
    ends, the lowest and the highest topic; frequent words beside them.  Against the
    oracle, and against dense rows for every word (whose prefix sums are associated differently)."""
    rng = np.random.default_rng(K)
    counts = np.r_[0, 1, 2, 33, 64, 65, 500, 900, 3000, 9000, 20_000, 400]
    words = np.repeat(np.arange(counts.size, dtype=np.int32), counts)
    rng.shuffle(words)
    lens = np.r_[0, 500, rng.integers(0, 200, 2 * words.size // 200)]
    doc_ptr = np.r_[0, np.minimum(np.cumsum(lens), words.size)].astype(np.int64)
    doc_ptr = np.r_[doc_ptr, np.arange(doc_ptr[-1], words.size, 199)[1:], words.size].astype(np.int64)
    few = np.r_[np.arange(31, 66), 0, K - 33, K - 2, K - 1, 1000, K // 2]
    z = np.where(rng.random(words.size) < 0.7, rng.choice(few, words.size), rng.integers(0, K, words.size)).astype(np.int32)
    pk, V, alpha = saber(), counts.size, 50.0 / K
    tok = rng.integers(0, words.size, 3000)
    g = pk.Saber(doc_ptr, words, V, K, alpha, 0.01, 3, light_word_tokens=9500)
    p = pk.Saber(doc_ptr, words, V, K, alpha, 0.01, 3, light_word_tokens=-1)
    o = oracle.Model(doc_ptr, words, V, K, alpha, 0.01, 3)
    assert g.get_stats()["light_tokens"] == counts[counts < 9500].sum()
    for m in (g, p):
        m.set_z(z, 1)
    o.set_z(z, it=1)
    phi, prefix = g.get_phi(np.arange(V, dtype=np.int32))
    assert np.array_equal(phi, o.phi)
    assert np.mean(prefix != o.c32) < 1e-5 and np.allclose(prefix, o.c32, rtol=1.2e-7, atol=0)
    for a, b in zip(g.token_probs(tok), p.token_probs(tok)):
        assert np.allclose(a, b, rtol=1.2e-7, atol=0)                # S the same sums, Q from totals of other association
    assert abs(g.loglik() - o.loglik()) <= 1e-6 * abs(o.loglik())
    assert_estep_parity(g, o)
    p.iterate(1)
    assert np.mean(g.get_z() != p.get_z()) <= 1e-4
    obs = (np.arange(words.size) % 2).astype(np.uint8)
    a, b = (m.holdout_loglik(doc_ptr, words, obs, 1, 5) for m in (g, p))
    assert a[1] == b[1] and np.mean(a[2] != b[2]) <= 1e-3 and abs(a[0] - b[0]) <= 1e-5 * abs(b[0])
    for m in (g, p, o):
        m.close()


@pytest.mark.parametrize("K", [63, 1024, 1025, 2049, 8192, 8193, 16385, 70000])
def test_dense_rows_counted_where_they_are_normalised(K):
    """Rows on both sides of what a workgroup holds in registers (4 assignments per thread), counts itself (32 per thread)
    and leaves to the slab histograms, for workgroups of 256, 512 and 1,024 threads and one or several ranges of topics."""
    block = 256 if K <= 1024 else 512 if K <= 2048 else 1024
    counts = np.array([0, 1, 7, 4 * block - 1, 4 * block, 4 * block + 1, 32 * block, 32 * block + 1, 33 * block + 5, 3])
    doc_ptr, words = corpus_of_word_counts(counts, 900, K)
    V, rng = counts.size, np.random.default_rng(K)
    z = np.where(rng.random(words.size) < 0.3, K - 1, (K * rng.random(words.size) ** 3).astype(np.int64)).astype(np.int32)
    pk = saber()
    for state in (0, 1):                       # rows of B are clear again after each M-step
        z = np.roll(z, 17 * state)
        if state == 0:
            g = pk.Saber(doc_ptr, words, V, K, 0.1, 0.01, 4, light_word_tokens=-1)
            o = oracle.Model(doc_ptr, words, V, K, 0.1, 0.01, 4)
        g.set_z(z, 1)
        o.set_z(z, it=1)
        phi, prefix = g.get_phi(np.arange(V, dtype=np.int32))
        assert np.array_equal(phi, o.phi)
        assert np.mean(prefix != o.c32) < 1e-5 and np.allclose(prefix, o.c32, rtol=1.2e-7, atol=0)
        assert np.array_equal(g.counts(want_cd=False)[3], o.cwk)
    g.close()
    o.close()


@pytest.mark.parametrize("T,K,opts", [(1, 5, {}), (131072, 50, {}), (131073, 300, {}), (2_500_000, 40, {}), (300_001, 70000, {}),
                                      (1_000_003, 2000, {"light_word_tokens": 1 << 16}), (700_000, 9000, {"light_word_tokens": -1}),
                                      (900_000, 100, {"stream_workers": 3, "n_chunks": 4}), (2 << 20, 50, {}), ((2 << 20) + 1, 50, {}),
                                      (2_300_000, 70000, {}), (2_500_000, 60000, {"light_word_tokens": -1}),
                                      (2_500_000, 60000, {"light_word_tokens": 1 << 16}),
                                      (9_000_000, 100, {"stream_workers": 3, "n_chunks": 4})])
def test_results_that_leave_in_pieces(T, K, opts):
    """Assignments and counts go to the caller by plain copies, or above 8 MB by pieces through staging, several
    at a time: some, many, more than the staging holds; documents longer than the others' average piece; repeated calls on
    one context."""
    rng = np.random.default_rng(T)
    V = 37
    most = (1 << (32 - max(1, (K - 1).bit_length()))) - 1        # tokens of the longest document that K leaves count bits for
    lens = np.r_[7, min(T // 3, most), rng.integers(0, 900, 2 + T // 440)]
    doc_ptr = np.r_[0, np.minimum(np.cumsum(lens), T)].astype(np.int64)
    T = int(doc_ptr[-1])
    words = np.minimum(rng.geometric(0.2, T), V).astype(np.int32) - 1
    z = np.minimum(rng.geometric(20.0 / K, T) % K, K - 1).astype(np.int32) if K > 20 else rng.integers(0, K, T).astype(np.int32)
    g = saber().Saber(doc_ptr, words, V, K, 0.1, 0.01, 3, **opts)
    z0 = g.get_z()
    g.set_z(z, 2)
    for _ in range(2):
        assert np.array_equal(g.get_z(), z)
        cd_ptr, topic, count, cwk, ck = g.counts()
        doc = np.repeat(np.arange(doc_ptr.size - 1), np.diff(doc_ptr))
        key, n = np.unique(doc * K + z, return_counts=True)
        assert np.array_equal(cd_ptr, np.searchsorted(key, np.arange(doc_ptr.size) * K))
        assert np.array_equal(topic, key % K) and np.array_equal(count, n)
        assert np.array_equal(cwk.reshape(-1), np.bincount(words.astype(np.int64) * K + z, minlength=V * K))
        assert np.array_equal(ck, np.bincount(z, minlength=K))
    g.set_z(z0, 0)
    assert np.array_equal(g.get_z(), z0)
    g.close()


@pytest.mark.parametrize("T,K,opts", [(11_000_000, 1000, {}), (11_000_000, 16384, {}), (17_300_000, 300, {}),
                                      (24_000_000, 2500, {"n_chunks": 2, "stream_workers": 2})])
def test_frequent_words_cut_by_ranges_of_documents(T, K, opts):
    """Tiles cut at the ends of sixteen ranges of documents, against the plain order of tiles (classes by size switch the
    ranges off).  Empty documents on both ends, one document longer than several ranges (some ranges are empty), words that
    occur in one range only, words with too few tokens to be cut."""
    rng = np.random.default_rng(K)
    lens = np.r_[0, 0, rng.integers(0, 700, T // 900), min(T // 5, (1 << (32 - (K - 1).bit_length())) - 1), rng.integers(0, 700, T // 600), 0]
    doc_ptr = np.r_[0, np.minimum(np.cumsum(lens), T)].astype(np.int64)
    T, V = int(doc_ptr[-1]), 900
    words = np.minimum(rng.geometric(0.01, T) - 1, V - 2).astype(np.int32)
    words[T // 3: T // 3 + 40000] = V - 1
    pk = saber()
    g = pk.Saber(doc_ptr, words, V, K, 50.0 / K, 0.01, 8, **opts)
    p = pk.Saber(doc_ptr, words, V, K, 50.0 / K, 0.01, 8, stage_min_tokens=2, light_block_threads=256, n_chunks=opts.get("n_chunks", 0))
    assert g.get_stats()["tiles"] > p.get_stats()["tiles"]
    for _ in range(2):
        g.iterate(1)
        p.iterate(1)
        assert np.array_equal(g.get_z(), p.get_z())
    assert abs(g.loglik() - p.loglik()) <= 1e-11 * abs(p.loglik())
    g.close()
    p.close()


@pytest.mark.parametrize("K,opts", [(60, {}), (1000, {}), (9000, {}), (40_000, {}), (1000, {"stage_phi": 0}), (70_000, {}), (300, {"n_chunks": 3}),
                                    (300, {"n_chunks": 3, "stream_workers": 2})])
def test_normalisers_of_a_few_tokens(K, opts):
    """Fewer than an eighth of the tokens are marked and worked on alone, in chunks of 400,000 tokens and more: the same numbers
    as where all are asked for, which the oracle checks; none in a tile or a batch, one, all of a run, a word's all; repeats;
    tokens on both sides of what a mark holds; both sides of an eighth; a large request between two small ones."""
    rng = np.random.default_rng(K)
    edges = [1, 2, 63, 64, 65, 129, 400, 700]
    heavy = 600_000 if opts.get("n_chunks") else 200_000
    doc_ptr, words = corpus_of_word_counts(np.r_[heavy, heavy, np.repeat(edges, 9), 4000, 9000], 4260, K)
    words[doc_ptr[7]: doc_ptr[7] + 40] = 3                            # runs of more than one token
    T, V = words.size, int(words.max()) + 1
    g = saber().Saber(doc_ptr, words, V, K, 50.0 / K, 0.01, 11, **opts)
    g.iterate(2)
    every = g.token_probs(np.arange(T))
    for tok in (np.array([T - 1]), np.array([0, 31, 32, 63, 64, T - 1, 0, 32]), rng.integers(0, T, 300), np.arange(doc_ptr[7], doc_ptr[8]),
                np.arange(T), np.nonzero(words == V - 1)[0][:T // 9], np.arange(T // 8 - 1), np.arange(T // 8), rng.permutation(T)[:T // 8 - 1]):
        for a, b in zip(g.token_probs(tok), every):
            assert np.array_equal(a, b[tok])
    g.close()


@pytest.mark.parametrize("K,opts", [(9000, {}), (20_011, {}), (9000, {"tile_tokens": 64}), (20_011, {"tile_tokens": 64})])
def test_workgroups_that_work_on_several_light_words(K, opts):
    """Enough tiles of light words for several per workgroup, against chunks with too few: words of one token to more than a
    workgroup has threads, whose topics it takes back one by one or by staging the row again; the numbers of tiles leave a
    remainder.  With tiles of 64 tokens most are of words with more topics than threads."""
    small, large = (2001, 1100) if opts else (45_001, 40)
    counts = np.r_[np.resize([1, 2, 3, 1, 5, 90], small), np.resize([2600, 300, 4200], large), 14_000]
    doc_ptr, words = corpus_of_word_counts(counts, counts.size // 10, K)
    pk, V, alpha = saber(), counts.size, 50.0 / K
    g = pk.Saber(doc_ptr, words, V, K, alpha, 0.01, 11, **opts)
    p = pk.Saber(doc_ptr, words, V, K, alpha, 0.01, 11, n_chunks=60)
    for _ in range(2):
        g.iterate(1)
        p.iterate(1)
        assert np.array_equal(g.get_z(), p.get_z())
    assert g.get_stats()["tiles"] > 32_768
    g.close()
    p.close()


@pytest.mark.parametrize("K", [20_011, 70_000])
def test_rows_of_many_blocks(K):
    """Rows of A of one block of 256 entries to 67, on both sides of two, three, four and 64: the draw's block is found from the
    sums through the blocks, from the 65th on by going through them."""
    lens = np.r_[255, 256, 257, 511, 512, 513, 767, 768, 769, 1024, 1025, 1281, 16_383, 16_384, 16_385, 17_000]
    doc_ptr = np.r_[0, np.cumsum(np.r_[lens, lens])].astype(np.int64)
    rng = np.random.default_rng(K)
    V, T = 300, int(doc_ptr[-1])
    words = rng.integers(0, V, T).astype(np.int32)
    # as many topics as tokens in the first half's documents, most mass on a document's last topics in the other's
    z = np.concatenate([rng.permutation(K)[:n] if i < lens.size else np.minimum(rng.integers(K - 700, K, n), np.arange(n) % K)
                        for i, n in enumerate(np.r_[lens, lens])]).astype(np.int32)
    g = saber().Saber(doc_ptr, words, V, K, 50.0 / K, 0.01, 3)
    o = oracle.Model(doc_ptr, words, V, K, 50.0 / K, 0.01, 3)
    g.set_z(z, 1)
    o.set_z(z, it=1)
    assert_estep_parity(g, o)
    g.close()
    o.close()


@pytest.mark.parametrize("K", [8256, 9216, 12_000, 20_011, 70_000])
def test_rows_of_bhat_by_parts(K):
    """Few rows of many topics have a workgroup per range of topics and their running sums added up afterwards, more rows a
    workgroup each: the same sums in the same order, so the same bits; rows that are counted where they are normalised, also with
    more assignments than a workgroup holds, and rows counted before."""
    counts = np.r_[np.resize([1, 3, 64, 700], 190), 4000, 5000, 20_000, 40_000, np.zeros(106, np.int64)]
    doc_ptr, words = corpus_of_word_counts(counts, 400, K)
    pk, V, used = saber(), counts.size, np.arange(194, dtype=np.int32)
    few = pk.Saber(doc_ptr, words, V, K, 0.1, 0.01, 4, light_word_tokens=1)      # (a word without tokens keeps no dense row)
    all_rows = pk.Saber(doc_ptr, words, V, K, 0.1, 0.01, 4, light_word_tokens=-1)
    o = oracle.Model(doc_ptr, words, V, K, 0.1, 0.01, 4)
    for _ in range(2):
        phi, prefix = few.get_phi(used)
        ref, ref_prefix = all_rows.get_phi(used)
        assert np.array_equal(phi, o.phi[:194]) and np.array_equal(phi, ref) and np.array_equal(prefix, ref_prefix)
        assert np.mean(prefix != o.c32[:194]) < 1e-5 and np.allclose(prefix, o.c32[:194], rtol=1.2e-7, atol=0)
        few.iterate(1)
        all_rows.iterate(1)
        z = few.get_z()
        assert np.array_equal(z, all_rows.get_z())
        o.set_z(z, 1)
    few.close(); all_rows.close(); o.close()


@pytest.mark.parametrize("K", [60, 1000, 8192, 8200])
@pytest.mark.parametrize("V", [16_380, 16_500])
def test_light_words_of_a_wavefront(K, V):
    """Four light words to a wavefront where rows are short and words many, one otherwise: words without tokens, with one, with one
    block of topics, with more non-zeros than lanes; a last wavefront with fewer words."""
    counts = np.r_[np.resize([0, 1, 2, 29], V - 9), 63, 64, 65, 128, 129, 200, 400, 0, 1]
    doc_ptr, words = corpus_of_word_counts(counts, 300, K)
    pk = saber()
    g = pk.Saber(doc_ptr, words, V, K, 0.1, 0.01, 4, light_word_tokens=1000)
    o = oracle.Model(doc_ptr, words, V, K, 0.1, 0.01, 4)
    assert g.get_stats()["light_words_present"] == np.count_nonzero(counts)
    some = np.r_[0:400, V - 30:V].astype(np.int32)
    for _ in range(2):
        phi, prefix = g.get_phi(some)
        assert np.array_equal(phi, o.phi[some])
        assert np.mean(prefix != o.c32[some]) < 1e-5 and np.allclose(prefix, o.c32[some], rtol=1.2e-7, atol=0)
        assert_estep_parity(g, o)
    g.close(); o.close()


@pytest.mark.parametrize("K", [11_000, 14_000, 20_500, 36_990, 37_013, 37_048, 37_049])
def test_short_rows_exchange_beside_a_long_row_in_lds(K):
    """Rows of Bhat that leave some of a CU's LDS to the wavefronts' parts, from K = 37,013 to 37,048 all but 144 bytes of it
    or fewer; from 37,049 on there is none left for them."""
    counts = np.r_[np.resize([1, 2, 5, 29, 40], 3000), 500, 3000]
    doc_ptr, words = corpus_of_word_counts(counts, 900, K)
    pk, V = saber(), counts.size
    g = pk.Saber(doc_ptr, words, V, K, 0.01, 0.01, 4)
    p = pk.Saber(doc_ptr, words, V, K, 0.01, 0.01, 4, quarter_row_entries=-1, half_row_entries=-1)
    o = oracle.Model(doc_ptr, words, V, K, 0.01, 0.01, 4)
    assert_estep_parity(g, o)
    p.iterate(1)
    assert np.array_equal(g.get_z(), p.get_z())
    g.iterate(2)
    p.iterate(2)
    assert np.array_equal(g.get_z(), p.get_z())
    g.close(); p.close(); o.close()


@pytest.mark.parametrize("K", [1000, 5000, 8200])
def test_light_words_of_many_tokens_among_others(K):
    """Words of more than 256 tokens have a wavefront each and come first among the light ones, wherever they are in the vocabulary:
    words on both sides of that line, of up to 12,000 tokens, between 16,400 of few."""
    rng = np.random.default_rng(K)
    counts = rng.permutation(np.r_[np.resize([0, 1, 2, 9], 16_400), 65, 128, 255, 256, 256, 257, 257, 300, 1000, 3000, 12_000])
    doc_ptr, words = corpus_of_word_counts(counts, 500, K)
    pk, V = saber(), counts.size
    g = pk.Saber(doc_ptr, words, V, K, 0.1, 0.01, 4, light_word_tokens=20_000)
    o = oracle.Model(doc_ptr, words, V, K, 0.1, 0.01, 4)
    assert g.get_stats()["light_tokens"] == o.T
    some = np.r_[np.nonzero(counts > 9)[0], 0:200, V - 30:V].astype(np.int32)
    for _ in range(2):
        phi, prefix = g.get_phi(some)
        assert np.array_equal(phi, o.phi[some])
        assert np.mean(prefix != o.c32[some]) < 1e-5 and np.allclose(prefix, o.c32[some], rtol=1.2e-7, atol=0)
        assert_estep_parity(g, o)
    h = np.array([0, 4000], dtype=np.int64)              # a context that borrows the model's rows
    hw, mask = rng.choice(words, 4000).astype(np.int32), (np.arange(4000) % 2).astype(np.uint8)
    got, ref = g.holdout_loglik(h, hw, mask, 0, 5), o.holdout_loglik(h, hw, mask, 0, 5)
    assert got[1] == ref[1] and abs(got[0] - ref[0]) <= 1e-6 * abs(ref[0])
    g.close(); o.close()
