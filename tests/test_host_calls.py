"""The library's host code without a GPU: what it does when a call of the runtime fails, which launches it makes."""
import pytest

import fake_hip


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    lib = fake_hip.build(tmp_path_factory.mktemp("fake_hip"))
    return lambda code, **kw: fake_hip.run(lib, code, **kw)


def test_a_failed_call_does_not_fail_the_next_one(host):
    """The runtime hands out a thread's last error until it is asked for; the library reports it once."""
    host("""
        words = np.zeros(50000, np.int32)
        g = pk.Saber(np.r_[0, 500, words.size], words, 1, 100, 0.1, 0.01, 3)
        for call, code, use in (("hipMalloc", -2, lambda: g.set_z(words, 0)), ("hipMemcpy:", -3, lambda: g.counts_nnz()),
                                ("estep_kernel", -2, lambda: g.iterate(1)), ("hipMalloc", -2, lambda: g.token_probs([3]))):
            fake.fake_fail(call.encode(), 1)
            assert code_of(use) == code, call
            g.iterate(1)
            assert g.loglik() == 0.0                # (no kernel has run)
    """)


@pytest.mark.parametrize("call,K", [("hipHostMalloc", 60000), ("hipEventCreate", 60000), ("hipMemcpyAsync", 60000),
                                    ("hipMemcpy:", 60000), ("hipEventRecord", 60000), ("hipMemcpy:", 100)])
def test_counts_after_an_export_that_failed(host, call, K):
    """saber_counts rebuilds B for the export; whatever fails on the way, later counts do not contain it."""
    host("""
        call = %r
        counts = [3, 40000, 900, 0, 9000] + 35 * [2]
        words = np.repeat(np.arange(40, dtype=np.int32), counts)
        fake.fake_imitate(1)                        # (no sampling: every token keeps topic 0)
        K = %d                                      # (rows of 40 words for one copy, and for several through staging)
        g = pk.Saber(np.r_[0, 500, words.size], words, 40, K, 0.1, 0.01, 3, light_word_tokens=-1)
        nth = 0
        while True:
            nth += 1
            fake.fake_fail(call.encode(), nth)
            code = code_of(lambda: g.counts(want_cd=False, want_ck=False))
            if fake.fake_fail_pending() > 0: break  # fewer calls than that
            assert code in (0, -2, -3)              # (memory refused: another kind is used)
            fake.fake_fail(b"", 0)
            if nth %% 2:
                g.iterate(1)
            cwk, ck = g.counts(want_cd=False)[3:]
            assert np.array_equal(cwk[:, 0], counts) and not cwk[:, 1:].any(), (nth, cwk)
            if nth == 1: g.set_z(np.zeros(words.size, np.int32), 0)
        assert nth > 1
    """ % (call, K))


def test_topic_totals_after_an_iteration_that_failed(host):
    """The accumulators of the M-step are clear at its start, also where the one before broke off."""
    host("""
        words = np.zeros(50000, np.int32)
        fake.fake_imitate(1)
        g = pk.Saber(np.r_[0, 500, words.size], words, 1, 100, 0.1, 0.01, 3, light_word_tokens=-1)
        for kernel in (b"denominators_kernel", b"phi_tree_kernel"):
            fake.fake_fail(kernel, 1)
            assert code_of(lambda: g.iterate(1)) == -2
            g.set_z(np.zeros(words.size, np.int32), 0)
            cwk, ck = g.counts(want_cd=False)[3:]
            assert ck[0] == 50000 and cwk[0, 0] == 50000, (kernel, ck[0], cwk[0, 0])
    """)


@pytest.mark.parametrize("K", [100, 70000])
def test_results_with_another_device_current(host, K):
    """Results are copied out on the context's own device, whichever the caller has current."""
    host("""
        words = np.arange(5_000_000, dtype=np.int32) %% 50
        doc_ptr = np.r_[0, np.arange(999, words.size, 1000), words.size]
        g = pk.Saber(doc_ptr, words, 50, %d, 0.1, 0.01, 3)
        first = pk.Saber(doc_ptr, words, 50, %d, 0.1, 0.01, 3)
        first.get_z()
        fake.hipSetDevice(1)
        now = ctypes.c_int()
        for use in (g.get_z, lambda: g.counts(want_cwk=False), g.counts, first.get_z,
                    lambda: first.holdout_loglik(np.arange(0, 5_000_001, 1000), words, words %% 4 > 0, 1, 5)):
            use()
            fake.hipGetDevice(ctypes.byref(now))
            assert now.value == 1
    """ % (K, K))


def test_rows_of_more_words_than_a_launch_takes(host):
    """saber_get_phi: one workgroup per word asked for, words in any number (repeats count)."""
    host("""
        words = np.zeros(100, np.int32)
        g = pk.Saber(np.r_[0, 50, 100], words, 3, 2, 0.1, 0.01, 3)
        m = (1 << 24) + 1
        g.get_phi(np.zeros(m, np.int32))
        n, blocks, most = launches("phi_export")
        assert blocks == m and most < 1 << 32
    """)


@pytest.mark.parametrize("V,K,threads", [(1 << 23, 1025, 512), (1 << 22, 2049, 1024)])
def test_dense_rows_of_more_words_than_a_launch_takes(host, V, K, threads):
    """One workgroup per dense row, of more threads the longer the row."""
    host("""
        V, K, threads = %d, %d, %d
        words = np.array([0, V - 1, 5], np.int32)
        g = pk.Saber(np.array([0, 1, 3]), words, V, K, 0.1, 0.01, 3, light_word_tokens=-1)
        n, blocks, most = launches("phi_tree")
        assert n == 2 and blocks == V + 1 and most < 1 << 32 and most %% threads == 0
    """ % (V, K, threads))


def test_more_documents_and_light_words_than_a_launch_takes(host):
    """Documents and light words share the launches of the segmented count, one wavefront each."""
    host("""
        D = (1 << 26) - 4
        doc_ptr = np.zeros(D + 1, np.int64)
        doc_ptr[D:] = 5
        g = pk.Saber(doc_ptr, np.arange(5, dtype=np.int32), 10, 40, 0.1, 0.01, 3)
        n, blocks, most = launches("count_dz")
        assert n == 2 and blocks == D + 10 and most < 1 << 32, (n, blocks, most)
    """)


def test_more_tiles_than_a_launch_takes(host):
    """One workgroup per tile; a word that occurs has at least one."""
    host("""
        V = (1 << 22) + 3
        words = np.arange(V, dtype=np.int32)
        doc_ptr = np.r_[np.arange(0, V, 1000), V]
        for opts in ({"stage_phi": 0, "block_threads": 1024}, {"block_threads": 1024}):
            g = pk.Saber(doc_ptr, words, V, 20, 0.1, 0.01, 3, **opts)
            for use in (lambda: g.iterate(1), g.loglik, lambda: g.token_probs([0, V - 1])):
                fake.fake_clear()
                use()
                n, blocks, most = launches("estep_kernel")
                assert blocks == V and most < 1 << 32, (n, blocks, most)
            g.close()
        fake.fake_imitate(1)                        # B of as many dense rows: a slab each, and the totals beside them
        g = pk.Saber(doc_ptr, words, V, 2, 0.1, 0.01, 3, light_word_tokens=-1)
        cwk, ck = g.counts(want_cd=False)[3:]
        assert (cwk[:, 0] == 1).all() and not cwk[:, 1].any() and ck[0] == V
        n, blocks, most = launches("count_slabs")
        assert most < 1 << 32
    """)


@pytest.mark.parametrize("K,threads", [(100, 256), (2048, 256), (2049, 1024), (60000, 1024), (70000, 1024)])
def test_threads_of_a_workgroup_whose_row_is_not_staged(host, K, threads):
    """Large workgroups are for rows too long for the first-level cache; with short ones they lose."""
    host("""
        words = np.arange(5000, dtype=np.int32) %% 40
        g = pk.Saber(np.r_[0, 2000, 5000], words, 40, %d, 0.1, 0.01, 3, stage_phi=0)
        g.iterate(1)
        assert fake.fake_block(b"estep_kernel") == %d
    """ % (K, threads))


@pytest.mark.parametrize("D,V,K,opts,joined", [(3, 40, 4096, {}, True), (3, 40, 4097, {}, False),
                                               ((384 << 10) - 40, 40, 400, {}, True), ((384 << 10) - 39, 40, 400, {}, False),
                                               (3, 40, 100, {"light_word_tokens": -1}, False),
                                               (3, 40, 400, {"stream_workers": 2}, False)])
def test_which_m_steps_take_two_launches(host, D, V, K, opts, joined):
    """Those of small resident corpora with light words."""
    host("""
        D, V, K, opts, joined = %r
        words = np.arange(5000, dtype=np.int32) %% V
        doc_ptr = np.zeros(D + 1, np.int64)
        doc_ptr[1:] = np.minimum(np.arange(1, D + 1) * 2000, words.size)
        g = pk.Saber(doc_ptr, words, V, K, 0.1, 0.01, 3, **opts)
        fake.fake_clear()
        g.iterate(2)
        assert launches("mstep_counts")[0] == launches("mstep_rows")[0] == (2 if joined else 0)
        assert (launches("denominators")[0], launches("phi_tree")[0], launches("stats_kernel")[0]) == 3 * (0 if joined else 2,)
    """ % ((D, V, K, opts, joined),))


@pytest.mark.parametrize("T,edges", [(5000, {64: 1724, 128: 3612, 256: 8024, 512: 20124}),
                                     (4_300_000, {64: 1220, 128: 2732, 256: 6640, 512: 13316})])
def test_threads_and_tiles_of_a_workgroup_whose_row_is_staged(host, T, edges):
    """The smallest workgroup with which LDS leaves a CU enough wavefronts, more of them in large chunks; a tile is a 32,768th of
    the chunk per wavefront.  Both sides of every line; a caller's tile_tokens keeps the size with the most wavefronts."""
    host("""
        T, edges = %d, %r
        words = np.zeros(T, np.int32)
        doc_ptr = np.r_[np.arange(0, T, 1000), T]
        for block, K in edges.items():
            for k, b in ((K, block), (K + 4, 2 * block)):
                tile = min(256, max(64, k // 16 & ~63), 1 << 15)
                tile = max(tile, (T * min(b // 64, 4) // 32768) & ~63)
                g = pk.Saber(doc_ptr, words, 1, k, 0.1, 0.01, 3)
                g.iterate(1)
                assert fake.fake_block(b"estep_kernel") == b, (k, b, fake.fake_block(b"estep_kernel"))
                assert g.get_stats()["tiles"] == -(-T // tile), (k, b, g.get_stats()["tiles"], tile)
                g.close()
        g = pk.Saber(doc_ptr, words, 1, 100, 0.1, 0.01, 3, tile_tokens=1024)
        g.iterate(1)
        assert fake.fake_block(b"estep_kernel") == 256
    """ % (T, edges))


@pytest.mark.parametrize("K,T,opts,light,block", [(70_000, 500_000, {}, True, 256), (70_000, 9_000_000, {}, True, 1024), (70_000, 500_000, {"light_word_tokens": -1}, False, 1024),
                                                  (70_000, 500_000, {"stage_phi": 0}, False, 1024), (37_000, 500_000, {}, True, 1024)])
def test_light_words_where_lds_cannot_hold_a_row(host, K, T, opts, light, block):
    """They are read with marks in LDS, unless the caller wants dense rows, or rows gathered from memory."""
    host("""
        K, T, opts, light, block = %r
        words = (np.arange(T) %% 400).astype(np.int32)
        words[:8500] = 0
        words[-100:] = 401
        g = pk.Saber(np.r_[np.arange(0, T, 1000), T], words, 402, K, 0.1, 0.01, 3, **opts)
        g.iterate(1)
        n = np.bincount(words)
        most = (8192 if K == 70_000 else K // 2) if T < 8 << 20 else 1 << 15
        assert g.get_stats()["light_tokens"] == (n[n < most].sum() if light else 0), g.get_stats()
        assert fake.fake_block(b"estep_kernel") == block
    """ % ((K, T, opts, light, block),))


@pytest.mark.parametrize("K,T,least,most", [(100, 1 << 20, 0, 0), (100, (1 << 20) + 1, 1, 1 << 19), (100, 2 << 20, 1, 1 << 19),
                                            (100, (2 << 20) + 1, 3 << 20, 13 << 20), (70000, 2 << 20, 0, 0),
                                            (70000, (2 << 20) + 1, 3 << 20, 13 << 20)])
def test_staging_grows_with_the_results(host, K, T, least, most):
    """Threads and a large pinned staging are for results that are worth them; those of a small model take little or none."""
    host("""
        words = np.zeros(%d, np.int32)
        g = pk.Saber(np.r_[np.arange(0, words.size, 1000), words.size], words, 1, %d, 0.1, 0.01, 3)
        fake.fake_clear()
        for i in range(3):
            g.get_z()
            assert %d <= fake.fake_host_bytes() <= %d
    """ % (T, K, least, most))


@pytest.mark.parametrize("what", ["small tiles", "one long document", "many words", "words within the limit of the cut"])
def test_tiles_of_a_chunk_stay_within_the_static_work_space(host, what):
    """saber_loglik_static takes 2^20 tiles per chunk: neither the cut by ranges of documents nor the automatic size of a tile
    goes beyond, for a corpus that plain tiles of 8,192 tokens, or the caller's size, keep within."""
    host("""
        import paper_1610_02496_amd.binding as binding
        what, opts, K = %r, {}, 1000
        if what == "small tiles":                    # as many as there may be, unless words are cut into pieces on top
            V, tile = 40, 9
            T = tile * ((1 << 20) - 200)
            words = np.arange(T, dtype=np.int32) %% V
            words[:T // 2] = words[:T // 2] * 7 %% 11 # (uneven counts)
            doc_ptr, opts = np.r_[np.arange(0, T, 32), T], {"tile_tokens": tile}
        elif what == "one long document":            # a chunk of 70 M tokens where a hundredth of the corpus is 0.7 M
            V, K, T = 3, 2, 70_000_000
            words = np.zeros(T, np.int32)
            doc_ptr, opts = np.r_[np.arange(200), T], {"n_chunks": 100}
        elif what == "many words":
            V, K, T = (1 << 19) + 1, 20, 3_000_000
            words = (np.arange(T) * 7919 %% V).astype(np.int32)
            doc_ptr = np.r_[np.arange(0, T, 100), T]
        else:                                        # 17 V + 2^16 = 2^20 - 15
            V, T = 57825, 9_000_000
            words = (np.random.default_rng(1).random(T) ** 3 * V).astype(np.int32)
            doc_ptr, opts = np.r_[np.arange(0, T, 32), T], {"light_word_tokens": -1}
        g = pk.Saber(doc_ptr, words, V, K, 0.1, 0.01, 3, **opts)
        out = ctypes.c_double()
        assert binding.load_library().saber_loglik_static(g._h, ctypes.addressof(out)) == 0
        tiles = g.get_stats()["tiles"]
        if what == "many words": assert tiles == V   # (8,192 tokens at least: none of these words has more)
        if what == "words within the limit of the cut":
            n = np.bincount(words, minlength=V)
            assert tiles >= np.count_nonzero(n) + 15 * np.count_nonzero(n >= 2048)
    """ % what)


@pytest.mark.parametrize("T,length,K,cut", [(9_000_000, 32, 999, True), (9_000_000, 32, 1000, True), (9_000_000, 32, 60, True),
                                            (8_300_000, 32, 1000, False), (9_000_000, 250, 100, False),
                                            (9_000_000, 250, 999, True), (9_000_000, 250, 16384, True),
                                            (9_000_000, 250, 16385, False)])
def test_which_chunks_are_cut_by_ranges_of_documents(host, T, length, K, cut):
    """Those with enough tokens and with more rows of A than the caches hold, whatever the number of topics below the limit."""
    host("""
        T, length, K, cut = %d, %d, %d, %r
        words = np.arange(T, dtype=np.int32) %% 50
        doc_ptr = np.r_[np.arange(0, T, length), T]
        tiles = []
        for opts in ({}, {"stage_min_tokens": 2, "light_block_threads": 256}):   # (the second: never cut)
            g = pk.Saber(doc_ptr, words, 50, K, 0.1, 0.01, 3, tile_tokens=1 << 20, **opts)
            tiles.append(g.get_stats()["tiles"])
            g.close()
        assert tiles == [800 if cut else 50, 50]
    """ % (T, length, K, cut))


def test_classes_of_light_words_have_launches_of_their_own(host):
    """Of the corpora that the GPU tests compare: one launch for each class, tiles and workgroups as they should be."""
    host("""
        sys.path.insert(0, "tests")
        from test_gpu_launch_shapes import CLASSES, corpus_of_three_classes, corpus_of_word_counts
        counts, doc_ptr, words = corpus_of_three_classes()
        for K, n in CLASSES.items():
            g = pk.Saber(doc_ptr, words, counts.size, K, 50 / K, 0.01, 11, tile_tokens=1024)
            for use in (lambda: g.iterate(1), g.loglik, lambda: g.token_probs([0])):
                fake.fake_clear()
                use()
                got, blocks, most = launches("estep_kernel")
                assert got == n and blocks == g.get_stats()["tiles"], (K, got, blocks)
            assert fake.fake_block(b"estep_kernel") == {1000: 64, 2000: 128, 9000: 512}[K]
            g.close()
    """)


def test_host_memory_that_runs_out_is_a_status(host):
    """No exception leaves the library: also where the list of rows of an inspection call does not fit."""
    host("""
        import resource
        import paper_1610_02496_amd.binding as binding
        words = np.zeros(1000, np.int32)
        g = pk.Saber(np.array([0, 1000]), words, 1, 10, 0.1, 0.01, 3, light_word_tokens=-1)
        out = np.zeros(10)
        size = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
        resource.setrlimit(resource.RLIMIT_AS, (size + (1 << 30), -1))
        L, m = binding.load_library(), 1 << 30
        assert L.saber_alias_build_probe(g._h, words.ctypes.data, m, out.ctypes.data, out.ctypes.data, out.ctypes.data, None) == -2
    """)


def test_held_out_calls_that_break_off(host):
    """The scored documents' layout is another thread's work from 32,768 tokens on: whatever fails meanwhile, the call ends with
    a status and the next one works."""
    host("""
        V, K = 50, 100
        words = np.arange(140_000, dtype=np.int32) % V
        doc_ptr = np.r_[0, np.arange(999, words.size, 1000), words.size]
        g = pk.Saber(doc_ptr, words, V, K, 0.1, 0.01, 3)
        for n in (1, 2, 3, 65_534, 65_536, 65_538, 140_000):
            dp = np.minimum(doc_ptr, n)
            observed = (np.arange(n) % 2).astype(np.uint8)
            bad = words[:n].copy()
            for i in (0, n - 1):
                bad[:] = words[:n]
                bad[i] = V
                assert code_of(lambda: g.holdout_loglik(dp, bad, observed, 1, 5)) == -1
            z = np.full(int(observed.sum()), K, np.int32)
            assert code_of(lambda: g.holdout_loglik(dp, words[:n], observed, 1, 5, z)) == (-1 if z.size else 0)
            for call in ("hipMalloc", "hipMemcpy:", "estep_kernel", "hipStreamCreate"):
                for nth in range(1, 60):
                    fake.fake_fail(call.encode(), nth)
                    code = code_of(lambda: g.holdout_loglik(dp, words[:n], observed, 1, 5))
                    if fake.fake_fail_pending(): break
                    assert code in (-2, -3), (call, nth, code)
                fake.fake_fail(b"", 0)
            assert g.holdout_loglik(dp, words[:n], observed, 1, 5)[1] == n - observed.sum()
    """)


def test_kept_work_space_is_the_contexts_device(host):
    """Inspection calls keep their work space for later ones: it lies on the context's device, also where the caller has
    another one current, which stays so."""
    host("""
        now = ctypes.c_int()
        for first in (lambda g: g.token_probs([3]), lambda g: g.get_phi([0]), lambda g: g.token_probs(np.arange(50_000)),
                      lambda g: g.get_phi(np.zeros(90_000, np.int32))):      # (more than is kept)
            words = np.zeros(50_000, np.int32)
            g = pk.Saber(np.r_[0, 500, words.size], words, 1, 100, 0.1, 0.01, 3)
            fake.fake_clear()
            assert fake.hipSetDevice(1) == 0
            first(g)
            assert (fake.fake_mallocs_on(0), fake.fake_mallocs_on(1)) == (1, 0)
            fake.hipGetDevice(ctypes.byref(now))
            assert now.value == 1
            assert fake.hipSetDevice(0) == 0
            g.close()
    """)


@pytest.mark.parametrize("opts,times", [({}, (1, 1, 0, 1)),                                    # two launches
                                        ({"light_word_tokens": -1}, (1, 1, 1, 2))])            # documents; totals; denominators and Bhat
def test_profile_times_of_the_kernel_groups(host, opts, times):
    """Each launch of an iteration is in the time of its group (here a launch takes a millisecond), also where a small corpus'
    M-step takes two."""
    host("""
        opts, times = %r
        words = np.arange(5000, dtype=np.int32) %% 40
        g = pk.Saber(np.r_[0, 400, 800, words.size], words, 40, 400, 0.1, 0.01, 3, profile=1, long_doc_tokens=5000, **opts)
        g.iterate(3)
        s = g.get_stats()
        assert (s["ms_sample"], s["ms_count_dz"], s["ms_ck"], s["ms_phi"]) == tuple(3.0 * t for t in times), s
        assert s["ms_total"] == 3.0 * sum(times)
    """ % ((opts, times),))


def test_normalisers_of_more_tokens_than_a_grid_was_cut_to(host):
    """Every request has a thread that gathers its result (it used to be the first 268 million)."""
    host("""
        import paper_1610_02496_amd.binding as binding
        L, m = binding.load_library(), 65535 * 16 * 256 + 1
        g = pk.Saber(np.array([0, 1000]), np.zeros(1000, np.int32), 1, 10, 0.1, 0.01, 3)
        tok = np.zeros(m, np.int64)                 # (read only: it takes no memory, its copy does)
        assert L.saber_token_probs(g._h, tok.ctypes.data, m, None, None, None) == 0
        assert fake.fake_blocks(b"gather_probs") == -(-m // 256)
    """)


def test_held_out_call_in_little_host_memory(host):
    """Where both parts' layouts do not fit they are made one after the other: 8.5 bytes per token of documents of 1,000 tokens,
    13.6 side by side."""
    host("""
        V, K, n = 50, 100, 1_000_000
        words = np.arange(n, dtype=np.int32) % V
        doc_ptr = np.r_[0, np.arange(999, n, 1000), n]
        observed = (np.arange(n) % 2).astype(np.uint8)
        g = pk.Saber(doc_ptr, words, V, K, 0.1, 0.01, 3)
        for per_token, code in ((9, 0), (7, -2), (9, 0), (20, 0)):
            fake.fake_new_limit(per_token * n)
            assert code_of(lambda: g.holdout_loglik(doc_ptr, words, observed, 1, 5)) == code, per_token
        fake.fake_new_limit(-1)
        assert g.holdout_loglik(doc_ptr, words, observed, 1, 5)[1] == n // 2
    """)


@pytest.mark.parametrize("T,opts,m,marked", [(400_000, {}, 49_999, 1), (400_000, {}, 50_000, 0), (399_999, {}, 100, 0), (399_999, {}, 49_999, 0),
                                             (1_200_000, {"n_chunks": 3}, 100, 3), (1_197_000, {"n_chunks": 3}, 100, 0)])
def test_which_requests_for_normalisers_are_marked(host, T, opts, m, marked):
    """Fewer than an eighth of the tokens, in chunks whose pass costs more than marking them."""
    host("""
        T, opts, m, marked = %r
        g = pk.Saber(np.r_[np.arange(0, T, 1000), T], np.zeros(T, np.int32), 1, 100, 0.1, 0.01, 3, **opts)
        fake.fake_clear()
        g.token_probs(np.arange(m))
        assert launches("mark_tokens")[0] == launches("number_tokens")[0] == marked
    """ % ((T, opts, m, marked),))


def test_first_inspection_calls_share_a_block(host):
    """Fresh device memory costs more than a call: a sampler's first inspection calls allocate once where they need more than
    a MB, and never more than what is kept."""
    host("""
        words = np.arange(500_000, dtype=np.int32) % 40
        def mallocs(*calls):
            g = pk.Saber(np.r_[np.arange(0, words.size, 1000), words.size], words, 40, 1000, 0.1, 0.01, 3)
            fake.fake_clear()
            for call in calls: call(g)
            g.close()
            return fake.fake_calls(b"hipMalloc")
        probs = lambda m: lambda g: g.token_probs(np.arange(m) % words.size)
        phi = lambda m: lambda g: g.get_phi(np.arange(m, dtype=np.int32) % 40)
        assert mallocs(probs(60_000), phi(400)) == 1                    # 1.8 MB, 3.2 MB
        assert mallocs(phi(400), probs(500_000), phi(1000)) == 2        # 14 MB the second
        assert mallocs(phi(8000), phi(8400), phi(400), phi(8400)) == 3  # 64 MB; more than that lives as long as its call
        assert mallocs(phi(8400), phi(8400)) == 2
        # memory that is short: the size asked for if not the block, what is kept goes if a call needs more
        for calls, refused, n in (((phi(400), phi(400)), 1, 2), ((phi(400), phi(8400)), 2, 3), ((phi(8400), phi(400)), 2, 3)):
            fake.fake_fail(b"hipMalloc", 0)
            g = pk.Saber(np.r_[np.arange(0, words.size, 1000), words.size], words, 40, 1000, 0.1, 0.01, 3)
            fake.fake_clear()
            fake.fake_fail(b"hipMalloc", refused)
            for call in calls: call(g)
            assert fake.fake_calls(b"hipMalloc") == n and fake.fake_fail_pending() == 0
            g.close()
    """)


@pytest.mark.parametrize("K,opts,cus,walkers", [(9000, {}, 256, 20_000), (9000, {}, 64, 5000), (9000, {}, 8, 2500), (3900, {}, 8, 20_000),
                                                (9000, {"stage_phi": 0}, 8, 20_000), (20_011, {}, 256, 10_000), (20_011, {}, 8, 2500)])
def test_workgroups_that_light_words_are_dealt_to(host, K, opts, cus, walkers):
    """20,000 tiles of light words, K = 9,000: four workgroups of 512 threads fit a CU, and every place gets 16 or more in turn; at
    most eight tiles each; one where rows are short or not staged.  K = 20,011: two of 1,024."""
    host("""
        K, opts, cus, walkers = %r
        fake.fake_cus(cus)
        words = np.repeat(np.arange(20_000, dtype=np.int32), 5)
        g = pk.Saber(np.r_[np.arange(0, words.size, 1000), words.size], words, 20_000, K, 0.1, 0.01, 3, **opts)
        fake.fake_clear()
        g.iterate(1)
        assert fake.fake_blocks(b"estep_kernel") == walkers
        fake.fake_clear()
        g.loglik()
        assert fake.fake_blocks(b"estep_kernel") == g.get_stats()["tiles"] == 20_000
    """ % ((K, opts, cus, walkers),))


@pytest.mark.parametrize("observed,scored,pack", [(16_383, 4000, 2), (16_384, 4000, 1), (20_000, 4000, 1), (4000, 20_000, 2), (16_383, 16_384, 2)])
def test_scored_parts_read_the_observed_parts_rows(host, observed, scored, pack):
    """The kernel that scores is the one for the counts in the rows of A that it reads, whatever length the scored parts have."""
    host("""
        observed, scored, pack = %r
        words = (np.arange(observed + scored) %% 40).astype(np.int32)
        g = pk.Saber(np.array([0, 1000]), words[:1000], 40, 300, 0.1, 0.01, 3)
        fake.fake_clear()
        mask = np.arange(observed + scored) < observed
        g.holdout_loglik(np.array([0, words.size]), words, mask, 0, 5)
        kernel = "estep_kernelILi2ELb1EtLi%%dE"      # log-likelihood, staged rows, 16-bit assignments
        assert [launches(kernel %% p)[0] for p in (0, 1, 2)] == [int(p == pack) for p in (0, 1, 2)]
    """ % ((observed, scored, pack),))


@pytest.mark.parametrize("K,opts,walkers", [(37_010, {}, 2500), (37_020, {}, 2500), (37_040, {}, 2500), (37_060, {}, 2500), (37_240, {"block_threads": 960}, 2500),
                                            (37_650, {"block_threads": 832}, 2500), (36_000, {"light_block_threads": 1024, "block_threads": 64}, 2500)])
def test_workgroups_whose_lds_is_all_a_cu_has(host, K, opts, walkers):
    """A staged row and the wavefronts' parts of LDS may fill a CU's to the last piece: one workgroup fits, and light words' tiles
    are dealt to as many as fit the chip."""
    host("""
        K, opts, walkers = %r
        fake.fake_cus(8)
        words = np.repeat(np.arange(20_000, dtype=np.int32), 5)
        g = pk.Saber(np.r_[np.arange(0, words.size, 1000), words.size], words, 20_000, K, 0.1, 0.01, 3, **opts)
        fake.fake_clear()
        g.iterate(1)
        assert fake.fake_blocks(b"estep_kernel") == walkers
    """ % ((K, opts, walkers),))


STREAMED = """
        V, K = 60, %d
        words = np.arange(30_000, dtype=np.int32) * 7 %% V
        lens = np.r_[np.resize([0, 40, 900, 3], 60), 1000]
        lens[-1] = words.size - lens[:-1].sum()
        doc_ptr = np.r_[0, np.cumsum(lens)]
        g = pk.Saber(doc_ptr, words, V, K, 0.1, 0.01, 3, stream_workers=%d, n_chunks=%d)
        z = np.zeros(words.size, np.int32)
        uses = {"iterate": lambda: g.iterate(2), "get_z": g.get_z, "loglik": g.loglik, "probs": lambda: g.token_probs([3, 29_000]),
                "set_z": lambda: g.set_z(z, 0), "counts": lambda: g.counts()}
"""


@pytest.mark.parametrize("workers,chunks", [(1, 5), (2, 5), (3, 5), (3, 2), (2, 1), (4, 3)])
@pytest.mark.parametrize("K", [100, 70_000])
def test_buffers_of_streamed_chunks_are_used_in_order(host, K, workers, chunks):
    """Copies of token lists, the expansion of their documents and the kernels that read them run on three streams, a checkpoint
    looks a chunk ahead: whatever call follows which, a buffer's uses are in order."""
    host(STREAMED % (K, workers, chunks) + """
        for first in uses.values():
            for second in uses.values():
                first()
                second()
        assert launches("expand_tok_doc")[0] and launches("scatter_zwm")[0] and launches("estep_kernel")[0]
        assert races() == (0, "")
    """)


@pytest.mark.parametrize("workers,chunks", [(1, 5), (2, 5), (3, 4)])
def test_buffers_of_streamed_chunks_after_a_call_that_broke_off(host, workers, chunks):
    """What a failed call has queued for a buffer may still run when the next call takes the buffer."""
    host(STREAMED % (100, workers, chunks) + """
        nth_max = 0
        for name, first in uses.items():
            for call in ("expand_tok_doc", "estep_kernel", "count_dz", "scatter_zwm", "fill_zwm", "hipEventRecord", "hipMemcpyAsync", "hipMemcpy:", "hipStreamWaitEvent"):
                for nth in range(1, 60):
                    fake.fake_fail(call.encode(), nth)
                    code = code_of(first)
                    if fake.fake_fail_pending(): break
                    nth_max = max(nth, nth_max)
                    fake.fake_fail(b"", 0)
                    assert code in (0, -2, -3), (name, call, nth, code)
                    for second in (uses["get_z"], uses["iterate"])[::1 if nth % 2 else -1]: second()
                    assert races() == (0, ""), (name, call, nth, races())
                fake.fake_fail(b"", 0)
        assert nth_max > 4
    """)


@pytest.mark.parametrize("K,few,wide,shares", [(5000, 16_384, 40, 40 + 4096), (5000, 16_383, 40, 16_423), (8192, 20_001, 3, 3 + 5001), (8193, 20_001, 3, 20_004),
                                               (1000, 16_386, 0, 4097), (1000, 16_386, 40, 40 + 4097), (1000, 16_383, 1, 16_384)])
def test_wavefronts_of_light_words(host, K, few, wide, shares):
    """Light words are four to a wavefront where rows are short and words many, those of more than 256 tokens alone."""
    host("""
        K, few, wide, shares = %r
        rng = np.random.default_rng(K)
        counts = np.r_[np.full(wide, 257), 256, np.ones(few - 1, int)]
        words = np.repeat(rng.permutation(counts.size).astype(np.int32), counts)
        g = pk.Saber(np.r_[np.arange(0, words.size, 1000), words.size], words, counts.size, K, 0.1, 0.01, 3, light_word_tokens=1000)
        fake.fake_clear()
        g.iterate(1)
        alone, joined = launches("light_tree")[1], launches("mstep_rows")[1]
        if K > 4096: assert (alone, joined) == (shares, 0)
        else: assert alone == 0 and joined == -(-shares // 4) + min(256, -(-counts.size // fake.fake_block(b"mstep_rows")))
    """ % ((K, few, wide, shares),))


@pytest.mark.parametrize("K,cus,rows,parts", [(8257, 256, 256, 2), (8257, 256, 257, 0), (8192, 256, 10, 0), (20_011, 64, 64, 3), (20_011, 64, 65, 0), (70_000, 256, 2, 9)])
def test_which_rows_of_bhat_are_worked_on_by_parts(host, K, cus, rows, parts):
    """Rows of several ranges of topics, where there are no more of them (with the base vector) than CUs."""
    host("""
        K, cus, rows, parts = %r
        fake.fake_cus(cus)
        words = np.repeat(np.arange(rows - 1 + 5, dtype=np.int32), np.r_[np.full(rows - 1, 20), np.full(5, 3)])
        g = pk.Saber(np.r_[np.arange(0, words.size, 1000), words.size], words, rows + 4, K, 0.1, 0.01, 3, light_word_tokens=10)
        fake.fake_clear()
        g.iterate(1)
        assert launches("phi_sums")[1] == (rows if parts else 0)
        assert launches("phi_tree")[1] == rows * max(parts, 1)
    """ % ((K, cus, rows, parts),))
