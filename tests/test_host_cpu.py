"""Host code of the library on the CPU, over a stand-in for the HIP runtime:
what is allocated, launched and captured, and what a call returns, without a
GPU and without running a kernel."""
import fake_hip


def test_graph_is_captured_again_when_its_reads_change(tmp_path):
    """The captured launch says whether the cells bypass the caches, which
    depends on which volumes read entries and which read values: 120 + 80 MB
    fit the caches, 480 + 20 MB do not, with the same kernel variants."""
    fake_hip.run(tmp_path, '''
    A, B = build(30_000_000), build(5_000_000)
    g = C.c_void_p()
    reqs = [request(A, 64), request(B, 64)]
    ok(L.dvl_graph_create((D.dvl_request * 2)(*reqs), 2, C.byref(g)))

    def captured(cached, values):
        ok(L.dvl_set_entry_cache(cached, D.ENTRY_CACHE_ALWAYS))
        ok(L.dvl_set_entry_cache(values, D.ENTRY_CACHE_NEVER))
        H.fake_reset()
        for _ in range(4):                     # two descriptor slots, twice
            ok(L.dvl_graph_launch(g, None))
        return H.fake_instantiated()

    assert captured(A, B) == 2
    assert captured(B, A) == 2
    assert captured(A, B) == 0                 # both forms are kept
    L.dvl_graph_destroy(g)
    for v in (A, B):
        L.dvl_destroy(v)
    ''')


def test_value_readers_of_one_volume_share_a_launch(tmp_path):
    """Requests that read the values of one large volume (320 MB): up to 8 in a
    launch, whose workgroups number a multiple of 8 (one per XCD) per request
    and fit the chip (5 to a compute unit here); the rest as before."""
    fake_hip.run(tmp_path, '''
    V, small = build(20_000_000, entry_cache=2), build(100_000, entry_cache=2)
    ex = executor()

    def sums(reqs):
        H.fake_reset()
        batch(ex, reqs)
        return [x for _, x, _ in launched("k_tile_sums")]

    for k in (2, 3, 8):
        g = sums([request(V, 64) for _ in range(k)])
        assert len(g) == 1 and g[0] % (8 * k) == 0 and 1000 <= g[0] <= 1280, (k, g)
    g = sums([request(V, 64) for _ in range(9)])
    assert len(g) == 2 and g[0] % 64 == 0, g                 # 8, and one alone
    assert len(sums([request(V, 64) for _ in range(16)])) == 2
    assert len(sums([request(small, 64) for _ in range(4)])) == 1
    assert len(sums([request(V, 64), request(small, 64), request(V, 64, scan_mode=1)])) == 2
    # readers of cached entries have their own launch
    ok(L.dvl_set_entry_cache(V, D.ENTRY_CACHE_ALWAYS))
    g = sums([request(V, 64) for _ in range(4)])
    assert [n for n, _, _ in launched("k_tile_sums")] == ["_ZN3dvl11k_tile_sumsILi4ENS_3F32ELi1EEEvNS_8BatchDevE"], launched()
    L.dvl_executor_destroy(ex)
    for v in (V, small):
        L.dvl_destroy(v)
    ''')


def test_failing_build_without_host_memory(tmp_path):
    """A build whose device allocation fails while the host has no memory left
    either returns its status: nothing on its way out allocates."""
    fake_hip.run(tmp_path, '''
    H.fake_fail_attribute(1)                   # a long message first: its buffer has its size then
    assert L.dvl_executor_create(C.byref(C.c_void_p())) == D.E_HIP
    H.fake_fail_attribute(0)
    v, f = C.c_void_p(), (C.c_void_p * 1)(mem(16))
    a = [mem(16) for _ in range(4)]
    for _ in range(12):                        # more than the library keeps pages for
        H.fake_fail_mallocs(1)
        H.fake_fail_new(1)
        st = L.dvl_build_order(1000, *a, 1, 0, C.cast(f, C.c_void_p), None, C.byref(v))
        H.fake_fail_new(0)
        assert st == D.E_NOMEM and not v.value, st
    assert H.fake_host_mallocs() <= 2
    ''')


def test_bins_of_one_volume_read_by_two_threads(tmp_path):
    """Two threads read different bins of one volume at the same time (both
    launches are enqueued before either wait returns): each gets its own.  What
    is pinned for it does not grow with the volumes."""
    fake_hip.run(tmp_path, '''
    import threading
    W = 64
    vols = [build(1000, M=1) for _ in range(12)]

    def device_bins(value):
        b, arrays = D.dvl_bins(), []
        for name, dt, n in (("first_cell", np.uint32, W), ("last_cell", np.uint32, W), ("mean", np.float32, W), ("vmin", np.float32, W),
                            ("vmax", np.float32, W), ("y", np.float32, W), ("f_total", np.float64, 1), ("vmax_used", np.float32, 1)):
            a = np.full(n, value, dt)
            KEEP.append(a)
            setattr(b, name, a.ctypes.data)
        return b

    def read(v, value):
        out = [np.zeros(W, np.uint32) for _ in range(3)] + [np.zeros(W, np.float32) for _ in range(4)]
        tot = [np.zeros(1, np.float64), np.zeros(1, np.float32)]
        b = device_bins(value)
        ok(L.dvl_read_bins(v, C.byref(b), W, None, *[a.ctypes.data for a in out + tot]))
        assert (out[0] == 1).all(), out[0]
        for a in out[1:] + tot:
            assert (a == value).all(), (value, a)

    fails = []
    def thread(v, value):
        try:
            read(v, value)
        except AssertionError as e:
            fails.append(e)

    for rnd in range(3):
        H.fake_sync_parties(2)
        ts = [threading.Thread(target=thread, args=(vols[0], x)) for x in (3 + rnd, 40 + rnd)]
        [t.start() for t in ts]
        [t.join() for t in ts]
        H.fake_sync_parties(0)
        assert not fails, fails
    H.fake_reset()
    for i, v in enumerate(vols):
        read(v, 100 + i)
    assert H.fake_host_mallocs() == 0
    ''')


def test_entry_cache_of_mixed_requests(tmp_path):
    """Requests on one volume decide about its entry cache eight at a time: a
    batch with one request of other windows builds and reads it for the others."""
    fake_hip.run(tmp_path, '''
    ex = executor()
    sums = "k_tile_sumsILi4ENS_3F32ELi%dE"

    def run(V, *his):
        H.fake_reset()
        batch(ex, [request(V, 64, hi=h) for h in his])
        return len(launched(sums % 1)), len(launched(sums % 0)), len(launched("k_build_index"))

    def cached(V):
        hi = np.zeros(4, np.float32)
        return hi[0] if L.dvl_entry_cache_info(V, None, hi.ctypes.data, None) else None

    V = build(1_000_000, entry_cache=D.ENTRY_CACHE_ALWAYS)
    assert run(V, *[1.0] * 8, 0.5) == (1, 1, 4) and cached(V) == 1.0
    assert run(V, *[1.0] * 8, 0.5) == (1, 1, 0)              # kept
    assert run(V, *[1.0] * 8, *[0.5] * 8) == (1, 1, 0) and cached(V) == 1.0
    assert run(V, 1.0, 0.5) == (0, 1, 0) and cached(V) == 1.0   # no eight agree
    assert run(V, *[0.5] * 3) == (1, 0, 4) and cached(V) == 0.5
    # the automatic policy: built when two updates in a row use the same windows
    W = build(1_000_000)
    assert run(W, *[1.0] * 8) == (0, 1, 0) and cached(W) is None
    assert run(W, *[1.0] * 8, 0.5) == (1, 1, 4) and cached(W) == 1.0
    ''')


def test_first_update_allocates_nothing(tmp_path):
    """A new volume, or a zoom, has room for the descriptors of any single
    update and for the workspace of plots up to 3840 wide (with stored f where
    a plot of 1920 stores it), with and without a caller's allocator."""
    fake_hip.run(tmp_path, '''
    live, calls = {}, [0]
    def get(ctx, n, stream):
        calls[0] += 1
        a = np.empty(1, np.uint8) if n > 1 << 26 else np.empty(n, np.uint8)
        live[a.ctypes.data] = a
        return a.ctypes.data
    def put(ctx, p, stream):
        del live[p]
    cb = (D.ALLOC_FN(get), D.RELEASE_FN(put))
    own = D.dvl_allocator(cb[0], cb[1], None)

    def first(v, W, n_tf, M):
        set_tfs(v, M, n_tf)
        H.fake_reset()
        before = calls[0]
        update(v, W, M)
        return H.fake_mallocs() + H.fake_frees() + calls[0] - before

    H.fake_reset()
    made = 0
    for al in (None, C.pointer(own)):
        for n, M, Ws in ((1000, 1, (1, 3840)), (262144, 4, (1024, 3840)), (1_000_000, 16, (1920,)), (31_000_000, 4, (1920, 3840)),
                         (60_000_000, 4, (1920,)), (200_000_000, 4, (3840,))):
            for W in Ws:
                for n_tf in (256, 16384 // M if M >= 4 else 4096):
                    v = build(n, M, allocator=al)
                    assert first(v, W, n_tf, M) == 0, (n, M, W, n_tf)
                    if W == Ws[0]:
                        z = zoom(v, 10, n // 2)
                        assert first(z, W, n_tf, M) == 0, ("zoom", n, M, W, n_tf)
                        L.dvl_destroy(z)
                    L.dvl_destroy(v)
    assert not live
    # wider plots and more stored f grow the workspace, and all of it is given back
    for al in (None, C.pointer(own)):
        H.fake_reset()
        v = build(300_000, allocator=al)
        set_tfs(v)
        for W in (3840, 100_000, 10, 200_000):
            update(v, W)
        ex = executor()
        batch(ex, [request(v, 5000)])
        L.dvl_executor_destroy(ex)
        L.dvl_destroy(v)
        assert H.fake_mallocs() == H.fake_frees() and not live
    ''')


def test_small_masks_take_one_launch(tmp_path):
    fake_hip.run(tmp_path, '''
    r = np.array([0, 5, 9, 9], np.uint64)
    for n, launches in ((1, 1), (65536, 1), (65537, 1), (4_000_000, 1), (4_000_001, 2)):
        v = build(n)
        H.fake_reset()
        ok(L.dvl_select_mask(v, r.ctypes.data, 2, mem(16), None))
        assert len(launched()) == launches, (n, launched())
        L.dvl_destroy(v)
    ''')


def test_histogram_variants(tmp_path):
    """Counter copies and loads by the cells of a bin."""
    fake_hip.run(tmp_path, '''
    def variant(n, W, H_):
        v = build(n, M=1)
        H.fake_reset()
        ok(L.dvl_bin_histograms(v, C.byref(bins(W, 1)), W, 0, H_, C.c_float(0.0), C.c_float(1.0), mem(16), None))
        (name, _, _), = launched()
        L.dvl_destroy(v)
        return name[name.index("F32E") + 4:name.index("EEEvPK")]

    single, quads, copies = "Li1ELb0", "Li1ELb1", "Li8ELb1"
    for n, W, h, want in ((3_000_000, 1 << 20, 64, single), (47_000, 1000, 1, single), (64_000, 1000, 1, copies), (255_000, 1000, 256, single),
                          (256_000, 1000, 256, quads), (1_023_999, 1000, 256, quads), (1_024_000, 1000, 256, copies),
                          (20_000_000, 1000, 513, quads), (11_800_000, 1920, 64, copies)):
        assert variant(n, W, h) == want, (n, W, h, variant(n, W, h))
    ''')
