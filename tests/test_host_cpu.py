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
