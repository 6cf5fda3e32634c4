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
