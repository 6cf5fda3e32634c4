"""The ordering's radix sort at the edges of its layout: digits of 8 and 9
bits, key and index in one word or apart, tiles and counting chunks with
remainders, aligned and unaligned inputs; bit-exact against the oracle."""
import numpy as np
import pytest
import torch

from gpu_cases import check_order, dvl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dvl()


def _cells(n, bits, seed):
    """n distinct finest-level cells of a 2^bits cube, its far corner among them, in random order."""
    import synth
    g = np.random.default_rng(seed)
    side = 1 << bits
    if bits <= 7:
        flat = g.permutation(side ** 3)[:n].astype(np.int64)
        flat[0] = side ** 3 - 1 if side ** 3 - 1 not in flat else flat[0]
    else:
        flat = np.unique(g.integers(0, side ** 3, n + n // 8 + 16))
        flat = g.permutation(flat)[:n]
        flat[0] = side ** 3 - 1
        assert np.unique(flat).size == n
    c = [torch.from_numpy(((flat >> (bits * k)) & (side - 1)).astype(np.int32)) for k in range(3)]
    f = torch.from_numpy(g.random(n).astype(np.float32))
    return synth.Volume(c[0], c[1], c[2], torch.zeros(n, dtype=torch.uint8), [f], ["f"], side, 1, [])


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("n,bits", [(1, 1), (8, 1), (60, 2), (4095, 4), (4096, 5), (4097, 6), (70000, 7), (131072, 9),
                                    (300001, 11), (4097, 12), (65537, 14), (20000, 16), (20000, 17), (9000, 18),
                                    (70001, 19), (4096, 20), (300001, 21), (5, 21), (2, 21)])
def test_order_bit_exact(n, bits, offset):
    D = dvl()
    vol = _cells(n, bits, seed=n + bits)

    def put(t):
        buf = torch.zeros(t.numel() + offset, dtype=t.dtype, device="cuda")
        buf[offset:] = t.to("cuda")
        return buf[offset:]

    V = D.build_order(put(vol.x), put(vol.y), put(vol.z), put(vol.level), [put(vol.fields[0])])
    try:
        check_order(V, vol)
    finally:
        V.close()


def test_order_of_a_large_volume_is_a_sorted_permutation():
    """More tiles than one counting chunk per column wave: 24 M cells of a
    regular grid in reversed order; keys increase along the permutation and
    the permutation holds every cell once."""
    D = dvl()
    s = 288
    i = torch.arange(s ** 3, device="cuda", dtype=torch.int64).flip(0)
    x, y, z = (i % s).int(), ((i // s) % s).int(), (i // (s * s)).int()
    V = D.build_order(x, y, z, torch.zeros_like(x, dtype=torch.uint8), [i.float()])
    try:
        keys, perm = V.export_order()
        k = keys[perm.long()]
        assert bool((k[1:] > k[:-1]).all())
        assert bool((torch.bincount(perm.long(), minlength=s ** 3) == 1).all())
    finally:
        V.close()


def test_duplicates_and_order_past_the_caches():
    """More than 2^25 cells (passes read as streams): the keys back in the
    original order belong to the sorted ones, and a repeated cell at either end
    or in the middle of the sorted order is refused."""
    D = dvl()
    s = 324
    n = s ** 3 + 1
    i = torch.arange(s ** 3, device="cuda", dtype=torch.int64).flip(0)
    x, y, z = (torch.cat([c, c.new_full((1,), s)]) for c in ((i % s).int(), ((i // s) % s).int(), (i // (s * s)).int()))
    level = torch.zeros(n, dtype=torch.uint8, device="cuda")
    field = torch.arange(n, device="cuda").float()
    V = D.build_order(x, y, z, level, [field])
    try:
        keys, perm = V.export_order()
        k = keys[perm.long()]
        assert bool((k[1:] > k[:-1]).all())
        assert bool((torch.bincount(perm.long(), minlength=n) == 1).all())
        alone = torch.empty_like(perm)
        import ctypes as C
        assert D.lib().dvl_export_order(V.handle, C.c_void_p(0), C.c_void_p(alone.data_ptr()), C.c_void_p(0)) == 0
        torch.cuda.synchronize()
        assert torch.equal(alone, perm)
        assert torch.equal(V.export_sorted()[1][0], field[perm.long()])
        ends = [int(perm[h]) for h in (0, 1, n // 2, n - 2, n - 1)]
    finally:
        V.close()
    for at in ends:
        c = [t.clone() for t in (x, y, z)]
        other = (at + 1) % n
        for t in c:
            t[other] = t[at].clone()
        with pytest.raises(D.DvlError) as e:
            D.build_order(*c, level, [field])
        assert e.value.status == D.E_OVERLAP


@pytest.mark.parametrize("n", [2, 3, 5, 8, 13, 514, 4099])
def test_a_repeated_cell_is_found_wherever_it_lies(n):
    D = dvl()
    vol = _cells(n, 7, seed=n).to("cuda")
    for at in range(n) if n < 20 else sorted({0, 1, n - 1, n - 2, *range(63, n, 1 + n // 17)}):
        c = [t.clone() for t in (vol.x, vol.y, vol.z)]
        for t in c:
            t[at] = t[(at + n // 2) % n].clone()
        with pytest.raises(D.DvlError) as e:
            D.build_order(*c, vol.level, vol.fields)
        assert e.value.status == D.E_OVERLAP, at


@pytest.mark.parametrize("n", [1023, 1024, 1025, 3 * 1024 + 1, (3 << 19) - 1023, 3 << 19, (3 << 19) + 1, (3 << 19) + 4095])
def test_tiles_of_both_sizes(n):
    """Edges of the small tiles, and of the volumes that take the large ones:
    the permutation sorts the exported keys."""
    D = dvl()
    vol = _cells(n, 7 if n < 100000 else 9, seed=n).to("cuda")
    V = D.build_order(vol.x, vol.y, vol.z, vol.level, vol.fields)
    try:
        keys, perm = V.export_order()
        assert torch.equal(perm.long(), torch.argsort(keys))
        assert torch.equal(V.export_sorted()[1][0], vol.fields[0][perm.long()])
    finally:
        V.close()
