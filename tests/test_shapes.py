"""The index rules that the kernels share with host code, run on the CPU: the
same header built by the host compiler."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("shapes") / "libshapes.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", out, os.path.join(HERE, "shapes_host.cpp")],
                   check=True)
    lib = ctypes.CDLL(out)
    u32, u64, P = ctypes.c_uint32, ctypes.c_uint64, ctypes.c_void_p
    lib.items_of.restype = u64
    lib.items_of.argtypes = [u32, u32, u32, u32, P, P]
    lib.xv_offsets.argtypes = [ctypes.c_int32, u64, u32, u32, u64, u32, P]
    lib.xv_offsets.restype = None
    lib.number_tiles.argtypes = [u32, P, P, P]
    lib.number_tiles.restype = None
    lib.copiers.argtypes = [u32, u64, u32]
    lib.copiers.restype = u32
    lib.slot_groups.argtypes = [u64, u32, u32, u32, u32, u32, u32, u32]
    lib.slot_groups.restype = u32
    lib.waves.argtypes = [u64, u64]
    lib.waves.restype = u64
    lib.alone.argtypes = [u64, u32, ctypes.c_int32]
    return lib


def _items(lib, kept, pieces, t, threads, seen=None):
    total = ctypes.c_uint64()
    n = lib.items_of(kept, pieces, t, threads, ctypes.byref(total), seen.ctypes.data if seen is not None else None)
    return n, total.value


@pytest.mark.parametrize("kept,pieces", [(0, 5), (1, 1), (3, 100), (256, 7), (255, 33), (17, (1 << 20) + 3)])
def test_record_items_take_every_piece_once(lib, kept, pieces):
    seen = np.zeros(max(1, kept * pieces), np.uint8)
    n = sum(_items(lib, kept, pieces, t, 256, seen)[0] for t in range(256))
    assert n == kept * pieces
    assert (seen[:n] == 1).all()


@pytest.mark.parametrize("kept,pieces", [(256, 1 << 24), (255, 16843009), (64, (1 << 26) + 1)])
def test_record_items_of_very_wide_records(lib, kept, pieces):
    """Items past 2^32: kept * pieces = 2^32, 2^32 - 1 and 2^32 + 64; each thread ends after its share."""
    counts = [_items(lib, kept, pieces, t, 256)[0] for t in (0, 1, 255)]
    for n in counts:
        assert abs(n - kept * pieces / 256) <= pieces / (1 << 20) + 1


@pytest.mark.parametrize("rows,words,whole", [(1, 3, 0), (5, 16, 1), (5, 16, 0), (3, 20, 1), (2, 4096, 1), (2, (1 << 31) + 21, 0),
                                              (3, (1 << 31) + 16, 1), (2, (1 << 32) - 16, 1), (2, (1 << 32) - 16, 0)])
def test_gathered_tables_tile_their_words(lib, rows, words, whole):
    """The X1 and V slices of neighbouring rows and slices follow one another without overlap, to the tables' end."""
    nb = (words + 15) // 16
    to = np.zeros(2, np.uint64)
    for row in range(rows):
        for b in sorted(b for b in {0, 1, nb // 2, nb - 2, nb - 1, (1 << 27) - 1, 1 << 27} if 0 <= b < nb):
            length = min(16, words - 16 * b)
            lib.xv_offsets(whole, row, b, length, rows, words, to.ctypes.data)
            at = 2 * row * words + 32 * b if whole else row * words + 16 * b
            assert to.tolist() == [at, at + length if whole else rows * words + at]


@pytest.mark.parametrize("tiles", [[5, 7, 1], [1 << 27] * 70, [0xFFFFFFF0, 1, 0xFFFFFFEF, 1, 1], [3] + [1 << 27] * 33])
def test_tiles_of_a_batch_are_numbered_launch_by_launch(lib, tiles):
    t = np.array(tiles, np.uint64)
    first, starts = np.zeros(t.size, np.uint32), np.zeros(t.size, np.uint8)
    lib.number_tiles(t.size, t.ctypes.data, first.ctypes.data, starts.ctypes.data)
    total = 0
    for i, k in enumerate(tiles):
        if starts[i]:
            assert i == 0 or total + k > 0xFFFFFFF0          # no launch ends early
            total = 0
        assert first[i] == total
        total += k
        assert total <= 0xFFFFFFF0


@pytest.mark.parametrize("rows,words", [(1, 1), (70, 1999), (300, 500), (1100, 999), (2000, 500), (8000, 256), (8000, 4),
                                        (100003, 20), (1 << 22, 16), (65, 1 << 24), (1 << 20, 1 << 16)])
def test_wide_records_are_copied_by_many_workgroups(lib, rows, words):
    """A compaction whose records hold 16 KB and more for every CU has a workgroup for each of the 256; no table takes
    more than a grid allows, and none a workgroup without a row's worth of pieces."""
    blocks = max(1, min(2048, rows // 256))
    y = lib.copiers(blocks, rows, words)
    assert 1 <= y <= 65535
    if rows * words * 4 >= 256 * 16384:
        assert blocks * y >= 256
    pieces = min(rows, 256) * (words if words % 4 else words // 4)
    assert y == 1 or y * 256 <= pieces


@pytest.mark.parametrize("kept,pieces,groups", [(256, 33, 3), (7, 500, 9), (1, 5, 2)])
def test_copiers_share_the_pieces(lib, kept, pieces, groups):
    seen = np.zeros(kept * pieces, np.uint8)
    for t in range(256 * groups):
        _items(lib, kept, pieces, t, 256 * groups, seen)
    assert (seen == 1).all()


def _slots(lib, lens, calls, wx):
    """Workgroups of each slot of a selection over these lists, as the library launches it."""
    n, lmax, nrec = len(lens), int(max(lens)), int(sum(lens))
    least = -(-n // 2048)
    most = max(least, min(-(-n // 64), 4096 // lmax + 1))
    m = 8 if calls > 4 else 4 if calls > 1 else 1
    v = 2 if m == 8 else 1 if m == 1 and wx <= 128 else 4
    got = [lib.slot_groups(n, lmax, m, v, wx, most, l, nrec) for l in range(lmax)]
    for c in got:
        assert least <= c <= most                           # within the grid, at most 2,048 candidates each
    return got, least, most


@pytest.mark.parametrize("n,length,wx,calls", [(3000, 24, 94, 1), (3000, 24, 94, 8), (200, 24, 250, 1), (30011, 24, 32, 3),
                                               (1000, 300, 32, 8), (60000, 4, 500, 1), (20000, 16, 4, 1)])
def test_slots_of_equal_lists_are_shared_alike(lib, n, length, wx, calls):
    """Lists of one length reach every slot alike, so every slot has as many workgroups (the float rule may differ by
    one), and together they fill the chip as far as the lists go."""
    got, least, most = _slots(lib, [length] * n, calls, wx)
    assert max(got) - min(got) <= 1
    assert sum(got) >= min(256, length * most)


@pytest.mark.parametrize("calls", [1, 3, 8])
@pytest.mark.parametrize("n,longest,wx", [(30011, 24, 250), (3000, 24, 94), (500, 300, 7), (1, 1, 1), (70, 9, 1000)])
def test_slots_of_skewed_lists(lib, n, longest, wx, calls):
    """Short lists mostly: the first slot has the most workgroups, later ones no more than the ones before."""
    lens = np.minimum(np.random.default_rng(1).zipf(1.8, n) - 1, longest)
    lens[-1] = longest
    got, least, most = _slots(lib, lens, calls, wx)
    assert got == sorted(got, reverse=True)
    assert got[-1] == least or got[-1] < got[0] or most < 8


@pytest.mark.parametrize("nrec", [0, 1, 2**32 - 1])
def test_slots_at_the_ends(lib, nrec):
    for n, lmax, most in ((1, 1, 1), (2**32 - 1, 65535, 2**21), (5, 65535, 1), (2**32 - 1, 1, 2**26)):
        for l in {0, lmax - 1}:
            c = lib.slot_groups(n, lmax, 8, 2, 3, max(most, -(-n // 2048)), l, nrec)
            assert -(-n // 2048) <= c <= max(most, -(-n // 2048))


@pytest.mark.parametrize("rows,words,shuffle,fetch", [(1, 1, 1, 1), (64, 1 << 20, 1, 1), (65, 16, 1, 1), (128, 32, 1, 1), (129, 2, 0, 0),
                                                      (100, 48, 0, 1), (107, 48, 0, 0), (128, 2**32 - 1, 0, 0)])
def test_one_workgroup_where_it_wins(lib, rows, words, shuffle, fetch):
    """The line between one workgroup's shuffle and launches over the chip, on both sides of the measured crossings."""
    assert (bool(lib.alone(rows, words, 0)), bool(lib.alone(rows, words, 1))) == (bool(shuffle), bool(fetch))


@pytest.mark.parametrize("tiles", [0, 1, 4, 511, 512, 2048, 2049, 5000, 8192, 8193, 1 << 31])
def test_aes_workgroups_have_waves_enough_for_their_tables(lib, tiles):
    w = lib.waves(tiles, 512)
    assert 4 <= w <= 16
    assert w in (4, 16) or 512 * (w - 1) < tiles <= 512 * w
