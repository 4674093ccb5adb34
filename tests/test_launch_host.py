"""The host side of wpm_enumerate on the CPU, with a double of the HIP runtime:
what it reads, what it refuses and what it launches."""
import pytest

import hipdouble as H


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return H.build(tmp_path_factory.mktemp("hipdouble"))


COMMON = r"""
words = np.zeros(64, np.uint64)
batch = L.Batch(num_instances=1, max_row_words=8, max_kp=24, d_tables=64, d_offsets=64)
def enumerate(kind=0, **kw):
    batch.flags = kind
    a = dict(mode=L.SCHED_DYNAMIC, wg_size=256, grid=0, d_items=64, num_items=5, d_scratch=64, d_bin_offsets=64)
    a.update(kw)
    s = L.Sched(**a)
    return L.lib().wpm_enumerate(ctypes.byref(batch), ctypes.byref(s), None, 0, words.ctypes.data,
                                 words.ctypes.data, None, None)
"""


def check(so, code):
    rc, out, err = H.run(so, COMMON + code)
    assert rc == 0 and out.endswith("fine\n"), (rc, out, err[-2000:])


def test_host_items_are_read_in_plain_mode_alone(so):
    # The host copy may be gone (a page that cannot be read stands for it): the
    # launches are those without one.
    check(so, r"""
import mmap
libc = ctypes.CDLL(None, use_errno=True)
libc.mmap.restype = ctypes.c_void_p
libc.mmap.argtypes = [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_long]
gone = libc.mmap(None, 1 << 16, 0, mmap.MAP_PRIVATE | mmap.MAP_ANONYMOUS, -1, 0)
for mode in (L.SCHED_STATIC, L.SCHED_DYNAMIC, L.SCHED_PACKED):
    for n in (1, 5, 300, 100000):
        grid = 512 if mode == L.SCHED_PACKED else 0
        runs = []
        for h in (None, gone):
            before = len(hip.launches())
            assert enumerate(mode=mode, num_items=n, grid=grid, h_items=h) == L.WPM_OK
            runs.append([l[:4] for l in hip.launches()[before:]])
        assert runs[0] == runs[1] and len(runs[0]) == 3, runs
assert enumerate(mode=L.SCHED_PLAIN, h_items=None) == L.WPM_EINVAL
print("fine")
""")


def test_scratch_beyond_four_words_only_where_it_is_said_exactly(so):
    # The field was reserved: a caller that left something in it is neither
    # refused nor written to beyond its 4 words.
    check(so, r"""
for sw in (0, 4, -1, -2**31, 1, 5, 287, 289, 1000, 2**31 - 1, 288):
    before = len(hip.launches())
    assert enumerate(num_items=1000, scratch_words=sw) == L.WPM_OK, sw
    clear, tree, walk = hip.launches()[before:]
    assert clear[0] == "" and "tree_kernel" in tree[0] and "sweep_kernel" in walk[0]
    cleared = int.from_bytes(clear[4][5][:8], "little")
    queues = int.from_bytes(tree[4][3][116:120], "little")
    assert (cleared, queues) == ((144, 8) if sw == 288 else (2, 1)), (sw, cleared, queues)
print("fine")
""")


def test_walk_flag_launches_the_walk_alone(so):
    check(so, r"""
for mode in (L.SCHED_STATIC, L.SCHED_DYNAMIC, L.SCHED_PACKED):
    for flags in (0, L.BATCH_TREE, L.BATCH_WALK):
        for sched in (0, L.FLAG_WALK, L.FLAG_WALK | L.FLAG_ACCUMULATE):
            before = len(hip.launches())
            got = enumerate(flags, mode=mode, num_items=9, grid=7, **{"flags": sched})
            assert got == L.WPM_OK
            kernels = [l for l in hip.launches()[before:] if l[0]]
            alone = [int.from_bytes(l[4][3][108:112], "little") for l in kernels]
            names = ["tree" if "tree_kernel" in l[0] else "walk" for l in kernels]
            if sched & L.FLAG_WALK:
                assert (names, alone) == (["walk"], [2])
            else:
                assert names == {0: ["tree", "walk"], L.BATCH_TREE: ["tree"], L.BATCH_WALK: ["walk"]}[flags]
                assert alone == ([1] if flags else [0, 0])
print("fine")
""")
