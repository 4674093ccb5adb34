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
def enumerate(flags=0, **kw):
    batch.flags = flags
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
