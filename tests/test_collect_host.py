"""wpm_collect on the CPU, with a double of the HIP runtime: canonical order
and places against Python's own sort, at the sizes where its path changes, and
the memory it takes."""
import pytest

import hipdouble as H


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return H.build(tmp_path_factory.mktemp("hipdouble"))


COMMON = r"""
import resource
lib = L.lib()

class Case:
    '''num instances of M facets, k basis rows, and `results` records each.'''
    def __init__(self, shapes, seed=1):
        rng = np.random.default_rng(seed)
        self.num = len(shapes)
        self.hosts = (L.HostInstance * max(1, self.num))()
        self.keep, recs, self.want, self.cnt = [], [], [], np.zeros(max(1, self.num), np.uint64)
        for i, (M, k, n, off) in enumerate(shapes):
            W = (M + 31) // 32
            facets = rng.permutation(1 << 20)[:M].astype(np.uint32) if M < 4000 else np.arange(M, dtype=np.uint32)
            bits = rng.random((k + 1, M)) < min(0.5, 8.0 / M)
            words = np.zeros((k + 1, 32 * W), bool)
            words[:, :M] = bits
            words = np.packbits(words.reshape(k + 1, W, 32), axis=2, bitorder="little").view(np.uint32).reshape(k + 1, W)
            basis, offset = np.ascontiguousarray(words[:k]), np.ascontiguousarray(words[k])
            if k == 0:
                basis = np.zeros((1, W), np.uint32)
            self.keep.append((facets, basis, offset))
            self.hosts[i] = L.HostInstance(M=M, k=k, facets=facets.ctypes.data, basis=basis.ctypes.data,
                                           offset=offset.ctypes.data if off else None)
            x = rng.integers(0, 1 << k, n, dtype=np.uint64)
            recs.append(np.column_stack([x, np.full(n, i, np.uint64)]))
            self.cnt[i] = n
            self.shape = shapes
            K = (bits[k] if off else np.zeros(M, bool))[None].repeat(n, 0)
            for t in range(k):
                K = K ^ (bits[t][None] & ((x >> np.uint64(t)) & np.uint64(1)).astype(bool)[:, None])
            self.want.append((facets, K))
        rec = np.concatenate(recs + [np.tile(np.array([[0, 2**64 - 1]], np.uint64), (37, 1))])
        self.rec = np.ascontiguousarray(rec[rng.permutation(len(rec))])
        self.total = np.array([self.cnt.sum(), len(self.rec), 0, 0], np.uint64)

    def expected(self):
        out, offs = [], [0]
        for facets, K in self.want:
            lists = sorted(tuple(sorted(int(f) for f in facets[k])) for k in K)
            for l in lists:
                out += [len(l), *l]
            offs.append(len(out))
        return np.array(out, np.uint32), offs

    def collect(self, out, cap):
        h = np.zeros(max(1, self.num), np.uint64)
        self.offs = np.full(self.num + 1, -7, np.int64)
        self.words = ctypes.c_int64(-7)
        return lib.wpm_collect(self.hosts, self.num, self.rec.ctypes.data, len(self.rec), self.cnt.ctypes.data,
                               self.total.ctypes.data, E._ptr(h, L.c_u64p), None if out is None else
                               E._ptr(out, L.c_u32p), cap, ctypes.byref(self.words), E._ptr(self.offs, L.c_i64p), None)
"""


def check(so, code):
    rc, out, err = H.run(so, COMMON + code, timeout=300)
    assert rc == 0 and out.endswith("fine\n"), (rc, out[-500:], err[-2000:])


@pytest.mark.parametrize("shapes", [
    "[]", "[(1, 0, 1, True)]", "[(5, 2, 0, False), (5, 3, 7, False)]",
    "[(33, 14, 4096, False), (33, 14, 4097, True)]",              # at the limit of one range
    "[(12, 10, 20000, False)]",                                     # many equal results, lists that are prefixes
    "[(300, 20, 9000, True), (130, 9, 3, False), (64, 16, 17000, False)]",  # beyond 128 facets
    "[(40, 16, 300, i % 2 == 0) for i in range(150)]",
    "[(31 + i, 12, 17 * i, i % 3 == 0) for i in range(120)] + [(70, 24, 30000, False)]",
])
def test_lists_match_a_plain_sort(so, shapes):
    check(so, f"""
c = Case({shapes})
want, offs = c.expected()
""" + r"""
assert c.collect(None, 0) == L.WPM_ECAP and c.words.value == len(want) and list(c.offs) == offs
out = np.zeros(max(1, len(want)), np.uint32)
if len(want):
    assert c.collect(out, len(want) - 1) == L.WPM_ECAP and not out.any()
assert c.collect(out, len(want)) == L.WPM_OK and list(c.offs) == offs
assert np.array_equal(out[:len(want)], want)
if c.num:
    c.cnt[0] += 1
    assert c.collect(out, len(want)) == L.WPM_EINVAL   # counts and total disagree
    c.total[0] += 1
    assert c.collect(out, len(want)) == L.WPM_EINVAL   # counts and records disagree
print("fine")
""")


def test_memory_of_a_batch_of_many_instances(so):
    # 16 bytes a result for the copy of the records and 8 for its coordinates,
    # the bit vectors, one instance's references for every thread, and nothing
    # else that grows with the results
    check(so, r"""
c = Case([(96, 20, 3000, False)] * 4)
# 400 instances alike: 1.2e6 results
num, W = 400, 3
hosts = (L.HostInstance * num)(*[c.hosts[i % 4] for i in range(num)])
real = c.rec[c.rec[:, 1] != 2**64 - 1]
rec = np.concatenate([real + np.array([0, 4 * j], np.uint64) for j in range(num // 4)])
cnt = np.full(num, 3000, np.uint64)
c.hosts, c.num, c.rec, c.cnt = hosts, num, rec, cnt
c.total = np.array([len(rec), len(rec), 0, 0], np.uint64)
assert c.collect(None, 0) == L.WPM_ECAP
out = np.ones(c.words.value, np.uint32)      # (pages touched)
small = Case([(5, 3, 2000, False)] * 70)     # (the threads' first start)
assert small.collect(None, 0) == L.WPM_ECAP
def resident(key):
    with open("/proc/self/status") as f:
        return next(int(l.split()[1]) << 10 for l in f if l.startswith(key))
with open("/proc/self/clear_refs", "w") as f:
    f.write("5")   # the high-water mark starts from here
before = resident("VmRSS")
assert c.collect(out, len(out)) == L.WPM_OK
used = resident("VmHWM") - before
n = len(rec)
assert used <= n * (16 + 8 + 4 * W) + 16 * 3000 * (32 + 4 * W) + (8 << 20), (used, used / n)
print("fine")
""")
