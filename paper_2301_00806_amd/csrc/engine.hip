// Device side of the ABI: launches of the sweep and collection of results.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include <sys/mman.h>

#include "internal.h"
#include "launch.h"
#include "tree_kernel.h"

namespace wpm {

namespace {
thread_local char g_hip_err[256] = "no HIP error";

// The words a sweep accumulates into, cleared in one launch: four separate
// fills were most of a small sweep's launches.
__global__ void clear_outputs(unsigned long long *counts, int64_t num, unsigned long long *total,
                              unsigned long long *stats, unsigned long long *head, int64_t head_words) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (counts && i < num) counts[i] = 0ull;
    if (total && i < WPM_TOTAL_WORDS) total[i] = 0ull;
    if (stats && i < 8) stats[i] = 0ull;
    if (head && i < head_words) head[i] = 0ull;
}

int hip_fail(const char *what, hipError_t e) {
    set_hip_error(what, (int)e, hipGetErrorString(e));
    return WPM_EHIP;
}

#define HIP_TRY(expr)                                   \
    do {                                                \
        hipError_t _e = (expr);                         \
        if (_e != hipSuccess) return hip_fail(#expr, _e); \
    } while (0)

// Which kernels a batch needs: the descent for tables with a level section,
// the walk for the others (a batch that does not say gets both).
bool wants_tree(const wpm_batch *b) { return !(b->flags & WPM_BATCH_WALK); }
bool wants_walk(const wpm_batch *b) { return !(b->flags & WPM_BATCH_TREE); }

// Waves per SIMD of the kernel a schedule asks for (0: the default, 8).
int pick_waves(int w) { return w == 7 ? 7 : 8; }
}  // namespace

void set_hip_error(const char *what, int code, const char *text) {
    std::snprintf(g_hip_err, sizeof(g_hip_err), "%s: %d (%s)", what, code, text ? text : "?");
}

const char *last_hip_error() { return g_hip_err; }

int device_query(int32_t *num_cus, int64_t *wallclock_khz, int32_t *lds_per_block) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    int v = 0;
    if (num_cus) {
        HIP_TRY(hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev));
        *num_cus = v;
    }
    if (wallclock_khz) {
        HIP_TRY(hipDeviceGetAttribute(&v, hipDeviceAttributeWallClockRate, dev));
        *wallclock_khz = v;
    }
    if (lds_per_block) {
        HIP_TRY(hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
        *lds_per_block = v;
    }
    return WPM_OK;
}

int persistent_grid_waves(const wpm_batch *b, int wg_size, int waves, bool tree, int32_t *grid);

int persistent_grid(const wpm_batch *b, int wg_size, int32_t *grid) {
    return b ? persistent_grid_waves(b, wg_size, 0, wants_tree(b), grid) : WPM_EINVAL;
}

int persistent_grid_waves(const wpm_batch *b, int wg_size, int waves, bool tree, int32_t *grid) {
    if (!grid || wg_size < 64 || wg_size > 512 || (wg_size % 64)) return WPM_EINVAL;
    if (b->max_row_words < 4 || b->max_row_words > WPM_MAX_ROW_WORDS || (b->max_row_words & 3)) return WPM_EINVAL;
    if (b->max_kp < 7 || b->max_kp > WPM_MAX_K) return WPM_EINVAL;
    int32_t cus = 0;
    int rc = device_query(&cus, nullptr, nullptr);
    if (rc) return rc;
    int nb = 0;
    if (tree)
        HIP_TRY(occupancy_tree(&nb, wg_size, tree_lds_bytes(b->max_kp, b->max_row_words, wg_size)));
    else
        HIP_TRY(occupancy_sweep(pick_waves(waves), &nb, wg_size,
                                sweep_lds_bytes(b->max_kp, b->max_row_words, wg_size)));
    *grid = std::max(1, nb) * cus;
    return WPM_OK;
}

namespace {
// The sweep with the dynamic queues' heads at d_head (device, `head_words` >= 2
// words: the descent's, the walk's and, from HEADS_AT on, the descent's eight
// where there is room for them and more than HEADS_ITEMS items).
constexpr int64_t HEADS_AT = 16, HEADS = 8, HEADS_ITEMS = 256;

int enumerate_with(const wpm_batch *b, const wpm_sched *s, uint64_t *d_surv, uint64_t cap,
                   uint64_t *d_counts, uint64_t *d_total, uint64_t *d_stats, uint64_t *d_head,
                   int64_t head_words, void *stream) {
    if (!b || !s || !d_counts || !d_total || (cap > 0 && !d_surv)) return WPM_EINVAL;
    if (b->num_instances < 0 || !b->d_tables || !b->d_offsets) return WPM_EINVAL;
    if (b->max_row_words < 4 || b->max_row_words > WPM_MAX_ROW_WORDS || (b->max_row_words & 3))
        return WPM_EINVAL;
    if (b->max_kp < 7 || b->max_kp > WPM_MAX_K) return WPM_EINVAL;
    if (s->wg_size < 64 || s->wg_size > 512 || (s->wg_size % 64)) return WPM_EINVAL;
    if (s->num_items < 0 || (s->num_items > 0 && !s->d_items)) return WPM_EINVAL;
    if (s->mode < WPM_SCHED_PLAIN || s->mode > WPM_SCHED_PACKED) return WPM_EINVAL;
    if (s->mode == WPM_SCHED_PACKED && (!s->d_bin_offsets || s->grid < 1)) return WPM_EINVAL;
    if (s->mode == WPM_SCHED_PLAIN && s->num_items > 0 && !s->h_items) return WPM_EINVAL;
    if (s->mode == WPM_SCHED_DYNAMIC && !d_head) return WPM_EINVAL;
    if (s->waves_per_simd != 0 && s->waves_per_simd != 7 && s->waves_per_simd != 8) return WPM_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    const int waves = pick_waves(s->waves_per_simd);
    if ((b->flags & WPM_BATCH_TREE) && (b->flags & WPM_BATCH_WALK)) return WPM_EINVAL;
    const bool all = (s->flags & WPM_FLAG_WALK) != 0;
    const bool tree = wants_tree(b) && !all, walk = wants_walk(b) || all;
    const size_t lds = walk ? sweep_lds_bytes(b->max_kp, b->max_row_words, s->wg_size) : 0;
    const size_t tree_lds = tree ? tree_lds_bytes(b->max_kp, b->max_row_words, s->wg_size) : 0;
    int32_t lds_max = 0;
    if (cap >= (UINT64_MAX >> 2)) return WPM_EINVAL;
    int rc = device_query(nullptr, nullptr, &lds_max);
    if (rc) return rc;
    if (std::max(lds, tree_lds) > (size_t)lds_max) return WPM_ELIMIT;

    const bool clear = !(s->flags & WPM_FLAG_ACCUMULATE);
    // (one head hands out a claim in 12 ns; clearing eight takes a sweep of five
    // items from 38.8 to 40.0 us)
    const bool eight = tree && s->mode == WPM_SCHED_DYNAMIC && s->num_items > HEADS_ITEMS &&
                       head_words >= HEADS_AT + HEADS * HEAD_STRIDE;
    if (clear || d_head) {
        const int64_t hw = eight ? HEADS_AT + HEADS * HEAD_STRIDE : 2;
        const int64_t n = std::max<int64_t>(clear ? b->num_instances : 0, std::max<int64_t>(hw, 8));
        hipLaunchKernelGGL(clear_outputs, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                           (unsigned long long *)(clear ? d_counts : nullptr), (int64_t)b->num_instances,
                           (unsigned long long *)(clear ? d_total : nullptr),
                           (unsigned long long *)(clear ? d_stats : nullptr), (unsigned long long *)d_head, hw);
        HIP_TRY(hipGetLastError());
    }
    if (s->num_items == 0) return WPM_OK;

    KArgs a;
    std::memset(&a, 0, sizeof(a));
    a.num_items = s->num_items;
    a.head = (unsigned long long *)d_head;
    a.surv = d_surv;
    a.cap = cap;
    a.counts = (unsigned long long *)d_counts;
    a.total = (unsigned long long *)d_total;
    a.stats = (unsigned long long *)d_stats;
    a.times = s->d_item_times;
    a.bins = s->d_bin_offsets;
    a.num_instances = b->num_instances;
    a.max_rs = b->max_row_words;
    a.max_kp = b->max_kp;
    a.split = 0;
    const dim3 block((unsigned)s->wg_size);
    // One launch of each kernel the batch needs over [item_base, num_items);
    // each takes the items of its tables and counts the malformed ones among them.
    // Persistent workgroups reserve record slots in blocks of at most 128 per
    // wave (few global atomics); the one-shot ones of the plain mode reserve
    // exactly.
    auto launch = [&](int64_t want_grid) -> hipError_t {
        if (tree) {
            KArgs t = a;
            int64_t grid = want_grid;
            t.chunk = (s->mode == WPM_SCHED_PLAIN) ? 0 : 2 * (uint64_t)s->wg_size;
            t.queues = eight ? (int)HEADS : 1;
            if (eight) t.head = a.head + HEADS_AT;
            t.count_bad = !walk;
            t.alone = !walk;
            if (t.mode == 1 || t.mode == 2) {
                // Fewer items than workgroups: hand each out in parts, one to a
                // workgroup (stamped items stay whole).  The items are in
                // device memory, so their lengths are not known here: the
                // descent keeps TREE_MIN_SPLIT vectors to a part, and the
                // workgroups of the parts that a short item does not have end
                // at once.
                if (!t.times)
                    while (t.split < 6 && (t.num_items << (t.split + 1)) <= grid) ++t.split;
                const int64_t parts = t.num_items << t.split;
                grid = std::min<int64_t>(grid, parts);
            }
            const hipError_t e = launch_tree(dim3((unsigned)grid), block, tree_lds, st, b->d_tables, b->d_offsets,
                                             s->d_items, t);
            if (e != hipSuccess) return e;
        }
        if (walk) {
            KArgs w = a;
            w.chunk = (s->mode == WPM_SCHED_PLAIN) ? 0 : 128;
            w.count_bad = 1;
            w.alone = all ? 2 : !tree;
            w.head = a.head ? a.head + 1 : nullptr;
            const int64_t grid = w.mode == 3 ? want_grid : std::min<int64_t>(want_grid, w.num_items - w.item_base);
            return launch_sweep(waves, dim3((unsigned)grid), block, lds, st, b->d_tables, b->d_offsets, s->d_items, w);
        }
        return hipSuccess;
    };
    if (s->mode == WPM_SCHED_PLAIN) {
        // One launch per instance: a grid of exactly that instance's items
        // (items naming an unknown instance are rejected before any launch;
        // the kernel skips and counts any other malformed item).
        for (int64_t i = 0; i < s->num_items; ++i)
            if ((int64_t)s->h_items[i].instance >= (int64_t)b->num_instances) return WPM_EINVAL;
        a.mode = 0;
        int64_t i = 0;
        while (i < s->num_items) {
            int64_t e = i;
            while (e < s->num_items && s->h_items[e].instance == s->h_items[i].instance) ++e;
            a.item_base = i;
            a.num_items = e;
            HIP_TRY(launch(e - i));
            i = e;
        }
        return WPM_OK;
    }
    int32_t grid = s->grid;
    if (grid <= 0 && (rc = persistent_grid_waves(b, s->wg_size, waves, tree, &grid))) return rc;
    a.mode = (s->mode == WPM_SCHED_STATIC) ? 1 : (s->mode == WPM_SCHED_DYNAMIC) ? 2 : 3;
    HIP_TRY(launch(grid));
    return WPM_OK;
}

// Scratch of the allocation-free entry point: the dynamic queue's head.
// Each device holds its own copy of this array (its host-side name is not a
// device address); its address on a device is looked up once, with that
// device current, and every call on the device shares it.
static __device__ __align__(256) unsigned long long scratch[WPM_STATIC_SCRATCH_WORDS];

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[MAX_DEVICES] = {};

int scratch_on_current_device(uint64_t **out) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return WPM_ELIMIT;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return WPM_EHIP;
        g_scratch_ptr[dev] = p;
    }
    *out = (uint64_t *)g_scratch_ptr[dev];
    return WPM_OK;
}
}  // namespace

int enumerate(const wpm_batch *b, const wpm_sched *s, uint64_t *d_surv, uint64_t cap,
              uint64_t *d_counts, uint64_t *d_total, uint64_t *d_stats, void *stream) {
    if (!s) return WPM_EINVAL;
    // (the field was reserved once: whatever else it holds means 4 words)
    const int64_t words = s->scratch_words == WPM_QUEUE_SCRATCH_WORDS ? WPM_QUEUE_SCRATCH_WORDS : 4;
    return enumerate_with(b, s, d_surv, cap, d_counts, d_total, d_stats, (uint64_t *)s->d_scratch, words / 2, stream);
}

int enumerate_noalloc(const wpm_batch *b, const wpm_sched *s, uint64_t *d_surv, uint64_t cap,
                      uint64_t *d_counts, uint64_t *d_total, uint64_t *d_stats, void *stream) {
    if (!s || s->d_scratch) return WPM_EINVAL;  // the scratch is the library's own
    // scratch words this schedule needs: the queue head of the dynamic mode
    const int64_t need = s->mode == WPM_SCHED_DYNAMIC ? 2 : 0;
    if (need > WPM_STATIC_SCRATCH_WORDS) return WPM_ELIMIT;
    uint64_t *head = nullptr;
    if (need) {
        const int rc = scratch_on_current_device(&head);
        if (rc) return rc;
    }
    return enumerate_with(b, s, d_surv, cap, d_counts, d_total, d_stats, head, need, stream);
}

namespace {

// The threads of one call: the calling one and up to 15 more run the same
// function, phase by phase, with a barrier between phases.  (Threads started
// and joined for each phase cost more than the phases of a small result.)
// Threads start each other as a tree: one thread starting 15 took 200 us.
class Team {
   public:
    // fn(t) on `want` threads (fewer if the system refuses some).
    template <class Fn>
    void run(int want, Fn fn) {
        grow(0, want, fn);
        // (threads start counting in before fn; refused ones are counted out)
        while (size_.load(std::memory_order_acquire) == 0) {
            const int n = started_.load(std::memory_order_acquire);
            if (n + refused_.load(std::memory_order_acquire) == want) size_.store(n, std::memory_order_release);
            std::this_thread::yield();
        }
        fn(0);
        for (int t = 1; t < MAX; ++t)
            if (th_[t].joinable()) th_[t].join();
    }
    void barrier() {
        const int g = gen_.load(std::memory_order_acquire);
        if (arrived_.fetch_add(1, std::memory_order_acq_rel) + 1 == size_.load(std::memory_order_relaxed)) {
            arrived_.store(0, std::memory_order_relaxed);
            gen_.store(g + 1, std::memory_order_release);
        } else {
            for (int i = 0; gen_.load(std::memory_order_acquire) == g; ++i)
                if (i > 256) std::this_thread::yield();
        }
    }
    // this thread's share of [0, num), `grain` at a time (one phase number per loop)
    template <class Fn>
    void share(int phase, int64_t num, int64_t grain, Fn fn) {
        for (;;) {
            const int64_t a = next_[phase].fetch_add(grain, std::memory_order_relaxed);
            if (a >= num) break;
            for (int64_t i = a; i < std::min(num, a + grain); ++i) fn(i);
        }
    }

   private:
    static constexpr int MAX = 16;
    // thread t of `want`: starts threads 2t + 1 and 2t + 2.  th_ is written by
    // the starter alone; the calling thread joins in increasing order, so a
    // thread's starter has ended, and its th_ entries are there, before it
    // is looked at.
    template <class Fn>
    void grow(int t, int want, Fn &fn) {
        started_.fetch_add(1, std::memory_order_acq_rel);
        for (int c = 2 * t + 1; c <= 2 * t + 2 && c < want; ++c) {
            try {
                th_[c] = std::thread([this, c, want, &fn] {
                    grow(c, want, fn);
                    while (size_.load(std::memory_order_acquire) == 0) std::this_thread::yield();
                    fn(c);
                });
            } catch (...) {
                refused_.fetch_add(subtree(c, want), std::memory_order_acq_rel);
            }
        }
    }
    static int subtree(int c, int want) {
        return c < want ? 1 + subtree(2 * c + 1, want) + subtree(2 * c + 2, want) : 0;
    }
    std::thread th_[MAX];
    std::atomic<int> started_{0}, refused_{0}, size_{0}, arrived_{0}, gen_{0};
    std::atomic<int64_t> next_[8] = {};
};

// Uninitialised host memory of one call, from 4 MB on in huge pages: the first
// touch of ordinary pages took longer than the phases that fill them.
template <class T>
class Buffer {
   public:
    Buffer() = default;
    ~Buffer() { std::free(p_); }
    Buffer(const Buffer &) = delete;
    Buffer &operator=(const Buffer &) = delete;
    bool reset(size_t n) {
        constexpr size_t HUGE_PAGE = (size_t)2 << 20;
        const size_t bytes = std::max<size_t>(1, n) * sizeof(T);
        std::free(p_);
        if (bytes >= 2 * HUGE_PAGE) {
            const size_t whole = (bytes + HUGE_PAGE - 1) & ~(HUGE_PAGE - 1);
            p_ = (T *)std::aligned_alloc(HUGE_PAGE, whole);
            if (p_) (void)madvise(p_, whole, MADV_HUGEPAGE);
        } else {
            p_ = (T *)std::malloc(bytes);
        }
        return p_ != nullptr;
    }
    void release() {
        std::free(p_);
        p_ = nullptr;
    }
    T *get() const { return p_; }
    T &operator[](size_t i) const { return p_[i]; }

   private:
    T *p_ = nullptr;
};

// A key whose order agrees with the canonical order wherever two keys differ:
// the first 128 positions, facet 0 first, a held facet below a missing one; the
// positions after a complex's last facet count as held, so that a list that is a
// prefix of another does not come after it.  Equal keys say nothing.
struct Key {
    uint64_t a, b;
    bool operator<(const Key &o) const { return a != o.a ? a < o.a : b < o.b; }
    bool operator==(const Key &o) const { return a == o.a && b == o.b; }
};

// One instance's part of a call: its facets in increasing vertex-mask order,
// its basis (and coset offset) with the facet bits moved to those positions --
// the set bits of a complex's bit vector, read in increasing position, are then
// its facets in increasing mask order -- and the places of its results.
struct Collected {
    int W = 0;
    uint32_t *mask = nullptr;   // [M] facet masks, increasing
    uint32_t *basis = nullptr;  // [k][W] permuted basis rows
    uint32_t *off = nullptr;    // [W] permuted offset (zero for a subspace)
    int64_t first = 0, n = 0;   // results [first, first + n) of the call
    uint32_t *kv = nullptr;     // [n][W] permuted bit vectors (in order, of an instance of one range)
    int buckets = 1;            // key ranges the results are sorted in
    int64_t chunk0 = 0, chunks = 0, bucket0 = 0;
    int64_t shared0 = 0;        // place of the first result in the arrays of instances of several ranges
    Key *split = nullptr;       // [buckets - 1] first keys of the ranges after the first
    int64_t words = 0;
};

// (arrays of the right size, zeroed)
void sort_facets(const wpm_host_instance &in, Collected &c) {
    const int M = in.M, W = c.W;
    int32_t order[WPM_MAX_M], pos[WPM_MAX_M];
    for (int j = 0; j < M; ++j) order[j] = j;
    std::sort(order, order + M, [&](int32_t a, int32_t b) { return in.facets[a] < in.facets[b]; });
    for (int r = 0; r < M; ++r) {
        pos[order[r]] = r;
        c.mask[r] = in.facets[order[r]];
    }
    auto permute = [&](const uint32_t *src, uint32_t *dst) {
        for (int w = 0; w < W; ++w)
            for (uint32_t v = src[w]; v; v &= v - 1) {
                const int r = pos[w * 32 + __builtin_ctz(v)];
                dst[r >> 5] |= 1u << (r & 31);
            }
    };
    for (int t = 0; t < in.k; ++t) permute(in.basis + (size_t)t * W, c.basis + (size_t)t * W);
    if (in.offset) permute(in.offset, c.off);
}

// The complex of x as a permuted bit vector.
inline void expand(const Collected &c, uint64_t x, uint32_t *K) {
    for (int q = 0; q < c.W; ++q) K[q] = c.off[q];
    for (uint64_t b = x; b; b &= b - 1) {
        const uint32_t *row = c.basis + (size_t)__builtin_ctzll(b) * c.W;
        for (int q = 0; q < c.W; ++q) K[q] ^= row[q];
    }
}

inline uint64_t reverse_bits(uint64_t v) {
    v = ((v >> 1) & 0x5555555555555555ull) | ((v & 0x5555555555555555ull) << 1);
    v = ((v >> 2) & 0x3333333333333333ull) | ((v & 0x3333333333333333ull) << 2);
    v = ((v >> 4) & 0x0F0F0F0F0F0F0F0Full) | ((v & 0x0F0F0F0F0F0F0F0Full) << 4);
    return __builtin_bswap64(v);
}

inline Key order_key(const uint32_t *K, int W) {
    auto two = [&](int q) -> uint64_t {
        return (q < W ? (uint64_t)K[q] : 0u) | (q + 1 < W ? (uint64_t)K[q + 1] << 32 : 0u);
    };
    uint64_t a = two(0), b = two(2);
    bool later = false;
    for (int q = 4; q < W && !later; ++q) later = K[q] != 0u;
    auto fill = [](uint64_t v) { return v ? v | (~0ull << (63 - __builtin_clzll(v))) : ~0ull; };
    if (!later) {
        if (!b) a = fill(a);
        b = fill(b);
    }
    return {~reverse_bits(a), ~reverse_bits(b)};
}

// Canonical order of two complexes given as permuted bit vectors (facets in
// increasing mask order): lexicographic order of their facet lists, a list
// that is a prefix of another coming first.  At the lowest differing position
// j the complex holding j continues with facet j; the other continues with a
// later facet (j comes first) or has ended (it comes first).
inline bool canon_less(const uint32_t *A, const uint32_t *B, int W) {
    for (int w = 0; w < W; ++w) {
        const uint32_t d = A[w] ^ B[w];
        if (!d) continue;
        const int b = __builtin_ctz(d);
        const bool a_has = (A[w] >> b) & 1u;
        const uint32_t *other = a_has ? B : A;
        const uint32_t above = b == 31 ? 0u : (other[w] >> (b + 1));
        bool more = above != 0u;
        for (int v = w + 1; v < W && !more; ++v) more = other[v] != 0u;
        return a_has == more;
    }
    return false;
}

}  // namespace

// Host expansion of the records into canonical facet lists, in phases that a
// team of threads shares:
//   the records are grouped by instance (histograms of record ranges, scatter);
//   every result is expanded into a permuted bit vector, and the words of its
//     list are counted.  An instance of one key range is sorted here, by one
//     thread in its own memory; in a larger one each result is assigned to one
//     of up to 256 key ranges, found by a sample, and then put to its range;
//   the lists' places follow;
//   the lists are written: an instance of one range as its bit vectors lie,
//     of a larger one each range is sorted and written.
// With a batch of many instances the whole is bound by passes over memory, with
// a single one by its sort.  Instances are cut into ranges from 4096 results
// on, or from as many as leave every thread 8 instances, at most 16384.  (Keys,
// references and ranges of every result in memory, 41 bytes each, made the
// headline batch, 5.4e7 results of 16384 instances on 16 cores, 951 ms, and
// sorting by instance alone 810; now 715.  128 instances 10.7 -> 8.5 ms, one of
// 31e3 results 4.1 by instance, 1.11 -> 1.00.)
int collect(const wpm_host_instance *insts, int32_t num, const uint64_t *d_surv, uint64_t cap,
            const uint64_t *d_counts, const uint64_t *d_total, uint64_t *h_counts, uint32_t *h_out,
            int64_t out_cap, int64_t *out_words, int64_t *h_offsets, void *stream) {
    if (num < 0 || !d_counts || !d_total || !h_counts || !out_words || !h_offsets ||
        (num > 0 && !insts))
        return WPM_EINVAL;
    for (int i = 0; i < num; ++i)
        if (insts[i].M < 0 || insts[i].M > WPM_MAX_M || insts[i].k < 0 || insts[i].k > WPM_MAX_K ||
            (insts[i].k > 0 && !insts[i].basis) || (insts[i].M > 0 && !insts[i].facets))
            return WPM_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    uint64_t tot[WPM_TOTAL_WORDS] = {0, 0, 0, 0};
    HIP_TRY(hipMemcpyAsync(h_counts, d_counts, sizeof(uint64_t) * (size_t)num, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipMemcpyAsync(tot, d_total, sizeof(tot), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    const uint64_t total = tot[0], slots = tot[1];
    if (tot[2] != 0) return WPM_EINVAL;  // the sweep skipped malformed items
    if (slots > cap) {
        *out_words = -(int64_t)slots;  // record slots needed
        return WPM_ECAP;
    }
    uint64_t sum = 0;
    for (int i = 0; i < num; ++i) sum += h_counts[i];
    if (sum != total) return WPM_EINVAL;  // counts and total disagree: corrupted buffers
    // the records: read in place when they are in host memory, else copied
    const uint64_t *rec = d_surv;
    Buffer<uint64_t> rec_copy;
    {
        hipPointerAttribute_t attr;
        const bool host = hipPointerGetAttributes(&attr, d_surv) == hipSuccess &&
                          attr.type == hipMemoryTypeHost;
        (void)hipGetLastError();
        if (!host && slots) {
            if (!rec_copy.reset(2 * slots)) return WPM_ELIMIT;
            HIP_TRY(hipMemcpyAsync(rec_copy.get(), d_surv, sizeof(uint64_t) * 2 * slots, hipMemcpyDefault, st));
            HIP_TRY(hipStreamSynchronize(st));
            rec = rec_copy.get();
        }
    }
    const int hw = (int)std::max(1u, std::min(16u, std::thread::hardware_concurrency()));
    const int want = (int)std::min<int64_t>(hw, 1 + (int64_t)(slots / 1024) + num / 64);
    // (no more histograms than there are records for)
    const int64_t ranges = std::max<int64_t>(
        1, std::min<int64_t>({64, (int64_t)(slots / 8192) + 1, (int64_t)(slots / std::max<uint64_t>(1, (uint64_t)num))}));
    const uint64_t per = (slots + ranges - 1) / (uint64_t)ranges;
    constexpr int64_t CHUNK = 1024;
    const bool write = h_out != nullptr;
    struct Task { int32_t inst; int32_t sub; };  // sub: a chunk or a range; -1: the whole instance
    struct Cell { int64_t n, words; };
    struct Ref { Key key; uint32_t idx; };
    std::vector<int64_t> hist;
    std::vector<Collected> cs;
    Buffer<uint64_t> xs;
    Buffer<uint32_t> kv;
    // of the instances of several ranges: each result's range, and the results
    // range by range
    Buffer<uint8_t> bucket_of;
    Buffer<uint32_t> order;
    std::vector<uint32_t> facet_words;
    std::vector<Key> splits;
    std::vector<Task> expand_tasks, write_tasks;
    std::vector<int64_t> cell0;   // first cell of each expand task that is a chunk
    std::vector<Cell> cells;      // per chunk and range
    std::vector<Cell> starts;     // per range: first result, first word (in the instance)
    size_t row_words = 0, rows = 0;  // of a thread's own memory
    std::atomic<int> bad{0}, failed{0};
    int rc = WPM_OK;
    bool stop = false;
    try {
        hist.assign((size_t)ranges * (size_t)num, 0);
        cs.resize((size_t)num);
    } catch (const std::bad_alloc &) {
        return WPM_ELIMIT;
    }
    auto plan = [&]() -> int {  // after the histograms, on one thread
        if (bad) return WPM_EINVAL;
        int64_t total_n = 0, fw = 0, kw = 0, sw = 0, shared = 0, nc = 0;
        const int64_t most = std::min<int64_t>(16 * CHUNK, std::max<int64_t>(4 * CHUNK, (int64_t)total / (8 * want)));
        for (int i = 0; i < num; ++i) {
            int64_t c = 0;
            for (int64_t r = 0; r < ranges; ++r) {
                int64_t &h = hist[(size_t)r * num + i];
                const int64_t v = h;
                h = total_n + c;  // this range's first position for instance i
                c += v;
            }
            if ((uint64_t)c != h_counts[i]) return WPM_EINVAL;
            Collected &ci = cs[i];
            ci.W = (insts[i].M + 31) / 32;
            ci.first = total_n;
            ci.n = c;
            total_n += c;
            if (!c) continue;
            if (c > most) {
                ci.buckets = (int)std::min<int64_t>(256, c / CHUNK);
                ci.chunks = (c + CHUNK - 1) / CHUNK;
                ci.chunk0 = (int64_t)expand_tasks.size();
                ci.bucket0 = (int64_t)starts.size();
                ci.shared0 = shared;
                shared += c;
                for (int64_t q = 0; q < ci.chunks; ++q) {
                    expand_tasks.push_back({i, (int32_t)q});
                    cell0.push_back(nc);
                    nc += ci.buckets;
                }
                for (int q = 0; q < ci.buckets; ++q) write_tasks.push_back({i, q});
                starts.resize(starts.size() + (size_t)ci.buckets, Cell{0, 0});
            } else {
                expand_tasks.push_back({i, -1});
                cell0.push_back(0);
                write_tasks.push_back({i, -1});
                row_words = std::max(row_words, (size_t)c * ci.W);
            }
            rows = std::max(rows, (size_t)(c > most ? std::min<int64_t>(c, 4 * CHUNK) : c));
            fw += insts[i].M + (int64_t)insts[i].k * ci.W + ci.W;
            kw += c * ci.W;
            sw += ci.buckets - 1;
        }
        facet_words.assign((size_t)fw, 0u);
        splits.assign((size_t)sw, Key{0, 0});
        cells.assign((size_t)nc, Cell{0, 0});
        if (!xs.reset((size_t)total_n) || !kv.reset((size_t)kw) || !bucket_of.reset((size_t)shared) ||
            (write && !order.reset((size_t)shared)))
            return WPM_ELIMIT;
        uint32_t *f = facet_words.data(), *v = kv.get();
        Key *sp = splits.data();
        for (int i = 0; i < num; ++i) {
            Collected &ci = cs[i];
            if (!ci.n) continue;
            ci.mask = f;
            ci.basis = ci.mask + insts[i].M;
            ci.off = ci.basis + (size_t)insts[i].k * ci.W;
            f = ci.off + ci.W;
            ci.kv = v;
            v += ci.n * ci.W;
            ci.split = sp;
            sp += ci.buckets - 1;
        }
        return WPM_OK;
    };
    // the facet list of a bit vector; returns the place after it
    auto put_list = [](const Collected &c, const uint32_t *K, uint32_t *out) {
        uint32_t *len = out++;
        for (int q = 0; q < c.W; ++q)
            for (uint32_t v = K[q]; v; v &= v - 1) *out++ = c.mask[q * 32 + __builtin_ctz(v)];
        *len = (uint32_t)(out - len - 1);
        return out;
    };
    auto list_words = [](const Collected &c, const uint32_t *K) {
        int64_t w = 1;
        for (int q = 0; q < c.W; ++q) w += __builtin_popcount(K[q]);
        return w;
    };
    // references in canonical order of the bit vectors at `base`
    auto sort_refs = [](const Collected &c, const uint32_t *base, Ref *r, size_t n) {
        const int W = c.W;
        std::sort(r, r + n, [&](const Ref &a, const Ref &b) {
            if (!(a.key == b.key)) return a.key < b.key;
            return canon_less(base + (size_t)a.idx * W, base + (size_t)b.idx * W, W);
        });
    };
    Team team;
    auto work = [&](int t) {
        Buffer<uint32_t> own;  // this thread's bit vectors of an instance, and references
        Buffer<Ref> refs;
        size_t refs_have = 0;
        team.share(0, ranges, 1, [&](int64_t r) {
            int64_t *h = hist.data() + (size_t)r * num;
            const uint64_t e = std::min<uint64_t>(slots, (uint64_t)(r + 1) * per);
            for (uint64_t q = (uint64_t)r * per; q < e; ++q) {
                const uint64_t inst = rec[2 * q + 1];
                if (inst == ~0ull) continue;
                if (inst >= (uint64_t)num) { bad = 1; return; }
                const uint64_t x = rec[2 * q];
                if (insts[inst].k < 64 && (x >> insts[inst].k)) { bad = 1; return; }
                ++h[inst];
            }
        });
        team.barrier();
        if (t == 0) {
            try {
                rc = plan();
            } catch (const std::bad_alloc &) {
                rc = WPM_ELIMIT;
            }
            stop = rc != WPM_OK;
        }
        team.barrier();
        if (stop) return;
        team.share(1, ranges, 1, [&](int64_t r) {
            int64_t *h = hist.data() + (size_t)r * num;
            const uint64_t e = std::min<uint64_t>(slots, (uint64_t)(r + 1) * per);
            for (uint64_t q = (uint64_t)r * per; q < e; ++q) {
                const uint64_t inst = rec[2 * q + 1];
                if (inst != ~0ull) xs[(size_t)h[inst]++] = rec[2 * q];
            }
        });
        refs_have = rows;
        if (!own.reset(row_words) || !refs.reset(refs_have)) failed = 1;
        team.barrier();
        if (failed) return;
        // facets, and key ranges by a sample of the instance's results
        if (t == 0) rec_copy.release();
        team.share(2, num, 4, [&](int64_t i) {
            Collected &c = cs[(size_t)i];
            if (!c.n) return;
            sort_facets(insts[i], c);
            if (c.buckets == 1) return;
            Key sample[1024];
            uint32_t K[WPM_MAX_M / 32];
            const int m = std::min(1024, c.buckets * 16);
            for (int q = 0; q < m; ++q) {
                expand(c, xs[(size_t)(c.first + c.n * q / m)], K);
                sample[q] = order_key(K, c.W);
            }
            std::sort(sample, sample + m);
            for (int q = 1; q < c.buckets; ++q) c.split[q - 1] = sample[(int64_t)m * q / c.buckets];
        });
        team.barrier();
        team.share(3, (int64_t)expand_tasks.size(), 2, [&](int64_t et) {
            const Task tk = expand_tasks[(size_t)et];
            Collected &c = cs[(size_t)tk.inst];
            const int W = c.W;
            if (tk.sub < 0) {
                int64_t words = 0;
                for (int64_t r = 0; r < c.n; ++r) {
                    uint32_t *K = own.get() + (size_t)r * W;
                    expand(c, xs[(size_t)(c.first + r)], K);
                    words += list_words(c, K);
                    if (write) refs[(size_t)r] = {order_key(K, W), (uint32_t)r};
                }
                c.words = words;
                if (!write) return;
                sort_refs(c, own.get(), refs.get(), (size_t)c.n);
                for (int64_t r = 0; r < c.n; ++r)
                    std::memcpy(c.kv + (size_t)r * W, own.get() + (size_t)refs[(size_t)r].idx * W, sizeof(uint32_t) * W);
                return;
            }
            Cell *cell = cells.data() + cell0[(size_t)et];
            const int64_t r1 = std::min<int64_t>(c.n, (tk.sub + 1) * CHUNK);
            for (int64_t r = tk.sub * CHUNK; r < r1; ++r) {
                uint32_t *K = c.kv + (size_t)r * W;
                expand(c, xs[(size_t)(c.first + r)], K);
                const Key key = order_key(K, W);
                const int b = (int)(std::upper_bound(c.split, c.split + c.buckets - 1, key) - c.split);
                bucket_of[(size_t)(c.shared0 + r)] = (uint8_t)b;
                ++cell[b].n;
                cell[b].words += list_words(c, K);
            }
        });
        team.barrier();
        if (t == 0) xs.release();
        // places: per instance of several ranges, range by range, chunk by chunk
        team.share(4, num, 16, [&](int64_t i) {
            Collected &c = cs[(size_t)i];
            if (c.buckets == 1) return;
            int64_t n = 0, w = 0;
            for (int b = 0; b < c.buckets; ++b) {
                starts[(size_t)(c.bucket0 + b)] = {n, w};
                for (int64_t q = 0; q < c.chunks; ++q) {
                    Cell &cell = cells[(size_t)(cell0[(size_t)(c.chunk0 + q)] + b)];
                    const int64_t m = cell.n;
                    cell.n = n;
                    n += m;
                    w += cell.words;
                }
            }
            c.words = w;
        });
        team.barrier();
        if (t == 0) {
            int64_t words = 0;
            for (int i = 0; i < num; ++i) {
                h_offsets[i] = words;
                words += cs[(size_t)i].words;
            }
            h_offsets[num] = words;
            *out_words = words;
            if (!write || out_cap < words) rc = WPM_ECAP;
            stop = rc != WPM_OK;
        }
        team.barrier();
        if (stop) return;
        team.share(5, (int64_t)expand_tasks.size(), 4, [&](int64_t et) {
            const Task tk = expand_tasks[(size_t)et];
            if (tk.sub < 0) return;
            const Collected &c = cs[(size_t)tk.inst];
            Cell *cell = cells.data() + cell0[(size_t)et];
            const int64_t r1 = std::min<int64_t>(c.n, (tk.sub + 1) * CHUNK);
            for (int64_t r = tk.sub * CHUNK; r < r1; ++r)
                order[(size_t)(c.shared0 + cell[bucket_of[(size_t)(c.shared0 + r)]].n++)] = (uint32_t)r;
        });
        team.barrier();
        team.share(6, (int64_t)write_tasks.size(), 1, [&](int64_t wt) {
            const Task tk = write_tasks[(size_t)wt];
            const Collected &c = cs[(size_t)tk.inst];
            uint32_t *out = h_out + h_offsets[tk.inst];
            if (tk.sub < 0) {
                for (int64_t r = 0; r < c.n; ++r) out = put_list(c, c.kv + (size_t)r * c.W, out);
                return;
            }
            const Cell &at = starts[(size_t)(c.bucket0 + tk.sub)];
            const size_t n = (size_t)((tk.sub + 1 < c.buckets ? starts[(size_t)(c.bucket0 + tk.sub) + 1].n : c.n) - at.n);
            const uint32_t *idx = order.get() + c.shared0 + at.n;
            if (n > refs_have) {  // (a range of very many equal keys)
                refs_have = n;
                if (!refs.reset(n)) {
                    refs_have = 0;
                    failed = 1;
                    return;
                }
            }
            for (size_t r = 0; r < n; ++r) refs[r] = {order_key(c.kv + (size_t)idx[r] * c.W, c.W), idx[r]};
            sort_refs(c, c.kv, refs.get(), n);
            out += at.words;
            for (size_t r = 0; r < n; ++r) out = put_list(c, c.kv + (size_t)refs[r].idx * c.W, out);
        });
    };
    team.run(want, work);
    return failed ? WPM_ELIMIT : rc;
}

}  // namespace wpm
