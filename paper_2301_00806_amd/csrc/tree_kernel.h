// The tree descent of the F2 kernel on gfx950 (device code): the sweep of
// every table that has a level section (the packer gives one to all).
//
// A range of Gray indices is descended as a tree of aligned sub-cubes with
// fan-out 64: blocks of 2^24 vectors, groups of 2^18, nodes of 2^12, children
// of 2^6, vectors.  While the low L coordinates of x run freely, a facet
// without any of them in its basis membership is constant, and at least 3 such
// parents of a ridge in K reject every vector of the sub-cube (Proposition
// 2.1; the packer's level rows hold these parents bit-sliced, 32 ridges per
// word, with nothing in the rows of the free coordinates).  Every vector is
// decided: a rejected sub-cube by a ridge that fails for each of its vectors,
// the others down to the vector, whose remaining ridges, facet bound and
// properties are checked exactly as in the walk (sweep_kernel.h).
//
//   block     its 64 groups are tested at once, group = lane.
//   group     its 64 nodes are tested at once, node = lane: the lane's own part
//             of the words (the rows of the Gray bits of lane << 12, the same
//             for every group, since Gray codes of aligned sums are linear)
//             with the group's words XORed in.
//   node      likewise, child = lane; the node's words are one lane of the
//             vectors above (v_readlane).  Surviving children are appended to
//             the wave's child list in LDS (ballot, mbcnt).
//   child     64 listed children at a time, child = lane: each lane rebuilds
//             its child's leaf words from LDS tables and walks its 64 vectors
//             in Gray order, passes collected as bits (no branch: 8 VALU ops
//             per 64 vectors, against about 130 cycles for one child expanded
//             on its own).  Then each lane lists its candidates.
//   vector    64 listed candidates at a time, candidate = lane: any state word
//             is the XOR of the window's row and seven Gray-bit table rows.
//
// What bounds it: instruction issue and the latency of the waves' dependent
// chains; the descent makes no memory accesses.  Survivors cluster (in the
// vectors with few high coordinates, and in small kernels), so a group with
// many surviving nodes is shared by the waves of the workgroup, and items are
// spread over the workgroups, in parts where there are few.
//
// Measured against the walk of every vector (ms a sweep, the same inputs and
// outputs, two seeds): 1024 maps of n = 5..8, 6e10 vectors 9.9, 7.5 -> 1.12, 0.90;
// 512 of n = 4..7 1.87, 1.45 -> 0.40, 0.34; 512 over convenient bases 1.88, 1.61 ->
// 0.50, 0.45; three facet sets of 7-subsets of [11], k = 32..36, 11.3, 5.2 -> 0.40,
// 0.70; a slice of 1.5e10 pruned vectors of an n = 9 orbit 1.70 -> 0.11.  16384
// maps of n = 5..8, k <= 36, 1.04e12 vectors: 113 -> 7.3.
#pragma once

#include "sweep_kernel.h"

namespace wpm {

// Level section rows (must match the packer): the slot words of the leaf
// filter, of the 2^6 test (two groups of 32 ridges), of the 2^12 and of the
// 2^18 test.
constexpr int DLV_WORDS = 20;
enum { DLV_LEAF = 0, DLV_SIX = 4, DLV_TWELVE = 12, DLV_EIGHTEEN = 16 };
constexpr int LVT_WORDS = 16;                   // of these in the Gray-bit tables: all but the last
constexpr int BLOCK_BITS = 24, GROUP_BITS = 18;
constexpr int WIN_BITS = 21;                    // lists are relative to an aligned window of this
constexpr int WIN_ROWS = 8 * (WIN_BITS / 3);    // tables of a window's Gray bits, 3 per table
constexpr int TREE_LIST = 192;                  // candidates a wave's list holds
constexpr int CHILD_LIST = 128;                 // children a wave's list holds
constexpr int TREE_MIN_SPLIT = 1 << 16;         // vectors a part of a split item keeps at least
constexpr uint32_t CLAIM_TIME = 5000;           // of a claim, in 10 ns
constexpr uint32_t LONG_TIME = 1000;            // into a claim a wave's checks go first, in 10 ns
constexpr int MAX_CLAIM = 16;                   // items of a claim, at most
constexpr int HEAD_STRIDE = 16;                 // words from queue head to queue head (128 bytes)
constexpr int QUEUE_BLOCK = 64;                 // (parts of) items a queue holds in a row
constexpr int DENSE_GROUP = 16;                 // surviving nodes that make a group dense
// The base of a block of record slots has 44 bits; the top one stands for any
// block from 2^43 on, past every buffer, of which nothing is written.  (Its other
// bits still differ from one block to the next, which waiting waves look for.)
constexpr uint64_t PAST_RECORDS = 1ull << 43;

// Row stride of the window tables: an odd number of 16-byte units, so that the
// 8 rows a wave's lanes pick from start in 8 different bank groups.
__host__ __device__ constexpr int tree_stride(int RS) { return RS | 4; }

// LDS of one workgroup (uint32 words), for row width RS, stride S, kp rows:
//   [nw][TREE_LIST]       a candidate list per wave
//   [nw][CHILD_LIST / 2]  a child list per wave (16-bit entries)
//   [56][16]              Gray-bit tables of the level words (bits 0-20)
//   [kp-17][20]           level rows of coordinates 17 and up
//   [56][S]               Gray-bit tables of the staged instance (bits 0-20)
//   [nw][S]               per-wave window rows
// For 256 threads, RS = 44, kp = 36 that is 19.3 KB, with the static part 20.2 KB:
// seven workgroups, as many as the registers allow, in the 160 KB of a CU.
__host__ __device__ constexpr size_t tree_lds_bytes(int max_kp, int max_row_words, int wg_size) {
    const size_t nw = (size_t)(wg_size / 64), kp = (size_t)max_kp;
    const size_t up = kp > GROUP_BITS - 1 ? kp - (GROUP_BITS - 1) : 0;
    return sizeof(uint32_t) * (nw * (TREE_LIST + CHILD_LIST / 2) + (size_t)WIN_ROWS * LVT_WORDS +
                               up * DLV_WORDS + (WIN_ROWS + nw) * (size_t)tree_stride(max_row_words));
}

__device__ __forceinline__ uint32_t rlane(uint32_t v, uint32_t l) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)l);
}

// Global memory through pointers read from LDS: said to be global, since a
// flat access would also hold up the wave's LDS counter.
typedef __attribute__((address_space(1))) unsigned long long gu64;
__device__ __forceinline__ uint64_t add64(unsigned long long *p, uint64_t v) {
    return __hip_atomic_fetch_add((gu64 *)p, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t look64(const unsigned long long *p) {
    return __hip_atomic_load((const gu64 *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put64(uint64_t *p, uint64_t v) { *(gu64 *)p = v; }

template <int WAVES>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(WAVES)))
void tree_kernel(const uint32_t *__restrict__ tables, const int64_t *__restrict__ offsets,
                 const wpm_item *__restrict__ items, KArgs a_in) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds_dyn[];
    // The launch arguments, read from LDS where they are used.
    __shared__ KArgs s_a;
    // Counters that every workgroup adds to serialise at about 12 ns an access on
    // this chip, whatever the access does: 8192 waves adding six statistics
    // words each took longer than the sweep of a thousand instances.  So a
    // workgroup takes several items from the queue at a time, reserves record
    // slots in blocks shared by its waves (one LDS
    // atomic per check), adds an instance's count once per run of its items and
    // its statistics once.
    struct Shared {
        uint64_t block;    // of record slots: base << 20 | log2 size << 16 | used (size 0: none yet)
        uint64_t taken;
        uint64_t results;  // those added to the instances' counts
        uint64_t item, since;  // of the last claim
        uint32_t claim, ticket, queue;
        __attribute__((aligned(16))) wpm_item items[MAX_CLAIM + 1];  // of the last claim
        uint64_t dense[3];  // dense groups of a block of 64, by turns
        __attribute__((aligned(16))) uint32_t head[16];  // the staged table's header
    };
    __shared__ Shared sh;
    struct Book {
        // Vectors past every resident ridge group, and results, so far (over
        // any number of items: 32 bits could wrap).  Those that the rest of the
        // check rejects are the difference: an LDS add of their own made the
        // smallest sweep 2% longer.
        uint64_t past, results;
        uint32_t n[8];  // other statistics, in the order of d_stats
    };
    __shared__ Book s_book[512 / 64];
    if (threadIdx.x == 0) {
        s_a = a_in;
        sh.since = __builtin_amdgcn_s_memrealtime();
        sh.block = sh.taken = sh.results = 0;
        sh.dense[0] = sh.dense[1] = sh.dense[2] = 0;
    }
    const int tid = threadIdx.x;
    const int bd = blockDim.x, nw = bd >> 6;
    const int wv = (int)__builtin_amdgcn_readfirstlane((uint32_t)(tid >> 6));
    Book &bk = s_book[wv];
    if ((tid & 63) < 8) bk.n[tid & 63] = 0;
    bk.past = bk.results = 0;
    __syncthreads();
    const KArgs &a = s_a;
    auto tid_now = [&]() { return wv * 64 + lane_now(); };

    // per launch, wave-uniform
    const int mode = (int)__builtin_amdgcn_readfirstlane((uint32_t)a.mode);
    const int split = (int)__builtin_amdgcn_readfirstlane((uint32_t)a.split);
    const bool timed = rfl64((uint64_t)(uintptr_t)a.times) != 0;
    const int64_t vnum = (int64_t)rfl64((uint64_t)a.num_items) << split;

    uint32_t *const lds_W = lds_dyn + wv * TREE_LIST;
    uint16_t *const lds_C = (uint16_t *)(lds_dyn + nw * TREE_LIST) + wv * CHILD_LIST;
    uint32_t *const lds_LT = lds_dyn + nw * (TREE_LIST + CHILD_LIST / 2);
    uint32_t *const lds_LR = lds_LT + WIN_ROWS * LVT_WORDS;

    // the staged instance, wave-uniform
    int64_t staged = -1;
    const uint32_t *tab = tables;
    int kp = 7, RS = 4, S = 4;
    uint32_t *lds_X = lds_LR;
    // the wave's lists: candidates and children, the window they are relative
    // to, and the window whose row is in LDS
    uint32_t tcnt = 0, ccnt = 0;
    uint64_t twin = 0, trow = ~0ull;
    // level word (lane & 15) of the group at Gray state lvx, of the window at lvwx
    uint32_t lvst = 0, lvw = 0;
    uint64_t lvx = 0, lvwx = 0;
    uint32_t turn = 0;  // blocks of groups done: which dense mask is in use
    auto tally = [&](int i, uint32_t v) {  // (an LDS add that nothing waits for)
        if (lane_now() == 0)
            __hip_atomic_fetch_add(&bk.n[i], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };

    auto flush_counts = [&]() {  // with every wave past its last result
        if (tid_now() == 0 && staged >= 0) {
            uint64_t n = 0;
            for (int q = 0; q < nw; ++q) n += s_book[q].results;
            if (n != sh.results) add64(a.counts + staged, n - sh.results);
            sh.results = n;
        }
    };
    for (int64_t round = 0;; ++round) {
        // ---- the (parts of) items this workgroup takes next.  In the
        // dynamic mode the first is fixed, the others come from the queue's
        // counter.
        int64_t vt, vend, vnext = 0;
        uint32_t rest = 0;
        if (mode == 0) {
            if (round > 0) break;
            vt = (int64_t)rfl64((uint64_t)a.item_base) + (int64_t)blockIdx.x;
            vend = vt + 1;
        } else if (mode == 1) {
            vt = (int64_t)blockIdx.x + round * (int64_t)gridDim.x;
            vend = vt + 1;
        } else if (mode == 3) {
            if (round > 0) break;
            vt = (int64_t)rfl64((uint64_t)a.bins[blockIdx.x]);
            vend = (int64_t)rfl64((uint64_t)a.bins[blockIdx.x + 1]);
        } else {
            if (round == 0) {
                vt = (int64_t)blockIdx.x;
                vend = vt + 1;
                if (tid_now() == 0) {
                    sh.claim = 1;
                    sh.queue = blockIdx.x & (uint32_t)(a.queues - 1);
                }
            } else {
                if ((int64_t)gridDim.x >= vnum) break;
                if (wv == 0) {
                    // so many items that they take CLAIM_TIME at the last
                    // claim's pace (their density is that of their
                    // neighbours in the queue), and no more than a share of
                    // what is left
                    const uint64_t now = __builtin_amdgcn_s_memrealtime();
                    const uint32_t n0 = __builtin_amdgcn_readfirstlane(sh.claim),
                                   pace = (uint32_t)(now - rfl64(sh.since)) / n0 + 1u;
                    const int64_t left = (vnum - (int64_t)rfl64(sh.item)) / (16 * (int64_t)gridDim.x);
                    uint32_t n = CLAIM_TIME / pace;
                    if ((int64_t)n > left) n = (uint32_t)left;
                    n = timed || n < 1u ? 1u : n > (uint32_t)MAX_CLAIM ? (uint32_t)MAX_CLAIM : n;
                    // The items go round the queues in blocks; ticket t of queue
                    // q is (part of) item v, v rising with t.  An empty queue is
                    // left for another.  One head hands out a claim in 12 ns:
                    // where items are cheap, so that claims are short, 14,641
                    // of them were 190 us and are 105 from eight heads (1024
                    // maps 940 -> 875 us a sweep, 512 maps 431 -> 406, three
                    // facet sets of k = 32..36 557 -> 494).
                    uint32_t q = __builtin_amdgcn_readfirstlane(sh.queue);
                    const uint32_t nq = __builtin_amdgcn_readfirstlane((uint32_t)a.queues);
                    auto place = [&](uint64_t t, uint32_t of) -> int64_t {
                        return (int64_t)gridDim.x +
                               (int64_t)((t / QUEUE_BLOCK * nq + of) * QUEUE_BLOCK + t % QUEUE_BLOCK);
                    };
                    int64_t v;
                    uint64_t t;
                    for (;;) {
                        t = 0;
                        if (lane_now() == 0) t = add64(a.head + HEAD_STRIDE * q, n);
                        t = rfl64(t);
                        v = place(t, q);
                        if (v < vnum) break;
                        const uint32_t ln = (uint32_t)lane_now();
                        const bool some = ln < nq && place(look64(a.head + HEAD_STRIDE * (ln < nq ? ln : 0u)), ln) < vnum;
                        const uint32_t m = (uint32_t)__builtin_amdgcn_ballot_w64(some);
                        if (m == 0) break;
                        const uint32_t after = m & (0u - (2u << q));  // the next such queue, round from q
                        q = (uint32_t)__builtin_ctz(after ? after : m);
                    }
                    if (lane_now() == 0) {
                        sh.claim = n;
                        sh.ticket = (uint32_t)(t % QUEUE_BLOCK);
                        sh.queue = q;
                        sh.item = (uint64_t)v;
                    }
                }
                if (wv == 0) {
                    // the claim's items at once (loaded one by one, two loads were
                    // on each item's path: 512 maps 428 -> 419 us a sweep, 1024
                    // maps 1122 -> 1104, three facet sets of k = 32..36 670 -> 635)
                    const int64_t i = (int64_t)(rfl64(sh.item) >> split) + lane_now();
                    if (lane_now() <= MAX_CLAIM && i < vnum >> split) sh.items[lane_now()] = items[i];
                }
                __syncthreads();
                __builtin_amdgcn_s_setprio(0);
                vt = (int64_t)rfl64(sh.item);
                const uint32_t n = __builtin_amdgcn_readfirstlane(sh.claim),
                               room = (uint32_t)QUEUE_BLOCK - __builtin_amdgcn_readfirstlane(sh.ticket);
                vend = vt + (int64_t)(n < room ? n : room);
                if (n > room) {  // it goes on in the queue's next block
                    rest = n - room;
                    vnext = vend + (int64_t)(__builtin_amdgcn_readfirstlane((uint32_t)a.queues) - 1) * QUEUE_BLOCK;
                }
            }
            if (tid_now() == 0) {
                sh.since = __builtin_amdgcn_s_memrealtime();
                if (round == 0) sh.item = (uint64_t)vt;
            }
        }
        if (vt >= vnum) break;
        if (vend > vnum) vend = vnum;
        const int64_t held = mode == 2 && round > 0 ? vt >> split : INT64_MAX - MAX_CLAIM;
        auto item_at = [&](int64_t i) -> wpm_item { return i >= held && i <= held + MAX_CLAIM ? sh.items[i - held] : items[i]; };
        for (;; ++vt) {
            if (vt >= vend) {
                if (rest == 0 || vnext >= vnum) break;
                vt = vnext;
                vend = vnext + rest < vnum ? vnext + (int64_t)rest : vnum;
                rest = 0;
            }
            // Parts: a workgroup has one (the host makes no more of them than
            // workgroups), and the first parts of all items come first.  Short
            // items have no others: with an item's parts side by side, the last of
            // 49 items of 128 vectors waited for 1500 workgroups without work
            // (45 us a sweep, now 36).
            int64_t it = vt;
            uint32_t part = 0;
            if (split != 0) {
                const uint32_t n = (uint32_t)(vnum >> split);
                part = (uint32_t)vt / n;
                it = (int64_t)((uint32_t)vt % n);
            }
            uint64_t t_start = 0;
            if (timed) t_start = __builtin_amdgcn_s_memrealtime();
            const wpm_item itm = item_at(it);
            const uint32_t inst = __builtin_amdgcn_readfirstlane(itm.instance);
            const int c = (int)__builtin_amdgcn_readfirstlane((uint32_t)itm.cbits);
            const int lanes = (int)__builtin_amdgcn_readfirstlane((uint32_t)itm.lanes);
            const uint64_t first = rfl64(itm.first);
            // Parts p..p1 of an item with first index lo and n + 1 vectors; past
            // its end they are empty.
            auto part_range = [&](uint64_t lo, uint64_t n, uint32_t p, uint32_t p1, uint64_t &b, uint64_t &e) {
                uint64_t q = ((n >> split) + 128) & ~127ull;
                if (q < (uint64_t)TREE_MIN_SPLIT) q = TREE_MIN_SPLIT;
                b = lo + q * p;
                e = p1 != (1u << split) - 1u && q * (p1 + 1) <= n ? lo + q * (p1 + 1) - 1 : lo + n;
                return p == 0 || q * p <= n;
            };
            const uint64_t len = c < 64 ? ((uint64_t)lanes << c) - 1 : ~0ull;  // (less one)
            if (part != 0) {  // an empty part: before anything is staged for it
                uint64_t b, e;
                if (!part_range(0, len, part, part, b, e)) continue;
            }
            auto fits = [&](int cc, int ll, uint64_t ff) {
                return cc >= 7 && cc <= kp && ll >= 1 && ll <= bd &&
                       (int)(ff & ((1u << LANE_BITS) - 1)) + ll <= (1 << LANE_BITS) &&
                       (cc == 0 || ff + (uint64_t)ll <= (1ull << (kp - cc)));
            };
            // ---- a new instance: its header, counts of the last one, tables.
            // Malformed items are skipped and counted (as in the walk); items
            // of tables without a level section belong to the walk, which
            // counts its own.
            bool bad = false, skip = false;
            const bool fresh = (int64_t)inst != staged;
            const uint32_t *ntab = tab;
            int nRS = RS;
            bool has_off = false;
            const int okp = kp;
            if (fresh) {
                bad = inst >= (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a.num_instances);
                if (!bad) {
                    ntab = tables + rfl64((uint64_t)offsets[inst]);
                    const int G = (int)ntab[D_G], Qp = (int)ntab[D_QS], W = (int)ntab[D_W];
                    kp = (int)ntab[D_KP];
                    nRS = (int)ntab[D_RS];
                    has_off = (ntab[D_FLAGS] & D_FLAG_OFFSET) != 0u;
                    skip = (ntab[D_FLAGS] & D_FLAG_TREE) == 0u;
                    bad = (skip && __builtin_amdgcn_readfirstlane((uint32_t)a.alone) != 0u) ||
                          ntab[D_MAGIC] != D_TABLE_MAGIC || kp < 7 ||
                          kp > (int)__builtin_amdgcn_readfirstlane((uint32_t)a.max_kp) ||
                          nRS > (int)__builtin_amdgcn_readfirstlane((uint32_t)a.max_rs) || (nRS & 3) || G < 1 ||
                          (Qp != 4 && Qp != 8) || 4 + (G - 1) * Qp + W > nRS;
                }
            }
            bad = bad || !fits(c, lanes, first);
            if (bad || skip) {
                kp = okp;
                const bool theirs = inst >= (uint32_t)a.num_instances ? !a.count_bad : skip && !a.alone;
                if (bad && !theirs && part == 0 && tid_now() == 0) {
                    add64(a.total + TOT_BAD_ITEMS, 1ull);
                    if (timed) a.times[2 * it] = a.times[2 * it + 1] = 0;
                }
                continue;
            }
            if (fresh) {
                __syncthreads();  // every wave is done with the last instance
                flush_counts();
                tab = ntab;
                RS = nRS;
                S = tree_stride(RS);
                const int up = kp > GROUP_BITS - 1 ? kp - (GROUP_BITS - 1) : 0;
                lds_X = lds_LR + up * DLV_WORDS;
                const uint32_t *rows = tab + DEV_HDR_WORDS;
                const uint32_t *lrows = rows + (kp + (has_off ? 1 : 0)) * RS;
                // Gray-bit tables: row v of table b = XOR of the rows 3b + j
                // over the set bits j of v (rows >= kp count as zero); a
                // thread takes one word of one table
                auto table3 = [&](const uint32_t *src, int stride, int b, int w, uint32_t *dst, int dstride) {
                    const int t0 = 3 * b;
                    const uint32_t r0 = t0 < kp ? src[t0 * stride + w] : 0u;
                    const uint32_t r1 = t0 + 1 < kp ? src[(t0 + 1) * stride + w] : 0u;
                    const uint32_t r2 = t0 + 2 < kp ? src[(t0 + 2) * stride + w] : 0u;
                    uint32_t *d = dst + 8 * b * dstride + w;
                    const uint32_t r01 = r0 ^ r1;
                    d[0] = 0u;
                    d[dstride] = r0;
                    d[2 * dstride] = r1;
                    d[3 * dstride] = r01;
                    d[4 * dstride] = r2;
                    d[5 * dstride] = r0 ^ r2;
                    d[6 * dstride] = r1 ^ r2;
                    d[7 * dstride] = r01 ^ r2;
                };
                if (tid_now() < DEV_HDR_WORDS) sh.head[tid_now()] = tab[tid_now()];
                for (int e = tid_now(); e < (WIN_BITS / 3) * LVT_WORDS; e += bd)
                    table3(lrows, DLV_WORDS, e / LVT_WORDS, e % LVT_WORDS, lds_LT, LVT_WORDS);
                for (int e = tid_now(); e < up * DLV_WORDS; e += bd)
                    lds_LR[e] = lrows[(GROUP_BITS - 1) * DLV_WORDS + e];
                for (int w = lane_now(); w < RS; w += 64)
                    for (int b = wv; b < WIN_BITS / 3; b += nw) table3(rows, RS, b, w, lds_X, S);
                lvst = lvw = has_off ? lrows[kp * DLV_WORDS + (lane_now() & 15)] : 0u;
                lvx = lvwx = 0;
                twin = 0;  // (lvw is the window's at index 0; the lists are empty)
                trow = ~0ull;
                staged = inst;
                __syncthreads();
            }
            // ---- the run: Gray indices [i0, i1] of this item's parts in the
            // claim, and of the claim's next items while they continue the
            // range (one set-up for all).
            const uint32_t plast = (1u << split) - 1u;
            const uint64_t lo0 = c < 64 ? first << c : 0;
            uint64_t i0, i1;
            bool some;
            {
                const int64_t left = vend - vt - 1;
                const uint32_t p1 = (int64_t)(plast - part) <= left ? plast : part + (uint32_t)left;
                some = part_range(lo0, len, part, p1, i0, i1);
                if (!timed) vt += p1 - part;
            }
            // the list is emptied when the instance or the claim ends
            bool last = true;
            while (!timed && vt + 1 < vend) {
                const wpm_item nx = item_at((vt + 1) >> split);
                const int nc = (int)__builtin_amdgcn_readfirstlane((uint32_t)nx.cbits);
                const int nl = (int)__builtin_amdgcn_readfirstlane((uint32_t)nx.lanes);
                const uint64_t nf = rfl64(nx.first);
                if ((int64_t)__builtin_amdgcn_readfirstlane(nx.instance) != staged || !fits(nc, nl, nf)) break;
                if (!some || nc >= 64 || i1 + 1 == 0 || nf << nc != i1 + 1) {
                    last = false;
                    break;
                }
                const int64_t left = vend - vt - 2;
                const uint32_t p1 = (int64_t)plast <= left ? plast : (uint32_t)left;
                uint64_t b;
                part_range(nf << nc, ((uint64_t)nl << nc) - 1, 0, p1, b, i1);
                vt += 1 + p1;
            }
            // every nw-th set bit of a mask, from this wave's place on
            auto my_turns = [&](uint64_t m) -> uint64_t {
                const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                return m & __builtin_amdgcn_ballot_w64(below % (uint32_t)nw == (uint32_t)wv);
            };
            // the rows of the set bits of d (at and above 17), word `w` each
            auto high_rows = [&](uint64_t d, int w) -> uint32_t {
                uint32_t v = 0;
                for (; d; d &= d - 1) v ^= lds_LR[((int)__builtin_ctzll(d) - (GROUP_BITS - 1)) * DLV_WORDS + w];
                return v;
            };
            // lane vectors, re-read from LDS after every check (so that they
            // hold no registers through it): what node `lane` of a group and
            // child `lane` of a node add; o12 with the group's words in
            uint32_t o12[12], o6[8];
            auto lane_vectors = [&]() {
                // Gray bits of 2 lane: bit j is bit s - 1 + j of the Gray code of lane << s
                const uint32_t ln = (uint32_t)lane_now(), gr = ln ^ (ln << 1);
                const uint32_t d0 = 4 * (gr & 1u), d1 = (gr >> 1) & 7u, d2 = (gr >> 4) & 7u;
                auto acc = [&](uint32_t *o, int nq, uint32_t ta, uint32_t tb, uint32_t tc) {
                    const uint32_t *pa = lds_LT + ta * LVT_WORDS + DLV_SIX, *pb = lds_LT + tb * LVT_WORDS + DLV_SIX,
                                   *pc = lds_LT + tc * LVT_WORDS + DLV_SIX;
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        if (q < nq) {
                            const uint4 u = *(const uint4 *)(pa + 4 * q), v = *(const uint4 *)(pb + 4 * q),
                                        w = *(const uint4 *)(pc + 4 * q);
                            o[4 * q] = xor3(u.x, v.x, w.x);
                            o[4 * q + 1] = xor3(u.y, v.y, w.y);
                            o[4 * q + 2] = xor3(u.z, v.z, w.z);
                            o[4 * q + 3] = xor3(u.w, v.w, w.w);
                        }
                };
                acc(o12, 3, 8 * 3 + d0, 8 * 4 + d1, 8 * 5 + d2);  // lane << 12: bits 11 (table 3), 12-14, 15-17
                acc(o6, 2, 8 * 1 + d0, 8 * 2 + d1, 8 * 3 + d2);   // lane << 6: bits 5 (table 1), 6-8, 9-11
#pragma unroll
                for (int q = 0; q < 12; ++q) o12[q] ^= rlane(lvst, (uint32_t)(DLV_SIX + q));
            };
            // ---- blocks of 64 groups: the groups that pass the 2^18 test go
            // round the waves; a wave that meets a dense one leaves it to all
            // of them, for after the others (a wave alone on it was the tail of
            // the launch).  Fewer groups than waves are shared at once.
            const uint64_t gfirst = i0 >> GROUP_BITS, gend = some ? (i1 >> GROUP_BITS) + 1 : gfirst;
            uint64_t gb0 = gfirst & ~63ull, m18 = 0, m12 = 0, gcur = 0;
            int phase = 0;        // 0: a new block, 1: own groups, 2: shared groups
            bool share6 = false;  // the nodes' children are shared by the waves
            uint32_t r12 = 0;
            uint32_t ca = 0, cb = 0, cbase = 0;  // a walked batch's candidates still to list, its place in lds_C
            bool drain = false;   // empty the child list
            bool done = gfirst >= gend;  // every group of the run has been visited
            bool pend = false;            // a walked batch still has candidates to list
            while (!done || pend || (last && (tcnt | ccnt) != 0u)) {
                bool full = false;
                pend = false;
                drain = drain || (done && last);
                auto append = [&](bool p, uint64_t m) -> uint32_t {  // this lane's place among the set bits
                    return p ? __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))
                             : 0u;
                };
                // ---- children: until fewer than 64 are listed (none, to drain
                // the list), or the candidate list is full
                for (;;) {
                    // candidates of a walked batch: every lane lists its next one
                    for (;;) {
                        const uint32_t w = ca ? ca : cb;
                        const uint64_t m = __builtin_amdgcn_ballot_w64(w != 0u);
                        if (!m) break;
                        const uint32_t n = (uint32_t)__builtin_popcountll(m);
                        if (tcnt + n > (uint32_t)TREE_LIST) {
                            full = pend = true;
                            tally(4, 1);
                            break;
                        }
                        // bit 31 - s of ca is step s, of cb step 32 + s
                        const uint32_t st = (uint32_t)__builtin_clz(w | 1u);
                        const uint32_t at = tcnt + append(w != 0u, m);
                        if (w) lds_W[at] = (uint32_t)lds_C[cbase + (uint32_t)lane_now()] << 6 | (ca ? st : st + 32u);
                        const uint32_t cleared = w & ~(0x80000000u >> st);
                        cb = ca ? cb : cleared;
                        ca = ca ? cleared : 0u;
                        tcnt += n;
                    }
                    if (full || !(ccnt >= 64u || (drain && ccnt != 0u))) break;
                    {
                        // the last (at most 64) listed children: each lane
                        // rebuilds its child's leaf words (Gray bits 5-20 of
                        // child << 6 in the window) and walks 64 vectors as two
                        // chains of 32 steps, which share the flipped rows
                        const uint32_t nb = ccnt < 64u ? ccnt : 64u;
                        ccnt -= nb;
                        cbase = ccnt;
                        tally(7, nb);
                        const bool mine = (uint32_t)lane_now() < nb;
                        const uint32_t e = mine ? (uint32_t)lds_C[cbase + (uint32_t)lane_now()] : 0u;
                        const uint32_t gr = (e << 6) ^ (e << 5);
                        auto leaf = [&](uint32_t row) { return *(const uint4 *)(lds_LT + row * LVT_WORDS + DLV_LEAF); };
                        const uint4 t1 = leaf(8 * 1 + ((gr >> 3) & 7u)), t2 = leaf(8 * 2 + ((gr >> 6) & 7u)),
                                    t3 = leaf(8 * 3 + ((gr >> 9) & 7u)), t4 = leaf(8 * 4 + ((gr >> 12) & 7u)),
                                    t5 = leaf(8 * 5 + ((gr >> 15) & 7u)), t6 = leaf(8 * 6 + ((gr >> 18) & 7u));
                        uint32_t s0[4], s1[4], rw[5][4];
                        s0[0] = xor3(xor3(t1.x, t2.x, t3.x), xor3(t4.x, t5.x, t6.x), rlane(lvw, 0));
                        s0[1] = xor3(xor3(t1.y, t2.y, t3.y), xor3(t4.y, t5.y, t6.y), rlane(lvw, 1));
                        s0[2] = xor3(xor3(t1.z, t2.z, t3.z), xor3(t4.z, t5.z, t6.z), rlane(lvw, 2));
                        s0[3] = xor3(xor3(t1.w, t2.w, t3.w), xor3(t4.w, t5.w, t6.w), rlane(lvw, 3));
#pragma unroll
                        for (int t = 0; t < 5; ++t) {  // the rows of coordinates 0-4
                            const uint4 r = leaf((uint32_t)(8 * (t / 3) + (1 << (t % 3))));
                            rw[t][0] = r.x, rw[t][1] = r.y, rw[t][2] = r.z, rw[t][3] = r.w;
                        }
                        const uint4 r5 = leaf(8 + 4);  // coordinate 5: step 32 has the Gray code 48
                        s1[0] = xor3(s0[0], rw[4][0], r5.x);
                        s1[1] = xor3(s0[1], rw[4][1], r5.y);
                        s1[2] = xor3(s0[2], rw[4][2], r5.z);
                        s1[3] = xor3(s0[3], rw[4][3], r5.w);
                        ca = cb = 0;
#pragma unroll
                        for (int st = 0; st < 32; ++st) {
                            const uint32_t f0 = fail4(s0[0], s0[1], s0[2], s0[3]);
                            const uint32_t f1 = fail4(s1[0], s1[1], s1[2], s1[3]);
                            ca = ca + ca + (f0 == 0u ? 1u : 0u);
                            cb = cb + cb + (f1 == 0u ? 1u : 0u);
                            if (st < 31) {
                                const int t = __builtin_ctz((unsigned)(st + 1));
#pragma unroll
                                for (int q = 0; q < 4; ++q) {
                                    s0[q] ^= rw[t][q];
                                    s1[q] ^= rw[t][q];
                                }
                            }
                        }
                        if (!mine) ca = cb = 0;
                    }
                }
                // ---- descend until 64 children are listed, or a list has to be
                // emptied, or every group has been visited
                if (!full && !done) {
                lane_vectors();
                while (ccnt < 64u) {
                    if (m12) {
                        // a node: its 64 children
                        r12 = (uint32_t)__builtin_ctzll(m12);
                        m12 &= m12 - 1;
                        uint32_t v[8];
#pragma unroll
                        for (int q = 0; q < 8; ++q) v[q] = o6[q] ^ rlane(o12[q], r12);
                        const uint32_t f = fail4(v[0], v[1], v[2], v[3]) | fail4(v[4], v[5], v[6], v[7]);
                        uint64_t m6 = __builtin_amdgcn_ballot_w64(f == 0u);
                        if (!m6) continue;
                        const uint64_t nb = (gcur << GROUP_BITS) + ((uint64_t)r12 << 12);
                        if (nb < i0 || i1 - nb < 4095) {  // a node that the range only partly covers
                            if (nb < i0) m6 &= ~0ull << ((i0 - nb) >> 6);
                            if (i1 - nb < 4095) m6 &= ~0ull >> (63 - ((i1 - nb) >> 6));
                        }
                        if (share6) m6 = my_turns(m6);
                        const bool p = (m6 >> lane_now()) & 1ull;
                        const uint32_t at = ccnt + append(p, m6);
                        if (p)
                            lds_C[at] = (uint16_t)(((uint32_t)gcur & ((1u << (WIN_BITS - GROUP_BITS)) - 1)) << 12 |
                                                   r12 << 6 | (uint32_t)lane_now());
                        ccnt += (uint32_t)__builtin_popcountll(m6);
                        continue;
                    }
                    if (phase == 1 && m18 == 0) {
                        // own groups done: the dense ones, once every wave is
                        if (tid_now() == 0) sh.dense[turn == 2 ? 0 : turn + 1] = 0;
                        __syncthreads();
                        m18 = rfl64(__hip_atomic_load(&sh.dense[turn], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                        turn = turn == 2 ? 0 : turn + 1;
                        phase = 2;
                    }
                    if (phase == 2 && m18 == 0) {
                        phase = 0;
                        gb0 += 64;
                    }
                    if (phase == 0) {
                        if (gb0 >= gend) {
                            done = true;
                            break;
                        }
                        // a block: its 64 groups.  The block's words, then
                        // the rows of the Gray bits of lane << 18 (bits 17-23).
                        const uint64_t xb = (gb0 << GROUP_BITS) ^ (gb0 << (GROUP_BITS - 1));
                        uint32_t e[4];
                        const bool off = (__builtin_amdgcn_readfirstlane(sh.head[D_FLAGS]) & D_FLAG_OFFSET) != 0u;
#pragma unroll
                        for (int q = 0; q < 4; ++q) e[q] = 0;
                        if (off) {
                            const uint32_t *r = opaque(tab) + DEV_HDR_WORDS + (kp + 1) * RS + kp * DLV_WORDS + DLV_EIGHTEEN;
#pragma unroll
                            for (int q = 0; q < 4; ++q) e[q] = gword(r + q);
                        }
                        for (uint64_t d = xb; d; d &= d - 1) {
                            const uint4 r = *(const uint4 *)(lds_LR + ((int)__builtin_ctzll(d) - (GROUP_BITS - 1)) * DLV_WORDS +
                                                             DLV_EIGHTEEN);
                            e[0] ^= r.x, e[1] ^= r.y, e[2] ^= r.z, e[3] ^= r.w;
                        }
                        const uint32_t ln = (uint32_t)lane_now(), gr = ln ^ (ln << 1);
#pragma unroll
                        for (int t = 1; t < 7; ++t) {  // (bit 17 is free)
                            if (GROUP_BITS - 1 + t >= kp) break;
                            const uint4 r = *(const uint4 *)(lds_LR + t * DLV_WORDS + DLV_EIGHTEEN);
                            const uint32_t on = 0u - ((gr >> t) & 1u);
                            e[0] ^= r.x & on, e[1] ^= r.y & on, e[2] ^= r.z & on, e[3] ^= r.w & on;
                        }
                        m18 = __builtin_amdgcn_ballot_w64(fail4(e[0], e[1], e[2], e[3]) == 0u);
                        if (gb0 < gfirst) m18 &= ~0ull << (gfirst - gb0);
                        if (gend - gb0 < 64) m18 &= ~0ull >> (64 - (gend - gb0));
                        if (__builtin_popcountll(m18) < nw) {
                            phase = 2;
                        } else {
                            phase = 1;
                            m18 = my_turns(m18);
                        }
                        continue;
                    }
                    // a group: its 64 nodes
                    const uint64_t gnext = gb0 + (uint64_t)__builtin_ctzll(m18);
                    const uint64_t win = gnext >> (WIN_BITS - GROUP_BITS);
                    if (win != twin) {
                        // the lists are emptied before the window moves
                        if (ccnt) {
                            drain = true;
                            break;
                        }
                        if (tcnt) {
                            full = true;
                            break;
                        }
                        drain = false;
                        twin = win;
                        const uint64_t xw = (win << WIN_BITS) ^ (win << (WIN_BITS - 1));
                        lvw ^= high_rows(xw ^ lvwx, lane_now() & 15);
                        lvwx = xw;
                    }
                    m18 &= m18 - 1;
                    gcur = gnext;
                    const uint64_t xg = (gcur << GROUP_BITS) ^ (gcur << (GROUP_BITS - 1));
                    const uint32_t dv = high_rows(xg ^ lvx, lane_now() & 15);
                    lvx = xg;
                    lvst ^= dv;
#pragma unroll
                    for (int q = 0; q < 12; ++q) o12[q] ^= rlane(dv, (uint32_t)(DLV_SIX + q));
                    m12 = __builtin_amdgcn_ballot_w64(fail4(o12[8], o12[9], o12[10], o12[11]) == 0u);
                    const uint64_t gb = gcur << GROUP_BITS;
                    if (gb < i0) m12 &= ~0ull << ((i0 - gb) >> 12);
                    if (i1 - gb < (1ull << GROUP_BITS) - 1) m12 &= ~0ull >> (63 - ((i1 - gb) >> 12));
                    const int left = __builtin_popcountll(m12);
                    // (counted by the wave that expands it, of a shared one by the first)
                    if ((phase == 1 ? left < DENSE_GROUP : wv == 0) && lane_now() == 0) {
                        __hip_atomic_fetch_add(&bk.n[5], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        __hip_atomic_fetch_add(&bk.n[6], (uint32_t)left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                    share6 = false;
                    if (phase == 1) {
                        if (left >= DENSE_GROUP) {
                            if (lane_now() == 0)
                                __hip_atomic_fetch_or(&sh.dense[turn], 1ull << (gcur - gb0), __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_WORKGROUP);
                            m12 = 0;
                        }
                    } else if (left >= 2 * nw) {
                        m12 = my_turns(m12);
                    } else {
                        // few nodes: every wave expands them all, and the waves
                        // share their children
                        share6 = true;
                    }
                }
                }
                if (full || (done && last && ccnt == 0u && tcnt != 0u)) {
                    // ---- check: lane j takes entry base + j
                    // A wave that is long into its claim has dense items, the last
                    // of the launch to end: it issues before its neighbours
                    // (512 maps 320 -> 303 us a sweep, 512 pruned 640 -> 600, three
                    // facet sets of k = 32..36 463 -> 453, 1024 maps 1112 -> 1097;
                    // 25 and 50 us and other priorities measured the same).
                    if (mode == 2 && !timed && (uint32_t)(__builtin_amdgcn_s_memrealtime() - rfl64(sh.since)) > LONG_TIME)
                        __builtin_amdgcn_s_setprio(1);
                    tally(0, tcnt);
                    tally(3, (tcnt + 63) / 64);
                    if (trow != twin) {
                        // the state at the window's start, one word per lane
                        const uint64_t wb = twin << WIN_BITS;
                        const uint64_t xw = (wb ^ (wb >> 1)) >> (WIN_BITS - 1);
                        const uint32_t *rw = opaque(tab) + DEV_HDR_WORDS;
                        const bool off = (__builtin_amdgcn_readfirstlane(sh.head[D_FLAGS]) & D_FLAG_OFFSET) != 0u;
                        for (int w = lane_now(); w < RS; w += 64) {
                            uint32_t s = off ? gword(rw + kp * RS + w) : 0u;
                            for (uint64_t d = xw; d; d &= d - 1)
                                s ^= gword(rw + (WIN_BITS - 1 + __builtin_ctzll(d)) * RS + w);
                            lds_X[(WIN_ROWS + wv) * S + w] = s;
                        }
                        trow = twin;
                    }
                    asm volatile("" ::: "memory");
                    const uint32_t *const lds_win = lds_X + (WIN_ROWS + wv) * S;
                    const uint4 *const hd = (const uint4 *)sh.head;
                    const uint4 h0 = hd[0], h1 = hd[1], h2 = hd[2], h3 = hd[3];
                    const uint32_t hk = __builtin_amdgcn_readfirstlane(h0.y), hw = __builtin_amdgcn_readfirstlane(h1.x),
                                   hg = __builtin_amdgcn_readfirstlane(h1.y), hq = __builtin_amdgcn_readfirstlane(h1.z),
                                   hm = __builtin_amdgcn_readfirstlane(h2.x), hf = __builtin_amdgcn_readfirstlane(h2.w),
                                   hp = __builtin_amdgcn_readfirstlane(h3.x), hn = __builtin_amdgcn_readfirstlane(h3.y),
                                   hd0 = __builtin_amdgcn_readfirstlane(h3.z), hdn = __builtin_amdgcn_readfirstlane(h3.w);
                    auto head = [&](int i) -> uint32_t {
                        return i == D_K ? hk : i == D_W ? hw : i == D_MAXF ? hm
                               : i == D_FLAGS ? hf : i == D_PROPS ? hp : i == D_NPROPS ? hn : i == D_DEFER ? hd0 : hdn;
                    };
#pragma unroll 1
                    for (uint32_t base = 0; base < tcnt; base += 64) {
                        const uint32_t ln = (uint32_t)lane_now();
                        const uint32_t ent = base + ln < tcnt ? lds_W[base + ln] : 0u;
                        const uint32_t gr = ent ^ (ent >> 1);
                        uint32_t o[WIN_BITS / 3];
#pragma unroll
                        for (int b = 0; b < WIN_BITS / 3; ++b)
                            o[b] = (8u * b + ((gr >> (3 * b)) & 7u)) * (uint32_t)S;
                        // All eight loads of a word are in flight: a check is a chain of
                        // LDS round trips, and three loads at a time made it
                        // three times as long (three facet sets, k = 32..36: 609
                        // -> 554 us a sweep; 1024 maps 1.32 -> 1.27 ms).
                        auto word4 = [&](int off) {
                            asm volatile("" : "+s"(off));  // (one set of addresses, not one per slot group)
                            uint4 p[WIN_BITS / 3];
                            uint4 r = *(const uint4 *)(lds_win + off);
#pragma unroll
                            for (int b = 0; b < WIN_BITS / 3; ++b) p[b] = *(const uint4 *)(lds_X + o[b] + off);
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int b = 0; b < WIN_BITS / 3; b += 2) {
                                uint4 q = {0u, 0u, 0u, 0u};
                                if (b + 1 < WIN_BITS / 3) q = p[b + 1];
                                r.x = xor3(r.x, p[b].x, q.x);
                                r.y = xor3(r.y, p[b].y, q.y);
                                r.z = xor3(r.z, p[b].z, q.z);
                                r.w = xor3(r.w, p[b].w, q.w);
                            }
                            return r;
                        };
                        auto word1 = [&](int off) {
                            uint32_t r = lds_win[off];
#pragma unroll
                            for (int b = 0; b < WIN_BITS / 3; ++b) r ^= lds_X[o[b] + off];
                            return r;
                        };
                        bool pass = groups_pass((int)hg, (int)hq, base + ln < tcnt, 0, word4);
                        const uint64_t i = (twin << WIN_BITS) + (uint64_t)ent;
                        const uint64_t x = i ^ (i >> 1);
                        // x = 0 is the empty complex, except in a coset (K = K*)
                        const int kk = (int)head(D_K);
                        pass = pass && (x != 0 || (head(D_FLAGS) & D_FLAG_OFFSET) != 0u) &&
                               (kk >= 64 || (x >> kk) == 0);
                        const uint64_t pball = __builtin_amdgcn_ballot_w64(pass);
                        if (!pball) continue;
                        const bool ok = properties_pass(tab, head, (int)hg, (int)hq, pass, word4, word1);
                        const uint64_t bal = __builtin_amdgcn_ballot_w64(ok);
                        if (lane_now() == 0)
                            __hip_atomic_fetch_add(&bk.past, (uint64_t)__builtin_popcountll(pball), __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WORKGROUP);
                        if (!bal) continue;
                        // Record slots from the workgroup's block.  The wave
                        // whose results cross its end takes what is left, gets
                        // a new block and puts the rest at its start, so slots
                        // stay unused only at the end of the last block; waves
                        // that come meanwhile (used > size) wait for the new
                        // block.  Relaxed order is enough, since a wave's LDS
                        // operations complete in order; acquire and release
                        // would wait for its record stores as well.  Blocks grow from 128 slots with what the
                        // workgroup has used, to a.chunk; the plain mode (0)
                        // reserves exactly.
                        const uint32_t nbal = (uint32_t)__builtin_popcountll(bal);
                        uint64_t pos0 = 0, next = 0;
                        uint32_t room = 0;
                        if (lane_now() == 0) {
                            __hip_atomic_fetch_add(&bk.results, (uint64_t)nbal, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                            const uint32_t most = (uint32_t)a.chunk;
                            if (most == 0) {
                                next = add64(a.total + TOT_SLOTS, nbal);
                            } else {
                                for (;;) {
                                    const uint64_t old = __hip_atomic_fetch_add(&sh.block, (uint64_t)nbal, __ATOMIC_RELAXED,
                                                                                __HIP_MEMORY_SCOPE_WORKGROUP);
                                    asm volatile("" ::: "memory");
                                    const uint32_t used = (uint32_t)old & 0xFFFFu, lg = (uint32_t)(old >> 16) & 15u;
                                    const uint32_t size = lg ? 1u << lg : 0u;
                                    if (used > size) {  // another wave is getting the next block
                                        // (base and size: the first block's base
                                        // is 0, as before it)
                                        const uint64_t was = old >> 16;
                                        while ((__hip_atomic_load(&sh.block, __ATOMIC_RELAXED,
                                                                  __HIP_MEMORY_SCOPE_WORKGROUP) >> 16) == was)
                                            __builtin_amdgcn_s_sleep(2);
                                        continue;
                                    }
                                    pos0 = (old >> 20) + used;
                                    room = size - used < nbal ? size - used : nbal;
                                    if (nbal > room) {
                                        const uint32_t over = nbal - room;
                                        const uint64_t taken = __hip_atomic_load(&sh.taken, __ATOMIC_RELAXED,
                                                                                  __HIP_MEMORY_SCOPE_WORKGROUP);
                                        uint32_t l2 = 7;
                                        while (l2 < 12 && (2ull << l2) <= taken && (2u << l2) <= most) ++l2;
                                        next = add64(a.total + TOT_SLOTS, 1ull << l2);
                                        __hip_atomic_store(&sh.taken, taken + (1ull << l2), __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                                        asm volatile("" ::: "memory");
                                        uint64_t base = next & (PAST_RECORDS - 1);
                                        if (next >= PAST_RECORDS) base |= PAST_RECORDS;
                                        __hip_atomic_store(&sh.block, base << 20 | (uint64_t)l2 << 16 | over,
                                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                                    }
                                    break;
                                }
                            }
                        }
                        pos0 = rfl64(pos0);
                        next = rfl64(next);
                        room = __builtin_amdgcn_readfirstlane(room);
                        if (ok) {
                            const uint32_t rk = __builtin_amdgcn_mbcnt_hi(
                                (uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                            const uint64_t pos = rk < room ? pos0 + rk : next + (rk - room);
                            if (pos < a.cap) {
                                put64(a.surv + 2 * pos, x);
                                put64(a.surv + 2 * pos + 1, (uint64_t)staged);
                            }
                        }
                    }
                    tcnt = 0;
                    asm volatile("" ::: "memory");
                }
            }
            if (timed) {
                __syncthreads();
                if (tid_now() == 0) {
                    put64(a.times + 2 * it, t_start);
                    put64(a.times + 2 * it + 1, __builtin_amdgcn_s_memrealtime());
                }
            }
        }
        if (mode == 2) __syncthreads();  // every wave has read the claim
    }
    // ---- publish the workgroup's totals and close its block of record slots
    __syncthreads();
    flush_counts();
    const uint32_t lg = (uint32_t)(sh.block >> 16) & 15u, used = (uint32_t)sh.block & 0xFFFFu;
    for (uint32_t e = used + (uint32_t)tid; lg != 0 && e < 1u << lg; e += (uint32_t)bd) {
        const uint64_t pos = (sh.block >> 20) + e;
        if (pos < a.cap) {
            put64(a.surv + 2 * pos, 0);
            put64(a.surv + 2 * pos + 1, ~0ull);
        }
    }
    if (tid == 0 && sh.results) add64(a.total + TOT_RESULTS, sh.results);
    if (a.stats && tid < 8) {
        uint64_t n = 0;
        for (int q = 0; q < nw; ++q) n += tid == 1 || tid == 2 ? s_book[q].past : s_book[q].n[tid];
        if (tid == 2) n -= sh.results;
        if (n) add64(a.stats + tid, n);
    }
}

}  // namespace wpm
