// Join of the partition pairs of a PHJ ("apply SHJ on each partition pair",
// Algorithm 2; steps b1-b4 and p1-p4 of Algorithm 1 inside each pair).
//
// Work item = (partition pair i, chunk of up to kJoinChunk S tuples of S_i),
// probed kJoinSub tuples at a time.  One workgroup per item:
//  * |R_i| <= lds_cap: R_i becomes a chained table in LDS.  The paper's
//    bucket header + key list + rid list (Section 3.1) is laid out without an
//    allocator: one head word per bucket, one 32-bit record (what the bucket
//    does not say of the key, link) and the rid per R tuple at its own row; a
//    tuple is pushed on its bucket's chain with one LDS exchange (the latch of
//    Section 3.3).  Probing walks the chain (p3) and compares keys (p4).
//  * |R_i| > lds_cap (few, large partitions: low radix bits, duplicate-heavy
//    R): the pair is joined through a partition-local open-addressing table
//    in HBM (2 |R_i| slots at twice R_i's offset, plus per-key row chains),
//    cleared by the last scatter (or a launch of its own: scatter_clears) and
//    built by the first join launch before it probes (compare-and-swap for a
//    new key, exchange pushes for duplicates; build_tables); S tuples on very
//    long chains are counted and written by the whole workgroup (hj_heavy.h).
// Workgroups take items in groups of 16 consecutive ones per XCD
// (item_of_block), so one partition's items share that XCD's L2.
// Output: count pass -> per-wave counts -> scan -> write pass, which re-runs
// the same item and stores its pairs at the scanned offset, or one pass that
// reserves each round's pairs on a running total (Section 3.3's dynamic
// output allocation replaced by counting or by block reservation).
#include <algorithm>
#include <type_traits>

#include "hj_device.h"
#include "hj_heavy.h"
#include "hj_internal.h"
#include "hj_side.h"

namespace hj {

namespace {

constexpr uint32_t kSubJ = kJoinSub / kJoinWaves;     // S tuples per wave of a probe round

__device__ __forceinline__ uint64_t region_slot(int32_t key, uint32_t H) {
    return ((uint64_t)slot_hash(key) * H) >> 32;
}

// A value that is equal in all lanes, as a scalar: loops and branches around
// barriers have to be on scalars, or the compiler may part a wave's lanes there.
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return uniform_word(x); }

// Build items of the HBM tables, or 0 when a chained scan of the call gave up
// (which the call reports): partitions made from wrong starts may share table
// slots, and a look-up in a table without an empty slot would not end.
// (Both words are read at once: one after the other, every workgroup of a join with
// tables waited for both.)
__device__ __forceinline__ uint32_t table_items(const OvfBuild& B) {
    const uint32_t n = *B.total;
    return *B.err & kErrLookback ? 0u : n;
}

__global__ void __launch_bounds__(256) k_ovf_clear(OvfBuild B, uint64_t* __restrict__ ovf_table) {
    const uint32_t nitems = table_items(B);
    for (uint32_t item = blockIdx.x; item < nitems; item += gridDim.x) {
        const uint32_t i = B.part[item];
        const uint32_t c = item - B.begin[i];
        const PartPair pp = B.pairs[i];
        uint64_t* region = ovf_table + 2ull * pp.r_off;
        const uint64_t H = 2ull * pp.r_len;
        const uint32_t chunk = ovf_chunk(pp.r_len);
        const uint64_t end = min(2ull * (c + 1) * chunk, H);
        for (uint64_t x = 2ull * c * chunk + threadIdx.x; x < end; x += blockDim.x) region[x] = kEmptySlot;
    }
}

struct RegionStep {
    uint32_t H;
    __device__ __forceinline__ uint64_t operator()(uint64_t s) const { return s + 1 == H ? 0 : s + 1; }
};

struct ItemLoc {
    uint32_t item;
    bool live;
    uint32_t r_off, r_len;
    uint32_t s_begin, s_n;
};

// Inserts one build item (ovf_chunk rows of a partition) into its HBM table.
// Every thread of the workgroup calls it.  runs, seen: LDS of a run per wave and
// of WavePush::kSeen bytes for this wave.
template <uint32_t kBlock>
__device__ __forceinline__ void build_item(const OvfBuild& B, uint32_t item, const Tuple* rt, uint64_t* ovf_table,
                                           uint32_t* ovf_next, HotKeys* hot, HeavyQueue* heavy, WavePush::Run* runs,
                                           uint8_t* seen) {
    const uint32_t i = uniform(B.part[item]);
    const uint32_t c = item - uniform(B.begin[i]);
    const PartPair pp{uniform(B.pairs[i].r_off), uniform(B.pairs[i].r_len), 0u, uniform(B.pairs[i].s_len)};
    uint64_t* region = ovf_table + 2ull * pp.r_off;
    uint32_t* next = ovf_next + pp.r_off;
    const RegionStep step{2u * pp.r_len};
    const uint32_t chunk = ovf_chunk(pp.r_len);
    const uint32_t end = min((c + 1) * chunk, pp.r_len);
    // a partition the one-pass write may queue tuples of: the write's helpers
    // wait until its work items are done
    if (heavy && c == 0 && threadIdx.x == 0 && pp.r_len > kQueueRows) {
        atomicAdd(&heavy->items_expected, items_of(pp));
        __hip_atomic_store(&heavy->wait, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    WavePush push;
    push.hot_keys = hot;
    for (uint32_t j0 = c * chunk; j0 < end; j0 += kBlock) {  // uniform trip count
        const uint32_t j = j0 + threadIdx.x;
        int32_t k = 0;
        if (j < end) k = key_of(rt[pp.r_off + j]);
        const uint64_t s = push.claim<2>(region, j < end, k, j, region_slot(k, step.H), step, seen);
        push.add(region, next, s, k, j);
    }
    push.flush_block<kBlock / kWave>(region, next, runs);
}

// The HBM tables in a launch of their own (tables_expected): workgroups of four
// waves, which fill a CU, where the join's LDS leaves it three quarters.  What
// bounds it is the chains of dependent accesses in flight.
constexpr uint32_t kBuildBlock = 256;
__global__ void __launch_bounds__(kBuildBlock) k_ovf_build(OvfBuild B, const Tuple* rt, uint64_t* ovf_table,
                                                          uint32_t* ovf_next, HotKeys* hot, HeavyQueue* heavy) {
    constexpr uint32_t kWaves = kBuildBlock / kWave;
    __shared__ WavePush::Run runs[kWaves];
    __shared__ uint8_t seen[kWaves * WavePush::kSeen];
    const uint32_t nitems = table_items(B);
    for (uint32_t item = blockIdx.x; item < nitems; item += gridDim.x)
        build_item<kBuildBlock>(B, item, rt, ovf_table, ovf_next, hot, heavy, runs,
                                seen + threadIdx.x / kWave * WavePush::kSeen);
}

// The HBM tables of the oversized partitions, built inside the join launch that
// probes them first (where few partitions have one, else by k_ovf_build): a
// workgroup claims build items until none is left and, with `wait`, returns
// only when every item is built.  A workgroup waits when all items are claimed,
// so each is in the hands of a running workgroup that waits for nothing before
// it is done.  Workgroups whose own item needs a table build and wait; of the
// others the first `nitems` build before they turn to their items (every claim
// is an atomic on one word: claims by all workgroups, after their items, took
// the one-pass write of 64K x 16M with a tenth of R on one key from 121 us to
// 226).  A build launch of its own cost every join 6 us, mostly for nothing to
// build.  What bounds a build is its chain of dependent accesses, about 3 us
// per 512 rows; the joins of other partitions run beside it.
// lds: kJoinWaves runs, a word and kJoinWaves * WavePush::kSeen bytes.
__device__ __forceinline__ void build_tables(const OvfBuild& B, const Tuple* rt, uint64_t* ovf_table,
                                             uint32_t* ovf_next, HotKeys* hot, HeavyQueue* heavy, uint32_t nitems,
                                             bool wait, uint32_t* lds) {
    WavePush::Run* runs = reinterpret_cast<WavePush::Run*>(lds);
    uint32_t* s_item = reinterpret_cast<uint32_t*>(runs + kJoinWaves);
    uint8_t* seen = reinterpret_cast<uint8_t*>(s_item + 1) + threadIdx.x / kWave * WavePush::kSeen;
    while (true) {
        if (threadIdx.x == 0) *s_item = atomicAdd(&B.words[1], 1u);
        __syncthreads();
        const uint32_t item = uniform(*s_item);
        if (item >= nitems) break;
        build_item<kJoinBlock>(B, item, rt, ovf_table, ovf_next, hot, heavy, runs, seen);
        await_memory();
        __syncthreads();
        if (threadIdx.x == 0) {  // (every wave's stores have reached this XCD's L2)
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            atomicAdd(&B.words[2], 1u);
        }
        // (and thread 0's branch here stays apart from the next claim's: joined
        // into one, thread 0 would stay behind while its wave went to the barrier)
        __syncthreads();
    }
    if (!wait) return;
    if (threadIdx.x == 0) {
        uint32_t polls = 0;
        while (__hip_atomic_load(&B.words[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < nitems) {
            if (++polls > 8 * kMaxStatusPolls) {  // (cannot happen; the launch ends all the same)
                atomicOr((unsigned long long*)B.err, (unsigned long long)kErrLookback);
                break;
            }
            __builtin_amdgcn_s_sleep(8);
        }
    }
    if (threadIdx.x < kWave) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    __syncthreads();
}

constexpr uint32_t kSU = kSubJ / kWave;  // S tuples per lane of a probe round
// Small work items (up to kJoinBlock R and kFewU kJoinBlock S tuples) have code of
// their own: one round of the build instead of RPT, and their S tuples spread
// over the waves, kFewU groups of 64 each, where kSU groups in the first wave
// left seven idle.  Items of 256 x 256 tuples (1M x 1M, 2^12 partitions): count
// 28.0 to 18.3 us, write 38.0 to 15.4.  Larger items keep full waves: every step
// of a chain reads for all kSU groups of a wave, whether they hold a tuple or not
// (1024 x 1024 spread over the waves: count 31 to 36 us, write 43 to 52).
constexpr uint32_t kFewU = 2;

static_assert(kRptLarge * kJoinBlock == kMaxLdsCap, "largest build covers kMaxLdsCap");

// Strided columns of the heavy-key scans (hj_heavy.h) over partitioned tuples.
typedef Column<2> TupleColumn;
__device__ __forceinline__ TupleColumn key_column(const Tuple* t) {
    return TupleColumn{reinterpret_cast<const int32_t*>(t)};
}
__device__ __forceinline__ TupleColumn rid_column(const Tuple* t) {
    return TupleColumn{reinterpret_cast<const int32_t*>(t) + 1};
}

// R_i's tuples of this thread, 1 <= n <= RPT * kJoinBlock (rows past n: the last).
// Plain loads: every S chunk (work item) of a partition reads R_i again.
template <uint32_t RPT>
__device__ __forceinline__ void load_r(const Tuple* __restrict__ rt, uint32_t n, int32_t* k, int32_t* rid) {
#pragma unroll
    for (uint32_t u = 0; u < RPT; ++u) {
        const Tuple t = rt[min(u * kJoinBlock + threadIdx.x, n - 1)];
        k[u] = key_of(t);
        rid[u] = rid_of(t);
    }
}
// The same from two columns (direct joins).
template <uint32_t RPT>
__device__ __forceinline__ void load_r(const int32_t* __restrict__ rk, const int32_t* __restrict__ rr, uint32_t n,
                                       int32_t* k, int32_t* rid) {
#pragma unroll
    for (uint32_t u = 0; u < RPT; ++u) {
        const uint32_t j = min(u * kJoinBlock + threadIdx.x, n - 1);
        k[u] = rk[j];
        rid[u] = rr[j];
    }
}

// LDS table of a work item: chain heads, one 32-bit record per R_i tuple at its
// row j -- what the bucket does not say of its key, and the link to the next row
// of the bucket's chain -- and its rid (the paper's bucket header, key list and
// rid list of Section 3.1, with row indices in place of pointers).
// A key is told by its radix hash (a bijection of the key).  Its low bits are
// the same in all of a partition; the high 32 - bits are mixed (again a
// bijection), the top log2H mixed bits are the bucket and the others, shifted
// to the top, the record's part: two keys of a bucket are equal exactly when
// those are.  A record's low link_bits are free for the link, as
// bits + log2H >= link_bits (table_shape).
// Layout: heads[H] | rec[cap + 128] | rid[cap + 128] (write); row cap ends every
// chain (its own link is cap), rows cap + 64 .. cap + 127 take what has no row.
// Against 64-bit records (key, link) with the rids read from HBM for matches
// the 16M x 16M one-pass write went from 94 to 91 us.
//
// One bucket per row, or two where three workgroups, as many as the registers
// of the write allow, still share a CU's LDS: shorter chains took 10M x 12M
// tuples, 2 rows to a key, from 71 + 143 to 65 + 130 us (count + write).
constexpr uint32_t kLdsOfThird = 160u * 1024u / 3u - 1536u;
struct TableShape {
    uint32_t log2H, link_bits;
};
__host__ __device__ inline TableShape table_shape(uint32_t cap, uint32_t bits) {
    uint32_t l = 6;  // floor(log2(cap)), cap >= 64
    while ((2u << l) <= cap) ++l;
    const bool twice = bits == 0 || 4u * ((2u << l) + 2u * (cap + 2u * kWave)) <= kLdsOfThird;
    return TableShape{twice ? l + 1 : l, l + 1};  // rows 0 .. cap fit l + 1 bits
}

struct LdsTable {
    uint32_t* heads;
    uint32_t* rec;
    uint32_t* rid;
    uint32_t cap, log2H, link_mask;
    uint32_t keep;  // the radix-hash bits above the partition's
};

// small: a table of up to kJoinBlock rows, with 1024 buckets to clear (or as many
// as leave the links their bits) whatever the capacity.
__device__ __forceinline__ LdsTable lds_table(uint32_t* lds, uint32_t cap, uint32_t bits, bool small = false) {
    TableShape t = table_shape(cap, bits);
    LdsTable v;
    v.heads = lds;
    v.rec = lds + (1u << t.log2H);
    if (small) t.log2H = min(t.log2H, t.link_bits > bits + 10 ? t.link_bits - bits : 10u);
    v.rid = v.rec + cap + 2 * kWave;
    v.cap = cap;
    v.log2H = t.log2H;
    v.link_mask = (1u << t.link_bits) - 1u;
    v.keep = ~0u << bits;  // (bits <= 20)
    return v;
}

// The mixed bits of a key: bucket in the top log2H, then the record's part.
template <uint32_t kHash>
__device__ __forceinline__ uint32_t mixed(const LdsTable& v, int32_t key) {
    uint32_t h = (radix_hash(key, kHash) & v.keep) * 0x9E3779B1u;  // odd factors and a right shift
    h ^= (h >> 15) & v.keep;                                       // within the kept bits: a bijection
    return h * 0x85EBCA6Bu;
}

// Builds the table over the n <= RPT * kJoinBlock tuples held in registers: b1-b2
// bucket of the key, b3-b4 the tuple is pushed on its bucket's chain with one
// LDS exchange (the latch of Section 3.3 is the exchange itself) and its record
// stored at its row.  kGroup rounds at a time (those past n are skipped as a
// whole, n is uniform over the block) without branches between their exchanges:
// a lane past n exchanges on a spare row.
template <uint32_t RPT, uint32_t kHash, bool kRids>
__device__ __forceinline__ void build_lds(const int32_t* k, const int32_t* rid, uint32_t n, const LdsTable& v) {
    constexpr uint32_t kGroup = RPT == 1 ? 1 : RPT % 4 == 0 ? 4 : 3;
    static_assert(RPT % kGroup == 0, "whole groups");
    uint4* heads = reinterpret_cast<uint4*>(v.heads);
    for (uint32_t x = threadIdx.x; x < (1u << v.log2H) / 4; x += kJoinBlock)
        heads[x] = make_uint4(v.cap, v.cap, v.cap, v.cap);
    if (threadIdx.x == 0) v.rec[v.cap] = v.cap;
    __syncthreads();
    const uint32_t sh = 32 - v.log2H;
    const uint32_t spare = v.cap + kWave + lane_id();
#pragma unroll
    for (uint32_t u0 = 0; u0 < RPT; u0 += kGroup) {
        if (u0 * kJoinBlock < n) {
            uint32_t m[kGroup], old[kGroup];
#pragma unroll
            for (uint32_t g = 0; g < kGroup; ++g) {
                const uint32_t j = (u0 + g) * kJoinBlock + threadIdx.x;
                m[g] = mixed<kHash>(v, k[u0 + g]);
                old[g] = atomicExch(j < n ? &v.heads[m[g] >> sh] : &v.rec[spare], j);
            }
#pragma unroll
            for (uint32_t g = 0; g < kGroup; ++g) {
                const uint32_t j = (u0 + g) * kJoinBlock + threadIdx.x;
                const uint32_t at = j < n ? j : spare;
                v.rec[at] = (m[g] << v.log2H) | old[g];
                if (kRids) v.rid[at] = (uint32_t)rid[u0 + g];
            }
        }
    }
    __syncthreads();
}

// The work item of this workgroup, one dependent load (the plan writes the
// records past the last item empty; an item has at least one S tuple).
// Workgroups go to the 8 XCDs round-robin; items are dealt to them in groups
// of kItemGroup consecutive items (the items of one partition share its table
// in the XCD's L2), so each XCD gets every 8th group, evenly however many
// items there are.  A bijection on a grid of a multiple of 8 kItemGroup.
__device__ __forceinline__ uint32_t item_of_block(uint32_t b) {
    const uint32_t x = b % 8, l = b / 8;
    return ((l / kItemGroup) * 8 + x) * kItemGroup + l % kItemGroup;
}

__device__ __forceinline__ ItemLoc locate_item(const ItemRec* __restrict__ item_rec) {
    ItemLoc L;
    L.item = item_of_block(blockIdx.x);
    const ItemRec r = item_rec[L.item];
    L.live = r.s_n != 0;
    L.r_off = r.r_off;
    L.r_len = r.r_len;
    L.s_begin = r.s_begin;
    L.s_n = r.s_n;
    return L;
}

// S keys and rids of this lane for the wave's range of the item from wb on,
// kU groups of 64 of the item's s_n >= 1 tuples.  Lanes past the end load the last tuple again:
// behind a branch each load would be awaited on its own (kNt: non-temporal loads, for large joins; see kNtMinTuples).
template <uint32_t kU, bool kNt>
__device__ __forceinline__ void load_s(const Tuple* __restrict__ st, uint32_t wb, uint32_t s_n, int32_t* q,
                                       int32_t* qr) {
#pragma unroll
    for (uint32_t u = 0; u < kU; ++u) {
        const uint32_t j = wb + u * kWave + lane_id();
        const Tuple* a = st + min(j, s_n - 1);
        const uint64_t t = kNt ? __builtin_nontemporal_load(a) : *a;
        q[u] = key_of(t);
        qr[u] = rid_of(t);
    }
}
// The same from two columns (direct joins).
template <uint32_t kU>
__device__ __forceinline__ void load_s(const int32_t* __restrict__ skp, const int32_t* __restrict__ srp, uint32_t wb,
                                       uint32_t s_n, int32_t* q, int32_t* qr) {
#pragma unroll
    for (uint32_t u = 0; u < kU; ++u) {
        const uint32_t j = wb + u * kWave + lane_id();
        const uint32_t i = min(j, s_n - 1);
        q[u] = skp[i];
        qr[u] = srp[i];
    }
}

// p1-p4 for the lane's kU S keys against the LDS table, without branches per
// key: the chain heads of all keys are read first, then the chains are walked
// in lockstep (each step reads the current record of every key; an ended chain
// stays at row cap), so each step keeps kU LDS reads in flight and a wave runs
// only as many steps as its longest chain.
// cf[u] = matches | first << 16 (16-bit halves: rows < 2^16), first = row of
// the first match met (cap when there is none).  m[u] becomes the record's part
// of the key.
template <uint32_t kU, uint32_t kHash>
__device__ __forceinline__ void probe_lds(const LdsTable& v, const int32_t* q, uint32_t wb, uint32_t we, uint32_t* m,
                                          uint32_t* cf) {
    uint32_t h[kU];
#pragma unroll
    for (uint32_t u = 0; u < kU; ++u) {
        const bool ok = wb + u * kWave + lane_id() < we;
        m[u] = mixed<kHash>(v, q[u]);
        const uint32_t head = v.heads[m[u] >> (32 - v.log2H)];
        h[u] = ok ? head : v.cap;
        m[u] <<= v.log2H;
        cf[u] = v.cap << 16;
    }
    while (true) {
        bool live = false;
#pragma unroll
        for (uint32_t u = 0; u < kU; ++u) live |= h[u] != v.cap;
        if (__ballot(live) == 0) break;
        uint32_t rc[kU];
#pragma unroll
        for (uint32_t u = 0; u < kU; ++u) rc[u] = v.rec[h[u]];
        __builtin_amdgcn_sched_barrier(0);  // keep the step's reads together, in flight at once
#pragma unroll
        for (uint32_t u = 0; u < kU; ++u) {
            const bool hit = (rc[u] ^ m[u]) <= v.link_mask && h[u] != v.cap;
            const uint32_t first = (cf[u] & 0xFFFFu) == 0 ? h[u] << 16 : cf[u];
            cf[u] = hit ? (first & 0xFFFF0000u) | ((cf[u] & 0xFFFFu) + 1u) : cf[u];
            h[u] = rc[u] & v.link_mask;
        }
    }
}

// LDS of a work item whose R partition has an HBM table: the heavy set of a
// probe round and the hot keys the table's build recorded.
struct HbmLds {
    HeavySet hs;
    int32_t hk[kHotKeys];
    uint32_t hr[kHotKeys];
    uint32_t nhk;
};

// Matches of the lane's kSU S keys in the partition-local HBM table (H = 2
// r_len slots).  A key with a chain longer than lim is registered in `hs`
// (c[u] = kHeavyBit | its index) when there is room, else counted by walking;
// a hot key whose recorded rows alone exceed lim is registered without the
// walk.  hs->n must be zero and visible to the block before the call.
__device__ __forceinline__ void probe_hbm(const uint64_t* __restrict__ region, const uint32_t* __restrict__ next,
                                          uint32_t H, uint32_t lim, const int32_t* q, const int32_t* qr, uint32_t wb,
                                          uint32_t we, uint32_t* c, uint32_t* at, HbmLds* sh) {
    const RegionStep step{H};
#pragma unroll
    for (uint32_t u = 0; u < kSU; ++u) {
        c[u] = 0;
        at[u] = kNotFound;
        if (wb + u * kWave + lane_id() < we) {
            at[u] = chain_find<2>(region, region_slot(q[u], H), q[u], step);
            if (at[u] != kNotFound) {
                const uint32_t hot = (at[u] & kLast) ? 0u : hot_rows_of(q[u], sh->hk, sh->hr, sh->nhk);
                c[u] = hot > lim ? register_heavy(next, at[u], q[u], qr ? qr[u] : 0, &sh->hs)
                                 : heavy_or_len(next, at[u], lim, q[u], qr ? qr[u] : 0, &sh->hs);
            }
        }
    }
}

// Rids of a table's rows: in LDS, or in R's column of n >= 1 rows (direct joins whose
// LDS would hold fewer workgroups with them).  Rows without a rid are readable too.
struct LdsRids {
    const uint32_t* rid;
    __device__ __forceinline__ int32_t operator()(uint32_t row) const { return (int32_t)rid[row]; }
};
struct ColumnRids {
    const int32_t* __restrict__ rid;
    uint32_t n;
    __device__ __forceinline__ int32_t operator()(uint32_t row) const { return rid[min(row, n - 1)]; }
};

// Writes the matches after the first of an S tuple (m: the record's part of its
// key, `first` the first match's row) to o_r/o_s[p ...], slots below `room` only.
template <typename Rids>
__device__ __forceinline__ void write_more(const LdsTable& v, Rids rids, uint32_t m, int32_t rs, uint32_t first,
                                           uint32_t p, uint32_t room, int32_t* __restrict__ o_r,
                                           int32_t* __restrict__ o_s) {
    for (uint32_t x = v.rec[first] & v.link_mask; x != v.cap;) {
        const uint32_t r = v.rec[x];
        if ((r ^ m) <= v.link_mask) {
            if (p < room) {
                o_r[p] = rids(x);
                o_s[p] = rs;
            }
            ++p;
        }
        x = r & v.link_mask;
    }
}

// Wave-uniform copy of a 64-bit value held equal in every active lane.
__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Block-wide output reservation for one probe round (the block allocator of
// Section 3.3 with a block sized to the round's pairs): one atomic add of the
// round's total on the running count.  `mine` = this lane's pairs.  Returns the
// first slot of this wave.  `again`: a previous round used `wtot` (uniform over
// the block).
// T: uint32_t for the LDS table (a round has at most kJoinSub x kMaxLdsCap
// pairs), uint64_t for the HBM table (duplicate-heavy R can exceed 2^32).
template <typename T>
__device__ __forceinline__ uint64_t block_reserve(T mine, unsigned long long* total, uint64_t* wtot,
                                                  bool again) {
    const uint32_t w = threadIdx.x / kWave;
    mine = wave_sum(mine);
    if (again) __syncthreads();  // every wave has read the previous round's offsets
    if (lane_id() == 0) wtot[w] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t t = 0;
        for (uint32_t i = 0; i < kJoinWaves; ++i) t += wtot[i];
        wtot[kJoinWaves] = t ? atomicAdd(total, (unsigned long long)t) : 0ull;
    }
    __syncthreads();
    uint64_t pos0 = wtot[kJoinWaves];
    for (uint32_t i = 0; i < w; ++i) pos0 += wtot[i];
    return pos0;
}

template <uint32_t kU>
__device__ __forceinline__ uint32_t lane_pairs_lds(const uint32_t* cf) {
    uint32_t m = 0;
#pragma unroll
    for (uint32_t u = 0; u < kU; ++u) m += cf[u] & 0xFFFFu;
    return m;
}

// Stores the round's pairs of this wave from output slot pos0 on (wave-compacted
// by match counts); returns the slot after the wave's last pair.  LDS table.
// A round of a wave has fewer than 2^32 pairs (kSubJ keys x kMaxLdsCap
// matches), so slots are 32-bit offsets from the wave's uniform base.
template <uint32_t kU, typename Rids>
__device__ __forceinline__ uint64_t write_round_lds(const LdsTable& v, Rids rids, const uint32_t* m, const int32_t* qr,
                                                    const uint32_t* cf, uint64_t pos0, uint64_t capacity,
                                                    int32_t* __restrict__ out_r, int32_t* __restrict__ out_s) {
    pos0 = uniform64(pos0);
    const uint64_t left = capacity > pos0 ? capacity - pos0 : 0ull;
    const uint32_t room = left > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)left;
    int32_t* __restrict__ o_r = out_r + pos0;
    int32_t* __restrict__ o_s = out_s + pos0;
    int32_t rid0[kU];
#pragma unroll
    for (uint32_t u = 0; u < kU; ++u) rid0[u] = rids(cf[u] >> 16);
    uint32_t done = 0;  // pairs of the wave written so far
#pragma unroll
    for (uint32_t u = 0; u < kU; ++u) {
        const uint32_t c = cf[u] & 0xFFFFu;
        uint32_t excl, wtotal;
        wave_offsets32(c, &excl, &wtotal);
        const uint32_t p = done + excl;
        if (c && p < room) {
            o_r[p] = rid0[u];
            o_s[p] = qr[u];
        }
        if (wtotal > kWave || __ballot(c > 1))  // uniform: some key has several matches
            if (c > 1) write_more(v, rids, m[u], qr[u], cf[u] >> 16, p + 1, room, o_r, o_s);
        done += wtotal;
    }
    return pos0 + done;
}

// The same for the partition-local HBM table: c[u] matches on the row chain
// that starts at at[u].
// Heavy entries (is_heavy(c[u])) take their count from hs and only publish
// their first slot in hs->pos; heavy_writes writes them.
__device__ __forceinline__ uint64_t write_round_hbm(const uint32_t* __restrict__ next,
                                                    TupleColumn rrp, const int32_t* qr,
                                                    const uint32_t* c, const uint32_t* at,
                                                    HeavySet* hs, uint64_t pos0, uint64_t capacity,
                                                    int32_t* __restrict__ out_r, int32_t* __restrict__ out_s) {
#pragma unroll
    for (uint32_t u = 0; u < kSU; ++u) {
        const bool heavy = is_heavy(c[u]);
        const uint32_t cu = heavy ? hs->cnt[c[u] & ~kHeavyBit] : c[u];
        uint64_t excl, wtotal;
        wave_offsets(cu, &excl, &wtotal);
        uint64_t pos = pos0 + excl;
        pos0 += wtotal;
        if (heavy) {
            hs->pos[c[u] & ~kHeavyBit] = pos;
        } else if (cu) {
            uint32_t h = at[u];
            while (true) {
                const uint32_t row = h & ~kLast;
                if (pos < capacity) {
                    out_r[pos] = rrp[row];
                    out_s[pos] = qr[u];
                }
                ++pos;
                if (h & kLast) break;
                h = next[row];
            }
        }
    }
    return pos0;
}

// Count pass over a partition whose R exceeds the LDS table: probes the
// partition-local HBM table and returns this lane's pair count.  hs takes the
// LDS the table would have used.
__device__ __forceinline__ uint64_t join_count_hbm(const ItemLoc L, uint32_t w, const Tuple* __restrict__ rt,
                                                   const Tuple* __restrict__ stp,
                                                   const uint64_t* __restrict__ ovf_table,
                                                   const uint32_t* __restrict__ ovf_next, const HotKeys* hot,
                                                   HbmLds* sh) {
    HeavySet* hs = &sh->hs;
    uint64_t cnt = 0;
    int32_t q[kSU], qr[kSU];
    load_hot(hot, sh->hk, sh->hr, &sh->nhk);  // read after the round's barrier
    for (uint32_t sb = 0; sb < L.s_n; sb += kJoinSub) {
        const uint32_t wb = sb + w * kSubJ, we = min(wb + kSubJ, L.s_n);
        load_s<kSU, false>(stp, wb, L.s_n, q, qr);
        if (threadIdx.x == 0) hs->n = 0;
        __syncthreads();
        uint32_t c[kSU], at[kSU];
        probe_hbm(ovf_table + 2ull * L.r_off, ovf_next + L.r_off, 2u * L.r_len, heavy_limit(L.r_len), q, nullptr, wb,
                  we, c, at, sh);
        heavy_counts<kJoinBlock, kHeavyV>(key_column(rt + L.r_off), L.r_len, hs);
#pragma unroll
        for (uint32_t u = 0; u < kSU; ++u) cnt += is_heavy(c[u]) ? hs->cnt[c[u] & ~kHeavyBit] : c[u];
        __syncthreads();  // the set is reused by the next round
    }
    return cnt;
}

// S tuples per wave of a small item: whole groups of 64.
__device__ __forceinline__ uint32_t small_share(uint32_t s_n) { return (s_n + kJoinBlock - 1) / kJoinBlock * kWave; }

__device__ __forceinline__ bool small_item(const ItemLoc& L) {
    return L.r_len <= kJoinBlock && L.s_n <= kFewU * kJoinBlock;
}

template <uint32_t RPT, bool kNt, uint32_t kHash>
__global__ void __launch_bounds__(kJoinBlock) __attribute__((amdgpu_waves_per_eu(6)))
k_join_count(const ItemRec* __restrict__ item_rec, const Tuple* __restrict__ rt, const Tuple* __restrict__ st,
             uint32_t lds_cap, uint32_t bits, uint64_t* ovf_table, uint32_t* ovf_next, HotKeys* hot,
             uint64_t* __restrict__ wave_cnt, OvfBuild B) {
    extern __shared__ uint32_t lds[];
    const uint32_t w = threadIdx.x / kWave;
    const uint32_t lane = lane_id();
    const ItemLoc L = locate_item(item_rec);
    const uint32_t novf = table_items(B);  // uniform
    const Tuple* __restrict__ stp = st + L.s_begin;
    const bool mine = novf && L.live && L.r_len > lds_cap;  // uniform
    if (B.words && (mine || blockIdx.x < novf)) {
        build_tables(B, rt, ovf_table, ovf_next, hot, nullptr, novf, mine, lds);
        __syncthreads();
    }
    uint64_t cnt = 0;
    if (L.live && L.r_len <= lds_cap) {
        auto run = [&](auto rounds, auto groups) {
            constexpr uint32_t kR = decltype(rounds)::value, kU = decltype(groups)::value;
            int32_t q[kU], qr[kU], k[kR], rid[kR];
            const uint32_t n = kR == 1 ? small_share(L.s_n) : kSubJ;  // per wave
            load_r<kR>(rt + L.r_off, L.r_len, k, rid);
            load_s<kU, kNt>(stp, w * n, L.s_n, q, qr);
            const LdsTable v = lds_table(lds, lds_cap, bits, kR == 1);
            build_lds<kR, kHash, false>(k, rid, L.r_len, v);
            for (uint32_t sb = 0; sb < L.s_n; sb += kJoinSub) {
                const uint32_t wb = sb + w * n, we = min(wb + n, L.s_n);
                if (sb) load_s<kU, kNt>(stp, wb, L.s_n, q, qr);
                uint32_t m[kU], cf[kU];
                probe_lds<kU, kHash>(v, q, wb, we, m, cf);
                cnt += lane_pairs_lds<kU>(cf);
            }
        };
        if (small_item(L)) run(std::integral_constant<uint32_t, 1>(), std::integral_constant<uint32_t, kFewU>());
        else run(std::integral_constant<uint32_t, RPT>(), std::integral_constant<uint32_t, kSU>());
        cnt = wave_sum(cnt);
    }
    if (mine)
        cnt = wave_sum(join_count_hbm(L, w, rt, stp, ovf_table, ovf_next, hot, reinterpret_cast<HbmLds*>(lds)));
    if (lane == 0) wave_cnt[(uint64_t)L.item * kJoinWaves + w] = cnt;
}

// Write pass over a partition whose R exceeds the LDS table (see
// join_count_hbm).  One-pass output with `heavy`: a heavy S tuple of a
// partition of more than kQueueRows rows is registered after
// a walk of at most kQueueWalk rows (none for a recorded hot key) and handed
// to the device-wide queue, whose chunks every workgroup of the launch helps
// write (help_heavy); tuples the queue has no room for stay with this
// workgroup's own scans.
template <bool kOnePass>
__device__ __forceinline__ void join_write_hbm(
    const ItemLoc L, uint32_t w, const Tuple* __restrict__ rt, const Tuple* __restrict__ stp,
    const uint64_t* __restrict__ ovf_table,
    const uint32_t* __restrict__ ovf_next, const HotKeys* hot, uint64_t base, unsigned long long* __restrict__ total,
    uint64_t* wtot, int32_t* __restrict__ out_r, int32_t* __restrict__ out_s, uint64_t capacity, HbmLds* sh,
    HeavyQueue* heavy) {
    HeavySet* hs = &sh->hs;
    const uint64_t* __restrict__ region = ovf_table + 2ull * L.r_off;
    const uint32_t* __restrict__ next = ovf_next + L.r_off;
    const TupleColumn rkp = key_column(rt + L.r_off), rrp = rid_column(rt + L.r_off);
    const bool queue = kOnePass && heavy && L.r_len > kQueueRows;  // uniform
    const uint32_t lim = queue ? min(heavy_limit(L.r_len), kQueueWalk) : heavy_limit(L.r_len);
    int32_t q[kSU], qr[kSU];
    load_hot(hot, sh->hk, sh->hr, &sh->nhk);  // read after the round's barrier
    for (uint32_t sb = 0; sb < L.s_n; sb += kJoinSub) {
        const uint32_t wb = sb + w * kSubJ, we = min(wb + kSubJ, L.s_n);
        load_s<kSU, false>(stp, wb, L.s_n, q, qr);
        if (threadIdx.x == 0) hs->n = hs->queued = 0;
        __syncthreads();
        uint32_t c[kSU], at[kSU];
        probe_hbm(region, next, 2u * L.r_len, lim, q, qr, wb, we, c, at, sh);
        if (queue) hand_off(heavy, hs, L.r_off, L.r_len);
        heavy_counts<kJoinBlock, kHeavyV, kOnePass>(rkp, L.r_len, hs);
        uint64_t mine = 0;
#pragma unroll
        for (uint32_t u = 0; u < kSU; ++u) mine += is_heavy(c[u]) ? hs->cnt[c[u] & ~kHeavyBit] : c[u];
        const uint64_t pos0 = kOnePass ? block_reserve(mine, total, wtot, sb != 0) : base;
        base = write_round_hbm(next, rrp, qr, c, at, hs, pos0, capacity, out_r, out_s);
        heavy_writes<kJoinBlock, kHeavyV>(rkp, rrp, L.r_len, hs, capacity, out_r, out_s);
        __syncthreads();  // the set is reused by the next round
    }
}

// Polls of the item count by a helper workgroup before it leaves anyway (its
// help is only a speed-up: every queued chunk is also taken by the workgroup
// that queued it).
constexpr uint32_t kHelpWaitPolls = 1u << 20;
constexpr uint32_t kMaxHelpers = 256;

// A helper's loop: help with the queued tuples until the items the build
// counted are done.
__device__ __forceinline__ void help_until_done(HeavyQueue* heavy, const Tuple* rt,
                                                         unsigned long long* total, uint64_t capacity, int32_t* out_r,
                                                         int32_t* out_s, uint32_t* lds, uint32_t* s_word) {
    const uint32_t expected =
        uniform(__hip_atomic_load(&heavy->items_expected, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    for (uint32_t polls = 0;; ++polls) {
        __syncthreads();
        if (threadIdx.x == 0)
            *s_word = __hip_atomic_load(&heavy->items_done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        const bool all_done = uniform(*s_word) >= expected;
        help_heavy<kJoinBlock, kHelpChunkPart>(heavy, key_column(rt), rid_column(rt), total, capacity, out_r, out_s,
                                               lds);
        if (all_done || polls >= kHelpWaitPolls) break;
        __builtin_amdgcn_s_sleep(32);
    }
}

struct WriteArgs {
    const Tuple *rt, *st;
    uint32_t lds_cap;
    uint64_t* ovf_table;
    uint32_t* ovf_next;
    HotKeys* hot;
    const uint64_t* wave_base;
    unsigned long long* total;
    int32_t *out_r, *out_s;
    uint64_t capacity;
    HeavyQueue* heavy;
    uint32_t item_grid;
};
// The part of a write workgroup that HBM tables need (novf != 0): its item if
// that has such a table and, one-pass, help with the heavy tuples any workgroup
// queued.  Helpers (`helper`, one-pass) are workgroups past the items: when a
// partition may queue tuples (heavy->wait, set by the build), the items of such
// partitions count themselves done and the helpers keep helping until all of
// them are (the build counted them in items_expected), so that a tuple queued
// late still finds helpers.  (Counting every item instead cost the write
// ~0.26 ms at 16M x 16M: thousands of atomics on the queue's line, which every
// workgroup also reads.)  The helpers are at most half of the workgroups the
// device holds at once, so items always have room to run, whatever order the
// workgroups start in.
template <bool kOnePass>
__device__ __forceinline__ void write_hbm_part(const ItemLoc& L, bool helper, const WriteArgs& A, uint32_t* lds,
                                               uint64_t* wtot, uint32_t* s_word) {
    const bool mine = !helper && L.live && L.r_len > A.lds_cap;  // uniform
    if (kOnePass && helper) {
        if (uniform(__hip_atomic_load(&A.heavy->wait, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)))  // (final by now)
            help_until_done(A.heavy, A.rt, A.total, A.capacity, A.out_r, A.out_s, lds, s_word);
        return;
    }
    if (mine) {
        const uint32_t w = threadIdx.x / kWave;
        join_write_hbm<kOnePass>(L, w, A.rt, A.st + L.s_begin, A.ovf_table, A.ovf_next, A.hot,
                                 kOnePass ? 0ull : A.wave_base[(uint64_t)L.item * kJoinWaves + w], A.total, wtot,
                                 A.out_r, A.out_s, A.capacity, reinterpret_cast<HbmLds*>(lds), A.heavy);
    }
    if (kOnePass && A.heavy) {
        if (mine && L.r_len > kQueueRows) {  // an item the helpers wait for (the build counted it)
            __syncthreads();  // the item's hand-offs are made
            if (threadIdx.x == 0) atomicAdd(&A.heavy->items_done, 1u);
        }
        help_heavy<kJoinBlock, kHelpChunkPart>(A.heavy, key_column(A.rt), rid_column(A.rt), A.total, A.capacity,
                                               A.out_r, A.out_s, lds);
    }
}

// Write pass.  kOnePass: instead of reading a scanned per-wave offset, each
// probe round reserves its pairs' output slots with block_reserve.
template <bool kOnePass, uint32_t RPT, bool kNt, uint32_t kHash>
__global__ void __launch_bounds__(kJoinBlock) __attribute__((amdgpu_waves_per_eu(RPT > kRptMid ? 4 : 6)))
k_join_write(const ItemRec* __restrict__ item_rec, uint32_t bits, WriteArgs A, OvfBuild B) {
    extern __shared__ uint32_t lds[];
    __shared__ uint64_t wtot[kJoinWaves + 1];
    __shared__ uint32_t s_word;
    const uint32_t w = threadIdx.x / kWave;
    const uint32_t novf = table_items(B);  // uniform
    const bool helper = kOnePass && blockIdx.x >= A.item_grid;
    if (helper && !novf) return;
    ItemLoc L{};
    if (!helper) {
        L = locate_item(item_rec);
    }
    if (kOnePass && novf && B.words) {
        const bool wait = helper || (L.live && L.r_len > A.lds_cap);  // uniform
        if (wait || blockIdx.x < novf) {
            build_tables(B, A.rt, A.ovf_table, A.ovf_next, A.hot, A.heavy, novf, wait, lds);
            __syncthreads();
        }
    }
    if (!helper) {
        if (L.live && L.r_len <= A.lds_cap) {
            const Tuple* __restrict__ stp = A.st + L.s_begin;
            uint64_t base = kOnePass ? 0ull : A.wave_base[(uint64_t)L.item * kJoinWaves + w];
            auto run = [&](auto rounds, auto groups) {
                constexpr uint32_t kR = decltype(rounds)::value, kU = decltype(groups)::value;
                int32_t q[kU], qr[kU], k[kR], rid[kR];
                const uint32_t n = kR == 1 ? small_share(L.s_n) : kSubJ;  // per wave
                load_r<kR>(A.rt + L.r_off, L.r_len, k, rid);
                load_s<kU, kNt>(stp, w * n, L.s_n, q, qr);
                const LdsTable v = lds_table(lds, A.lds_cap, bits, kR == 1);
                build_lds<kR, kHash, true>(k, rid, L.r_len, v);
                for (uint32_t sb = 0; sb < L.s_n; sb += kJoinSub) {
                    const uint32_t wb = sb + w * n, we = min(wb + n, L.s_n);
                    if (sb) load_s<kU, kNt>(stp, wb, L.s_n, q, qr);
                    uint32_t m[kU], cf[kU];
                    probe_lds<kU, kHash>(v, q, wb, we, m, cf);
                    const uint64_t pos0 = kOnePass ? block_reserve(lane_pairs_lds<kU>(cf), A.total, wtot, sb != 0) : base;
                    base = write_round_lds<kU>(v, LdsRids{v.rid}, m, qr, cf, pos0, A.capacity, A.out_r, A.out_s);
                }
            };
            if (small_item(L)) run(std::integral_constant<uint32_t, 1>(), std::integral_constant<uint32_t, kFewU>());
            else run(std::integral_constant<uint32_t, RPT>(), std::integral_constant<uint32_t, kSU>());
        }
    }
    if (novf) {
        __syncthreads();  // the table is free
        write_hbm_part<kOnePass>(L, helper, A, lds, wtot, &s_word);
    }
}

// Joins whose whole R fits one LDS table, several jobs per launch: one
// workgroup per (job, chunk of S tuples) builds the table over
// the job's R and writes the chunk's pairs to the job's output with one-pass
// reservation.
// kOne: the only job is `one`; a grid of one workgroup clears its count and
// err_clear.  kRids: rids in LDS (direct_rids_in_lds).
template <uint32_t RPT, bool kOne, bool kRids>
__global__ void __launch_bounds__(kJoinBlock) __attribute__((amdgpu_waves_per_eu(RPT > kRptMid ? 4 : 6)))
k_direct_join(const DirectJob* __restrict__ jobs, const uint32_t* __restrict__ item_job, DirectJob one,
              uint64_t* err_clear, uint32_t lds_cap) {
    extern __shared__ uint32_t lds[];
    __shared__ uint64_t wtot[kJoinWaves + 1];
    const uint32_t w = threadIdx.x / kWave;
    const uint32_t item = xcd_remap(blockIdx.x, gridDim.x);
    const DirectJob J = kOne ? one : jobs[item_job[item]];
    if (kOne && gridDim.x == 1 && threadIdx.x == 0) {  // (the thread that reserves later)
        *J.count = 0;
        if (err_clear) *err_clear = 0;
    }
    const uint32_t s_begin = (item - J.item0) * J.chunk;
    const uint32_t s_n = min(J.chunk, J.n_s - s_begin);
    const uint32_t r_len = min(J.n_r, lds_cap);  // the planner guarantees n_r <= lds_cap
    const int32_t* __restrict__ skp = J.sk + s_begin;
    const int32_t* __restrict__ srp = J.sr + s_begin;
    int32_t k[RPT], rid[RPT];
    load_r<RPT>(J.rk, J.rr, r_len, k, rid);
    int32_t q[kSU], qr[kSU];
    load_s<kSU>(skp, srp, w * kSubJ, s_n, q, qr);
    const LdsTable v = lds_table(lds, lds_cap, 0u);
    build_lds<RPT, 0, kRids>(k, rid, r_len, v);
    for (uint32_t sb = 0; sb < s_n; sb += kJoinSub) {
        const uint32_t wb = sb + w * kSubJ, we = min(wb + kSubJ, s_n);
        if (sb) load_s<kSU>(skp, srp, wb, s_n, q, qr);
        uint32_t m[kSU], cf[kSU];
        probe_lds<kSU, 0>(v, q, wb, we, m, cf);
        const uint64_t pos0 = block_reserve(lane_pairs_lds<kSU>(cf), (unsigned long long*)J.count, wtot, sb != 0);
        if (kRids) write_round_lds<kSU>(v, LdsRids{v.rid}, m, qr, cf, pos0, J.capacity, J.out_r, J.out_s);
        else write_round_lds<kSU>(v, ColumnRids{J.rr, r_len}, m, qr, cf, pos0, J.capacity, J.out_r, J.out_s);
    }
}

__global__ void k_direct_zero(const DirectJob* __restrict__ jobs, uint32_t njobs) {
    for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < njobs; j += gridDim.x * blockDim.x)
        *jobs[j].count = 0;
}

__global__ void k_write_zero(uint64_t* p, uint64_t* err_clear) {
    if (threadIdx.x == 0) {
        *p = 0;
        if (err_clear) *err_clear = 0;
    }
}

}  // namespace

size_t join_lds_bytes(uint32_t lds_cap, uint32_t bits, bool write) {
    static_assert(sizeof(HbmLds) <= sizeof(uint32_t) * (256 + 256 + 2 * kWave),
                  "the heavy-key set and the hot keys fit the smallest table area");
    const size_t rows = (size_t)lds_cap + 2 * kWave;
    return sizeof(uint32_t) * (((size_t)1 << table_shape(lds_cap, bits).log2H) + (write ? 2 : 1) * rows);
}

void direct_zero(const DirectJob* jobs, uint32_t njobs, Recorder& rec) {
    if (njobs == 0) return;
    rec.before("direct_zero");
    hipLaunchKernelGGL(k_direct_zero, dim3((njobs + 255) / 256), dim3(256), 0, rec.stream, jobs, njobs);
    rec.after();
}

static void allow_lds(const void* fn, size_t lds) {
    if (lds > 65536) (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

namespace {

// Workgroups of a direct join that a CU holds: by LDS, and by the waves the
// register budget allows.
uint32_t direct_blocks(uint32_t lds_cap, bool rids) {
    const uint32_t by_lds = (uint32_t)(160u * 1024u / (join_lds_bytes(lds_cap, 0, rids) + 512u));
    const uint32_t by_waves = (join_rpt(lds_cap) > kRptMid ? 4u : 6u) * 4u / kJoinWaves;
    return std::max(1u, std::min(by_lds, by_waves));
}

// Rids in LDS unless the device holds more of the items at once without them, whose
// matches then read R's column: with the two buckets per row that a direct table
// needs (its links have no partition's bits to use), rids leave a CU one workgroup
// instead of two from 6016 rows on, two instead of three at 4096 to 4608.  6500 x
// 16M: 123 us with rids in LDS, 87.5 without; 4608 x 2M (455 items) 18.0 and 18.7.
bool direct_rids_in_lds(uint32_t lds_cap, uint32_t nitems) {
    if (nitems <= 256) return true;
    const uint32_t with = direct_blocks(lds_cap, true);
    return nitems <= 256 * with || with == direct_blocks(lds_cap, false);
}

template <uint32_t RPT, bool kOne, bool kRids>
void direct_join_t(const DirectJob* jobs, const uint32_t* item_job, const DirectJob& one, uint32_t nitems,
                   uint32_t lds_cap, Recorder& rec) {
    const size_t lds = join_lds_bytes(lds_cap, 0, kRids);
    allow_lds((const void*)k_direct_join<RPT, kOne, kRids>, lds);
    rec.before("direct_join");
    hipLaunchKernelGGL((k_direct_join<RPT, kOne, kRids>), dim3(nitems), dim3(kJoinBlock), lds, rec.stream, jobs,
                       item_job, one, rec.err_clear, lds_cap);
    rec.after();
}

template <bool kOne>
void direct_join_rpt(const DirectJob* jobs, const uint32_t* item_job, const DirectJob& one, uint32_t nitems,
                     uint32_t lds_cap, Recorder& rec) {
    const bool rids = direct_rids_in_lds(lds_cap, nitems);
    switch (join_rpt(lds_cap)) {
        case kRptSmall: direct_join_t<kRptSmall, kOne, true>(jobs, item_job, one, nitems, lds_cap, rec); break;
        case kRptMid:
            if (rids) direct_join_t<kRptMid, kOne, true>(jobs, item_job, one, nitems, lds_cap, rec);
            else direct_join_t<kRptMid, kOne, false>(jobs, item_job, one, nitems, lds_cap, rec);
            break;
        default:
            if (rids) direct_join_t<kRptLarge, kOne, true>(jobs, item_job, one, nitems, lds_cap, rec);
            else direct_join_t<kRptLarge, kOne, false>(jobs, item_job, one, nitems, lds_cap, rec);
            break;
    }
}

}  // namespace

uint32_t direct_chunk(uint64_t n_s, uint32_t lds_cap) {
    if (n_s <= 256ull * kJoinSub) return kJoinSub;
    const uint64_t slots = 256ull * std::max(direct_blocks(lds_cap, true), direct_blocks(lds_cap, false));
    return n_s <= slots * kJoinSub ? kJoinSub : kJoinChunk;
}

void direct_join(const DirectJob* jobs, const uint32_t* item_job, uint32_t nitems, uint32_t lds_cap,
                 Recorder& rec) {
    if (nitems == 0) return;
    direct_join_rpt<false>(jobs, item_job, DirectJob{}, nitems, lds_cap, rec);
}

void direct_join_one(const DirectJob& j, uint32_t lds_cap, Recorder& rec) {
    const uint32_t nitems = (j.n_s + j.chunk - 1) / j.chunk;
    if (nitems > 1) write_zero_count(j.count, rec);
    direct_join_rpt<true>(nullptr, nullptr, j, nitems, lds_cap, rec);
}

void write_zero_count(uint64_t* d_count, Recorder& rec) {
    rec.before("zero_count");
    hipLaunchKernelGGL(k_write_zero, dim3(1), dim3(64), 0, rec.stream, d_count, rec.err_clear);
    rec.after();
}

// (an upper bound: the plan runs in workgroups of at least kMinPartBlock threads)
size_t plan_state_words(uint32_t P) { return 1 + plan_blocks(P, kMinPartBlock); }

uint32_t ovf_grid(uint32_t P, uint64_t n_r) {
    return (uint32_t)(P + (n_r + kOvfChunk - 1) / kOvfChunk);  // the smaller chunk bounds both
}

uint32_t join_grid(uint32_t P, uint64_t n_s) {
    const uint64_t items = P + (n_s + kJoinChunk - 1) / kJoinChunk;
    return (uint32_t)((items + 8 * kItemGroup - 1) / (8 * kItemGroup) * (8 * kItemGroup));  // item_of_block
}

void join_ovf_clear(const OvfBuild& b, uint32_t grid, uint64_t* ovf_table, Recorder& rec) {
    if (grid == 0) return;
    grid = grid < kOvfGrid ? grid : kOvfGrid;  // grid-stride: few chunks in the common case
    rec.before("ovf_clear");
    hipLaunchKernelGGL(k_ovf_clear, dim3(grid), dim3(256), 0, rec.stream, b, ovf_table);
    rec.after();
}

void join_ovf_build(const OvfBuild& b, uint32_t grid, const Tuple* rt, uint64_t* ovf_table, uint32_t* ovf_next,
                    HotKeys* hot, HeavyQueue* heavy, Recorder& rec) {
    if (grid == 0) return;
    grid = grid < kOvfGrid ? grid : kOvfGrid;
    rec.before("ovf_build");
    hipLaunchKernelGGL(k_ovf_build, dim3(grid), dim3(kBuildBlock), 0, rec.stream, b, rt, ovf_table, ovf_next, hot,
                       heavy);
    rec.after();
}

namespace {

struct JoinArgs {
    const ItemRec* item_rec;
    uint32_t grid;
    const Tuple *rt, *st;
    uint32_t lds_cap, bits;
    OvfBuild ovf;
    uint64_t* ovf_table;
    uint32_t* ovf_next;
    HotKeys* hot;
    uint64_t* wave;   // per-wave counts (count), or their scan (write; nullptr: one-pass)
    uint64_t* total;
    int32_t *out_r, *out_s;
    uint64_t capacity;
    HeavyQueue* heavy;
};

template <uint32_t RPT, bool kNt, uint32_t kHash>
void join_count_t(const JoinArgs& a, Recorder& rec) {
    const size_t lds = join_lds_bytes(a.lds_cap, a.bits, false);
    allow_lds((const void*)k_join_count<RPT, kNt, kHash>, lds);
    rec.before("join_count");
    hipLaunchKernelGGL((k_join_count<RPT, kNt, kHash>), dim3(a.grid), dim3(kJoinBlock), lds, rec.stream, a.item_rec, a.rt,
                       a.st, a.lds_cap, a.bits, a.ovf_table, a.ovf_next, a.hot, a.wave, a.ovf);
    rec.after();
}

template <bool kOnePass, uint32_t RPT, bool kNt, uint32_t kHash>
void join_write_t(const JoinArgs& a, Recorder& rec) {
    const size_t lds = join_lds_bytes(a.lds_cap, a.bits, true);
    allow_lds((const void*)k_join_write<kOnePass, RPT, kNt, kHash>, lds);
    rec.before(kOnePass ? "join_write_1pass" : "join_write");
    uint32_t grid = a.grid;
    if (kOnePass && a.heavy) {
        // helpers: at most half the workgroups resident at once (by LDS and by
        // the waves the register budget allows: 6 per SIMD, 4 for the large build)
        const uint32_t by_lds = (uint32_t)(160u * 1024u / (lds + 1024u));  // lds: this launch's dynamic bytes
        const uint32_t by_waves = (RPT > kRptMid ? 4u : 6u) * 4u / kJoinWaves;
        const uint32_t resident = 256u * std::max(1u, std::min(by_lds, by_waves));
        grid += std::max(1u, std::min(kMaxHelpers, resident / 2));
    }
    const WriteArgs args{a.rt, a.st, a.lds_cap, a.ovf_table, a.ovf_next, a.hot, a.wave, (unsigned long long*)a.total,
                         a.out_r, a.out_s, a.capacity, a.heavy, a.grid};
    hipLaunchKernelGGL((k_join_write<kOnePass, RPT, kNt, kHash>), dim3(grid), dim3(kJoinBlock), lds, rec.stream,
                       a.item_rec, a.bits, args, a.ovf);
    rec.after();
}

template <bool kNt, uint32_t kHash>
void join_count_n(const JoinArgs& a, Recorder& rec) {
    switch (join_rpt(a.lds_cap)) {
        case kRptSmall: join_count_t<kRptSmall, kNt, kHash>(a, rec); break;
        case kRptMid: join_count_t<kRptMid, kNt, kHash>(a, rec); break;
        default: join_count_t<kRptLarge, kNt, kHash>(a, rec); break;
    }
}

template <bool kOnePass, bool kNt, uint32_t kHash>
void join_write_n(const JoinArgs& a, Recorder& rec) {
    switch (join_rpt(a.lds_cap)) {
        case kRptSmall: join_write_t<kOnePass, kRptSmall, kNt, kHash>(a, rec); break;
        case kRptMid: join_write_t<kOnePass, kRptMid, kNt, kHash>(a, rec); break;
        default: join_write_t<kOnePass, kRptLarge, kNt, kHash>(a, rec); break;
    }
}

template <bool kOnePass, bool kNt>
void join_write_h(const JoinArgs& a, uint32_t hash, Recorder& rec) {
    if (hash) join_write_n<kOnePass, kNt, 1>(a, rec);
    else join_write_n<kOnePass, kNt, 0>(a, rec);
}

}  // namespace

void join_count(const ItemRec* item_rec, uint32_t grid, const Tuple* rt, const Tuple* st, uint32_t lds_cap,
                uint32_t bits, uint32_t hash, const OvfBuild& ovf, uint64_t* ovf_table, uint32_t* ovf_next, HotKeys* hot,
                uint64_t* wave_cnt, bool nt_s, Recorder& rec) {
    if (grid == 0) return;
    const JoinArgs a{item_rec, grid, rt, st, lds_cap, bits, ovf, ovf_table, ovf_next, hot, wave_cnt, nullptr, nullptr,
                     nullptr, 0, nullptr};
    if (nt_s && hash) join_count_n<true, 1>(a, rec);
    else if (nt_s) join_count_n<true, 0>(a, rec);
    else if (hash) join_count_n<false, 1>(a, rec);
    else join_count_n<false, 0>(a, rec);
}

void join_write(const ItemRec* item_rec, uint32_t grid, const Tuple* rt, const Tuple* st, uint32_t lds_cap,
                uint32_t bits, uint32_t hash, const OvfBuild& ovf, uint64_t* ovf_table, uint32_t* ovf_next, HotKeys* hot,
                const uint64_t* wave_base, uint64_t* total, int32_t* out_r, int32_t* out_s, uint64_t capacity,
                HeavyQueue* heavy, bool nt_s, Recorder& rec) {
    if (grid == 0) return;
    const JoinArgs a{item_rec, grid, rt, st, lds_cap, bits, ovf, ovf_table, ovf_next, hot,
                     const_cast<uint64_t*>(wave_base), total, out_r, out_s, capacity, wave_base ? nullptr : heavy};
    if (wave_base) {
        if (nt_s) join_write_h<false, true>(a, hash, rec);
        else join_write_h<false, false>(a, hash, rec);
    } else {
        if (nt_s) join_write_h<true, true>(a, hash, rec);
        else join_write_h<true, false>(a, hash, rec);
    }
}

}  // namespace hj
