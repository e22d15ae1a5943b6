// Radix partitioning for the partitioned hash join (Algorithm 2, "Partition",
// steps n1-n3; Section 3.1: passes on the low bits of the integer hash value).
//
// Launches of a partitioning (R and S together, tiles of R first):
//   hist     n1: partition number of every tuple, counted in LDS over all tiles
//            of a persistent workgroup (at low fan-out the tuples of one wave
//            that share a partition are grouped with one ballot per radix bit)
//            and written as the workgroup's row of counts.
//   starts   sums of the rows, and their exclusive scan: partition starts and,
//            for each replica (one per XCD), a cursor at its part of every
//            partition.  Small joins skip it (self_starts).
//   scatter  n2-n3: a tile is read, every tuple gets its rank inside its
//            partition (value returned by its LDS atomic, or leader atomic +
//            popcount of lower group lanes at low fan-out), the tile reserves its
//            run of every partition with one atomic on its replica's cursor, is
//            reordered by partition in LDS and written out run by run as 64-bit
//            tuples.  The order of tiles inside a partition is that of their
//            reservations; no consumer depends on it.
// Two passes of up to kFuseBits bits in all run as one such scatter.  With more
// bits pass 2 splits every pass-1 partition of R and of S (a segment) again,
// by the same scatter with cursors per segment; the final partitions are
// counted by the one histogram up to 15 bits, above by a histogram of pass 2.
// The paper's partition "buckets" with dynamically allocated storage
// (Section 3.1, Section 3.3) become contiguous partitions at counted offsets.
#include <algorithm>

#include "hj_device.h"
#include "hj_internal.h"
#include "hj_side.h"

namespace hj {

namespace {

// Up to this many radix bits (8 partitions) the lanes of a wave that share a
// partition are grouped with ballots and one leader atomic per group: at such
// low fan-out most lanes of a wave hit the same few LDS counters.  Above it,
// one LDS atomic per tuple is faster on gfx950 (measured at 64 partitions:
// histogram 2x, scatter 1.2x).
constexpr uint32_t kBallotMaxBits = 3;

struct TileLoc {
    uint32_t seg, start, len;  // segment, first tuple (position in the copy), tuples
};

// tile_seg: the segment of every tile, written by the pass's setup.
__device__ __forceinline__ TileLoc locate(const PartSeg* __restrict__ segs, const uint32_t* __restrict__ tile_begin,
                                          const uint32_t* __restrict__ tile_seg, uint32_t tile, uint32_t T) {
    TileLoc t;
    t.seg = tile_seg[tile];
    const PartSeg g = segs[t.seg];
    const uint32_t off = (tile - tile_begin[t.seg]) * T;
    t.start = g.base + off;
    t.len = min(T, g.n - off);
    return t;
}

// kHash: the radix hash (hj_hash), a template argument of the kernels: a branch
// per tuple would part the LDS accesses of a tile, which then wait one by one.
template <uint32_t kHash>
__device__ __forceinline__ uint32_t part_of(int32_t key, uint32_t shift, uint32_t P) {
    return (radix_hash(key, kHash) >> shift) & (P - 1u);
}

// Lanes of this wave whose `p` equals this lane's (only lanes with `valid`).
__device__ __forceinline__ uint64_t match_mask(uint32_t p, uint32_t bits, bool valid) {
    uint64_t m = __ballot(valid);
    for (uint32_t b = 0; b < bits; ++b) {
        const bool bit = (p >> b) & 1u;
        const uint64_t bal = __ballot(bit);
        m &= bit ? bal : ~bal;
    }
    return valid ? m : 0ull;
}

// A tile of len <= BLOCK * IPT elements from p on (4-byte aligned, all that the
// hardware asks of a 16-byte global load, so a key and a rid column may start
// at different offsets of a line): thread t, slot 4 k + e is element
// 4 (t + k BLOCK) + e of the len / 4 whole chunks, loaded 16 bytes at a time;
// the up to 3 elements after them are slot IPT of threads 0..2.  Nothing outside
// the tile is read, and no load is behind a branch (a thread without a chunk
// loads the last one again): behind branches every load was awaited on its own.
// Pointers into device memory taken from tables in memory are generic; read
// through the global address space the loads are global loads, which unlike
// generic (flat) ones are not counted against LDS accesses (a wait for LDS
// would otherwise also wait for the tile's loads).  kStream: the vector loads
// are marked non-temporal (PassCfg::nt, large joins: each launch reads its
// input once).
typedef __attribute__((address_space(1))) const int32_t gint32;
typedef int32_t i32x4 __attribute__((ext_vector_type(4), aligned(4)));
typedef __attribute__((address_space(1))) const i32x4 gi32x4;
typedef __attribute__((address_space(1))) const uint64_t gtuple;

// any: 16 readable bytes, loaded where a tile has no whole chunk.
template <uint32_t BLOCK, uint32_t IPT, bool kStream>
__device__ __forceinline__ void load_tile(const int32_t* pg, uint32_t len, const void* any, int32_t* v, int32_t& x) {
    static_assert(IPT % 4 == 0, "vector tile slots");
    const uint32_t chunks = len / 4;
    gint32* p = (gint32*)pg;
    gint32* c = chunks ? p : (gint32*)any;
    const uint32_t last = chunks ? chunks - 1 : 0u;
#pragma unroll
    for (uint32_t k = 0; k < IPT / 4; ++k) {
        gi32x4* a = reinterpret_cast<gi32x4*>(c + 4 * min(threadIdx.x + k * BLOCK, last));
        const i32x4 w = kStream ? __builtin_nontemporal_load(a) : *a;
        v[4 * k] = w.x;
        v[4 * k + 1] = w.y;
        v[4 * k + 2] = w.z;
        v[4 * k + 3] = w.w;
    }
    x = p[min(4 * chunks + threadIdx.x, len - 1)];
}

// Whether slot s of this thread holds an element of a tile of len elements.
template <uint32_t BLOCK, uint32_t IPT>
__device__ __forceinline__ bool slot_in(uint32_t s, uint32_t len) {
    return s < IPT ? threadIdx.x + s / 4 * BLOCK < len / 4 : threadIdx.x < len % 4;
}

// kFine: counters of the final partitions (bits + fine_bits bits), which
// go to `rows` and, summed per pass-1 partition, to rows1.  What bounds it: the
// key read (2^25 tuples at 2^12 counters: 29 us, 4.6 TB/s).  Persistent
// workgroups write one row for all their tiles: a row per tile would be 64 MB
// there, and counters in memory added to with atomics cost 26 us per 8M of them.
template <uint32_t BLOCK, uint32_t IPT, bool kNt, uint32_t kHash, bool kFine>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(8))) k_part_hist(Pass1 A, PassCfg cfg) {
    extern __shared__ uint32_t cnt[];  // [P], then [64] for slots without an element
    constexpr uint32_t T = BLOCK * IPT;
    const uint32_t P1 = 1u << cfg.bits;
    const uint32_t fine = kFine ? A.fine_bits : 0u, bits = cfg.bits + fine;
    const uint32_t P = P1 << fine;
    const uint32_t shift = cfg.shift - fine;  // pass 1 takes the bits above the fine ones
    const uint64_t lt = lanemask_lt();
    // the words later launches expect to be zero
    for (uint64_t i = (uint64_t)blockIdx.x * BLOCK + threadIdx.x; i < A.nzero; i += (uint64_t)gridDim.x * BLOCK)
        A.zero[i] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0 && A.err_clear) *A.err_clear = 0;
    const uint32_t grid = A.self ? A.ntiles : A.h.grid();
    if (blockIdx.x >= grid) return;  // (many words to clear for few tiles)
    for (uint32_t i = threadIdx.x; i < P; i += BLOCK) cnt[i] = 0;
    const uint32_t nx = A.self ? 1u : A.h.nx();
    const uint32_t x = A.self ? 0u : blockIdx.x & (nx - 1), q = blockIdx.x >> A.h.log_nx;
    const uint32_t of = A.h.tiles_of(x, A.ntiles);
    const uint32_t j0 = A.self ? blockIdx.x : A.h.first(of, q), j1 = A.self ? blockIdx.x + 1 : A.h.first(of, q + 1);
    uint32_t row = blockIdx.x;
    for (uint32_t rel = 0; rel < 2; ++rel) {
        const uint32_t t0 = rel ? A.nt_r : 0u, t1 = rel ? A.ntiles : A.nt_r;
        const int32_t* col = rel ? A.sk : A.rk;
        const uint32_t n = rel ? A.n_s : A.n_r;
        const uint32_t a = max(j0, A.self ? t0 : A.h.tiles_of(x, t0)), b = min(j1, A.self ? t1 : A.h.tiles_of(x, t1));
        if (a >= b && (rel == 0 || row != blockIdx.x)) continue;  // (a workgroup without tiles writes an empty row)
        __syncthreads();  // counters cleared
        for (uint32_t j = a; j < b; ++j) {
            const uint32_t off = (x + j * nx - t0) * T, len = min(T, n - off);
            int32_t keys[IPT + 1];
            load_tile<BLOCK, IPT, kNt>(col + off, len, A.rows, keys, keys[IPT]);
            if (bits <= kBallotMaxBits) {  // uniform
#pragma unroll
                for (uint32_t k = 0; k <= IPT; ++k) {
                    const bool ok = slot_in<BLOCK, IPT>(k, len);
                    const uint32_t p = part_of<kHash>(keys[k], shift, P);
                    const uint64_t m = match_mask(p, bits, ok);
                    if (ok && (m & lt) == 0) atomicAdd(&cnt[p], (uint32_t)__popcll(m));
                }
            } else {
#pragma unroll
                for (uint32_t k = 0; k <= IPT; ++k)
                    atomicAdd(&cnt[slot_in<BLOCK, IPT>(k, len) ? part_of<kHash>(keys[k], shift, P) : P + lane_id()], 1u);
            }
        }
        __syncthreads();
        if (kFine) {
            uint32_t* __restrict__ r1 = A.rows1 + (uint64_t)row * P1;
            const uint32_t F = 1u << fine;
            if (F >= kWave) {  // a wave per partition (a thread each took 360 us at 2 partitions of 8192 counters)
                for (uint32_t i = threadIdx.x / kWave; i < P1; i += BLOCK / kWave) {
                    uint32_t v = 0;
                    for (uint32_t j = lane_id(); j < F; j += kWave) v += cnt[(i << fine) | j];
                    v = wave_sum(v);
                    if (lane_id() == 0) r1[i] = v;
                }
            } else {
                for (uint32_t i = threadIdx.x; i < P1; i += BLOCK) {
                    uint32_t v = 0;
                    for (uint32_t j = 0; j < F; ++j) v += cnt[(i << fine) | ((j + i) & (F - 1))];  // (apart in banks)
                    r1[i] = v;
                }
            }
            __syncthreads();
        }
        uint32_t* __restrict__ r = A.rows + (uint64_t)row * P;
        for (uint32_t i = threadIdx.x; i < P; i += BLOCK) {
            r[i] = cnt[i];
            cnt[i] = 0;
        }
        row = grid + x;  // S's, after R's
    }
}

// Partition starts and cursors from the rows: a workgroup sums kStartCols
// columns (partitions; R's, then S's) of all rows, and one wave scans the sums,
// chained over the workgroups in ticket order (see scan.hip).  What bounds it:
// the latency of the rows, written by other XCDs just before; 64 threads share
// a column group of 4 and keep 8 loads of 16 bytes in flight (with 16 threads
// per column and 4-byte loads it took 19 us at 512 rows, 29 us at 1024).
// cur: per replica; cnt: the sums themselves (fine job), which the second
// scatter counts down.
struct StartJob {
    const uint32_t* rows;
    uint32_t P;
    uint32_t* cur;
    uint32_t* cnt;
    uint32_t* start;
    uint64_t* state;
    uint32_t nblocks;
    bool big;  // the final partitions: look for oversized ones
};

__global__ void __launch_bounds__(1024) k_part_starts(Pass1 A, StartArgs S, StartJob J1, StartJob J2) {
    constexpr uint32_t kPh = 1024 / (kStartCols / 4);  // 64 threads per 4 columns
    __shared__ uint32_t part[kPh][kStartCols];
    __shared__ uint32_t red[8][kStartCols];
    __shared__ uint32_t s_blk;
    const StartJob J = blockIdx.x < J1.nblocks ? J1 : J2;
    if (threadIdx.x == 0) s_blk = (uint32_t)atomicAdd((unsigned long long*)J.state, 1ull);
    __syncthreads();
    const uint32_t blk = s_blk;
    const uint32_t nx = A.h.nx(), P = J.P;
    {
        const uint32_t g = threadIdx.x % (kStartCols / 4), ph = threadIdx.x / (kStartCols / 4);
        const uint32_t x = ph & (nx - 1), sub = ph >> A.h.log_nx, subs = kPh >> A.h.log_nx;
        const uint32_t c = blk * kStartCols + 4 * g;
        uint32_t sum[4] = {0, 0, 0, 0};
        if (c < 2 * P) {
            const uint32_t of = A.h.tiles_of(x, A.ntiles), nr = A.h.tiles_of(x, A.nt_r);
            const uint32_t rel = c >= P, p = rel ? c - P : c;
#pragma unroll 8
            for (uint32_t q = sub; q < A.h.groups(); q += subs) {
                const uint32_t j0 = A.h.first(of, q), j1 = A.h.first(of, q + 1);
                const bool has_r = j0 < min(j1, nr), has_s = j1 > max(j0, nr);
                const uint32_t row = has_r && has_s ? A.h.grid() + x : x + (q << A.h.log_nx);  // S's row
                if (P >= 4) {  // (loaded in any case: eight in flight)
                    const uint4 v = *reinterpret_cast<const uint4*>(
                        J.rows + (uint64_t)(rel ? row : x + (q << A.h.log_nx)) * P + p);
                    const bool has = rel ? has_s : has_r;
                    sum[0] += has ? v.x : 0u;
                    sum[1] += has ? v.y : 0u;
                    sum[2] += has ? v.z : 0u;
                    sum[3] += has ? v.w : 0u;
                } else {  // P == 2: the four columns are R's two and S's two
                    const uint32_t* r = J.rows + (uint64_t)(x + (q << A.h.log_nx)) * P;
                    const uint32_t* s = J.rows + (uint64_t)row * P;
                    sum[0] += has_r ? r[0] : 0u;
                    sum[1] += has_r ? r[1] : 0u;
                    sum[2] += has_s ? s[0] : 0u;
                    sum[3] += has_s ? s[1] : 0u;
                }
            }
        }
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e) part[ph][4 * g + e] = sum[e];
    }
    __syncthreads();
    const uint32_t c0 = threadIdx.x % kStartCols;
    if (threadIdx.x < nx * kStartCols) {  // the replicas' sums
        const uint32_t x = threadIdx.x / kStartCols;
        uint32_t v = 0;
        for (uint32_t k = x; k < kPh; k += nx) v += part[k][c0];
        red[x][c0] = v;
    }
    __syncthreads();
    if (threadIdx.x >= kWave) return;
    const uint32_t c = blk * kStartCols + c0;
    uint32_t v = 0;
    for (uint32_t x = 0; x < nx; ++x) v += red[x][c0];
    const uint32_t incl = wave_incl_scan(v);
    const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
    uint32_t run = (uint32_t)lookback_wave(J.state + 1, blk, tot, S.ctl) + incl - v;
    if (c < 2 * P) {
        const uint32_t rel = c >= P, p = rel ? c - P : c;
        J.start[c] = run;
        if (c == 2 * P - 1) J.start[c + 1] = A.n_r + A.n_s;
        if (J.cnt) J.cnt[c] = v;
        if (J.cur)
            for (uint32_t x = 0; x < nx; ++x) {
                J.cur[(uint64_t)(rel * nx + x) * P + p] = run;
                run += red[x][c0];
            }
        if (J.big && rel == 0 && (S.r_pairs ? S.r_pairs[p].r_len : v) > S.lds_cap) *S.big = 1;
    }
}

// Histogram of a second pass, per tile of a segment.
template <uint32_t BLOCK, uint32_t IPT, uint32_t kHash>
__global__ void __launch_bounds__(BLOCK) k_part_hist2(const Tuple* __restrict__ in, const PartSeg* __restrict__ segs,
                                                      const uint32_t* __restrict__ tile_begin,
                                                      const uint32_t* __restrict__ tile_seg, uint32_t nseg,
                                                      PassCfg cfg, uint32_t* __restrict__ cnt2) {
    extern __shared__ uint32_t cnt[];  // [P], then [64] for slots without a tuple
    const uint32_t P = 1u << cfg.bits;
    const uint32_t ntiles = tile_begin[nseg];
    const uint32_t tile = live_remap(blockIdx.x, ntiles);
    if (tile >= ntiles) return;
    const TileLoc t = locate(segs, tile_begin, tile_seg, tile, BLOCK * IPT);
    const gtuple* src = (const gtuple*)in + t.start;
    uint64_t v[IPT];
#pragma unroll
    for (uint32_t k = 0; k < IPT; ++k) v[k] = src[min(k * BLOCK + threadIdx.x, t.len - 1)];
    for (uint32_t i = threadIdx.x; i < P; i += BLOCK) cnt[i] = 0;
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < IPT; ++k)
        atomicAdd(&cnt[k * BLOCK + threadIdx.x < t.len ? part_of<kHash>(key_of(v[k]), cfg.shift, P) : P + lane_id()], 1u);
    __syncthreads();
    uint32_t* __restrict__ out = cnt2 + ((uint64_t)t.seg << cfg.bits);
    for (uint32_t i = threadIdx.x; i < P; i += BLOCK) {
        const uint32_t c = cnt[i];
        if (c) atomicAdd(&out[i], c);
    }
}

// Clears share c of n of the HBM tables of R's oversized partitions: the slots
// of R positions [a, b), a partition at a time.  begin(i): the first position
// of R's partition i (i == npart: its end); probed(i): whether S has tuples
// for it (else its table is neither built nor read).
template <typename Begin, typename Probed>
__device__ __forceinline__ void clear_tables(const ClearTables& C, uint32_t c, uint32_t n, Begin begin, Probed probed) {
    const uint32_t per = (uint32_t)(((uint64_t)C.n_r + n - 1) / n);
    const uint32_t a = (uint32_t)min((uint64_t)c * per, (uint64_t)C.n_r);
    const uint32_t b = (uint32_t)min((uint64_t)a + per, (uint64_t)C.n_r);
    if (a >= b) return;
    uint32_t lo = 0, hi = C.npart;  // the last partition that starts at or before a (uniform)
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (begin(mid) <= a) lo = mid; else hi = mid;
    }
    uint4* __restrict__ slots = reinterpret_cast<uint4*>(C.table);  // the 2 slots of an R position
    for (uint32_t i = lo; i < C.npart; ++i) {
        const uint32_t s = begin(i), e = begin(i + 1);
        if (s >= b) break;
        if (e - s <= C.lds_cap || !probed(i)) continue;
        for (uint32_t j = max(s, a) + threadIdx.x; j < min(e, b); j += blockDim.x)
            slots[j] = make_uint4(~0u, ~0u, ~0u, ~0u);
    }
}

// Sums of the rows [r0, r1) of P <= BLOCK counters each (self_starts): tot[p]
// over all, bef[p] over those below `mine`, added to LDS arrays that are zero
// and visible to the block.  Needs a barrier before they are read.
template <uint32_t BLOCK>
__device__ __forceinline__ void sum_rows(const uint32_t* __restrict__ rows, uint32_t P, uint32_t r0, uint32_t r1,
                                         uint32_t mine, uint32_t* tot, uint32_t* bef) {
    const uint32_t p = threadIdx.x & (P - 1), ph = threadIdx.x / P, phases = BLOCK / P;
    uint32_t t = 0, b = 0;
#pragma unroll 8
    for (uint32_t r = r0 + ph; r < r1; r += phases) {
        const uint32_t v = rows[(uint64_t)r * P + p];
        t += v;
        b += r < mine ? v : 0u;
    }
    if (t) atomicAdd(&tot[p], t);
    if (bef && b) atomicAdd(&bef[p], b);
}

// Scatter of one tile per workgroup.  kSeg: a tile of a segment of `in` (pass
// 2), else of the input's columns.  kCols: two columns out instead of tuples.
// What bounds it: HBM traffic at few partitions (128M x 256M, 2^7 partitions:
// 1.22 ms, 5.3 TB/s of its 16 bytes per tuple), at 2^12 the lines that leave the
// L2 before a partition's next run fills them (16M x 16M: 425-442 MB written for
// 268, 283 read, 4.6 TB/s in 155 us with 16384-tuple tiles, where two
// scatters of 2^6 took 107 us each before the tuples were one word, the cursors
// per XCD and the tile's loads and LDS accesses free of branches).  kSelf:
// partition starts from the rows (self_starts).
// Registers: at most 64 up to 8 tuples per thread, so that LDS alone limits
// the workgroups of a CU (two of 8192 tuples).
template <uint32_t BLOCK, uint32_t IPT, bool kSeg, bool kNt, bool kCols, bool kSelf, uint32_t kHash>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(IPT <= 8 ? 8 : 4)))
k_part_scatter(Pass1 A, const Tuple* __restrict__ in, const PartSeg* __restrict__ segs,
               const uint32_t* __restrict__ tile_begin, const uint32_t* __restrict__ tile_seg, uint32_t nseg, PassCfg cfg,
               const uint32_t* __restrict__ start2, uint32_t* __restrict__ cur1, Tuple* __restrict__ out,
               int32_t* __restrict__ key_out, int32_t* __restrict__ rid_out, ClearTables clr, SideJob side,
               uint32_t lds_words) {
    extern __shared__ uint64_t lds64[];
    uint32_t* lds = reinterpret_cast<uint32_t*>(lds64);
    if (blockIdx.x >= gridDim.x - side.blocks) {  // extra workgroups: the side job
        if (kSelf) {  // the join plan, from starts made here (P <= 2^kSelfBits: one workgroup)
            const uint32_t P = 1u << cfg.bits;
            for (uint32_t i = threadIdx.x; i < 2 * P; i += BLOCK) lds[i] = 0;
            __syncthreads();
            sum_rows<BLOCK>(A.rows, P, 0u, A.nt_r, 0u, lds, nullptr);
            sum_rows<BLOCK>(A.rows, P, A.nt_r, A.ntiles, 0u, lds + P, nullptr);
            __syncthreads();
            uint32_t* wt = lds + 2 * (P < kWave ? kWave : P);
            for (uint32_t i = 2 * P + threadIdx.x; i < kWave; i += BLOCK) lds[i] = 0;  // (the scan takes 64 at a time)
            __syncthreads();
            lds_excl_scan(lds, 2 * P < kWave ? kWave : 2 * P, wt);
            __syncthreads();
            join_plan_block(side.plan, lds, A.n_r + A.n_s);
            return;
        }
        run_side_job(side, blockIdx.x - (gridDim.x - side.blocks), lds, lds_words);
        return;
    }
    constexpr uint32_t T = BLOCK * IPT;
    constexpr bool kLoop = !kSeg && IPT > 8;
    constexpr uint32_t kOwn = kSelf ? 1 : 4;  // partitions per thread whose reservation stays in registers
    const uint32_t P = 1u << cfg.bits;
    const uint32_t Pp = P < kWave ? kWave : P;  // scan length, a multiple of 64
    Tuple* stage = lds64;                              // [T], then [64] for slots without a tuple
    uint32_t* cnt = lds + 2 * (T + kWave);             // [Pp] counts, local starts, then global - local
    uint32_t* none = cnt + Pp;                         // [64] counts of slots without a tuple
    uint32_t* wt = none + kWave;                       // [kScanScratch]
    uint32_t* resv = wt + kScanScratch;                // [P] (P > kOwn BLOCK only): reservations
    uint32_t* tot = wt + kScanScratch;                 // [Pp] (kSelf): the relation's counts, then starts
    uint32_t* bef = tot + Pp;                          // [Pp] (kSelf): counts of the tiles before this one

    // kLoop: workgroups stay for several tiles (blk, blk + G, ...: one replica), and the
    // next tile's keys are loaded while this one is written out
    const uint32_t ntiles = kSeg ? tile_begin[nseg] : A.ntiles;
    const uint32_t G = gridDim.x - side.blocks;
    uint32_t tile = kSeg ? live_remap(blockIdx.x, ntiles)  // an XCD's tiles are contiguous: it writes whole segments
                         : blockIdx.x;
    constexpr bool kMore = IPT <= 8;  // (tiles of 16384 tuples: one per CU at least, as many as clear_share)
    // share c of the HBM tables' clearing (rare; uniform)
    auto clear = [&](uint32_t c) {
        const uint32_t n = kMore ? max(ntiles, clr.share) : ntiles;
        if (kSelf && !clr.r_pairs) {  // R's tiles know R's partitions, and share the clearing among them
            clear_tables(clr, c, A.nt_r, [&](uint32_t i) { return i < P ? tot[i] : clr.n_r; },
                         [](uint32_t) { return true; });
            return;
        }
        if constexpr (!kMore) {  // (one copy of the code: three would cost the kernel registers)
            clear_tables(clr, c, n,
                         [&](uint32_t i) {
                             return i >= clr.npart ? clr.n_r : clr.r_pairs ? clr.r_pairs[i].r_off : clr.start[i];
                         },
                         [&](uint32_t i) { return clr.start[clr.npart + i + 1] != clr.start[clr.npart + i]; });
            return;
        }
        auto cleared = [&](auto begin) {
            if (kSelf)
                clear_tables(clr, c, n, begin, [&](uint32_t i) { return (i + 1 < P ? tot[i + 1] : A.n_s) != tot[i]; });
            else
                clear_tables(clr, c, n, begin, [&](uint32_t i) {
                    return clr.start[clr.npart + i + 1] != clr.start[clr.npart + i];
                });
        };
        if (clr.r_pairs) cleared([&](uint32_t i) { return i < clr.npart ? clr.r_pairs[i].r_off : clr.n_r; });
        else cleared([&](uint32_t i) { return i < clr.npart ? clr.start[i] : clr.n_r; });
    };
    if (tile >= ntiles) {  // a workgroup that only clears
        if (!kMore || !clr.table || tile >= clr.share) return;
        if (!kSelf) {
            if (*clr.big != 0) clear(tile);
            return;
        }
        if (!clr.r_pairs || !__syncthreads_or(threadIdx.x < P && clr.r_pairs[threadIdx.x].r_len > clr.lds_cap)) return;
        for (uint32_t i = threadIdx.x; i < Pp; i += BLOCK) tot[i] = 0;
        __syncthreads();
        sum_rows<BLOCK>(A.rows, P, A.nt_r, A.ntiles, 0u, tot, nullptr);
        __syncthreads();
        lds_excl_scan(tot, Pp, wt);
        __syncthreads();
        clear(tile);
        return;
    }
    uint32_t len, lo, n;  // tuples; positions [lo, lo + n) they may take
    uint32_t* cur;
    const uint32_t* st = nullptr;
    const int32_t* rin = nullptr;
    // slots: as load_tile; a segment's tile (kSeg) has element k BLOCK + t in thread t's slot k
    constexpr uint32_t kSlots = kSeg ? IPT : IPT + 1;
    int32_t keys[kSlots], rids[kSlots];
    auto in_tile = [&](uint32_t k) { return kSeg ? k * BLOCK + threadIdx.x < len : slot_in<BLOCK, IPT>(k, len); };
    auto load = [&](uint32_t t) {  // (kSeg: keys and rids; else the keys)
        if constexpr (kSeg) {
            const TileLoc L = locate(segs, tile_begin, tile_seg, t, T);
            const PartSeg g = segs[L.seg];
            len = L.len;
            lo = g.base;
            n = g.n;
            cur = cur1 + ((uint64_t)L.seg << cfg.bits);  // (pass 2: the counts)
            st = start2 + ((uint64_t)L.seg << cfg.bits);
            const gtuple* src = (const gtuple*)in + L.start;
#pragma unroll
            for (uint32_t k = 0; k < IPT; ++k) {
                const gtuple* a = src + min(k * BLOCK + threadIdx.x, len - 1);
                const uint64_t v = kNt ? __builtin_nontemporal_load(a) : *a;
                keys[k] = key_of(v);
                rids[k] = rid_of(v);
            }
        } else {
            const bool s1 = t >= A.nt_r;  // field by field: no dynamic index into the arguments
            const uint32_t off = (s1 ? t - A.nt_r : t) * T;
            lo = s1 ? A.n_r : 0u;
            n = s1 ? A.n_s : A.n_r;
            len = min(T, n - off);
            if (!kSelf) cur = cur1 + (uint64_t)((s1 ? A.h.nx() : 0u) + (t & (A.h.nx() - 1))) * P;
            rin = (s1 ? A.sr : A.rr) + off;
            load_tile<BLOCK, IPT, kNt>((s1 ? A.sk : A.rk) + off, len, A.rows, keys, keys[IPT]);
        }
    };
    load(tile);
    const uint64_t lt = lanemask_lt();
    while (true) {
        // the rids are needed last: in flight while the tile is counted
        if constexpr (!kSeg) load_tile<BLOCK, IPT, kNt>(rin, len, A.rows, rids, rids[IPT]);
        // counters cleared while the loads are in flight
        for (uint32_t i = threadIdx.x; i < (kSelf ? Pp + kWave + kScanScratch + 2 * Pp : Pp); i += BLOCK) cnt[i] = 0;
        __syncthreads();
        bool big = false;
        if (kSelf)
            sum_rows<BLOCK>(A.rows, P, tile < A.nt_r ? 0u : A.nt_r, tile < A.nt_r ? A.nt_r : A.ntiles, tile, tot, bef);
        uint32_t rank[kSlots];
        if (cfg.bits <= kBallotMaxBits) {  // uniform
#pragma unroll
            for (uint32_t k = 0; k < kSlots; ++k) {
                const bool ok = in_tile(k);
                const uint32_t p = part_of<kHash>(keys[k], cfg.shift, P);
                const uint64_t m = match_mask(p, cfg.bits, ok);
                const uint32_t below = (uint32_t)__popcll(m & lt);
                uint32_t old = 0;
                if (ok && below == 0) old = atomicAdd(&cnt[p], (uint32_t)__popcll(m));
                const uint32_t leader = m ? (uint32_t)(__ffsll((long long)m) - 1) : 0u;
                old = __shfl(old, (int)leader, kWave);
                rank[k] = old + below;
            }
        } else {
            // the returned old value is the tuple's rank; lanes hitting the same
            // counter in one instruction get distinct values
#pragma unroll
            for (uint32_t k = 0; k < kSlots; ++k)
                rank[k] = atomicAdd(in_tile(k) ? &cnt[part_of<kHash>(keys[k], cfg.shift, P)] : &none[lane_id()], 1u);
        }
        __syncthreads();
        // The tile's run of every partition is reserved on the partition's cursor;
        // the answers are awaited only after the tile is reordered below.
        auto reserve = [&](uint32_t p) -> uint32_t {
            const uint32_t c = cnt[p];
            if (c == 0) return 0u;
            if (!kSeg) return atomicAdd(&cur[p], c);
            return st[p] + atomicSub(&cur[p], c) - c;  // counted down to the partition's start
        };
        uint32_t own[kOwn];
        if (kSelf) {
            if (clr.table) {  // (uniform) R's tiles know R's partitions; a built table's are looked up
                if (clr.r_pairs) big = threadIdx.x < P && clr.r_pairs[threadIdx.x].r_len > clr.lds_cap;
                else big = tile < A.nt_r && threadIdx.x < P && tot[threadIdx.x] > clr.lds_cap;
                big = __syncthreads_or(big);
            }
            lds_excl_scan(tot, Pp, wt);
            __syncthreads();
            own[0] = threadIdx.x < P ? lo + tot[threadIdx.x] + bef[threadIdx.x] : 0u;
        } else {
#pragma unroll
            for (uint32_t o = 0; o < kOwn; ++o) {
                const uint32_t p = o * BLOCK + threadIdx.x;
                own[o] = p < P ? reserve(p) : 0u;
            }
            for (uint32_t p = kOwn * BLOCK + threadIdx.x; p < P; p += BLOCK) resv[p] = reserve(p);
            __syncthreads();
        }
        lds_excl_scan(cnt, Pp, wt);
        __syncthreads();
#pragma unroll
        for (uint32_t k = 0; k < kSlots; ++k) rank[k] += cnt[part_of<kHash>(keys[k], cfg.shift, P)];
#pragma unroll
        for (uint32_t k = 0; k < kSlots; ++k)
            stage[in_tile(k) ? rank[k] : T + lane_id()] = (uint32_t)keys[k] | (uint64_t)(uint32_t)rids[k] << 32;
        // the reservations are back by now; waiting for them here keeps the waits
        // out of the store loop below
#pragma unroll
        for (uint32_t o = 0; o < kOwn; ++o) settle(own[o]);
        __syncthreads();
#pragma unroll
        for (uint32_t o = 0; o < kOwn; ++o) {
            const uint32_t p = o * BLOCK + threadIdx.x;
            if (p < P) cnt[p] = own[o] - cnt[p];
        }
        if (!kSelf)
            for (uint32_t p = kOwn * BLOCK + threadIdx.x; p < P; p += BLOCK) cnt[p] = resv[p] - cnt[p];
        __syncthreads();
        const uint32_t w_len = len, w_lo = lo, w_n = n;
        const uint32_t next = tile + G;
        const bool more = kLoop && next < ntiles;  // uniform
        if (more) load(next);
        // kOut tuples per thread at a time: their LDS reads in flight together
        constexpr uint32_t kOut = IPT > 8 || IPT < 8 ? 4 : 8;
#pragma unroll
        for (uint32_t k0 = 0; k0 < IPT; k0 += kOut) {
            uint64_t v[kOut];
            uint32_t dst[kOut];
#pragma unroll
            for (uint32_t k = 0; k < kOut; ++k) v[k] = stage[(k0 + k) * BLOCK + threadIdx.x];
#pragma unroll
            for (uint32_t k = 0; k < kOut; ++k) dst[k] = cnt[part_of<kHash>(key_of(v[k]), cfg.shift, P)];
#pragma unroll
            for (uint32_t k = 0; k < kOut; ++k) {
                const uint32_t j = (k0 + k) * BLOCK + threadIdx.x, d = dst[k] + j;
                // (the second test holds for consistent counts; it keeps stores in the relation or segment)
                if (j < w_len && d - w_lo < w_n) {
                    if (kCols) {
                        key_out[d] = key_of(v[k]);
                        rid_out[d] = rid_of(v[k]);
                    } else {
                        out[d] = v[k];
                    }
                }
            }
        }
        if (clr.table && (kSelf ? big : *clr.big != 0)) clear(tile);
        if (!more) break;
        tile = next;
        __syncthreads();  // the tile's LDS is free again
    }
}

template <typename F>
void allow_lds(F fn, size_t lds) {
    if (lds > 65536) (void)hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

template <uint32_t BLOCK, uint32_t IPT, uint32_t kHash>
void launch_hist(const Pass1& p1, const PassCfg& cfg, Recorder& rec) {
    static_assert(BLOCK * IPT >= 1024 && BLOCK * IPT <= kMaxScatterTile && BLOCK / kWave <= kScanScratch, "tile shape");
    const size_t lds = sizeof(uint32_t) * (((size_t)1 << (cfg.bits + p1.fine_bits)) + kWave);
    // (workgroups past the tiles' clear words only: 4096 rows in 2^18 partitions, one tile, 2 MB to clear)
    const uint32_t grid =
        std::max(p1.self ? p1.ntiles : p1.h.grid(), (uint32_t)std::min<uint64_t>(256, p1.nzero / 4096));
    const auto fine = cfg.nt ? k_part_hist<BLOCK, IPT, true, kHash, true> : k_part_hist<BLOCK, IPT, false, kHash, true>;
    const auto flat = cfg.nt ? k_part_hist<BLOCK, IPT, true, kHash, false> : k_part_hist<BLOCK, IPT, false, kHash, false>;
    const auto fn = p1.fine_bits ? fine : flat;
    allow_lds(fn, lds);
    rec.before("part_hist");
    hipLaunchKernelGGL(fn, dim3(grid), dim3(BLOCK), lds, rec.stream, p1, cfg);
    rec.after();
}

constexpr uint32_t kScatterLoopGrid = 256;

template <uint32_t kHash>
void hist_tiles(const Pass1& p1, const PassCfg& cfg, Recorder& rec) {
    switch (cfg.tile) {
        case 1024: launch_hist<256, 4, kHash>(p1, cfg, rec); break;
        case 2048: launch_hist<256, 8, kHash>(p1, cfg, rec); break;
        case 4096: launch_hist<512, 8, kHash>(p1, cfg, rec); break;
        case 8192: launch_hist<1024, 8, kHash>(p1, cfg, rec); break;
        default: launch_hist<1024, 16, kHash>(p1, cfg, rec); break;
    }
}

template <uint32_t BLOCK, uint32_t IPT>
void launch_hist2(const Tuple* in, const PartSeg* segs, const uint32_t* tile_begin, const uint32_t* tile_seg,
                  uint32_t nseg, uint32_t grid, const PassCfg& cfg, uint32_t* cnt2, Recorder& rec) {
    const size_t lds = sizeof(uint32_t) * (((size_t)1 << cfg.bits) + kWave);
    const auto fn = cfg.hash_kind ? k_part_hist2<BLOCK, IPT, 1> : k_part_hist2<BLOCK, IPT, 0>;
    hipLaunchKernelGGL(fn, dim3(grid), dim3(BLOCK), lds, rec.stream, in, segs, tile_begin, tile_seg, nseg, cfg, cnt2);
}

struct ScatterArgs {
    Pass1 p1;
    const Tuple* in;
    const PartSeg* segs;
    const uint32_t *tile_begin, *tile_seg;
    uint32_t nseg, grid;
    const uint32_t* start2;
    uint32_t* cur;
    Tuple* out;
    int32_t *key_out, *rid_out;
};

template <uint32_t BLOCK, uint32_t IPT, bool kSeg, bool kNt, bool kCols, bool kSelf, uint32_t kHash>
void launch_scatter(const ScatterArgs& a, const PassCfg& cfg, const ClearTables& clr, const SideJob& side,
                    Recorder& rec) {
    const size_t P = (size_t)1 << cfg.bits;
    const size_t Pp = P < kWave ? kWave : P;
    size_t lds = sizeof(Tuple) * (BLOCK * IPT + kWave) +
                 sizeof(uint32_t) * (Pp + kWave + kScanScratch + (kSelf ? 2 * Pp : P > 4 * BLOCK ? P : 0));
    if (side.kind == kSideSetup2) {
        // room for the pass-2 segment tile offsets (else the setup fills the tile map from HBM)
        const size_t want = sizeof(uint32_t) * (kScanScratch + 2 * ((size_t)1 << side.setup2.bits1) + 1);
        if (want > lds && want <= 65536) lds = want;
    }
    allow_lds(k_part_scatter<BLOCK, IPT, kSeg, kNt, kCols, kSelf, kHash>, lds);
    // one workgroup per CU for tiles of more than 8 tuples per thread (kLoop)
    uint32_t grid = !kSeg && IPT > 8 && a.grid > kScatterLoopGrid ? kScatterLoopGrid : a.grid;
    if (IPT <= 8 && clr.table && grid < clr.share) grid = clr.share;
    rec.before("part_scatter");
    hipLaunchKernelGGL((k_part_scatter<BLOCK, IPT, kSeg, kNt, kCols, kSelf, kHash>), dim3(grid + side.blocks), dim3(BLOCK), lds,
                       rec.stream, a.p1, a.in, a.segs, a.tile_begin, a.tile_seg, a.nseg, cfg, a.start2, a.cur, a.out,
                       a.key_out, a.rid_out, clr, side, (uint32_t)(lds / sizeof(uint32_t)));
    rec.after();
}

template <bool kSeg, bool kNt, bool kSelf, uint32_t kHash>
void scatter_tiles(const ScatterArgs& a, const PassCfg& cfg, const ClearTables& clr, const SideJob& side,
                   Recorder& rec) {
    switch (cfg.tile) {  // workgroup size by tile: scatter_block()
        case 1024: launch_scatter<256, 4, kSeg, kNt, false, kSelf, kHash>(a, cfg, clr, side, rec); break;
        case 2048: launch_scatter<256, 8, kSeg, kNt, false, kSelf, kHash>(a, cfg, clr, side, rec); break;
        case 4096: launch_scatter<512, 8, kSeg, kNt, false, kSelf, kHash>(a, cfg, clr, side, rec); break;
        case 8192: launch_scatter<1024, 8, kSeg, kNt, false, kSelf, kHash>(a, cfg, clr, side, rec); break;
        default:  // (self_starts joins have no tiles of more than 8192 tuples)
            if constexpr (!kSelf) launch_scatter<1024, 16, kSeg, kNt, false, kSelf, kHash>(a, cfg, clr, side, rec);
            break;
    }
}

template <bool kSeg, bool kNt, bool kSelf = false>
void scatter_hash(const ScatterArgs& a, const PassCfg& cfg, const ClearTables& clr, const SideJob& side,
                  Recorder& rec) {
    if (cfg.hash_kind) scatter_tiles<kSeg, kNt, kSelf, 1>(a, cfg, clr, side, rec);
    else scatter_tiles<kSeg, kNt, kSelf, 0>(a, cfg, clr, side, rec);
}

// Two columns out: one tile and MurmurHash 2.0 only (the out-of-core partition pass).
template <bool kNt>
void scatter_columns(const ScatterArgs& a, const PassCfg& cfg, const ClearTables& clr, const SideJob& side,
                     Recorder& rec) {
    if (cfg.tile != kColumnsTile || !cfg.hash_kind) {
        if (rec.err == hipSuccess) rec.err = hipErrorInvalidConfiguration;
        return;
    }
    static_assert(kColumnsTile == 1024 * 8, "tile of the column kernels");
    launch_scatter<1024, 8, false, kNt, true, false, 1>(a, cfg, clr, side, rec);
}

// (grid > 0 or side workgroups, and a tile the kernels are built for)
bool scatter_ok(const ScatterArgs& a, const PassCfg& cfg, const SideJob& side, Recorder& rec) {
    if (a.grid + side.blocks == 0) return false;
    const uint32_t t = cfg.tile;
    if (t != 1024 && t != 2048 && t != 4096 && t != 8192 && t != kMaxScatterTile) {
        if (rec.err == hipSuccess) rec.err = hipErrorInvalidConfiguration;
        return false;
    }
    return true;
}

}  // namespace

Pass1 make_pass1(const int32_t* rk, const int32_t* rr, uint32_t n_r, const int32_t* sk, const int32_t* sr,
                 uint32_t n_s, uint32_t tile) {
    Pass1 a{};
    a.rk = rk;
    a.rr = rr;
    a.sk = sk;
    a.sr = sr;
    a.n_r = n_r;
    a.n_s = n_s;
    a.nt_r = (uint32_t)(((uint64_t)n_r + tile - 1) / tile);
    a.ntiles = a.nt_r + (uint32_t)(((uint64_t)n_s + tile - 1) / tile);
    return a;
}

void part_starts(const Pass1& p1, const PassCfg& cfg, const StartArgs& st, Recorder& rec) {
    if (p1.ntiles == 0 || p1.self) return;
    const uint32_t P1 = 1u << cfg.bits, P = P1 << p1.fine_bits;
    auto blocks = [](uint32_t parts) { return (2 * parts + kStartCols - 1) / kStartCols; };
    const bool fine = p1.fine_bits != 0;
    const StartJob j1{fine ? p1.rows1 : p1.rows, P1, st.cur1, nullptr, st.start1, st.state1, blocks(P1),
                      !fine && st.npart != 0};
    const StartJob j2{p1.rows, P, nullptr, st.cnt2, st.start2, st.state2, fine ? blocks(P) : 0u, st.npart != 0};
    rec.before("part_starts");
    hipLaunchKernelGGL(k_part_starts, dim3(j1.nblocks + j2.nblocks), dim3(1024), 0, rec.stream, p1, st, j1, j2);
    rec.after();
}

void part_hist(const Pass1& p1, const PassCfg& cfg, Recorder& rec) {
    if (p1.ntiles == 0) return;
    if (cfg.hash_kind) hist_tiles<1>(p1, cfg, rec);
    else hist_tiles<0>(p1, cfg, rec);
}

void part_hist2(const Tuple* in, const PartSeg* segs, const uint32_t* tile_begin, const uint32_t* tile_seg,
                uint32_t nseg, uint32_t grid, const PassCfg& cfg, uint32_t* cnt2, Recorder& rec) {
    if (grid == 0) return;
    rec.before("part_hist2");
    switch (cfg.tile) {
        case 1024: launch_hist2<256, 4>(in, segs, tile_begin, tile_seg, nseg, grid, cfg, cnt2, rec); break;
        case 2048: launch_hist2<256, 8>(in, segs, tile_begin, tile_seg, nseg, grid, cfg, cnt2, rec); break;
        case 4096: launch_hist2<512, 8>(in, segs, tile_begin, tile_seg, nseg, grid, cfg, cnt2, rec); break;
        case 8192: launch_hist2<1024, 8>(in, segs, tile_begin, tile_seg, nseg, grid, cfg, cnt2, rec); break;
        default: launch_hist2<1024, 16>(in, segs, tile_begin, tile_seg, nseg, grid, cfg, cnt2, rec); break;
    }
    rec.after();
}

void part_scatter(const Pass1& p1, const PassCfg& cfg, uint32_t* cur1, Tuple* out, int32_t* key_out,
                  int32_t* rid_out, const ClearTables& clr, const SideJob& side, Recorder& rec) {
    const ScatterArgs a{p1, nullptr, nullptr, nullptr, nullptr, 0, p1.ntiles, nullptr, cur1, out, key_out, rid_out};
    if (!scatter_ok(a, cfg, side, rec)) return;
    if (!out) {
        if (cfg.nt) scatter_columns<true>(a, cfg, clr, side, rec);
        else scatter_columns<false>(a, cfg, clr, side, rec);
    } else if (p1.self) {
        scatter_hash<false, false, true>(a, cfg, clr, side, rec);
    } else if (cfg.nt) {
        scatter_hash<false, true>(a, cfg, clr, side, rec);
    } else {
        scatter_hash<false, false>(a, cfg, clr, side, rec);
    }
}

void part_scatter2(const Tuple* in, const PartSeg* segs, const uint32_t* tile_begin, const uint32_t* tile_seg,
                   uint32_t nseg, uint32_t grid, const PassCfg& cfg, const uint32_t* start2, uint32_t* cnt2,
                   Tuple* out, const ClearTables& clr, const SideJob& side, Recorder& rec) {
    const ScatterArgs a{Pass1{}, in, segs, tile_begin, tile_seg, nseg, grid, start2, cnt2, out, nullptr, nullptr};
    if (!scatter_ok(a, cfg, side, rec)) return;
    if (cfg.nt) scatter_hash<true, true>(a, cfg, clr, side, rec);
    else scatter_hash<true, false>(a, cfg, clr, side, rec);
}

}  // namespace hj
