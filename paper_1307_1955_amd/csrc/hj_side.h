// Work that rides along with another launch ("side jobs"): extra workgroups
// at the end of a radix-scatter grid run the next pass's setup or the join
// plan.  Both only read data that was complete before the hosting launch
// started (the partition starts) and write tables that only later launches
// read, so they need no ordering with the scatter's own workgroups and cost no
// launch of their own.
#pragma once

#include "hj_device.h"
#include "hj_internal.h"

namespace hj {

constexpr uint32_t kMaxPlanWaves = 16;  // waves of the largest workgroup that runs the join plan

// Everything the pass-2 setup reads and writes.
struct Setup2Args {
    const uint32_t* start1;  // pass-1 partition starts of R, then of S, [2 << bits1] = the end
    uint32_t bits1, tile, n_r, n_s;
    uint32_t tiles_ub;       // tiles there is room for
    PartSeg* segs2;
    uint32_t* tile_begin2;
    uint32_t* tile_seg2;
};

// Everything the join plan reads and writes (see join_plan_block).
struct PlanArgs {
    const uint32_t* start;  // final partition starts of R, then of S (S's from n_r on)
    uint32_t n_r, n_s, total_bits, lds_cap;
    PartPair* pairs;
    uint32_t* item_begin;
    uint32_t* ovf_begin;
    ItemRec* item_rec;
    uint32_t* ovf_part;
    uint64_t* zero_total;
    uint64_t* state;
    // R's partition ranges from an earlier build (hj_build); nullptr: from `start` like S's
    const PartPair* r_pairs;
    ScanCtl ctl;  // the chained scan of the plan reports a give-up here
    // records of item_rec up to here that have no item are written empty (the
    // join kernels' workgroup b takes record b)
    uint32_t items_ub, ovf_ub;  // records of item_rec, of ovf_part
};

enum SideKind : uint32_t { kSideNone = 0, kSideSetup2 = 1, kSidePlan = 2 };

struct SideJob {
    uint32_t kind;
    uint32_t blocks;  // extra workgroups at the end of the grid
    union {
        Setup2Args setup2;
        PlanArgs plan;
    };
    SideJob() : kind(kSideNone), blocks(0), plan() {}
};

// Join-plan workgroups of `block` threads (one partition pair per thread).
inline uint32_t plan_blocks(uint32_t P, uint32_t block) { return (P + block - 1) / block; }

__device__ __forceinline__ uint32_t items_of(const PartPair& pp) {
    return (pp.r_len && pp.s_len) ? (pp.s_len + kJoinChunk - 1) / kJoinChunk : 0u;
}

__device__ __forceinline__ uint32_t ovf_chunks_of(const PartPair& pp, uint32_t lds_cap) {
    const uint32_t chunk = ovf_chunk(pp.r_len);
    return (pp.r_len > lds_cap && pp.s_len) ? (pp.r_len + chunk - 1) / chunk : 0u;
}

// Plan (one thread per partition pair, workgroups in ticket order): ranges of
// R_i and S_i from the partition starts, the pair's work items and HBM-table
// build chunks, their exclusive scans over all pairs (one chained scan of both
// counts packed in one word), the work-item records and the chunk -> pair map.
// state[0]: ticket; state[1 + b]: status of workgroup b (cleared beforehand).
// Run by plan_blocks(P, blockDim.x) workgroups.  When the chained scan gives
// up, its prefixes come out too small, never too large: records overlap, and
// the last workgroup still empties everything past the last one.  No record is
// written past its array, whatever the prefix.
// start, end: the starts and their end ([2^(total_bits + 1)]); `start` may be LDS.
__device__ __forceinline__ void join_plan_block(const PlanArgs& A, const uint32_t* start, uint32_t end) {
    const uint32_t n_r = A.n_r, n_s = A.n_s;
    const uint32_t total_bits = A.total_bits, lds_cap = A.lds_cap;
    PartPair* __restrict__ pairs = A.pairs;
    uint32_t* __restrict__ item_begin = A.item_begin;
    uint32_t* __restrict__ ovf_begin = A.ovf_begin;
    ItemRec* __restrict__ item_rec = A.item_rec;
    uint32_t* __restrict__ ovf_part = A.ovf_part;
    uint64_t* __restrict__ zero_total = A.zero_total;
    uint64_t* state = A.state;
    __shared__ uint64_t wt[kMaxPlanWaves];
    __shared__ uint32_t s_blk;
    __shared__ uint64_t s_prefix;
    if (threadIdx.x == 0) s_blk = (uint32_t)atomicAdd((unsigned long long*)state, 1ull);
    __syncthreads();
    const uint32_t blk = s_blk;
    const uint32_t P = 1u << total_bits;
    const uint32_t i = blk * blockDim.x + threadIdx.x;
    if (i == 0 && zero_total) *zero_total = 0;
    PartPair pp{0, 0, 0, 0};
    uint32_t ni = 0, no = 0;
    if (i < P) {
        // clamped: a partition never extends past its relation or runs backwards
        const uint32_t e = i + 1 < P ? start[P + i + 1] : end;
        const uint32_t s0 = min(start[P + i] - n_r, n_s), s1 = max(s0, min(e - n_r, n_s));
        if (A.r_pairs) {
            const PartPair q = A.r_pairs[i];
            pp.r_off = q.r_off;
            pp.r_len = q.r_len;
        } else {
            const uint32_t r0 = min(start[i], n_r), r1 = max(r0, min(start[i + 1], n_r));
            pp.r_off = r0;
            pp.r_len = r1 - r0;
        }
        pp.s_off = s0;
        pp.s_len = s1 - s0;
        ni = items_of(pp);
        no = ovf_chunks_of(pp, lds_cap);
    }
    // items and chunks are each below 2^31: packed as items | chunks << 31
    uint64_t tot;
    const uint64_t excl = block_excl_scan((uint64_t)ni | ((uint64_t)no << 31), wt, &tot);
    if (threadIdx.x < kWave) {
        const uint64_t prefix = lookback_wave(state + 1, blk, tot, A.ctl);
        if (threadIdx.x == 0) s_prefix = prefix;
    }
    __syncthreads();
    const uint64_t run = s_prefix + excl;
    const uint32_t ib = (uint32_t)(run & 0x7FFFFFFFu), ob = (uint32_t)(run >> 31);
    if (i < P) {
        pairs[i] = pp;
        item_begin[i] = ib;
        ovf_begin[i] = ob;
        for (uint32_t x = 0; x < ni && ib + x < A.items_ub; ++x)
            item_rec[ib + x] = ItemRec{pp.r_off, pp.r_len, pp.s_off + x * kJoinChunk,
                                       min(kJoinChunk, pp.s_len - x * kJoinChunk)};
        for (uint32_t x = 0; x < no && ob + x < A.ovf_ub; ++x) ovf_part[ob + x] = i;
    }
    if (i == P - 1) {  // the last pair also writes the totals
        item_begin[P] = ib + ni;
        ovf_begin[P] = ob + no;
    }
    // the workgroup of the last pair marks the records past the last item empty
    __shared__ uint32_t s_live;
    const bool last_blk = blk * blockDim.x <= P - 1 && P - 1 < (blk + 1) * blockDim.x;  // uniform
    if (last_blk) {
        if (i == P - 1) s_live = ib + ni;
        __syncthreads();
        for (uint32_t x = s_live + threadIdx.x; x < A.items_ub; x += blockDim.x) item_rec[x] = ItemRec{0, 0, 0, 0};
    }
}



// Pass-2 segment table (every pass-1 partition of R and of S), its tile
// offsets and the tile -> segment map, from the pass-1 partition starts.  Run
// by one workgroup of any size; `lds` holds lds_words scratch words (the
// segment tile offsets are kept there for the tile map when they fit).
__device__ __forceinline__ void setup_pass2_block(const Setup2Args& A, uint32_t* lds, uint32_t lds_words) {
    const uint32_t tile = A.tile;
    PartSeg* __restrict__ segs2 = A.segs2;
    uint32_t* __restrict__ tile_begin2 = A.tile_begin2;
    uint32_t* __restrict__ tile_seg2 = A.tile_seg2;
    uint32_t* wt = lds;                   // [kScanScratch]
    uint32_t* tb = lds + kScanScratch;    // [nseg + 1] when it fits
    const uint32_t nseg = 2u << A.bits1;
    const uint32_t per = (nseg + blockDim.x - 1) / blockDim.x;
    const uint32_t a = min(threadIdx.x * per, nseg);
    const uint32_t b = min(a + per, nseg);
    // clamped (starts from a scan that gave up): a segment lies inside its
    // relation, and there are no more tiles than fit the map
    auto range = [&](uint32_t s, uint32_t* len) {
        const uint32_t lo = s < nseg / 2 ? 0u : A.n_r, hi = s < nseg / 2 ? A.n_r : A.n_r + A.n_s;
        const uint32_t base = min(max(A.start1[s], lo), hi);
        *len = max(base, min(A.start1[s + 1], hi)) - base;
        return base;
    };
    uint32_t ntiles = 0;
    for (uint32_t s = a; s < b; ++s) {
        uint32_t len;
        range(s, &len);
        ntiles += (len + tile - 1) / tile;
    }
    uint32_t total;
    uint32_t run = block_excl_scan(ntiles, wt, &total);
    const bool in_lds = nseg + 1 + kScanScratch <= lds_words;
    for (uint32_t s = a; s < b; ++s) {
        uint32_t len;
        const uint32_t base = range(s, &len);
        if (run >= A.tiles_ub || len / tile >= A.tiles_ub - run) len = 0;
        segs2[s] = PartSeg{base, len};
        tile_begin2[s] = run;
        if (in_lds) tb[s] = run;
        const uint32_t nt = (len + tile - 1) / tile;
        if (!in_lds)
            for (uint32_t x = 0; x < nt; ++x) tile_seg2[run + x] = s;
        run += nt;
    }
    if (threadIdx.x == 0) {
        total = min(total, A.tiles_ub);
        tile_begin2[nseg] = total;
        if (in_lds) tb[nseg] = total;
    }
    if (in_lds) {
        // every thread maps its share of the tiles to segments (binary search in LDS)
        __syncthreads();
        for (uint32_t t = threadIdx.x; t < min(total, A.tiles_ub); t += blockDim.x)
            tile_seg2[t] = upper_index(tb, nseg, t);
    }
}

// Runs the side job on workgroup `b` of its extra workgroups.  `lds`: the
// hosting kernel's dynamic LDS (lds_words words).
__device__ __forceinline__ void run_side_job(const SideJob& J, uint32_t b, uint32_t* lds, uint32_t lds_words) {
    if (J.kind == kSideSetup2) {
        if (b == 0) setup_pass2_block(J.setup2, lds, lds_words);
    } else if (J.kind == kSidePlan) {
        join_plan_block(J.plan, J.plan.start, J.plan.n_r + J.plan.n_s);
    }
}

}  // namespace hj
