// Internal declarations shared by the engine (hj_api.cpp) and the kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <cmath>

namespace hj {

// Partitioned tuples are 64-bit words: the key in the low 32 bits, the rid in
// the high 32, so that a run of a partition is one stream of 8-byte stores and
// a join reads key and rid of a tuple with one load.  Measured on MI355X
// (2^25 tuples, 8192-tuple tiles): the scatter takes 92 us at 64 partitions
// and 105 us at 1024 with such words, 99 and 120 us with two columns.
typedef uint64_t Tuple;

// One segment of a second partitioning pass (a pass-1 partition of R or of S):
// tuples [base, base + n) of the first copy, which become the same positions
// of the second one, grouped by partition number.
struct PartSeg {
    uint32_t base, n;
};

// One join work item: an R partition and a chunk of its S partition
// (positions relative to each relation's base in the scratch arrays).
struct ItemRec {
    uint32_t r_off, r_len;
    uint32_t s_begin, s_n;
};

// One final partition pair of a PHJ: ranges in the partitioned R and S arrays
// (positions relative to each relation's base in the scratch arrays).
struct PartPair {
    uint32_t r_off, r_len;
    uint32_t s_off, s_len;
};

// Bound on the polls of one unset status in a chained scan (decoupled
// look-back): predecessors always publish (they took their tickets earlier and
// wait on nothing later), the bound only guarantees that a kernel ends.
constexpr uint32_t kMaxStatusPolls = 1u << 20;
// Bits of a call's device error word (the first 8 bytes of its workspace; the
// call's first kernel clears it).
constexpr uint64_t kErrLookback = 1;  // a chained scan gave up waiting for a predecessor
// How the chained scans of one call wait, and where a scan that gives up says so.
struct ScanCtl {
    uint64_t* err;       // the call's error word (kErrLookback is or-ed in)
    uint32_t max_polls;  // polls of one unset status before giving up
    uint32_t stall;      // failure injection: the first tile of every chained scan never publishes
};

// Launch recorder: the stream, the call's error word, optional per-launch HIP
// event timing, and the first launch error.
struct Recorder {
    hipStream_t stream = nullptr;
    ScanCtl ctl{nullptr, kMaxStatusPolls, 0};
    // the call's first kernel clears this word (nullptr: the word belongs to an
    // enclosing batch that cleared it already)
    uint64_t* err_clear = nullptr;
    // failure injection: the launch of this phase reports a launch failure
    const char* fail_phase = nullptr;
    const char* cur = nullptr;
    bool timed = false;
    uint32_t n = 0, cap = 0;
    const char** names = nullptr;
    hipEvent_t* ev = nullptr;  // 2 per launch
    hipError_t err = hipSuccess;
    void before(const char* name);
    void after();
};

// ---- scan.hip ----
// Exclusive scans in one launch.  `state` needs scan_state_words(n) words that
// are zero when the scan starts (it leaves them non-zero).  `in` may equal `out`.
size_t scan_state_words(uint64_t n);
void scan_u32(const uint32_t* in, uint32_t* out, uint64_t n, uint64_t* state, uint32_t* total, Recorder& rec);
void scan_u64(const uint64_t* in, uint64_t* out, uint64_t n, uint64_t* state, uint64_t* total, Recorder& rec);
// Clears the words a and b (either may be nullptr) in one small launch.
void zero_pair(uint64_t* a, uint64_t* b, Recorder& rec);

// ---- shj.hip ----
constexpr uint32_t kShjBlock = 256;
constexpr uint32_t kShjTile = 2048;  // S tuples per probe tile
constexpr uint32_t kShjWavesPerBlock = kShjBlock / 64;
// Slots of the SHJ table per R row (linear probing, load factor 1 / this).
constexpr double kShjSlotsPerRow = 2.0;
// Slots of the SHJ table over n_r rows: kShjSlotsPerRow per row, rounded up to
// whole 128-byte lines.
inline uint64_t shj_slots(uint64_t n_r) {
    const uint64_t s = (uint64_t)(kShjSlotsPerRow * (double)(n_r < 1 ? 1 : n_r) + 0.999999);
    return (s + 15) / 16 * 16;
}
struct HotKeys;  // keys the build saw in long push runs (hj_device.h)
struct HeavyQueue;
// Fills the table with empty slots, clears the hot-key record and the call's
// error word (rec.err_clear); total, queue (or nullptr): a one-pass join's count
// and queue, cleared with them.
void shj_fill(uint64_t* table, uint64_t nslots, HotKeys* hot, uint64_t* total, HeavyQueue* queue, Recorder& rec);
// nt: R's keys read with non-temporal loads (kNtMinBuild).
void shj_build(const int32_t* key, uint64_t n, uint64_t* table, uint32_t* next, uint64_t nslots,
               HotKeys* hot, bool nt, Recorder& rec);
// Heavy S tuples of a one-pass probe (SHJ, and the HBM-table partitions of
// PHJ) are handed to a device-wide queue: any workgroup that has finished its
// own work claims chunks of the tuple's R rows and writes their matches (one
// 64-byte record per tuple; the queue is zeroed before each probe).
constexpr uint32_t kHeavyJobs = 256;
// R rows per claimed chunk of a table over all of R (SHJ) and of a partition's,
// and how many R rows a tuple must have to be queued at all.  A partition's
// queue holds few tuples: 2 steps of a workgroup per chunk spread them over the
// device (1M x 16M, a tenth of R on one key, one-pass write: 237 us with chunks
// of 65536 rows, 200 with 8192); SHJ's is full, where more claims and more
// reservations cost (1M x 16M: 1157 us and 1404).
constexpr uint32_t kHelpChunk = 1u << 16;
constexpr uint32_t kHelpChunkPart = 1u << 13;
constexpr uint32_t kQueueRows = 1u << 16;
struct HeavyJob {
    int32_t key, srid;
    uint32_t valid;        // 1 once the fields below are written
    uint32_t write_next;   // next chunk to claim
    uint32_t r_off, r_len; // the R rows that hold the tuple's matches (SHJ: all of R)
    uint32_t pad[10];
};
struct HeavyQueue {
    uint32_t n;            // tuples handed in (may exceed kHeavyJobs: the rest stay with their workgroup)
    // PHJ one-pass write: the HBM-table build sets `wait` when a partition can
    // hand tuples in (more than kQueueRows rows) and adds that partition's
    // work items to items_expected; those items count themselves done, and the
    // write's helper workgroups help the queue until items_done reaches
    // items_expected
    uint32_t wait;
    uint32_t items_expected;
    uint32_t items_done;
    uint32_t pad[12];
    HeavyJob job[kHeavyJobs];
};
static_assert(sizeof(HeavyJob) == 64 && sizeof(HeavyQueue) % 8 == 0, "queue layout");
// Sets *d_count to zero and empties the queue (one-pass SHJ probes); clears
// the call's error word (rec.err_clear).
void shj_zero_one_pass(uint64_t* d_count, HeavyQueue* q, Recorder& rec);

// The probe kernels read R's columns (r_key, r_rid, n_r rows, the ones the
// table was built from) for keys with long chains.  shj_count also clears the
// call's error word (rec.err_clear) and the count scan's state: it runs before
// that scan.
void shj_count(const int32_t* s_key, uint64_t n_s, const uint64_t* table, const uint32_t* next,
               uint64_t nslots, const int32_t* r_key, uint64_t n_r, const HotKeys* hot, uint64_t* wave_cnt,
               uint64_t* scan_state, uint64_t scan_words, Recorder& rec);
void shj_write(const int32_t* s_key, const int32_t* s_rid, uint64_t n_s, const uint64_t* table,
               const uint32_t* next, uint64_t nslots, const int32_t* r_key, const int32_t* r_rid,
               uint64_t n_r, const HotKeys* hot, const uint64_t* wave_base, uint64_t* total, HeavyQueue* heavy,
               int32_t* out_r, int32_t* out_s, uint64_t capacity,
               Recorder& rec);  // wave_base == nullptr: one-pass output into *total

// ---- phj_partition.hip ----
constexpr uint32_t kMinPartBlock = 256;
// Default partitioning tile: 8192 tuples when the join has enough tuples to
// fill the chip several times over with such tiles and needs the longer
// partition runs they give (2^25 tuples or more, or 2^24 or more in one pass of
// 8 or more radix bits), else 4096 (measured on MI355X).
inline uint32_t default_tile(uint64_t n_r, uint64_t n_s, uint32_t passes, uint32_t bits1) {
    const uint64_t n = n_r + n_s;
    return (n >= (1ull << 25) || (n >= (1ull << 24) && passes == 1 && bits1 >= 8)) ? 8192u : 4096u;
}
struct PassCfg {
    uint32_t shift;      // radix bits taken from (hash >> shift)
    uint32_t bits;       // partitions = 1 << bits
    uint32_t hash_kind;  // hj_hash
    uint32_t tile;       // tuples per workgroup of the pass (scatter_tile)
    uint32_t nt;         // input read with non-temporal loads
};
// Non-temporal loads of data a launch reads once pay only once a join's
// relations outgrow the caches; below that, plain loads leave lines that a
// later launch reads again.  Measured on MI355X (PHJ, one-pass output):
// partitioning tiles from |R| + |S| = 2^24 on (8M x 16M: -3.7%, 16M x 16M:
// -5.8%; 1M x 4M: +5.7%, 4M x 8M: +1.6%), the join's S chunks only while
// also |S| <= 2 |R| (16M x 16M: -1.2%; 2M x 16M and 16M x 64M: +1.5%), the
// SHJ build's R keys from |R| = 2^23 (16M: -7% build time; the probe's S
// loads gained nothing and stay plain).
constexpr uint64_t kNtMinTuples = 1ull << 24;
constexpr uint64_t kNtMinBuild = 1ull << 23;
// Two passes of 4..kCountedMaxBits radix bits in all.  (A statement about plans
// only, kept for those who ask it: which histogram counts what is counts_final.)
constexpr uint32_t kCountedMaxBits = 13;
inline bool counted_pass2(uint32_t passes, uint32_t b1, uint32_t b2) {
    return passes == 2 && b1 + b2 >= 4 && b1 + b2 <= kCountedMaxBits;
}
// How the partitions of a plan are made.  Up to kFuseBits radix bits in all,
// two passes run as one scatter straight into the final partitions: a
// workgroup's runs stay long enough (4 tuples of 16384 at 4096 partitions,
// the lines of one XCD's runs fit its L2) that one scatter beats two.
// Measured on MI355X, 2^25 tuples: one scatter into 2^12 partitions 151 us,
// two of 2^6 each 92 us; 2^13 partitions at once would need runs of 2.
constexpr uint32_t kFuseBits = 12;
inline bool one_scatter(uint32_t passes, uint32_t b1, uint32_t b2) { return passes == 1 || b1 + b2 <= kFuseBits; }
// Whether the histogram of the input counts the final partitions (up to 2^15
// counters of a workgroup in LDS, 128 KiB); else pass 2 has its own.  Plans of
// two scatters do so while the workgroups' rows fit the first copy (8 bytes a
// tuple), where they lie until it is written: up to 520 rows of 4 bytes for each
// final partition and half as many for pass 1.  (With fewer rows for fewer tuples
// 64K x 64K at 7+6 bits took 135 us, 130 with the second histogram.)
constexpr uint32_t kWideCountBits = 15;
inline bool counts_final(uint32_t passes, uint32_t b1, uint32_t b2, uint64_t n) {
    return one_scatter(passes, b1, b2) || (b1 + b2 <= kWideCountBits && n >= 400ull << (b1 + b2));
}
// Whether the last scatter clears the HBM tables of oversized partitions (it
// needs the final partitions' sizes before it starts), else a launch of its own.
inline bool counted_clears_tables(uint32_t b2) { return b2 <= 6; }
inline bool scatter_clears(uint32_t passes, uint32_t b1, uint32_t b2, uint64_t n) {
    return one_scatter(passes, b1, b2) || (counts_final(passes, b1, b2, n) && counted_clears_tables(b2));
}
// Tuples per workgroup of a pass into 2^bits partitions: the plan's tile, or
// more, as long as every CU still has a workgroup: at a high fan-out, where a
// 4096-tuple tile's runs would be too short, and instead of tiles below 4096,
// each of which reserves its runs as a large one does.  Measured, 2^25 tuples:
// 2^10 partitions 117 / 105 / 122 us with 4096 / 8192 / 16384 tuples, 2^11 149 /
// 123 / 132 us, 2^12 186 / 190 / 151 us; 2^6 partitions and
// 268 MB of HBM tables cleared beside, 200 us with 1024 and 131 with 4096.
constexpr uint32_t kMaxScatterTile = 16384;
inline uint32_t scatter_tile(uint32_t tile, uint32_t bits, uint64_t n) {
    while (tile < 4096 && n >= 256ull * 2 * tile) tile *= 2;
    const uint32_t want = bits == 12 ? kMaxScatterTile : bits >= 10 ? 8192u : tile;
    return tile < 4096 || want <= tile || n < 256ull * want ? tile : want;
}
// Threads of a partitioning workgroup that takes `tile` tuples.
inline uint32_t scatter_block(uint32_t tile) { return tile >= 8192 ? 1024u : tile >= 4096 ? 512u : kMinPartBlock; }
// Replicas of a pass-1 partition's cursor: one for each of the 8 XCDs (tile t
// reserves in replica t mod 8, and workgroups go to the XCDs round-robin), so that
// the tuples that one XCD writes to a partition are contiguous and lines are
// written by one L2.  Measured on MI355X, 2^25
// tuples, 8192-tuple tiles: 92 against 113 us at 2^6 partitions with one
// cursor for all, 105 against 146 us at 2^10.  Small joins keep one.
inline uint32_t cursor_replicas(uint64_t tiles) { return tiles >= 64 ? 8u : 1u; }

// The histogram's workgroups and their count rows.  Workgroup (x, q) = x + q nx
// counts a contiguous share of the tiles x, x + nx, ... of replica x and writes
// its counts as row x + q nx; a workgroup that meets both relations writes R's
// there and S's to row grid + x (only one of a replica does).
struct HistRows {
    uint32_t log_nx, log_groups;  // log2 of the replicas, of the workgroups per replica
    __host__ __device__ uint32_t nx() const { return 1u << log_nx; }
    __host__ __device__ uint32_t groups() const { return 1u << log_groups; }
    __host__ __device__ uint32_t grid() const { return 1u << (log_nx + log_groups); }
    __host__ __device__ uint32_t rows() const { return grid() + nx(); }
    // tiles of replica x below tile t
    __host__ __device__ uint32_t tiles_of(uint32_t x, uint32_t t) const {
        return t > x ? (t - x + nx() - 1) >> log_nx : 0u;
    }
    // first tile (in the replica's count) of workgroup q of a replica of `of` tiles
    __host__ __device__ uint32_t first(uint32_t of, uint32_t q) const {
        return (uint32_t)(((uint64_t)of * q) >> log_groups);
    }
};
// At most one workgroup per tile; fewer at many counters, whose rows the next
// launch sums.
inline HistRows hist_rows(uint64_t tiles, uint32_t nx, uint32_t count_bits) {
    const uint32_t cap = count_bits > 13 ? 256u : count_bits > 10 ? 512u : 1024u;
    HistRows h{nx == 8 ? 3u : 0u, 0};
    while (2ull * h.grid() <= cap && 2ull * h.grid() <= tiles) ++h.log_groups;
    return h;
}
// Small joins: the histogram writes one row per tile and every workgroup of the
// scatter sums the rows itself, which saves the launch that makes the starts.
// The rows (kSelfWords words at most) are read by every scatter workgroup, up to
// 32 words a thread (256 rows of 64 counters by 256 threads: a build of 262144
// rows 24.4 us, 15.0 with the launch).
constexpr uint32_t kSelfBits = 8;
constexpr uint32_t kSelfWords = 16384;
inline bool self_starts(uint64_t tiles, uint32_t bits, uint32_t tile) {
    const uint64_t most = 32ull * scatter_block(tile);
    return bits <= kSelfBits && (tiles << bits) <= (most < kSelfWords ? most : kSelfWords);
}

// The input of a join's first pass and what its histogram leaves for later
// launches.  R's tiles are numbered first; all positions are those of the
// partitioned copies (R's tuples, then S's).
struct Pass1 {
    const int32_t* rk;
    const int32_t* rr;
    const int32_t* sk;
    const int32_t* sr;
    uint32_t n_r, n_s;
    uint32_t nt_r, ntiles;  // tiles of R, of both
    uint32_t self;          // self_starts: rows per tile
    uint32_t fine_bits;     // bits of pass 2 when pass 1 counts its partitions too, else 0
    HistRows h;
    uint32_t* rows;         // [h.rows() (self: ntiles)][2^(bits + fine_bits)] counts
    uint32_t* rows1;        // fine_bits: [h.rows()][2^bits] the same per pass-1 partition
    uint64_t* zero;         // words the histogram clears for later launches
    uint64_t nzero;
    uint64_t* err_clear;    // the call's error word, cleared too (or nullptr)
};
// What the starts launch makes of the rows.
struct StartArgs {
    uint32_t* cur1;         // [rel][x][p]: first free position of replica x in pass-1 partition p
    uint32_t* start1;       // [2 << bits, + 1] partition starts of pass 1
    uint32_t* cnt2;         // fine_bits: tuples per final partition,
    uint32_t* start2;       //   and their starts
    uint64_t* state1;       // scan states (start_state_words; cleared by the histogram)
    uint64_t* state2;
    uint32_t* big;          // set when an R partition has more than lds_cap tuples (cleared by the histogram)
    const PartPair* r_pairs;  // R's partitions come from a built table (then n_r == 0 here)
    uint32_t lds_cap;       // (npart == 0: the final partitions are not known yet)
    uint32_t npart;
    ScanCtl ctl;
};
constexpr uint32_t kStartCols = 64;  // partitions per workgroup of the starts launch
inline size_t start_state_words(uint64_t partitions) { return 1 + (2 * partitions + kStartCols - 1) / kStartCols; }

Pass1 make_pass1(const int32_t* rk, const int32_t* rr, uint32_t n_r, const int32_t* sk, const int32_t* sr,
                 uint32_t n_s, uint32_t tile);
// Histogram of the input into rows.
void part_hist(const Pass1& p1, const PassCfg& cfg, Recorder& rec);
// Partition starts and cursors from the rows.
void part_starts(const Pass1& p1, const PassCfg& cfg, const StartArgs& st, Recorder& rec);
// Histogram of a second pass over the tuples `in` of the segments, into
// cnt2[seg << bits | p] (zero before).
void part_hist2(const Tuple* in, const PartSeg* segs, const uint32_t* tile_begin, const uint32_t* tile_seg,
                uint32_t nseg, uint32_t grid, const PassCfg& cfg, uint32_t* cnt2, Recorder& rec);
// HBM tables a scatter clears (two slots per R tuple at twice its position):
// those of R's partitions of more than lds_cap tuples that S has tuples for,
// when *big is set (self_starts: the scatter's workgroups see for themselves).
struct ClearTables {
    uint64_t* table;          // nullptr: nothing to clear
    const uint32_t* big;
    const uint32_t* start;    // starts of R's npart partitions (positions in R), then of S's, and their end
    const PartPair* r_pairs;  // instead of R's starts, for a built table
    uint32_t npart, n_r, lds_cap;
    // Workgroups that share the clearing: the tiles, or more, which then only clear (a probe of a
    // large table by few tuples: 16M rows in 256 partitions by one tuple, one tile: 1.9 ms, so 0.08).
    uint32_t share;
};
// (one per CU at most, and 4096 rows, one round of 64 KB, at least)
inline uint32_t clear_share(uint64_t n_r) { return (uint32_t)(n_r < 4096ull * 256 ? (n_r + 4095) / 4096 : 256); }
// `side`: extra workgroups appended to the grid that run the next step's setup
// (hj_side.h: the pass-2 segment table or the join plan).
struct SideJob;
// First pass: the input's tuples to `out`, or to two columns (key_out, rid_out)
// when out is nullptr (tiles of kColumnsTile, MurmurHash 2.0).
constexpr uint32_t kColumnsTile = 8192;
// cur1: the starts launch's cursors (self_starts: unused).
void part_scatter(const Pass1& p1, const PassCfg& cfg, uint32_t* cur1, Tuple* out, int32_t* key_out,
                  int32_t* rid_out, const ClearTables& clr, const SideJob& side, Recorder& rec);
// Second pass over segments of `in`: partition p of segment s starts at
// start2[s << bits | p], cnt2 holds its tuples and is counted down.
void part_scatter2(const Tuple* in, const PartSeg* segs, const uint32_t* tile_begin, const uint32_t* tile_seg,
                   uint32_t nseg, uint32_t grid, const PassCfg& cfg, const uint32_t* start2, uint32_t* cnt2,
                   Tuple* out, const ClearTables& clr, const SideJob& side, Recorder& rec);

// ---- phj_join.hip ----
constexpr uint32_t kJoinBlock = 512;
constexpr uint32_t kJoinWaves = kJoinBlock / 64;
constexpr uint32_t kJoinSub = 4608;     // S tuples per probe round of a work item (9 per lane)
constexpr uint32_t kJoinChunk = 2 * kJoinSub;  // S tuples per work item (probed kJoinSub at a time)
// R tuples per HBM-table build item: 4 rounds of a workgroup, more in a
// partition of more than kOvfBigPart tuples, about 128 items of it, up to 32
// rounds.  Small items keep the build's latency low (a round is a chain of
// dependent accesses, about 3 us); in a large partition, which is large because
// a key is heavy as often as not, each item's pushes of that key end in one
// exchange on its slot, and those exchanges serialize.  A partition of 106K
// rows (1M x 16M, a tenth of R on one key) took 98 us in items of 16384.
constexpr uint32_t kOvfChunk = 2048;
constexpr uint32_t kOvfChunkBig = 16384;
constexpr uint32_t kOvfBigPart = 1u << 16;
constexpr uint32_t kOvfGrid = 2048;  // workgroups of the HBM-table clear and build launches (8 per CU)
__host__ __device__ inline uint32_t ovf_chunk(uint32_t r_len) {
    uint32_t c = kOvfChunk;
    if (r_len > kOvfBigPart)
        while (c < kOvfChunkBig && c < r_len / 128) c *= 2;
    return c;
}
constexpr uint32_t kMaxLdsCap = 8192;   // largest R partition held in LDS
// R tuples per thread of the LDS build (a kernel template argument: the build
// keeps them in registers), by lds_cap class.
constexpr uint32_t kRptSmall = 4, kRptMid = 9, kRptLarge = kMaxLdsCap / kJoinBlock;
inline uint32_t join_rpt(uint32_t lds_cap) {
    return lds_cap <= kRptSmall * kJoinBlock ? kRptSmall : (lds_cap <= kRptMid * kJoinBlock ? kRptMid : kRptLarge);
}
// The join plan (final partition table, work-item and overflow-chunk scans and
// maps) runs as a side job of the last scatter (hj_side.h); its state needs
// plan_state_words(2^total_bits) words that are zero when it starts.
size_t plan_state_words(uint32_t P);
// Upper bounds of the HBM-table build items and of the join work items.
uint32_t ovf_grid(uint32_t P, uint64_t n_r);
uint32_t join_grid(uint32_t P, uint64_t n_s);  // (a multiple of 8 kItemGroup)
constexpr uint32_t kItemGroup = 16;  // consecutive join items dealt to one XCD
// Dynamic LDS bytes of the join kernels for tables of up to lds_cap tuples of a
// partition on `bits` radix bits (0: a direct join).
size_t join_lds_bytes(uint32_t lds_cap, uint32_t bits, bool write);
// Whether the tables are built by a launch of their own before the join: when
// partitions three standard deviations above the mean do not fit LDS, many have
// tables and the build is worth a launch; else only a skewed R has any, and the
// join launch that probes them first builds them.  Measured: 16M x 16M at 8 bits
// (every partition a table) 2237 us with the build inside the join and 1764
// before it; 1M x 16M with a tenth of R on one key 237 against 243.
inline bool tables_expected(uint64_t n_r, uint32_t P, uint32_t lds_cap) {
    if (n_r <= lds_cap) return false;
    const double mean = (double)n_r / P;
    return mean + 3.0 * std::sqrt(mean) > (double)lds_cap;
}
// The HBM tables of R's oversized partitions (from the join plan): build items
// by partition, their number, and the words (zero before) [1], [2] that count
// items taken and built (nullptr: built by join_ovf_build).
struct OvfBuild {
    const PartPair* pairs;
    const uint32_t* begin;  // [P + 1]
    const uint32_t* part;   // partition of every item
    const uint32_t* total;  // begin + P
    uint32_t* words;
    uint64_t* err;          // the call's error word
};
// Clears the HBM tables where the last scatter did not (ClearTables).
void join_ovf_clear(const OvfBuild& b, uint32_t grid, uint64_t* ovf_table, Recorder& rec);
// Builds them (tables_expected).
void join_ovf_build(const OvfBuild& b, uint32_t grid, const Tuple* rt, uint64_t* ovf_table, uint32_t* ovf_next,
                    HotKeys* hot, HeavyQueue* heavy, Recorder& rec);
// rt, st: partitioned R and S.  The first of a plan's join launches (the count,
// or the one-pass write) builds the HBM tables before it probes them, when they
// are not yet built (OvfBuild::words).
// hot: where the build records its hot keys (zeroed before); heavy: the
// one-pass queue (nullptr for count -> scan -> write), whose `wait` it sets.
// item_rec comes from the join plan; grid: join_grid; bits, hash: how R and S are
// partitioned (all radix bits).
void join_count(const ItemRec* item_rec, uint32_t grid, const Tuple* rt, const Tuple* st, uint32_t lds_cap,
                uint32_t bits, uint32_t hash, const OvfBuild& ovf, uint64_t* ovf_table, uint32_t* ovf_next,
                HotKeys* hot, uint64_t* wave_cnt, bool nt_s, Recorder& rec);
void join_write(const ItemRec* item_rec, uint32_t grid, const Tuple* rt, const Tuple* st, uint32_t lds_cap,
                uint32_t bits, uint32_t hash, const OvfBuild& ovf, uint64_t* ovf_table, uint32_t* ovf_next,
                HotKeys* hot, const uint64_t* wave_base, uint64_t* total, int32_t* out_r, int32_t* out_s, uint64_t capacity,
                HeavyQueue* heavy, bool nt_s, Recorder& rec);
// nt_s: S chunks read with non-temporal loads (LDS-table items).
// wave_base == nullptr selects the one-pass write: `total` must be zero on entry
// and ends as the number of pairs; `heavy` (one-pass only, zeroed before the
// HBM-table build, or nullptr) takes the heavy S tuples of HBM-table
// partitions of more than kQueueRows rows.  `hot`: the keys the
// HBM-table build recorded (their S tuples skip the chain walk).
// Writes zero to *d_count (joins with an empty side) and clears the call's
// error word (rec.err_clear).
void write_zero_count(uint64_t* d_count, Recorder& rec);

// ---- direct joins (no partitioning: R fits one LDS table) ----
// One job of the direct kernels.  Work item = (job, `chunk` S tuples); items of
// job j are [item0, item0 + ceil(n_s / chunk)).
struct DirectJob {
    const int32_t* rk;
    const int32_t* rr;
    const int32_t* sk;
    const int32_t* sr;
    int32_t* out_r;
    int32_t* out_s;
    uint64_t capacity;
    uint64_t* count;  // running total of the job's pairs (zeroed by direct_zero)
    uint32_t n_r, n_s, item0, chunk;
};
// S tuples per work item of a single direct join: one probe round while every
// item still runs at once (direct_blocks a CU), else kJoinChunk.  An item is a chain of
// dependent steps and a second round adds a load, a probe and a reservation to
// it; on idle CUs building R's table again costs nothing (2.2K x 26.7K:
// 18.3 to 13.7 us, 4K x 2M 23.3 to 19.0).  Batches keep kJoinChunk: their items fill the device.
uint32_t direct_chunk(uint64_t n_s, uint32_t lds_cap);
// A single direct join, its job a kernel argument.  One work item zeroes the
// job's count and the call's error word (rec.err_clear) itself; more need a
// launch before them (1K x 3K, two launches and one: 13.9 and 11.0 us).
void direct_join_one(const DirectJob& j, uint32_t lds_cap, Recorder& rec);
void direct_zero(const DirectJob* jobs, uint32_t njobs, Recorder& rec);
// lds_cap >= every job's n_r (<= kMaxLdsCap).
void direct_join(const DirectJob* jobs, const uint32_t* item_job, uint32_t nitems, uint32_t lds_cap,
                 Recorder& rec);

}  // namespace hj
