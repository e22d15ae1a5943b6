// Join engine: argument validation, workspace layouts and the launch
// sequences of the simple (SHJ, Algorithm 1) and radix-partitioned (PHJ,
// Algorithm 2) hash joins, shared by the single-join ABI and the batch
// executor.
//
// SHJ: fill table -> build -> count -> scan -> write (or build -> one-pass write).
// PHJ: hist -> starts -> scatter (R and S in the same launches; with more than
// kFuseBits radix bits a second scatter, the partition pairs planned beside the
// last one; small joins without the starts launch) -> count -> scan -> write
// (or one-pass write); the first join launch builds the HBM tables of oversized
// R partitions (where many are expected, a launch before it).
// Everything is enqueued on one stream; no host synchronisation, no
// host<->device copy and no allocation happen here.
#include "engine.h"
#include "hj_side.h"

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <string>

namespace hj {
namespace eng {

namespace {
thread_local std::string g_err;
}  // namespace

const char* last_error() { return g_err.c_str(); }
void clear_error() { g_err.clear(); }

hj_status fail(hj_status s, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return s;
}

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

uint32_t ceil_log2(uint64_t v) {
    uint32_t l = 0;
    while ((1ull << l) < v) ++l;
    return l;
}

uint64_t cdiv(uint64_t a, uint64_t b) { return (a + b - 1) / b; }

// Bump-carves aligned sub-buffers out of one workspace.
struct Carver {
    char* base;
    size_t off = 0;
    explicit Carver(void* b) : base((char*)b) {}
    template <typename T>
    T* take(uint64_t count) {
        T* p = base ? (T*)(base + off) : nullptr;
        off += align_up(sizeof(T) * (size_t)std::max<uint64_t>(count, 1));
        return p;
    }
};


// LDS per CU on gfx950, and what a join workgroup is planned with: 12 bytes per
// tuple and 1.5 KB (static LDS plus allocation rounding; measured: a 54,080-byte
// table set no longer fits three workgroups per CU, 53,312 bytes does).  Tables
// with one bucket per row (join_lds_bytes) take at most that; with two, which
// they have where three workgroups still share a CU, up to a third of a CU's LDS
// each: three workgroups are as many as the write kernels' registers allow, so
// the capacities that the plan tells apart by more than three share the figure.
constexpr size_t kLdsPerCu = 160 * 1024;

uint32_t join_blocks_per_cu(uint32_t cap) { return (uint32_t)(kLdsPerCu / (12ull * cap + 1536)); }

// Default LDS table capacity: room for a partition three standard deviations
// above the mean size (uniform hashing), then grown to the largest capacity
// that keeps the same number of write-kernel workgroups per CU and the same
// build kernel (registers per thread grow with the build's tuples per thread).
uint32_t auto_lds_cap(uint64_t n_r, uint32_t P) {
    const double avg = std::ceil((double)n_r / (double)P);
    const double need = avg + 3.0 * std::sqrt(avg) + 32.0;
    uint32_t cap = (uint32_t)std::min<double>(hj::kMaxLdsCap, std::max(256.0, need));
    cap = (cap + 63) / 64 * 64;
    if (cap > hj::kMaxLdsCap) cap = hj::kMaxLdsCap;
    const uint32_t bpc = join_blocks_per_cu(cap);
    while (cap + 64 <= hj::kMaxLdsCap && join_blocks_per_cu(cap + 64) == bpc &&
           hj::join_rpt(cap + 64) == hj::join_rpt(cap))
        cap += 64;
    return cap;
}

namespace {
// The parameters a plan runs with, every size-dependent choice filled in.
void fill_resolved(const hj_params* p, Plan* pl) {
    hj_params& r = pl->res;
    r = *p;
    r.algo = pl->phj ? HJ_PHJ : HJ_SHJ;
    r.tile = pl->tile;
    if (!pl->phj) return;
    r.passes = pl->passes;
    r.bits[0] = pl->b1;
    r.bits[1] = pl->b2;
    r.lds_cap = pl->lds_cap;
    if (pl->one_pass) r.flags |= HJ_FLAG_ONE_PASS;
}
}  // namespace

hj_status check_params(const hj_params* p, uint64_t n_r, uint64_t n_s, Plan* pl) {
    if (!p) return fail(HJ_ERR_INVALID, "params is NULL");
    if (p->algo == HJ_AUTO) {
        hj_params q = *p;
        auto_params(n_r, n_s, &q);
        return check_params(&q, n_r, n_s, pl);
    }
    if (p->flags & ~HJ_FLAG_ONE_PASS) return fail(HJ_ERR_INVALID, "unknown flags 0x%x", p->flags);
    if (p->algo != HJ_SHJ && p->algo != HJ_PHJ) return fail(HJ_ERR_INVALID, "unknown algo %u", p->algo);
    if (p->hash != HJ_HASH_IDENTITY && p->hash != HJ_HASH_MURMUR2)
        return fail(HJ_ERR_INVALID, "unknown hash %u", p->hash);
    if (p->tile != 0 && p->tile != 1024 && p->tile != 2048 && p->tile != 4096 && p->tile != 8192)
        return fail(HJ_ERR_INVALID, "tile must be 0 or a power of two in 1024..8192 (got %u)", p->tile);
    pl->phj = p->algo == HJ_PHJ;
    pl->one_pass = (p->flags & HJ_FLAG_ONE_PASS) != 0;
    pl->tile = p->tile ? p->tile : 4096;  // PHJ with partitioning: chosen below
    pl->hash = p->hash;
    pl->passes = 0;
    pl->b1 = pl->b2 = pl->B = 0;
    pl->P1 = pl->P2 = pl->P = 1;
    pl->lds_cap = 0;
    pl->nt_part = n_r + n_s >= hj::kNtMinTuples;
    pl->nt_s = pl->nt_part && n_s <= 2 * n_r;
    if (!pl->phj) {
        fill_resolved(p, pl);
        return HJ_OK;
    }
    if (p->passes == 0) {
        // no partitioning: R must fit one LDS table
        if (n_r > hj::kMaxLdsCap)
            return fail(HJ_ERR_INVALID, "passes 0 needs |R| <= %u (got %llu)", hj::kMaxLdsCap,
                        (unsigned long long)n_r);
        pl->passes = 0;
        pl->one_pass = true;
        const uint32_t need = (uint32_t)std::max<uint64_t>(256, (n_r + 63) / 64 * 64);
        pl->lds_cap = p->lds_cap ? std::max(p->lds_cap, need) : need;
        if (pl->lds_cap > hj::kMaxLdsCap) return fail(HJ_ERR_INVALID, "lds_cap above %u", hj::kMaxLdsCap);
        fill_resolved(p, pl);
        return HJ_OK;
    }
    if (p->passes != 1 && p->passes != 2)
        return fail(HJ_ERR_INVALID, "passes must be 0, 1 or 2 (got %u)", p->passes);
    pl->passes = p->passes;
    pl->b1 = p->bits[0];
    pl->b2 = p->passes == 2 ? p->bits[1] : 0;
    if (pl->b1 < 1 || pl->b1 > 13) return fail(HJ_ERR_INVALID, "bits[0] must be in 1..13 (got %u)", pl->b1);
    if (p->passes == 2 && (pl->b2 < 1 || pl->b2 > 13))
        return fail(HJ_ERR_INVALID, "bits[1] must be in 1..13 (got %u)", pl->b2);
    pl->B = pl->b1 + pl->b2;
    if (pl->B > kMaxRadixBits)
        return fail(HJ_ERR_INVALID, "total radix bits must be <= %u (got %u)", kMaxRadixBits, pl->B);
    pl->P1 = 1u << pl->b1;
    pl->P2 = 1u << pl->b2;
    pl->P = 1u << pl->B;
    if (p->lds_cap) {
        if (p->lds_cap % 64 || p->lds_cap < 256 || p->lds_cap > 8192)
            return fail(HJ_ERR_INVALID, "lds_cap must be 0 or a multiple of 64 in 256..8192 (got %u)",
                        p->lds_cap);
        pl->lds_cap = p->lds_cap;
    } else {
        pl->lds_cap = auto_lds_cap(n_r, pl->P);
    }
    if (!p->tile) pl->tile = hj::default_tile(n_r, n_s, pl->passes, pl->b1);
    fill_resolved(p, pl);
    return HJ_OK;
}

// Every workspace layout starts with the call's error word (kErrLookback;
// hj_workspace_status reads it), then its own buffers.
// Workspace layout; with base == nullptr only the size is computed.
struct PhjWs {
    uint64_t* err;
    hj::Tuple* A;        // partitioned R, then S: of pass 1, or of a plan's only scatter
    hj::Tuple* B;        //   of pass 2 (two scatters)
    hj::PartSeg* segs2;  // two scatters
    uint32_t* tb2;
    uint32_t* tseg2;
    uint32_t* start1;    // pass-1 partition starts (two scatters)
    uint32_t* start;     // final partition starts
    hj::PartPair* pairs;
    uint32_t* item_begin;
    uint32_t* ovf_begin;
    hj::ItemRec* item_rec;
    uint32_t* ovf_part;
    uint64_t* wave_cnt;
    uint64_t* ovf_table;
    uint32_t* ovf_next;
    uint32_t tile1, tile2;  // tuples per scatter workgroup
    uint64_t tiles1, tiles2_ub, items_ub, ovf_ub;
    bool self;              // self_starts
    bool clears;            // the last scatter clears the HBM tables
    hj::HistRows h;
    uint32_t* rows;         // the histogram's count rows, and the pass-1 ones (fine counts)
    uint32_t* rows1;
    uint32_t* cur1;         // first scatter's cursors
    uint32_t* cnt2;         // second scatter's counts
    // the block the histogram clears, `nzero` words from `zero` on:
    uint64_t* zero;
    uint64_t nzero;
    hj::HeavyQueue* heavy;  // one-pass heavy-tuple queue
    hj::HotKeys* hot;       // hot keys of the HBM-table build
    uint32_t* words;        // [0]: an R partition is oversized, [1], [2]: HBM-table build items taken, built
    uint64_t *st1, *st2;    // scan states: partition starts (pass 1, final),
    uint64_t* stw;          //   per-wave match counts,
    uint64_t* stp;          //   join plan
    size_t bytes;
};

// n_r, n_s: tuples partitioned by this call (either may be 0 for a table
// build or a probe); n_r_tab: tuples of the R that is joined (sizes the HBM
// tables of oversized R partitions).
PhjWs phj_layout(const Plan& pl, uint64_t n_r, uint64_t n_s, uint64_t n_r_tab, void* base) {
    PhjWs w{};
    Carver c(base);
    const uint64_t n = n_r + n_s;
    const bool one = hj::one_scatter(pl.passes, pl.b1, pl.b2);
    const bool hist2 = !hj::counts_final(pl.passes, pl.b1, pl.b2, n);
    w.clears = n_r_tab && hj::scatter_clears(pl.passes, pl.b1, pl.b2, n);
    const uint64_t Pc = one ? pl.P : pl.P1;  // partitions of the first scatter
    w.tile1 = hj::scatter_tile(pl.tile, one ? pl.B : pl.b1, n);
    w.tiles1 = cdiv(n_r, w.tile1) + cdiv(n_s, w.tile1);
    const uint32_t bits1 = one ? pl.B : pl.b1, cbits = hist2 ? pl.b1 : pl.B;
    w.self = one && hj::self_starts(w.tiles1, pl.B, w.tile1);
    w.h = hj::hist_rows(w.tiles1, hj::cursor_replicas(w.tiles1), cbits);
    w.err = c.take<uint64_t>(1);
    w.A = c.take<hj::Tuple>(n);
    // (plans of two passes have always reserved two copies: one scatter leaves
    // the second unused, and HJ_AUTO asks for one pass where one will do)
    if (pl.passes == 2) w.B = c.take<hj::Tuple>(n);
    if (!one) {
        w.tile2 = hj::scatter_tile(pl.tile, pl.b2, n);
        w.tiles2_ub = cdiv(n, w.tile2) + 2ull * pl.P1;
        w.segs2 = c.take<hj::PartSeg>(2ull * pl.P1);
        w.tb2 = c.take<uint32_t>(2ull * pl.P1 + 1);
        w.tseg2 = c.take<uint32_t>(w.tiles2_ub);
        w.start1 = c.take<uint32_t>(2 * Pc + 1);
    }
    w.pairs = c.take<hj::PartPair>(pl.P);
    w.item_begin = c.take<uint32_t>(pl.P + 1ull);
    w.ovf_begin = c.take<uint32_t>(pl.P + 1ull);
    w.items_ub = hj::join_grid(pl.P, n_s);
    w.ovf_ub = hj::ovf_grid(pl.P, n_r_tab);
    w.item_rec = c.take<hj::ItemRec>(w.items_ub);
    w.ovf_part = c.take<uint32_t>(w.ovf_ub);
    w.wave_cnt = c.take<uint64_t>(w.items_ub * hj::kJoinWaves);
    // the partition starts (2 P + 1 words of 32 bits) are last read by the
    // launch before the first that writes wave counts (at least 8 P words of 64)
    w.start = reinterpret_cast<uint32_t*>(w.wave_cnt);
    w.ovf_table = c.take<uint64_t>(2 * n_r_tab);
    w.ovf_next = c.take<uint32_t>(n_r_tab);
    static_assert(sizeof(hj::HotKeys) % sizeof(uint64_t) == 0, "hot keys in whole words");
    constexpr uint64_t kHeavyWords = sizeof(hj::HeavyQueue) / sizeof(uint64_t);
    constexpr uint64_t kHotWords = sizeof(hj::HotKeys) / sizeof(uint64_t);
    // Words that only launches before the first join launch use lie in the wave
    // counts' too, past the starts (at least 13 rows of P words are free there):
    // the first scatter's cursors, and the histogram's rows.  Rows that the
    // starts launch sums lie where copy A will when they fit; a histogram of few
    // tuples into many partitions makes fewer rows rather than grow the workspace.
    uint64_t spare = (2ull * pl.P + 1 + kAlign / 4 - 1) / (kAlign / 4) * (kAlign / 4);
    const uint64_t spare_end = w.items_ub * hj::kJoinWaves * 2;
    auto take_spare = [&](uint64_t words) {
        if (words > spare_end - spare) return c.take<uint32_t>(words);
        uint32_t* p = w.start ? w.start + spare : nullptr;
        spare += (words + kAlign / 4 - 1) / (kAlign / 4) * (kAlign / 4);
        return p;
    };
    if (w.self) {
        const uint64_t words = w.tiles1 << cbits;
        w.rows = pl.passes == 2 && words <= 2 * n ? reinterpret_cast<uint32_t*>(w.B) : take_spare(words);
    } else {
        w.cur1 = take_spare(2ull * w.h.nx() * Pc);
        const uint64_t fine = !one && !hist2 ? (uint64_t)1 << bits1 : 0, row = ((uint64_t)1 << cbits) + fine;
        while (w.h.log_groups && w.h.rows() * row > std::max(2 * n, spare_end - spare)) --w.h.log_groups;
        const uint64_t words = w.h.rows() * row;
        w.rows = words <= 2 * n ? reinterpret_cast<uint32_t*>(w.A) : take_spare(words);
        if (fine) w.rows1 = w.rows ? w.rows + ((uint64_t)w.h.rows() << cbits) : nullptr;
    }
    if (!one && !hist2) w.cnt2 = c.take<uint32_t>(2ull * pl.P);
    const uint64_t c2 = hist2 ? pl.P : 0;  // 64-bit words of a pass-2 histogram's counts
    const uint64_t n1 = w.self ? 0 : hj::start_state_words(Pc);
    const uint64_t n2 = one ? 0 : hist2 ? hj::scan_state_words(2ull * pl.P) : hj::start_state_words(pl.P);
    const uint64_t nw = hj::scan_state_words(w.items_ub * hj::kJoinWaves);
    const uint64_t np = hj::plan_state_words(pl.P);
    w.nzero = kHeavyWords + kHotWords + 2 + c2 + n1 + n2 + nw + np;
    w.zero = c.take<uint64_t>(w.nzero);
    w.bytes = c.off;
    if (w.zero) {  // (sizing only when there is no base: no arithmetic on a null pointer)
        uint64_t* z = w.zero;
        auto part = [&](uint64_t words) {
            uint64_t* p = z;
            z += words;
            return p;
        };
        w.heavy = reinterpret_cast<hj::HeavyQueue*>(part(kHeavyWords));
        w.hot = reinterpret_cast<hj::HotKeys*>(part(kHotWords));
        w.words = reinterpret_cast<uint32_t*>(part(2));
        uint64_t* c2p = part(c2);
        if (hist2) w.cnt2 = reinterpret_cast<uint32_t*>(c2p);
        w.st1 = part(n1);
        w.st2 = part(n2);
        w.stw = part(nw);
        w.stp = part(np);
    }
    return w;
}

// SHJ: the table over R (slots and row chains), then the probe's per-wave counts.
struct ShjTableWs {
    uint64_t* err;
    uint64_t* table;
    uint32_t* next;
    hj::HotKeys* hot;
    uint64_t nslots;
    size_t bytes;
};

ShjTableWs shj_table_layout(uint64_t n_r, void* base) {
    ShjTableWs w{};
    Carver c(base);
    w.nslots = hj::shj_slots(n_r);
    w.err = c.take<uint64_t>(1);
    w.table = c.take<uint64_t>(w.nslots);
    w.next = c.take<uint32_t>(n_r);
    w.hot = c.take<hj::HotKeys>(1);
    w.bytes = c.off;
    return w;
}

struct ShjProbeWs {
    uint64_t* err;
    hj::HeavyQueue* heavy;  // one-pass: heavy S tuples shared by all workgroups
    uint64_t* wave_cnt;
    uint64_t* st;  // scan state of the per-wave counts
    uint64_t nst;
    uint64_t tiles;
    size_t bytes;
};

ShjProbeWs shj_probe_layout(uint64_t n_s, void* base) {
    ShjProbeWs w{};
    Carver c(base);
    w.tiles = cdiv(n_s, hj::kShjTile);
    w.err = c.take<uint64_t>(1);
    w.heavy = c.take<hj::HeavyQueue>(1);
    w.wave_cnt = c.take<uint64_t>(w.tiles * hj::kShjWavesPerBlock);
    w.nst = hj::scan_state_words(w.tiles * hj::kShjWavesPerBlock);
    w.st = c.take<uint64_t>(w.nst);
    w.bytes = c.off;
    return w;
}

size_t shj_bytes(uint64_t n_r, uint64_t n_s) {
    return shj_table_layout(n_r, nullptr).bytes + shj_probe_layout(n_s, nullptr).bytes;
}

// Direct join (PHJ with no partitioning pass): the error word alone.
size_t direct_bytes() {
    Carver c(nullptr);
    c.take<uint64_t>(1);
    return c.off;
}

size_t ws_bytes_for(const Plan& pl, uint64_t n_r, uint64_t n_s) {
    if (pl.phj && pl.passes == 0) return direct_bytes();
    return pl.phj ? phj_layout(pl, n_r, n_s, n_r, nullptr).bytes : shj_bytes(n_r, n_s);
}

size_t table_bytes_for(const Plan& pl, uint64_t n_r) {
    if (pl.phj && pl.passes == 0) return kAlign;  // the table is R itself (nothing is stored)
    return pl.phj ? phj_layout(pl, n_r, 0, 0, nullptr).bytes : shj_table_layout(n_r, nullptr).bytes;
}

size_t probe_bytes_for(const Plan& pl, uint64_t n_r, uint64_t n_s) {
    if (pl.phj && pl.passes == 0) return direct_bytes();
    return pl.phj ? phj_layout(pl, 0, n_s, n_r, nullptr).bytes : shj_probe_layout(n_s, nullptr).bytes;
}

void run_direct(const Plan& pl, const hj_rel& R, const hj_rel& S, const hj_out& out,
                uint64_t* d_count, hj::Recorder& rec) {
    hj::DirectJob j{};
    j.rk = R.key;
    j.rr = R.rid;
    j.sk = S.key;
    j.sr = S.rid;
    j.out_r = out.rid_r;
    j.out_s = out.rid_s;
    j.capacity = out.capacity;
    j.count = d_count;
    j.n_r = (uint32_t)R.n;
    j.n_s = (uint32_t)S.n;
    j.chunk = hj::direct_chunk(S.n, pl.lds_cap);
    hj::direct_join_one(j, pl.lds_cap, rec);
}

hj_status check_call(const hj_params* p, const hj_rel* R, const hj_rel* S, const hj_out* out, void* ws,
                     size_t ws_bytes, uint64_t* d_count, Plan* pl) {
    if (!R || !S || !out) return fail(HJ_ERR_INVALID, "R, S and out must not be NULL");
    hj_status st = check_params(p, R->n, S->n, pl);
    if (st != HJ_OK) return st;
    if (R->n > kMaxRows || S->n > kMaxRows)
        return fail(HJ_ERR_INVALID, "relations must have fewer than 2^31 tuples");
    if (R->n && (!R->key || !R->rid)) return fail(HJ_ERR_INVALID, "R has tuples but a NULL array");
    if (S->n && (!S->key || !S->rid)) return fail(HJ_ERR_INVALID, "S has tuples but a NULL array");
    if (out->capacity && (!out->rid_r || !out->rid_s))
        return fail(HJ_ERR_INVALID, "out has capacity but a NULL array");
    if (!d_count) return fail(HJ_ERR_INVALID, "d_count is NULL");
    const size_t need = ws_bytes_for(*pl, R->n, S->n);
    if (!ws || ws_bytes < need)
        return fail(HJ_ERR_WORKSPACE, "workspace of %zu bytes needed, %zu given", need, ws ? ws_bytes : 0);
    if ((uintptr_t)ws % kAlign) return fail(HJ_ERR_INVALID, "workspace must be 256-byte aligned");
    return HJ_OK;
}

// SHJ build (Algorithm 1, b1-b4): empty slots, then R inserted.
// total, queue: see shj_fill.
void shj_build_table(const hj_rel& R, const ShjTableWs& t, uint64_t* total, hj::HeavyQueue* queue, hj::Recorder& rec) {
    hj::shj_fill(t.table, t.nslots, t.hot, total, queue, rec);
    hj::shj_build(R.key, R.n, t.table, t.next, t.nslots, t.hot, R.n >= hj::kNtMinBuild, rec);
}

// SHJ probe (Algorithm 1, p1-p4) of a table built over R.  cleared: the one-pass
// count and queue already are.
void shj_probe_table(const Plan& pl, const ShjTableWs& t, const hj_rel& R, const hj_rel& S,
                     const hj_out& out, const ShjProbeWs& w, uint64_t* d_count, bool cleared, hj::Recorder& rec) {
    if (!pl.one_pass) {
        hj::shj_count(S.key, S.n, t.table, t.next, t.nslots, R.key, R.n, t.hot, w.wave_cnt, w.st, w.nst,
                      rec);
        hj::scan_u64(w.wave_cnt, w.wave_cnt, w.tiles * hj::kShjWavesPerBlock, w.st, d_count, rec);
    } else if (!cleared) {
        hj::shj_zero_one_pass(d_count, w.heavy, rec);
    }
    hj::shj_write(S.key, S.rid, S.n, t.table, t.next, t.nslots, R.key, R.rid, R.n, t.hot,
                  pl.one_pass ? nullptr : w.wave_cnt, d_count, pl.one_pass ? w.heavy : nullptr, out.rid_r,
                  out.rid_s, out.capacity, rec);
}

void run_shj(const Plan& pl, const hj_rel& R, const hj_rel& S, const hj_out& out, void* ws,
             uint64_t* d_count, hj::Recorder& rec) {
    const ShjTableWs t = shj_table_layout(R.n, ws);
    const ShjProbeWs w = shj_probe_layout(S.n, (char*)ws + t.bytes);
    shj_build_table(R, t, pl.one_pass ? d_count : nullptr, pl.one_pass ? w.heavy : nullptr, rec);
    shj_probe_table(pl, t, R, S, out, w, d_count, true, rec);
}

// PHJ partitioning (Algorithm 2, n1-n3) of R and S (either may be empty) into
// w, with the join plan of the partition pairs riding on the last scatter.
// r_pairs: R's partition ranges from a built table (R is then empty here).
// n_r_tab: tuples of the R that is joined (0: a table build, nothing joined yet).
// Returns the partitioned tuples (R first, S from n_r on).
hj::Tuple* phj_partition(const Plan& pl, const hj_rel& R, const hj_rel& S, const PhjWs& w, uint64_t n_r_tab,
                         const hj::PartPair* r_pairs, uint64_t* zero_total, hj::Recorder& rec) {
    const uint32_t n_r = (uint32_t)R.n, n_s = (uint32_t)S.n;
    const bool one = hj::one_scatter(pl.passes, pl.b1, pl.b2);
    const bool fine = !one && hj::counts_final(pl.passes, pl.b1, pl.b2, R.n + S.n);
    const hj::PassCfg c1{one ? 0u : pl.b2, one ? pl.B : pl.b1, pl.hash, w.tile1, pl.nt_part};
    const hj::PassCfg c2{0, pl.b2, pl.hash, w.tile2, pl.nt_part};
    hj::Pass1 p1 = hj::make_pass1(R.key, R.rid, n_r, S.key, S.rid, n_s, w.tile1);
    p1.self = w.self;
    p1.fine_bits = fine ? pl.b2 : 0;
    p1.h = w.h;
    p1.rows = w.rows;
    p1.rows1 = w.rows1;
    p1.zero = w.zero;
    p1.nzero = w.nzero;
    p1.err_clear = rec.err_clear;
    const hj::StartArgs starts{w.cur1, one ? w.start : w.start1, fine ? w.cnt2 : nullptr, w.start, w.st1, w.st2,
                               w.words, r_pairs, pl.lds_cap, one || fine ? pl.P : 0, rec.ctl};
    // The plan's records are written at offsets from its chained scan and read
    // without a clamp, so its wait keeps the full bound and no injected stall
    // (every consumer of the other scans clamps what it reads and writes).
    const hj::ScanCtl plan_ctl{rec.ctl.err, hj::kMaxStatusPolls, 0};
    hj::SideJob plan;
    plan.kind = hj::kSidePlan;
    plan.blocks = hj::plan_blocks(pl.P, hj::scatter_block(one ? w.tile1 : w.tile2));
    plan.plan = hj::PlanArgs{w.start, n_r, n_s, pl.B, pl.lds_cap, w.pairs, w.item_begin, w.ovf_begin, w.item_rec,
                             w.ovf_part, zero_total, w.stp, r_pairs, plan_ctl, (uint32_t)w.items_ub, (uint32_t)w.ovf_ub};
    const hj::ClearTables clr{w.clears ? w.ovf_table : nullptr, w.words, w.start, r_pairs, pl.P, (uint32_t)n_r_tab,
                              pl.lds_cap, hj::clear_share(n_r_tab)};
    hj::part_hist(p1, c1, rec);
    hj::part_starts(p1, c1, starts, rec);
    if (one) {
        hj::part_scatter(p1, c1, w.cur1, w.A, nullptr, nullptr, clr, plan, rec);
        return w.A;
    }
    hj::SideJob setup2;
    setup2.kind = hj::kSideSetup2;
    setup2.blocks = 1;
    setup2.setup2 = hj::Setup2Args{w.start1, pl.b1, w.tile2, n_r, n_s, (uint32_t)w.tiles2_ub, w.segs2, w.tb2, w.tseg2};
    hj::part_scatter(p1, c1, w.cur1, w.A, nullptr, nullptr, hj::ClearTables{}, setup2, rec);
    if (!fine) {
        hj::part_hist2(w.A, w.segs2, w.tb2, w.tseg2, 2 * pl.P1, (uint32_t)w.tiles2_ub, c2, w.cnt2, rec);
        // R's counters come first, so the sums are positions; the total is the end
        hj::scan_u32(w.cnt2, w.start, 2ull * pl.P, w.st2, w.start + 2ull * pl.P, rec);
    }
    hj::part_scatter2(w.A, w.segs2, w.tb2, w.tseg2, 2 * pl.P1, (uint32_t)w.tiles2_ub, c2, w.start, w.cnt2, w.B, clr,
                      plan, rec);
    return w.B;
}

// PHJ join of the planned partition pairs (Algorithm 1 per pair): count -> scan
// -> write (or one-pass write).
// rt: partitioned R, st: partitioned S.
void phj_join_pairs(const Plan& pl, const PhjWs& w, uint64_t n_r, const hj::Tuple* rt, const hj::Tuple* st,
                    const hj_out& out, uint64_t* d_count, hj::Recorder& rec) {
    const bool before = hj::tables_expected(n_r, pl.P, pl.lds_cap);
    // (no partition of fewer rows queues tuples: no helper workgroups then)
    hj::HeavyQueue* heavy = pl.one_pass && n_r > hj::kQueueRows ? w.heavy : nullptr;
    const hj::OvfBuild ovf{w.pairs, w.ovf_begin, w.ovf_part, w.ovf_begin + pl.P, before ? nullptr : w.words, rec.ctl.err};
    if (!w.clears) hj::join_ovf_clear(ovf, (uint32_t)w.ovf_ub, w.ovf_table, rec);
    if (before)
        hj::join_ovf_build(ovf, (uint32_t)w.ovf_ub, rt, w.ovf_table, w.ovf_next, w.hot, heavy, rec);
    if (!pl.one_pass) {
        hj::join_count(w.item_rec, (uint32_t)w.items_ub, rt, st, pl.lds_cap, pl.B, pl.hash, ovf, w.ovf_table,
                       w.ovf_next, w.hot, w.wave_cnt, pl.nt_s, rec);
        hj::scan_u64(w.wave_cnt, w.wave_cnt, w.items_ub * hj::kJoinWaves, w.stw, d_count, rec);
    }
    hj::join_write(w.item_rec, (uint32_t)w.items_ub, rt, st, pl.lds_cap, pl.B, pl.hash, ovf, w.ovf_table, w.ovf_next, w.hot,
                   pl.one_pass ? nullptr : w.wave_cnt, d_count, out.rid_r, out.rid_s, out.capacity,
                   heavy, pl.nt_s, rec);
}

void run_phj(const Plan& pl, const hj_rel& R, const hj_rel& S, const hj_out& out, void* ws,
             uint64_t* d_count, hj::Recorder& rec) {
    const PhjWs w = phj_layout(pl, R.n, S.n, R.n, ws);
    const hj::Tuple* t = phj_partition(pl, R, S, w, R.n, nullptr, pl.one_pass ? d_count : nullptr, rec);
    phj_join_pairs(pl, w, R.n, t, t + R.n, out, d_count, rec);
}

void run_join(const Plan& pl, const hj_rel& R, const hj_rel& S, const hj_out& out, void* ws,
              uint64_t* d_count, Recorder& rec) {
    if (R.n == 0 || S.n == 0) {
        hj::write_zero_count(d_count, rec);
    } else if (pl.phj && pl.passes == 0) {
        run_direct(pl, R, S, out, d_count, rec);
    } else if (pl.phj) {
        run_phj(pl, R, S, out, ws, d_count, rec);
    } else {
        run_shj(pl, R, S, out, ws, d_count, rec);
    }
}

void run_build(const Plan& pl, const hj_rel& R, void* ws, hj::Recorder& rec) {
    if (R.n == 0 || (pl.phj && pl.passes == 0)) {  // passes 0: the table is R itself
        hj::zero_pair(rec.err_clear, nullptr, rec);
        return;
    }
    if (!pl.phj) {
        shj_build_table(R, shj_table_layout(R.n, ws), nullptr, nullptr, rec);
        return;
    }
    const PhjWs w = phj_layout(pl, R.n, 0, 0, ws);
    const hj_rel none{nullptr, nullptr, 0};
    phj_partition(pl, R, none, w, 0, nullptr, nullptr, rec);
}

void run_probe(const Plan& pl, const hj_table& t, const hj_rel& S, const hj_out& out, void* ws,
               uint64_t* d_count, hj::Recorder& rec) {
    const hj_rel R{t.r_key, t.r_rid, t.n_r};
    if (t.n_r == 0 || S.n == 0) {
        hj::write_zero_count(d_count, rec);
    } else if (pl.phj && pl.passes == 0) {
        run_direct(pl, R, S, out, d_count, rec);
    } else if (!pl.phj) {
        const ShjTableWs tw = shj_table_layout(t.n_r, t.ws);
        const ShjProbeWs w = shj_probe_layout(S.n, ws);
        shj_probe_table(pl, tw, R, S, out, w, d_count, false, rec);
    } else {
        // R's partitions and pair ranges are in the table; only S is partitioned here
        const PhjWs tw = phj_layout(pl, t.n_r, 0, 0, t.ws);
        const PhjWs w = phj_layout(pl, 0, S.n, t.n_r, ws);
        const hj_rel none{nullptr, nullptr, 0};
        const hj::Tuple* s = phj_partition(pl, none, S, w, t.n_r, tw.pairs, pl.one_pass ? d_count : nullptr, rec);
        phj_join_pairs(pl, w, t.n_r, hj::one_scatter(pl.passes, pl.b1, pl.b2) ? tw.A : tw.B, s, out, d_count, rec);
    }
}

// The plan a table was built with, after checking the table's own fields.
hj_status table_plan(const hj_table* t, uint64_t n_s, Plan* pl) {
    if (!t) return fail(HJ_ERR_INVALID, "table is NULL");
    if (t->n_r > kMaxRows) return fail(HJ_ERR_INVALID, "table: relations must have fewer than 2^31 tuples");
    hj_status st = check_params(&t->params, t->n_r, n_s, pl);
    if (st != HJ_OK) return st;
    if (t->params.algo == HJ_AUTO || (pl->phj && t->params.tile == 0))
        return fail(HJ_ERR_INVALID, "table parameters are not the ones hj_build filled in");
    if (!t->ws || t->ws_bytes < table_bytes_for(*pl, t->n_r))
        return fail(HJ_ERR_INVALID, "table: build workspace missing or too small");
    // SHJ probes read R's rids for every match and scan R's keys for the S
    // tuples of duplicate-heavy keys; PHJ probes without partitioning read both
    const bool reads_r = !pl->phj || pl->passes == 0;
    if (t->n_r && reads_r && (!t->r_rid || !t->r_key))
        return fail(HJ_ERR_INVALID, "table: R's key and rid arrays are needed by this probe");
    return HJ_OK;
}

void init_recorder(Recorder& rec, hipStream_t stream, uint64_t* err, bool clear) {
    rec.stream = stream;
    rec.ctl.err = err;
    rec.err_clear = clear ? err : nullptr;
    rec.ctl.max_polls = kMaxStatusPolls;
    rec.ctl.stall = 0;
    rec.fail_phase = nullptr;
    // HJ_DEBUG_FAIL_PHASE (tests of the failure paths, read per call):
    //   scan_stall     the first tile of every chained scan but the join plan's
    //                  never publishes and waits give up after 64 polls (every
    //                  kernel still ends; the call's error word reports it)
    //   launch:<name>  the launch of phase <name> reports a launch failure
    thread_local std::string phase;
    const char* v = getenv("HJ_DEBUG_FAIL_PHASE");
    if (!v || !*v) return;
    phase = v;
    if (phase == "scan_stall") {
        rec.ctl.max_polls = 64;
        rec.ctl.stall = 1;
    } else if (phase.rfind("launch:", 0) == 0) {
        rec.fail_phase = phase.c_str() + 7;
    }
}

hj_status launch_join(const hj_params* p, const hj_rel* R, const hj_rel* S, const hj_out* out, void* ws,
                      size_t ws_bytes, uint64_t* d_count, hj::Recorder& rec) {
    Plan pl;
    hj_status st = check_call(p, R, S, out, ws, ws_bytes, d_count, &pl);
    if (st != HJ_OK) return st;
    (void)hipGetLastError();  // clear a stale error left by unrelated work
    run_join(pl, *R, *S, *out, ws, d_count, rec);
    if (rec.err != hipSuccess)
        return fail(HJ_ERR_DEVICE, "launch failed: %s", hipGetErrorString(rec.err));
    g_err.clear();
    return HJ_OK;
}


}  // namespace eng
}  // namespace hj
