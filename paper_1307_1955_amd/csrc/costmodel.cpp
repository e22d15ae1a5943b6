// Per-step cost model of a join on MI355X (Section 4, Eq. 2-3) and the
// planner that evaluates it (HJ_AUTO).
//
// The paper sums, over a step series, each step's computation time, memory
// stall time and pipelined delay.  One GPU runs every step here, and a step is
// one kernel launch of the plan (engine.cpp's launch sequence):
//     T = sum over launches k of  D + d + max(M_k, W_k)
// D: delay of a dependent launch behind the previous kernel; d: a kernel's
// fixed ramp-up and drain; M_k: the launch's algorithmic bytes over the
// bandwidth of its access pattern (streaming read, scatter whose bandwidth
// grows with the run length tile / 2^bits, random table lines served from the
// caches or from HBM); W_k: rounds of resident workgroups times one
// workgroup's duration (the latency-bound join items; for the partitioning
// tiles the first round's and a share q_part of every later round's, as
// later rounds overlap the ones before).  The constants come
// from per-kernel HIP-event times of a grid of joins on MI355X (generated
// include calib_mi355x.inc; the Python twin paper_1307_1955_amd/costmodel.py
// fits them and is kept equal to this file by a test).
#include <algorithm>
#include <cmath>

#include "../../include/hj.h"
#include "engine.h"
#include "hj_internal.h"

namespace hj {
namespace eng {

namespace {

#include "calib_mi355x.inc"

constexpr double kCus = 256;
constexpr double kLdsPerCu = 160.0 * 1024;
constexpr double kChunk = kJoinChunk;
constexpr double kShjTileD = kShjTile;

double scatter_slots(uint32_t bits, uint32_t tile) {
    const double P = std::ldexp(1.0, (int)bits);
    const double lds = 8.0 * (tile + 64) + 4 * (std::max(P, 64.0) + 128);
    const double by_lds = std::floor(kLdsPerCu / lds);
    const double by_threads = std::floor(2048.0 / scatter_block(tile));
    return kCus * std::max(1.0, std::min(by_lds, by_threads));
}

// Join work items resident at once: workgroups per CU by LDS and by the waves
// the kernels' register budget allows (6 per SIMD, 4 with the largest build).
double join_slots(uint32_t cap) {
    const double by_waves = (join_rpt(cap) > kRptMid ? 4.0 : 6.0) * 4.0 / kJoinWaves;
    const double lds = (double)join_lds_bytes(cap, 1, true) + 512;
    return kCus * std::max(1.0, std::min(std::floor(kLdsPerCu / lds), std::floor(by_waves)));
}

double nonempty(double mean) { return mean < 30 ? 1.0 - std::exp(-mean) : 1.0; }

// Change of a random access's cost with the table size (1 up to base bytes).
double table_factor(double table_bytes, double gamma, double base = 1048576.0) {
    return std::pow(std::max(table_bytes, base) / base, gamma);
}

double rounds(double items, double slots) { return std::ceil(std::max(items, 1.0) / slots); }

// (a^p + b^p)^(1/p): max(a, b) as p grows, more than it when a and b are close.
double smooth_max(double a, double b, double p) {
    const double m = std::max(a, b);
    if (m <= 0) return 0;
    return m * std::pow(std::pow(a / m, p) + std::pow(b / m, p), 1.0 / p);
}

// Latency term of a partitioning launch: the first round of tiles, then a
// share q_part of each later round (rounds overlap).
double part_lat(double rounds, double per_tile) { return per_tile * (1.0 + (rounds - 1.0) * k_q_part); }

// grid: workgroups; bins: counters each clears and writes
double hist_s(double n, double grid, double bins) {
    if (grid == 0) return k_d_kernel;
    const double per = k_t_hist_tile * (n / grid) / 8192.0 + k_t_count_bin * bins;
    return k_d_kernel + smooth_max(4.0 * n / k_bw_hist, part_lat(std::ceil(grid / 1024.0), per), k_p_part);
}

// extra: bytes beyond the tuples' (HBM tables cleared); words: counts that every
// workgroup sums itself
double scatter_s(double n, double tiles, uint32_t tile, uint32_t bits, double extra, double words) {
    if (tiles == 0) return k_d_kernel;
    const double P = std::ldexp(1.0, (int)bits);
    const double run = tile / P;
    const double bw = k_bw_scatter * run / (run + k_run_half);
    const double per_tile = k_t_scatter_tile * tile / 8192.0 + k_t_reserve * P / 4096.0 + k_t_self_word * words;
    return k_d_kernel + smooth_max((16.0 * n + extra) / bw,
                                   part_lat(std::ceil(tiles / scatter_slots(bits, tile)), per_tile), k_p_part);
}

double scan_s(double entries) { return k_d_kernel + entries * k_t_scan_entry; }

// f: the kernel's work-item latency against the write pass (k_f_count, k_f_1pass, or 1)
// least: what the reservations on the output count take (one-pass write)
double join_s(double items, double r, double s, uint32_t cap, bool hbm, double bytes, double f, double least = 0) {
    const double lat = f * (hbm ? k_l_hbm0 + k_l_hbm_s * s : k_l_join0 + k_l_join_r * r + k_l_join_s * s);
    // the first round, then its later ones beside the memory traffic
    const double later = (rounds(items, join_slots(cap)) - 1.0) * lat;
    return k_d_kernel + smooth_max(lat + smooth_max(bytes / k_bw_join, later, k_p_join), least, 4.0);
}

}  // namespace

double model_seconds(const Plan& pl, uint64_t n_r_, uint64_t n_s_, double m) {
    const double n_r = (double)n_r_, n_s = (double)n_s_, n = n_r + n_s;
    const double gap = k_d_gap, d = k_d_kernel;
    if (n_r_ == 0 || n_s_ == 0) return gap + d;
    double t = 0;
    int nl = 0;
    if (!pl.phj) {
        const double slots = (double)shj_slots(n_r_);
        const double tb = 8 * slots;
        const double ins = k_t_ins * table_factor(tb, k_gamma_ins);
        const double probe = k_t_probe * table_factor(tb, k_gamma_probe);
        const double b_floor = k_t_bround * table_factor(tb, k_gamma_bround, 32768.0);
        const double p_floor = k_t_pround * table_factor(tb, k_gamma_pround, 32768.0);
        const double probe_s = std::max(n_s * probe, p_floor);
        const double write_s = std::max(n_s * probe + m * k_t_match, p_floor);
        t += d + 8 * slots / k_bw_fill;            // fill
        t += d + std::max(n_r * ins, b_floor);     // build
        nl += 2;
        if (pl.one_pass) {
            t += d + write_s;  // write
            nl += 1;
        } else {
            t += d + probe_s;                             // count
            t += scan_s(4 * std::ceil(n_s / kShjTileD));  // scan of the per-wave counts
            t += d + write_s;                             // write
            nl += 3;
        }
        return t + nl * gap;
    }
    if (pl.passes == 0) {
        const double chunk = direct_chunk(n_s_, pl.lds_cap), items = std::ceil(n_s / chunk);
        if (items > 1) t += d;  // zero the count
        t += join_s(items, n_r, std::min(n_s, chunk), pl.lds_cap, false, 8 * n + 8 * m, 1.0);
        return t + (items > 1 ? 2 : 1) * gap;
    }
    const uint32_t tile = pl.tile, b1 = pl.b1, b2 = pl.passes == 2 ? pl.b2 : 0;
    const double P = std::ldexp(1.0, (int)(b1 + b2)), P1 = std::ldexp(1.0, (int)b1);
    const uint64_t nn = n_r_ + n_s_;
    const bool one = one_scatter(pl.passes, b1, b2), final = counts_final(pl.passes, b1, b2, nn);
    const uint32_t tile1 = scatter_tile(tile, one ? b1 + b2 : b1, nn);
    const uint64_t tiles1 = (n_r_ + tile1 - 1) / tile1 + (n_s_ + tile1 - 1) / tile1;
    const bool self = one && self_starts(tiles1, b1 + b2, tile1);
    const uint32_t cbits = final ? b1 + b2 : b1;  // what the histogram counts
    const double hist_grid = self ? (double)tiles1 : (double)hist_rows(tiles1, cursor_replicas(tiles1), cbits).grid();
    const double r_part = n_r / P, s_part = n_s / P;
    const bool hbm = r_part > pl.lds_cap;
    const double ovf_r = hbm ? n_r : 0;
    const bool clears = scatter_clears(pl.passes, b1, b2, nn);  // the last scatter clears the HBM tables
    const double cleared = clears ? 16 * ovf_r : 0.0;
    t += hist_s(n, hist_grid, std::ldexp(1.0, (int)cbits));
    nl += 1;
    if (!self) {
        const double columns = std::ldexp(1.0, (int)cbits) + (final && !one ? P1 : 0.0);
        t += d + k_l_starts + 2 * hist_grid * columns * k_t_start_entry;
        nl += 1;
    }
    t += scatter_s(n, (double)tiles1, tile1, one ? b1 + b2 : b1, one ? cleared : 0.0,
                   self ? std::ldexp((double)tiles1, (int)(b1 + b2)) : 0.0);
    nl += 1;
    if (!one) {
        const uint32_t tile2 = scatter_tile(tile, b2, nn);
        const double seg = n / (2 * P1);
        const double tiles2 = seg > 0 ? 2 * P1 * std::max(1.0, std::ceil(seg / tile2)) : 0;
        if (!final) {
            t += hist_s(2 * n, tiles2, std::ldexp(1.0, (int)b2)) + scan_s(2 * P);
            nl += 2;
        }
        t += scatter_s(n, tiles2, tile2, b2, cleared, 0.0);
        nl += 1;
    }
    const double items = P * nonempty(r_part) * nonempty(s_part) * std::max(1.0, std::ceil(s_part / kChunk));
    const double grid = P + std::ceil(n_s / kChunk);
    const double s_item = std::min(std::max(s_part, 1.0), kChunk);
    const double r_item = std::min(r_part, (double)pl.lds_cap);
    if (!clears) {
        t += d + 16 * ovf_r / k_bw_fill;  // clear the HBM tables
        nl += 1;
    }
    if (tables_expected(n_r_, (uint32_t)P, pl.lds_cap)) {  // a launch before the join builds them
        t += d;
        nl += 1;
    }
    if (hbm) {  // inserts, or rounds of items of ovf_chunk() tuples
        const double chunk = ovf_chunk((uint32_t)std::min(r_part, 4294967295.0));
        const double turns = std::ceil(P * std::ceil(r_part / chunk) / (3.0 * kCus));
        t += std::max(ovf_r * k_t_ovf_insert, turns * std::ceil(std::min(r_part, chunk) / 512) * k_l_ovf_round);
    }
    if (!pl.one_pass) {
        t += join_s(items, r_item, s_item, pl.lds_cap, hbm, 4 * n, k_f_count);
        t += scan_s(8 * grid);
        t += join_s(items, r_item, s_item, pl.lds_cap, hbm, 8 * n + 8 * m, 1.0);
        nl += 3;
    } else {
        t += join_s(items, r_item, s_item, pl.lds_cap, hbm, 8 * n + 8 * m, k_f_1pass,
                    items * std::ceil(s_item / kJoinSub) * k_t_out);
        nl += 1;
    }
    return t + nl * gap;
}

// HJ_AUTO: the plan with the least modelled time among SHJ, the direct LDS join
// (|R| <= 8192) and PHJ in one or two radix passes around ~4096 R tuples per
// partition.  Bits that one scatter makes are weighed once, not in each of their
// splits (a call's plan is chosen anew each time: 10.1 us on the host at 1M x 1M,
// 3.1 so).  The partitioning tile is the caller's, else the measured size
// rule (default_tile): between the two tiles the model cannot see which pass
// loses by shorter runs (pass 1 reads the inputs cold; 16M x 16M ran 9% slower
// with 4096-tuple tiles, which the model priced faster).  Hash, lds_cap and
// flags are the caller's.  The output size is taken as |S|
// (one match per probe tuple), the same for every candidate.  Partitions that
// all need HBM tables (a small lds_cap) are weighed only past kOneTableRows:
// below, one table over all of R is cached as well and needs no partitioning
// (measured with lds_cap 256: 8.8K x 15M 195 us against 266 and more, 300K x 4.8M
// 134 against 161, 1M x 4M 160 against 181; past 1M rows either wins), which the model's per-access
// constants do not see.
constexpr uint64_t kOneTableRows = 1ull << 20;
void auto_params(uint64_t n_r, uint64_t n_s, hj_params* p) {
    const hj_params base = *p;
    const double m = (double)n_s;
    double best_t = 1e300;
    hj_params best = base;
    best.algo = HJ_PHJ;
    best.passes = 1;
    best.bits[0] = 1;
    best.bits[1] = 0;
    auto consider = [&](const hj_params& q) {
        Plan pl;
        const hj_status st = check_params(&q, n_r, n_s, &pl);
        if (st != HJ_OK) return;
        if (pl.phj && pl.passes && n_r <= kOneTableRows && (n_r >> pl.B) > pl.lds_cap) return;
        const double t = model_seconds(pl, n_r, n_s, m);
        if (t < best_t) {
            best_t = t;
            best = q;
        }
    };
    hj_params q = base;
    q.algo = HJ_SHJ;
    q.passes = 0;
    q.bits[0] = q.bits[1] = 0;
    consider(q);
    q.algo = HJ_PHJ;
    if (n_r <= kMaxLdsCap) consider(q);  // passes 0: one LDS table
    uint32_t B = 0;
    while (B < kMaxRadixBits && (n_r >> B) > 4096) ++B;
    for (uint32_t b = (B > 2 ? B - 2 : 1); b <= std::min(B + 2, kMaxRadixBits); ++b) {
        q.tile = base.tile;  // 0: the size rule
        if (b <= 13) {
            q.passes = 1;
            q.bits[0] = b;
            q.bits[1] = 0;
            consider(q);
        }
        if (b < 2) continue;
        if (b <= kFuseBits) {
            // one scatter however the bits are split: another plan only by the tile that the rule gives two
            // passes (one pass with that tile: two passes reserve a second copy of the tuples)
            const uint32_t two = default_tile(n_r, n_s, 2, b / 2);
            if (base.tile || two == default_tile(n_r, n_s, 1, b)) continue;
            q.tile = two;
            consider(q);
            continue;
        }
        q.passes = 2;
        for (uint32_t b1 = std::max(1u, b / 2 - 1); b1 <= std::min(13u, b / 2 + 2); ++b1) {
            if (b - b1 < 1 || b - b1 > 13) continue;
            q.bits[0] = b1;
            q.bits[1] = b - b1;
            consider(q);
        }
    }
    *p = best;
    p->tile = base.tile ? base.tile : best.tile;
}

}  // namespace eng
}  // namespace hj
