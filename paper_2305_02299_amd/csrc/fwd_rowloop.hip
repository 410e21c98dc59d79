// ROWLOOP forward kernel: launch shapes and their estimates (the kernel: fwd_rowloop.inl).
#include "srigl_internal.h"

namespace srigl {

// Bytes of x, and of W_c / idx.
static double x_bytes(const FwdArgs& a) { return (double)a.B * a.d_in * (a.x_bf16 ? 2 : 4); }
static double term_bytes(const FwdArgs& a) { return (double)a.n_active * a.K * ((a.x_bf16 ? 2 : 4) + (a.idx_u16 ? 2 : 4)); }

// Columns of a tile: whole units of its staging.
static int tile_columns_of(const FwdArgs& a, int BT) { return BT < 16 ? (a.d_in + 31) / 32 * 32 : (a.d_in + 15) / 16 * 16; }

// Estimated time (us) of a launch shape: per round of workgroups on the busiest XCD a constant, the tile (words staged; beyond 16 K words
// more from the second round on, when no wavefronts start under its loads any more), and per stored row of a wavefront a step
// per 16 terms (32 in 8-row tiles) and a constant (another where terms beyond 256 are walked in a loop); the bytes of y; the bytes the XCDs' L2 caches
// fetch (all of them the one array, each its share of the other).  Non-negative least squares on the relative error of 2600 launches
// (each tile, shapes within 1.6 times the fastest; 67 layers 112 to 2400 wide, fan-ins 6 to 384, both types, batches 8 to 2048, cached
// operands; 8-row tiles: 2800 launches, 297 layers 700 to 4096 wide, fan-ins to 806): standard deviation 6.5 to 9 %.  The 8-row launches were measured apart from the others and came
// out 7 % higher: on 1300 later points, where every tile was timed beside the others (300 to 4096 wide, batches 2 to 1200), 0.935 of their estimate at small,
// middle and large batches alike, so their constants are the fit's times 0.93.  The tile of smallest estimate is then 0.2 % behind the fastest up to 64 batch
// rows and 0.9 % above (7.9 % and 2.0 % before: 16-row tiles were taken where 8-row ones are ahead, 1280 -> 1008, K = 256, 625 stored at 24, 16-bit indices 6.6 us, 5.8).
// second_pass: workgroups make a second pass over their tile where it has more columns than one pass holds (2048 * wavefronts / rows of
// the tile: 4096, 2048, 1024 and 512 at 16), another trip to the L2 and back, which later rounds
// hide behind one another's arithmetic: the step in time at those widths on 2200 and, of 64-row tiles, 108 launches.  With it
// the tile taken on inputs of 1024 to 2600 columns at batches above 64 is 0.9 % behind the fastest (2.1 % without: 2160 -> 768, K = 216 at 256 in 16-row tiles 9.7 us, 8.2 in 8-row ones).
static double rowloop_us(const FwdArgs& a, const RowloopPlan& p) {
    struct Fit { double fixed, round, word, big, step, row, y, fetched, long_row, second_pass; };
    static const Fit fits[4] = {{2.620, 1.863, 0.2704e-4, 0.272e-4, 0.0635, 0.0866, 2.371e-6, 0.0314e-6, 0.1509, 0.0},
                                {2.231, 2.147, 0.2049e-4, 0.585e-4, 0.0545, 0.0423, 2.128e-6, 0.0585e-6, 0.2256, 1.4},
                                {3.522, 1.023, 0.1370e-4, 1.2465e-4, 0.0866, 0.0701, 1.613e-6, 0.0430e-6, 0.5675, 0.6},
                                {3.131, 1.348, 0.2724e-4, 0.3693e-4, 0.1745, 0.0951, 1.378e-6, 0.0448e-6, 0.0, 0.7}};
    const Fit& f = fits[p.BT == 8 ? 0 : p.BT == 16 ? 1 : p.BT == 32 ? 2 : 3];
    const int steps = a.K <= 256 ? p.ST : p.BT == 8 ? 8 + 2 * ((a.K - 256 + 63) / 64) : 16 + 4 * ((a.K - 256 + 63) / 64);
    const int rows = std::min((p.NG + p.NW - 1) / p.NW, (a.n_active + p.NW - 1) / p.NW);   // of the busiest wavefront
    const double fetched = p.bt_major ? x_bytes(a) + 8 * term_bytes(a) : 8 * x_bytes(a) + term_bytes(a);
    const double words = (double)p.BT * ((a.d_in + 15) / 16 * 16);
    const double again = tile_columns_of(a, p.BT) > 2048 / p.BT * p.NW ? f.second_pass : 0.0;
    return f.fixed + again + p.rounds * (f.round + f.word * words + rows * (f.step * steps + f.row + (a.K > 256 ? f.long_row : 0.0)) * p.NW / 16.0) +
           (p.rounds - 1) * f.big * std::max(0.0, words - 16384) + f.y * a.B * a.d_out + f.fetched * fetched;
}

// Rows per workgroup the result tile (and, with an active list, a column table of twice as many columns) has room for.
static long long rowloop_room(const FwdArgs& a, size_t tile, int BT) {
    if (tile >= kLdsMax) return 0;
    const size_t per_row = (size_t)BT * sizeof(float) + (a.active ? 2 * (sizeof(int) + sizeof(float)) : sizeof(float));
    return std::min<long long>((long long)((kLdsMax - tile) / per_row) - 2, 4096);
}

// The launch of p.BT batch rows x NG stored rows per workgroup.
static RowloopPlan rowloop_shape(const FwdArgs& a, RowloopPlan p, int NG, int xcd_order) {
    p.NG = NG;
    const int steps = p.BT == 8 ? std::min((a.K + 31) / 32, 8) : (a.K + 15) / 16;
    p.ST = steps <= 8 ? steps : std::min((steps + 1) / 2 * 2, 16);   // (the kernel has these; a row one step short of an even number walks one of padding)
    p.n_btiles = (a.B + p.BT - 1) / p.BT;
    p.n_groups = (a.n_active + NG - 1) / NG;
    const long long by_groups = (long long)((p.n_groups + 7) / 8) * p.n_btiles, by_tiles = (long long)((p.n_btiles + 7) / 8) * p.n_groups;
    // batch tiles to XCDs when every XCD gets a tile and either that takes no more rounds and x is the larger operand (an XCD's L2 then
    // fetches its own rows of x and all of W_c / idx, else all of x and its groups' W_c / idx), or x is more than an L2 of 4 MB holds,
    // which every group would fetch again (2400 -> 12000, K = 48 at batch 800 157 -> 143 us, 1792 -> 8192, K = 90 at 1024 87 -> 79,
    // 2048 -> 4096, K = 328 at 1500 193 -> 183; at batch 512, x of 4.2 MB, 65 -> 64; below, groups are level or up to 15 % ahead)
    const bool by_x = x_bytes(a) > 4.1e6 ? 10 * by_tiles <= 11 * by_groups : by_tiles <= by_groups && x_bytes(a) >= term_bytes(a);
    p.bt_major = xcd_order ? (xcd_order == 2) : (p.n_btiles >= 8 && by_x);
    p.rounds = (int)(((p.bt_major ? by_tiles : by_groups) + 31) / 32);
    return p;
}

// The rest of a plan whose tile and groups are set: what of a row is preloaded, and the LDS behind the tile (result tile; the bias of
// the workgroup's columns; with an active list the bias and the column table of a run of up to span_cap columns).
static RowloopPlan rowloop_finish(const FwdArgs& a, RowloopPlan p) {
    p.ok = false;
    const int C = tile_columns_of(a, p.BT);
    p.out_off = (C + 1) * p.BT;
    const size_t used = ((size_t)p.out_off + (size_t)p.BT * (p.NG | 1) + (a.active ? 0 : (size_t)p.NG)) * sizeof(float);
    if (used > kLdsMax) return p;
    p.span_cap = a.active ? (int)std::min<size_t>((kLdsMax - used) / (sizeof(int) + sizeof(float)), 1u << 20) : 0;
    p.lds = used + (size_t)p.span_cap * (sizeof(int) + sizeof(float));
    if (8LL * ((p.n_groups + 7) / 8) * ((p.n_btiles + 7) / 8 * 8) > 0x7fffffffLL) return p;
    p.ok = true;
    return p;
}

// As many groups as fill the compute units, fewer rows per workgroup where that costs no round; or rows_per_wave (> 0) as asked.
static RowloopPlan rowloop_best(const FwdArgs& a, RowloopPlan p, long long ng_max, int rows_per_wave, int xcd_order, double* us) {
    p.ok = false;
    if (ng_max < p.NW || rows_per_wave < 0 || (long long)rows_per_wave * p.NW > ng_max) return p;
    RowloopPlan best = p;
    for (int rpw = rows_per_wave ? rows_per_wave : 1; (long long)rpw * p.NW <= ng_max; ++rpw) {
        const RowloopPlan q = rowloop_shape(a, p, rpw * p.NW, xcd_order);
        const double t = rowloop_us(a, q);
        if (!best.ok || t < *us) { best = q; best.ok = true; *us = t; }
        if (rows_per_wave || q.n_groups == 1) break;
    }
    return best.ok ? rowloop_finish(a, best) : best;
}

// SRIGL_FWD_ROWLOOP as a caller can ask for it: tiles of 32 or 64 rows (term_slices 4 or 2) on rows of whole 16-column units.
RowloopPlan plan_rowloop(const FwdArgs& a, const srigl_fwd_tuning* t, double* us) {
    RowloopPlan p{};
    if (a.B <= 0 || a.n_active <= 0 || a.K <= 0) return p;
    if (t && t->rows_per_lane != 0 && t->rows_per_lane != 2) return p;
    const int H = t && t->term_slices ? t->term_slices : 4;
    if (H != 2 && H != 4) return p;
    p.BT = 128 / H;
    const size_t xal = (a.x_bf16 ? 2 : 4) * 4;
    if (a.d_in % 16 != 0 || reinterpret_cast<uintptr_t>(a.x) % xal != 0) return p;
    if (((long long)a.n_active + 256) * a.K + 4096 >= (1LL << 29)) return p;
    if ((long long)(p.BT + 1) * a.d_in * 4 >= (1LL << 32)) return p;
    p.NW = t && t->waves ? t->waves : 16;
    if (p.NW < 1 || p.NW > 16) return p;
    const int xo = t ? t->xcd_order : 0;
    if (xo < 0 || xo > 2) return p;
    const size_t tile = (size_t)(a.d_in + 1) * (p.BT + 4) * sizeof(float);   // (its documented room: the tile takes 4 words per column less)
    double best_us = 0.0;
    p = rowloop_best(a, p, rowloop_room(a, tile, p.BT), t ? t->neurons_per_wave : 0, xo, &best_us);
    if (us) *us = best_us;
    return p;
}

// The library's own choice of a tile: 8, 16, 32 or 64 batch rows, rows of any length.
RowloopPlan plan_tile(const FwdArgs& a, int tile_rows, int rows_per_wave, int xcd_order, double* us) {
    RowloopPlan best{};
    if (a.B <= 0 || a.n_active <= 0 || a.K <= 0 || a.d_in < 16 || a.d_in > 4096) return best;
    for (int BT = 8; BT <= 64; BT *= 2) {
        if (tile_rows && tile_rows != BT) continue;
        RowloopPlan p{};
        p.BT = BT;
        p.NW = 16;
        const size_t tile = (size_t)(tile_columns_of(a, BT) + 1) * BT * sizeof(float);
        double t = 0.0;
        p = rowloop_best(a, p, rowloop_room(a, tile, BT), rows_per_wave, xcd_order, &t);
        if (p.ok && (!best.ok || t < *us)) { best = p; *us = t; }
    }
    return best;
}

srigl_status launch_fwd_rowloop(const FwdArgs& a, const srigl_fwd_tuning* t, hipStream_t st) {
    if (a.B == 0 || a.n_active == 0) return SRIGL_OK;
    return launch_rowloop_plan(a, plan_rowloop(a, t, nullptr), st);
}

srigl_status launch_rowloop_plan(const FwdArgs& a, const RowloopPlan& p, hipStream_t st) {
    if (!p.ok) return SRIGL_ERR_UNSUPPORTED;
    if (a.idx_u16) return a.x_bf16 ? launch_rowloop_bf16_i16(a, p, st) : launch_rowloop_f32_i16(a, p, st);
    return a.x_bf16 ? launch_rowloop_bf16(a, p, st) : launch_rowloop_f32(a, p, st);
}

}  // namespace srigl
