// C ABI of libtplinear (see include/tp_linear.h): argument validation, the partition map
// (paper Section 2.2: chunk shapes [P/q, Q/q], N = S^2 D, [P/p^2, Q/p]; device-count rule),
// launch planning (macro-tile, split of K across workgroups, tile order) and kernel launches.
// Everything is checked before the first launch; nothing is allocated or synchronised here.
#include <algorithm>
#include <atomic>
#include <cstdint>
#include <cstring>

#include "tp_internal.h"

using namespace tpl;

namespace {

constexpr int kCUs = 256;                       // MI355X compute units (8 XCDs x 32): the tile order and the plan assume it
constexpr int64_t kMaxLd = (int64_t)1 << 21;    // keeps every in-tile byte offset below 2^31

// Launch-plan options of one call, resolved from the caller's tp_plan_opts_t (NULL = automatic).
// rotate: -1 automatic (on for the eight-wave kernel, off for the four-wave stream kernel: its workgroups
// of one XCD share operand panels through the L2 only while they walk K in step), 0 off, 1 on.
struct Opts { int tile, split, group, rotate, trim; bool eight_wave; };
int resolve_opts(const tp_plan_opts_t* o, Opts* r) {
    *r = Opts{0, 0, 0, -1, 1, false};
    if (!o) return TP_OK;
    if (o->tile < 0 || o->tile > 5 || o->split_k < 0 || o->split_k > 8 || o->group_m < 0 || o->group_m > 64 ||
        o->rotate < 0 || o->rotate > 2 || o->trim < 0 || o->trim > 2)
        return TP_ERR_MODE;
    r->tile = o->tile == 5 ? (int)TILE_256x256 : o->tile;
    r->eight_wave = o->tile == 5;
    r->split = o->split_k; r->group = o->group_m;
    r->rotate = o->rotate == 0 ? -1 : (o->rotate == 1); r->trim = o->trim != 2;
    return TP_OK;
}

// The device must be the one the kernels are laid out for: checked once per device.
int check_device() {
    static std::atomic<uint64_t> ok_mask{0}, bad_mask{0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return TP_ERR_HIP;
    const uint64_t bit = 1ull << (dev & 63);
    if (ok_mask.load(std::memory_order_relaxed) & bit) return TP_OK;
    if (bad_mask.load(std::memory_order_relaxed) & bit) return TP_ERR_HIP;
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return TP_ERR_HIP;
    (cus == kCUs ? ok_mask : bad_mask).fetch_or(bit, std::memory_order_relaxed);
    return cus == kCUs ? TP_OK : TP_ERR_HIP;
}

struct Chunks { int rc, kc, cc; };              // row chunks of X/Y, col chunks of X (= row chunks of W), col chunks of W/Y

int check_grid(const tp_grid_t* g, Chunks* c) {
    if (g->q < 1 || g->d < 1 || g->p < 1) return TP_ERR_GRID;
    int li = 1, lj = 1, lk = 1;
    switch (g->mode) {
        case TP_MODE_1D_COL: li = g->p; *c = {1, 1, g->p}; if (g->q != 1 || g->d != 1) return TP_ERR_GRID; break;
        case TP_MODE_1D_ROW: li = g->p; *c = {1, g->p, 1}; if (g->q != 1 || g->d != 1) return TP_ERR_GRID; break;
        case TP_MODE_2D:     li = lj = g->q; *c = {g->q, g->q, g->q}; if (g->p != 1 || g->d != 1) return TP_ERR_GRID; break;
        case TP_MODE_2P5D:   li = lj = g->q; lk = g->d; *c = {g->q * g->d, g->q, g->q}; if (g->p != 1) return TP_ERR_GRID; break;
        case TP_MODE_3D:     li = lj = lk = g->p; *c = {g->p * g->p, g->p, g->p}; if (g->q != 1 || g->d != 1) return TP_ERR_GRID; break;
        case TP_MODE_3D_GATHERED: li = lj = lk = g->p; *c = {g->p, g->p, g->p}; if (g->q != 1 || g->d != 1) return TP_ERR_GRID; break;
        default: return TP_ERR_MODE;
    }
    if (g->ri < 0 || g->ri >= li || g->rj < 0 || g->rj >= lj || g->rk < 0 || g->rk >= lk) return TP_ERR_GRID;
    return TP_OK;
}

struct Share {           // one pass of one rank
    int n_steps; int64_t m, n, k;
    int a_row[TP_MAX_STEPS], a_col[TP_MAX_STEPS], b_row[TP_MAX_STEPS], b_col[TP_MAX_STEPS];
    int out_row, out_col, partial;
};

int build_share(const tp_grid_t* g, const tp_dims_t* d, int pass, Share* s) {
    if (!g || !d || !s) return TP_ERR_NULL;
    if (pass != TP_PASS_FWD && pass != TP_PASS_DX && pass != TP_PASS_DW) return TP_ERR_MODE;
    Chunks c;
    if (int e = check_grid(g, &c)) return e;
    if (d->M < 1 || d->H < 1 || d->F < 1) return TP_ERR_SHAPE;
    if (d->M % c.rc || d->H % c.kc || d->F % c.cc) return TP_ERR_SHAPE;
    // the gathered slabs are made of p stored chunks [M/p^2, .]
    if (g->mode == TP_MODE_3D_GATHERED && d->M % ((int64_t)g->p * g->p)) return TP_ERR_SHAPE;
    const int64_t mb = d->M / c.rc, hb = d->H / c.kc, fb = d->F / c.cc;
    std::memset(s, 0, sizeof(*s));
    if (g->mode == TP_MODE_3D_GATHERED) {
        const int i = g->ri, j = g->rj, l = g->rk;
        s->n_steps = 1; s->partial = g->p > 1;
        if (pass == TP_PASS_FWD)     { s->m = mb; s->n = fb; s->k = hb; s->a_row[0] = i; s->a_col[0] = l; s->b_row[0] = l; s->b_col[0] = j; s->out_row = i; s->out_col = j; }
        else if (pass == TP_PASS_DX) { s->m = mb; s->n = hb; s->k = fb; s->a_row[0] = i; s->a_col[0] = j; s->b_row[0] = l; s->b_col[0] = j; s->out_row = i; s->out_col = l; }
        else                         { s->m = hb; s->n = fb; s->k = mb; s->a_row[0] = i; s->a_col[0] = l; s->b_row[0] = i; s->b_col[0] = j; s->out_row = l; s->out_col = j; }
        return TP_OK;
    }
    int steps = 1, row = 0, col = 0, wrow = 0;     // own row chunk, own column index, dW's row chunk
    int first_row = 0;                             // first row chunk of the group dW sums over
    switch (g->mode) {
        case TP_MODE_1D_COL: case TP_MODE_1D_ROW: steps = 1; break;
        case TP_MODE_2D:   steps = g->q; row = g->ri; col = g->rj; wrow = g->ri; first_row = 0; break;
        case TP_MODE_2P5D: steps = g->q; row = g->rk * g->q + g->ri; col = g->rj; wrow = g->ri; first_row = g->rk * g->q; break;
        case TP_MODE_3D:   steps = g->p; row = g->ri * g->p + g->rk; col = g->rj; wrow = g->rk; first_row = g->ri * g->p; break;
    }
    if (steps > TP_MAX_STEPS) return TP_ERR_GRID;
    s->n_steps = steps;
    if (g->mode == TP_MODE_1D_COL) {
        const int r = g->ri;
        if (pass == TP_PASS_FWD)      { s->m = mb; s->n = fb; s->k = hb; s->a_col[0] = 0; s->b_col[0] = r; s->out_col = r; }
        else if (pass == TP_PASS_DX)  { s->m = mb; s->n = hb; s->k = fb; s->a_col[0] = r; s->b_col[0] = r; s->partial = g->p > 1; }
        else                          { s->m = hb; s->n = fb; s->k = mb; s->b_col[0] = r; s->out_col = r; }
        return TP_OK;
    }
    if (g->mode == TP_MODE_1D_ROW) {
        const int r = g->ri;
        if (pass == TP_PASS_FWD)      { s->m = mb; s->n = fb; s->k = hb; s->a_col[0] = r; s->b_row[0] = r; s->partial = g->p > 1; }
        else if (pass == TP_PASS_DX)  { s->m = mb; s->n = hb; s->k = fb; s->b_row[0] = r; s->out_col = r; }
        else                          { s->m = hb; s->n = fb; s->k = mb; s->a_col[0] = r; s->out_row = r; }
        return TP_OK;
    }
    for (int k = 0; k < steps; ++k) {
        if (pass == TP_PASS_FWD)     { s->a_row[k] = row; s->a_col[k] = k; s->b_row[k] = k; s->b_col[k] = col; }
        else if (pass == TP_PASS_DX) { s->a_row[k] = row; s->a_col[k] = k; s->b_row[k] = col; s->b_col[k] = k; }
        else                         { s->a_row[k] = first_row + k; s->a_col[k] = wrow; s->b_row[k] = first_row + k; s->b_col[k] = col; }
    }
    if (pass == TP_PASS_FWD)     { s->m = mb; s->n = fb; s->k = hb; s->out_row = row; s->out_col = col; }
    else if (pass == TP_PASS_DX) { s->m = mb; s->n = hb; s->k = fb; s->out_row = row; s->out_col = col; }
    else {
        s->m = hb; s->n = fb; s->k = mb; s->out_row = wrow; s->out_col = col;
        s->partial = (g->mode == TP_MODE_2P5D && g->d > 1) || (g->mode == TP_MODE_3D && g->p > 1);
    }
    return TP_OK;
}

struct PartialsShare {   // the backward products as partials for other owners (2D, 2.5D)
    int n_steps; int64_t m, n, k;
    int own_row, own_col;
    int other_row[TP_MAX_STEPS], other_col[TP_MAX_STEPS], out_row[TP_MAX_STEPS], out_col[TP_MAX_STEPS];
};

int build_partials(const tp_grid_t* g, const tp_dims_t* d, int pass, PartialsShare* s) {
    if (!g || !d || !s) return TP_ERR_NULL;
    if (pass != TP_PASS_DX_PARTIALS && pass != TP_PASS_DW_PARTIALS) return TP_ERR_MODE;
    if (g->mode != TP_MODE_2D && g->mode != TP_MODE_2P5D) return TP_ERR_MODE;
    Chunks c;
    if (int e = check_grid(g, &c)) return e;
    if (d->M < 1 || d->H < 1 || d->F < 1) return TP_ERR_SHAPE;
    if (d->M % c.rc || d->H % c.kc || d->F % c.cc) return TP_ERR_SHAPE;
    if (g->q > TP_MAX_STEPS) return TP_ERR_GRID;
    const int64_t mb = d->M / c.rc, hb = d->H / c.kc, fb = d->F / c.cc;
    std::memset(s, 0, sizeof(*s));
    const int row = (g->mode == TP_MODE_2P5D ? g->rk * g->q : 0) + g->ri, col = g->rj;
    s->n_steps = g->q; s->own_row = row; s->own_col = col;
    for (int k = 0; k < g->q; ++k) {
        if (pass == TP_PASS_DX_PARTIALS) { s->other_row[k] = k; s->other_col[k] = col; s->out_row[k] = row; s->out_col[k] = k; }
        else                             { s->other_row[k] = row; s->other_col[k] = k; s->out_row[k] = k; s->out_col[k] = col; }
    }
    if (pass == TP_PASS_DX_PARTIALS) { s->m = mb; s->n = hb; s->k = fb; }
    else                             { s->m = hb; s->n = fb; s->k = mb; }
    return TP_OK;
}

struct Plan {
    int tile_id, bm, bn, tiles_m, tiles_n, split_k, group_m, groups;
    // Tail trimming: when the tile count is a little more than a whole number of rounds of the 256
    // persistent workgroups, the last tile rows are cut off and run as a second, small launch with a
    // plan of their own, so that the main launch ends on a full round.  m_main = rows of the main launch
    // (0 = not trimmed); the tail covers rows [m_main, m).
    int64_t m_main;
    int tail_tile_id, tail_tiles_m, tail_tiles_n, tail_split;
    size_t need;               // bytes of workspace the call asks for (at least what the plan uses)
};

// Costs in shader cycles, by macro-tile area (256 x 256; half; quarter).  k_tile: one 64-deep K tile of one
// workgroup; c_tile: what a C tile costs besides (epilogue, filling the pipeline).  plane: cycles x 1667 per element
// and plane of a K split; launch: the fix-up launch; trim: a tail launch.
struct Costs { double k_tile[3], c_tile[3], plane, launch, trim; };
// What the kernels take, fitted together with small_cost below to every admissible tile and split of 3700 drawn products
// (0.2 .. 250 GFLOP, all forms, grouped ones too), each timed with its operands in rotation over 450 MB, i.e. from
// memory as a step of a model finds its weights, and again with them in the caches.  Over those products the pick takes 1 %
// (from memory) and 1.6 % (cached) more than the best of them; constants fitted to cached operands alone took 7 % and left 345 of
// the 3700 slower than the eight-wave kernel's plan, up to 1.45 x: from memory a K tile of few workgroups takes its full time,
// and a split that spreads it pays (4 products of 678 x 4240 x 168: 46.5 us whole, 28.5 split in five).
// (The half tiles' K tile fits 1670 to 1870; the upper end, as over many rounds their extra traffic costs clock: dW 14744 x 13568 x 1640
// 710 us in three rounds of 256 x 128, 660 in two of 256 x 256.)
// (trim: since the outputs stream past the L2 a second launch waits for no write-back, and its line fell from 52000.  Whole / trimmed, us:
// forward 32896 x 2560, K = 2 x 640 242 / 220; 8448 x 2048, K = 1024 66 / 53; 32863 x 440, K = 600 62 / 54; dX 32802 x 512, K = 1072 56 / 45;
// dW 720 x 512, K = 33008 48 / 42; where it loses, short tiles: dX 4632 x 4024, K = 208 25.2 / 26.5, 32986 x 440, K = 136 22.6 / 24.1.)
constexpr Costs kRunCosts{{2730.0, 1870.0, 1200.0}, {21000.0, 15000.0, 10000.0}, 4.5, 6500.0, 18000.0};
// What the workspace query has always been computed from.  Callers size and keep workspaces by it, so it goes on
// deciding how many bytes a call needs (and which calls are refused); the plan that runs stays within them.
constexpr Costs kQueryCosts{{2730.0, 2220.0, 1410.0}, {12000.0, 20000.0, 20000.0}, 8.0, 12000.0, 15000.0};

int area_class(int bm, int bn) { return bm * bn == 65536 ? 0 : (bm * bn == 32768 ? 1 : 2); }

size_t ws_bytes_for(const Plan& p, int64_t m, int64_t n) {
    if (p.m_main > 0)              // the main launch never splits K; the tail may
        return p.tail_split > 1 ? (size_t)p.tail_split * (size_t)(m - p.m_main) * (size_t)n * sizeof(float) : 0;
    return p.split_k > 1 ? (size_t)p.split_k * (size_t)p.groups * (size_t)m * (size_t)n * sizeof(float) : 0;
}

// Pick the macro-tile and the split of K so that the launch fills whole rounds of the 256 CUs, with at most `limit`
// bytes of partial planes: rounds of workgroups x (K tiles per workgroup x cost + fixed cost), plus the fp32 round
// trip of the partials when K is split.
// groups > 1: that many products of the same extents share one launch (tiles_m, tiles_n stay per product).
Plan plan_whole(const Costs& cs, const Opts& o, int64_t m, int64_t n, int64_t k, int n_steps, int groups, size_t limit, double* cost_out) {
    const int64_t T = (int64_t)n_steps * ((k + 63) / 64);
    Plan best{};
    double best_cost = 1e300;
    const int tile_ids[4] = {TILE_256x256, TILE_128x256, TILE_256x128, TILE_128x128};
    const int forced_split = o.split, forced_tile = o.tile;
    for (int ti = 0; ti < 4; ++ti) {
        if (forced_tile && tile_ids[ti] != forced_tile) continue;
        int bm, bn;
        tile_shape(tile_ids[ti], &bm, &bn);
        const int64_t tm = (m + bm - 1) / bm, tn = (n + bn - 1) / bn;
        const int64_t tiles = tm * tn * groups;
        const int cls = area_class(bm, bn);
        for (int z = 1; z <= 8; ++z) {
            if (forced_split && z != forced_split) continue;
            if (z > T) break;
            Plan c{tile_ids[ti], bm, bn, (int)tm, (int)tn, z, 4, groups, 0, 0, 0, 0, 0, 0};
            if (ws_bytes_for(c, m, n) > limit) break;
            const int64_t rounds = (tiles * z + kCUs - 1) / kCUs;
            const double main_cost = (double)rounds * ((double)((T + z - 1) / z) * cs.k_tile[cls] + cs.c_tile[cls]);
            const double fix = z > 1 ? ((double)m * n * cs.plane * z / 1667.0 + cs.launch) * groups : 0.0;
            const double cost = main_cost + fix;
            if (cost < best_cost) {
                best_cost = cost;
                best = c;
            }
        }
    }
    if (best.tile_id == 0) {           // overrides left nothing admissible: fall back to the safe default
        best = Plan{TILE_256x256, 256, 256, (int)((m + 255) / 256), (int)((n + 255) / 256), 1, 4, groups, 0, 0, 0, 0, 0, 0};
    }
    best.group_m = o.group > 0 ? o.group : 4;
    if (cost_out) *cost_out = best_cost;
    return best;
}

Plan plan_by(const Costs& cs, const Opts& o, int64_t m, int64_t n, int64_t k, int n_steps, int groups, size_t limit,
             double* cost_out = nullptr) {
    double whole_cost = 0.0;
    Plan best = plan_whole(cs, o, m, n, k, n_steps, groups, limit, &whole_cost);
    if (cost_out) *cost_out = whole_cost;
    if (groups != 1 || !o.trim || o.split > 1) return best;
    const int64_t T = (int64_t)n_steps * ((k + 63) / 64);
    const int tile_ids[4] = {TILE_256x256, TILE_128x256, TILE_256x128, TILE_128x128};
    const int forced_tile = o.tile;
    double best_cost = whole_cost;
    for (int ti = 0; ti < 4; ++ti) {
        if (forced_tile && tile_ids[ti] != forced_tile) continue;
        int bm, bn;
        tile_shape(tile_ids[ti], &bm, &bn);
        const int64_t tm = (m + bm - 1) / bm, tn = (n + bn - 1) / bn;
        const int64_t tiles = tm * tn, rem = tiles % kCUs;
        if (tiles <= kCUs || rem == 0 || rem % tn != 0) continue;      // the tail must be whole tile rows
        const int64_t tail_rows_tiles = rem / tn;
        if (tail_rows_tiles >= tm) continue;
        const int64_t m_main = (tm - tail_rows_tiles) * bm;
        double tail_cost = 0.0;
        const Plan tail = plan_whole(cs, o, m - m_main, n, k, n_steps, 1, limit, &tail_cost);
        const int cls = area_class(bm, bn);
        const double cost = (double)((tiles - rem) / kCUs) * ((double)T * cs.k_tile[cls] + cs.c_tile[cls]) + tail_cost + cs.trim;
        if (cost < best_cost) {
            best_cost = cost;
            if (cost_out) *cost_out = cost;
            best = Plan{tile_ids[ti], bm, bn, (int)(tm - tail_rows_tiles), (int)tn, 1, best.group_m, 1,
                        m_main, tail.tile_id, tail.tiles_m, tail.tiles_n, tail.split_k, 0};
        }
    }
    return best;
}

// The same for the kernel that splits K over the waves of a workgroup (no partial planes, one launch): `wgs` workgroups of bm
// rows, T chunks of 64 k each, operands of `bytes` in all.  Its few bytes in flight per wave make a chunk's time a matter of where
// the operands are and of how many workgroups ask (0.07 us a chunk cached and alone, 0.18 from memory, 0.5 with two rounds):
// fitted with kRunCosts, up to 512 workgroups and 256 chunks.  Both sides, from memory, in us: 128 x 2048 x 1024 forward 8.1
// against 12.4 (128 x 128, split 8 and fix-up), 7 x 9128 x 4360 dX 28.4 / 31.5, 40 x 1192 x 4064 dW 11.7 / 13.6; and where it loses,
// many workgroups with many chunks: 2176 x 7760 x 32 dW, four products, 58.6 / 37.3, 57 x 2552 x 320 dX, four steps, 32.8 / 23.5.
//   At most 16 rows (bm) leave room for a third slot a wave: one more chunk on its way, hardly any time a chunk of its own.
//   dW of less than 1 MB of operands finds them in the L2 (32 x 1736 x 16, three steps, 8.3 / 12.1).
//   NN stops at 64 chunks whatever the costs say.  It reads 64-byte pieces of weight rows, and the line depends on where
//   they are: 16 x K x 4096 from memory is even at K = 3072 (13.6 / 13.7; 4096: 20.1 / 15.2), from L2 at 5000 (4608: 14.6 / 15.4;
//   5120: 16.5 / 16.0); 16 x K x 1024 at 4096 (12.9 / 12.5) and beyond 12288 (14.0 / 19.3).
double small_cost(int form, int bm, int64_t wgs, int64_t T, double bytes) {
    if (wgs > 2 * kCUs || T > (form == FORM_NN ? 64 : 256)) return 1e300;
    struct C { double launch, round, chunk, crowd; };
    const C c = form == FORM_NN   ? C{1500.0, 4500.0, 155.0, 290.0}
                : form == FORM_TN ? C{150.0, 7300.0, bytes < 1e6 ? 60.0 : 260.0, 160.0}
                : bm == 16        ? C{2200.0, 6900.0, 10.0, 320.0}
                                  : C{300.0, 8400.0, 200.0, 50.0};
    return c.launch + (double)((wgs + kCUs - 1) / kCUs) * c.round + (double)T * (c.chunk + c.crowd * (double)wgs / kCUs);
}

// The same kernel for a forward of at most 32 rows, with tiles of 64 columns (whole cache lines of weight rows) and K split
// over z workgroups too where there are few of them: z > 1 writes planes and takes the fix-up launch.  A wave then has one or
// two chunks, with 16 rows all on their way at once, instead of a chain of them.  Fitted to 16 rows, in us, mean of operands from memory
// and cached (1900 cycles); from memory, against the better of 32 columns and 128 x 128 tiles: 4096 x 4096 19.9 -> 13.6 (z = 4), 4096 x
// 1024 18.9 -> 9.7 (8), 8192 x 2048 17.1 -> 13.4 (8), 1024 x 16384 16.0 -> 11.1 (1), 4096 x 8192 21.0 -> 19.5 (2); 3 steps of
// 392 x 5568 stay with 32 columns (7.9 against 9.1), 4 of 6144 x 6144 with 128 x 128 tiles (58 / 71).
// 32 rows leave a wave one slot, so its chunks do not overlap: 1.15 x a chunk of 16 rows where a wave has nine or more (1.50 us against 1.31,
// medians of 370 and 290 draws; both below the constants, which were fitted on another card: the line is on the safe side).
double wide_cost(int bm, int64_t strips, int z, int64_t T) {
    const int64_t chunks = (T + 8 * z - 1) / (8 * z), rounds = (strips * z + kCUs - 1) / kCUs;
    const double wgs = (double)(strips * z) / (double)rounds, chunk = bm == 16 ? 1.95 : 2.2;
    return 1900.0 * (2.8 + (z > 1 ? 2.8 : 0.0) + (double)(rounds * chunks) * (chunk + 1.2 * std::max(0.0, wgs / (kCUs / 2) - 1.0)));
}

// Bytes of workspace a call needs, and the plan the eight-wave kernel runs: its costs are those the query is made of.
Plan query_plan(const Opts& o, int64_t m, int64_t n, int64_t k, int n_steps, int groups = 1) {
    Plan p = plan_by(kQueryCosts, o, m, n, k, n_steps, groups, SIZE_MAX);
    p.need = ws_bytes_for(p, m, n);
    return p;
}

// four_wave: the product runs on the kernels of tp_gemm4.hip, tp_gemm_ms.hip and tp_small.hip
Plan make_plan(const Opts& o, int form, int64_t m, int64_t n, int64_t k, int n_steps, int groups, bool four_wave) {
    const Plan q = query_plan(o, m, n, k, n_steps, groups);
    if (!four_wave) return q;
    const size_t need = q.need;
    double cost = 0.0;
    Plan p = plan_by(kRunCosts, o, m, n, k, n_steps, groups, need, &cost);
    if (!o.tile && !o.split) {
        const int bm = m <= 16 && form != FORM_TN ? 16 : 32;
        const int64_t tm = (m + bm - 1) / bm, T = (int64_t)n_steps * ((k + 63) / 64), wgs = tm * ((n + 31) / 32) * groups;
        const int group_m = o.group > 0 ? o.group : 4;
        // (the products of a grouped launch share one operand)
        const double bytes = 2.0 * (double)k * (form == FORM_NT ? (double)m * n_steps + (double)n * n_steps * groups
                                                                : (double)m * n_steps * groups + (double)n * n_steps);
        const double small = small_cost(form, bm, wgs, T, bytes);
        if (small < cost) {
            // dX with half the chip's workgroups or fewer and a long K: tiles of 16 columns, twice the workgroups (16 x 4096, K = 4096:
            // 12.4 -> 10.1 us; 16 x 2048, K = 8192 18.2 -> 13.3; 128 x 512, K = 2 x 2048 8.6 -> 7.9; short of that it loses: 128 x 1000, K = 1000
            // 5.1 / 5.4; 300 x 136, K = 2 x 328 4.9 / 5.1)
            const int bn = form == FORM_NT && wgs <= kCUs / 2 && T >= 32 ? 16 : 32;
            p = Plan{bn == 32 ? (bm == 16 ? TILE_16x32_SMALL : TILE_32x32_SMALL) : (bm == 16 ? TILE_16x16_SMALL : TILE_32x16_SMALL), bm, bn,
                     (int)tm, (int)((n + bn - 1) / bn), 1, group_m, groups, 0, 0, 0, 0, 0, 0};
            cost = small;
        }
        if (form == FORM_NN && m <= 32 && groups == 1) {
            const int64_t strips = (n + 63) / 64;
            for (int z = 1; z <= 8 && z * strips <= (z > 1 ? kCUs : 4 * kCUs); ++z) {
                Plan c{bm == 16 ? TILE_16x64_SMALL : TILE_32x64_SMALL, bm, 64, 1, (int)strips, z, group_m, 1, 0, 0, 0, 0, 0, 0};
                const double wide = wide_cost(bm, strips, z, T);
                // Whole K in one workgroup: its chain of chunks is in the open where the strips do not fit one round of workgroups, and
                // is long beyond eight chunks a wave.  Time of the best other plan over this one's, from memory and cached, 280 drawn products:
                // strips in one round, up to 8 chunks a wave 0.86 - 1.63 and 1.12 - 1.79, more chunks 0.58 - 1.16 and 0.59 - 1.22; strips in
                // several, up to 2 chunks 0.88 - 1.02 and 0.97 - 1.41, more 0.59 - 1.01 and 0.59 - 1.10.  (30 x 16992, K = 2360: 31.1 and 24.2 us with,
                // 23.0 and 21.0 without; 32 x 10896, K = 3 x 1624: 33.6 and 23.4, 26.7 and 24.5.)
                if (z == 1 && T > (strips > kCUs ? 16 : 64)) continue;
                if (ws_bytes_for(c, m, n) > need || wide >= cost) continue;
                p = c;
                cost = wide;
            }
        }
    }
    p.need = need;
    return p;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_cblk(const tp_cblk_t& b, int64_t cols) {
    if (!b.ptr) return TP_ERR_NULL;
    if (!aligned16(b.ptr) || (b.ld & 7) || (cols & 7)) return TP_ERR_ALIGN;
    if (b.ld < cols || b.ld > kMaxLd) return TP_ERR_SHAPE;
    return TP_OK;
}
int check_oblk(const tp_oblk_t& b, int64_t cols, bool f32_only) {
    if (!b.ptr) return TP_ERR_NULL;
    if (b.dtype != TP_BF16 && b.dtype != TP_F32) return TP_ERR_DTYPE;
    if (f32_only && b.dtype != TP_F32) return TP_ERR_DTYPE;
    if (!aligned16(b.ptr) || (b.ld & 7) || (cols & 7)) return TP_ERR_ALIGN;
    if (b.ld < cols) return TP_ERR_SHAPE;
    return TP_OK;
}

struct Product {                 // one validated GEMM ready to launch
    int form; Plan plan; GemmArgs args; bool active;
    bool four_wave;              // on the four-wave (and workgroup-split) kernels; else on the eight-wave one
};

// The four-wave kernels and the workgroup-split one keep one buffer descriptor per (C tile, step) and move
// 32-bit lane offsets along K: every offset they can form must stay below 2^31.
bool w4_eligible(int form, const GemmArgs& a) {
    const bool a_kc = form != FORM_TN, b_kc = form == FORM_NT;
    const int slots = a.n_groups > 1 ? a.n_groups : a.n_steps;
    for (int s = 0; s < slots; ++s) {
        const int64_t lda = a.lda[s], ldb = a.ldb[s], K = a.K;
        if (a_kc ? (255 * lda + K) * 2 >= ((int64_t)1 << 31) : (K * lda + 256) * 2 >= ((int64_t)1 << 31)) return false;
        if (b_kc ? (255 * ldb + K) * 2 >= ((int64_t)1 << 31) : (K * ldb + 256) * 2 >= ((int64_t)1 << 31)) return false;
    }
    // its epilogue addresses a wave's 128 rows of every output (and of the GeLU' operand) the same way
    const int64_t lim = (int64_t)1 << 31, N = a.N;
    const int groups = a.n_groups > 1 ? a.n_groups : 1;
    for (int g = 0; g < groups; ++g) {
        const int64_t ldo = a.n_groups > 1 ? a.ldos[g] : a.ldo;
        if ((128 * ldo + N) * 4 >= lim) return false;
    }
    if (a.pre && (128 * a.ldp + N) * 2 >= lim) return false;
    if (a.dg && (128 * a.lddg + N) * 2 >= lim) return false;
    if (129 * N * 4 >= lim) return false;          // split-K planes
    return true;
}

int run_one(const Opts& o, int form, bool four_wave, int tile_id, int split_k, const GemmArgs& a, hipStream_t stream) {
    // 256 x 256 tiles run on the four-wave stream kernel unless the eight-wave one is asked for, smaller ones on
    // the four-wave kernel with a ring of stages; the eight-wave kernel keeps what their 32-bit offsets cannot reach
    GemmArgs la = a;
    if (four_wave) {
        switch (tile_id) {
            case TILE_256x256: tile_id = TILE_256x256_W4; break;
            case TILE_128x256: tile_id = TILE_128x256_MS; break;
            case TILE_256x128: tile_id = TILE_256x128_MS; break;
            case TILE_128x128: tile_id = TILE_128x128_MS; break;
            default: break;
        }
    }
    la.rotate = o.rotate < 0 ? !four_wave : o.rotate;
    if (launch_gemm(form, tile_id, la, stream) != hipSuccess) return TP_ERR_HIP;
    if (split_k > 1) {
        const int groups = a.n_groups > 1 ? a.n_groups : 1;
        const int64_t mn = (int64_t)a.M * a.N;
        for (int g = 0; g < groups; ++g) {
            void* out = groups > 1 ? a.outs[g] : a.out;
            const int64_t ldo = groups > 1 ? a.ldos[g] : a.ldo;
            ReduceArgs r{a.ws + g * mn, mn * groups, a.split_k, a.M, a.N, out, ldo, a.out_f32, a.pre, a.ldp, a.bias, a.gelu, a.dg, a.lddg};
            if (launch_reduce(r, stream) != hipSuccess) return TP_ERR_HIP;
        }
    }
    return TP_OK;
}

int run_product(const Opts& o, const Product& pr, void* workspace, hipStream_t stream) {
    GemmArgs a = pr.args;
    a.ws = static_cast<float*>(workspace);
    const Plan& pl = pr.plan;
    if (pl.m_main <= 0) return run_one(o, pr.form, pr.four_wave, pl.tile_id, pl.split_k, a, stream);
    // main launch: rows [0, m_main), a whole number of rounds
    const int64_t m = a.M, m0 = pl.m_main;
    GemmArgs mainp = a;
    mainp.M = (int32_t)m0;
    if (int e = run_one(o, pr.form, pr.four_wave, pl.tile_id, 1, mainp, stream)) return e;
    // tail launch: rows [m_main, m) through shifted pointers, with its own tile shape and K split
    GemmArgs tail = a;
    tail.M = (int32_t)(m - m0);
    tail.tiles_m = pl.tail_tiles_m; tail.tiles_n = pl.tail_tiles_n; tail.split_k = pl.tail_split;
    for (int k = 0; k < a.n_steps; ++k) {
        const char* ap = static_cast<const char*>(a.a[k]);
        tail.a[k] = pr.form == FORM_TN ? ap + m0 * 2 : ap + m0 * (int64_t)a.lda[k] * 2;    // TN: A is [k][m], else [m][k]
    }
    tail.out = static_cast<char*>(a.out) + m0 * a.ldo * (a.out_f32 ? 4 : 2);
    if (a.pre) tail.pre = static_cast<char*>(a.pre) + m0 * a.ldp * 2;
    if (a.dg) tail.dg = static_cast<const char*>(a.dg) + m0 * a.lddg * 2;
    return run_one(o, pr.form, pr.four_wave, pl.tail_tile_id, pl.tail_split, tail, stream);
}

// Bytes a product reads or writes: the span of one block of rows x cols (es bytes an element)
struct Range { uintptr_t lo, hi; };
Range span(const void* p, int64_t ld, int64_t rows, int64_t cols, int es) {
    const uintptr_t lo = reinterpret_cast<uintptr_t>(p);
    return Range{lo, lo + (uintptr_t)(((rows - 1) * ld + cols) * es)};
}
bool overlap(const Range& a, const Range& b) { return a.lo < b.hi && b.lo < a.hi; }

// whether `w` writes anything that `r` reads or writes
bool writes_into(const GemmArgs& w, int form, const GemmArgs& r) {
    const int outs = w.n_groups > 1 ? w.n_groups : 1, slots = r.n_groups > 1 ? r.n_groups : r.n_steps, r_outs = r.n_groups > 1 ? r.n_groups : 1;
    for (int g = 0; g < outs; ++g) {
        const Range o = w.n_groups > 1 ? span(w.outs[g], w.ldos[g], w.M, w.N, 4) : span(w.out, w.ldo, w.M, w.N, w.out_f32 ? 4 : 2);
        for (int s = 0; s < slots; ++s) {
            if (overlap(o, form == FORM_TN ? span(r.a[s], r.lda[s], r.K, r.M, 2) : span(r.a[s], r.lda[s], r.M, r.K, 2))) return true;
            if (overlap(o, form == FORM_NT ? span(r.b[s], r.ldb[s], r.N, r.K, 2) : span(r.b[s], r.ldb[s], r.K, r.N, 2))) return true;
        }
        if (r.dg && overlap(o, span(r.dg, r.lddg, r.M, r.N, 2))) return true;
        for (int h = 0; h < r_outs; ++h)
            if (overlap(o, r.n_groups > 1 ? span(r.outs[h], r.ldos[h], r.M, r.N, 4) : span(r.out, r.ldo, r.M, r.N, r.out_f32 ? 4 : 2))) return true;
    }
    return false;
}

// The two products of a backward call, dX first.  Where both run on the workgroup-split kernel they share one launch, unless one
// writes what the other reads or writes: there the order shows, and the header promises it.
int run_backward(const Opts& o, const Product& px, const Product& pw, void* workspace, hipStream_t stream) {
    auto small = [](const Product& p) { return p.active && p.plan.tile_id >= TILE_32x32_SMALL; };
    if (small(px) && small(pw) && !writes_into(px.args, pw.form, pw.args) && !writes_into(pw.args, px.form, px.args))
        return launch_gemm_pair(px.plan.tile_id, px.args, pw.plan.tile_id, pw.args, stream) == hipSuccess ? TP_OK : TP_ERR_HIP;
    if (px.active) if (int e = run_product(o, px, workspace, stream)) return e;
    if (pw.active) if (int e = run_product(o, pw, workspace, stream)) return e;
    return TP_OK;
}

void fill_common(const Opts& o, GemmArgs& a, int64_t m, int64_t n, int64_t k, int n_steps) {
    std::memset(&a, 0, sizeof(a));
    a.M = (int32_t)m; a.N = (int32_t)n; a.K = (int32_t)k; a.n_steps = n_steps;
    a.max_workgroups = kCUs;
    a.rotate = o.rotate;                       // (run_one resolves "automatic" once it knows the kernel)
}

// The plan of a product whose blocks, epilogue and groups are filled in.  The offsets that its strides ask for come first:
// they decide which kernels can run it, and so whose costs count.
void plan_product(const Opts& o, Product& pr) {
    GemmArgs& a = pr.args;
    const int groups = a.n_groups > 1 ? a.n_groups : 1;
    pr.four_wave = !o.eight_wave && w4_eligible(pr.form, a);
    pr.plan = make_plan(o, pr.form, a.M, a.N, a.K, a.n_steps, groups, pr.four_wave);
    const Plan& p = pr.plan;
    a.tiles_m = p.tiles_m; a.tiles_n = p.tiles_n; a.split_k = p.split_k; a.group_m = p.group_m;
    if (a.n_groups > 0) {                      // the products of a grouped launch lie side by side along N or M
        a.group_tiles = a.group_along_n ? p.tiles_n : p.tiles_m;
        (a.group_along_n ? a.tiles_n : a.tiles_m) *= groups;
    }
}

bool ws_ok(size_t need, const void* workspace, size_t bytes) {
    return need == 0 || (workspace && bytes >= need && aligned16(workspace));
}

// ---------------------------------------------------------------------------------------------
// Built-in scratch for tp_linear_fwd_static: a fixed array in device memory (every GPU the library
// runs on holds its own copy until the process ends).  Host code never uses the array's name as an
// address: the address on the current device is asked for once per device and kept.
// ---------------------------------------------------------------------------------------------
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
static std::atomic<void*> g_scratch_ptr[kMaxDevices];

int static_scratch(void** out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return TP_ERR_HIP;
    void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!ptr) {
        if (hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return TP_ERR_HIP;
        g_scratch_ptr[dev].store(ptr, std::memory_order_release);      // (two threads racing here store the same address)
    }
    *out = ptr;
    return TP_OK;
}

int linear_fwd(const tp_grid_t* grid, const tp_dims_t* dims, int n_steps, const tp_cblk_t* x_blocks,
               const tp_cblk_t* w_blocks, const void* bias, int epi, tp_oblk_t y, tp_oblk_t preact,
               void* workspace, size_t workspace_bytes, void* hip_stream, const tp_plan_opts_t* opts,
               bool use_static_scratch) {
    Opts o;

    if (int e = resolve_opts(opts, &o)) return e;
    Share s;
    if (int e = build_share(grid, dims, TP_PASS_FWD, &s)) return e;
    if (!x_blocks || !w_blocks) return TP_ERR_NULL;
    if (n_steps < 1 || n_steps > s.n_steps) return TP_ERR_SHAPE;
    if (epi != TP_EPI_NONE && epi != TP_EPI_BIAS && epi != TP_EPI_BIAS_GELU) return TP_ERR_MODE;
    if (epi != TP_EPI_NONE && !bias) return TP_ERR_NULL;
    if (bias && !aligned16(bias)) return TP_ERR_ALIGN;
    if (s.partial) {                    // an additive partial: bias and GeLU come after the summation
        if (epi != TP_EPI_NONE || preact.ptr) return TP_ERR_MODE;
        if (y.ptr && y.dtype != TP_F32) return TP_ERR_DTYPE;
    }
    if (s.m > INT32_MAX || s.n > INT32_MAX || s.k > INT32_MAX) return TP_ERR_SHAPE;
    for (int k = 0; k < n_steps; ++k) {
        if (int e = check_cblk(x_blocks[k], s.k)) return e;
        if (int e = check_cblk(w_blocks[k], s.n)) return e;
    }
    if (int e = check_oblk(y, s.n, false)) return e;
    if (preact.ptr) {
        if (int e = check_oblk(preact, s.n, false)) return e;
        if (preact.dtype != TP_BF16) return TP_ERR_DTYPE;
    }
    Product pr{};
    pr.form = FORM_NN;
    fill_common(o, pr.args, s.m, s.n, s.k, n_steps);
    for (int k = 0; k < n_steps; ++k) {
        pr.args.a[k] = x_blocks[k].ptr; pr.args.lda[k] = (int32_t)x_blocks[k].ld;
        pr.args.b[k] = w_blocks[k].ptr; pr.args.ldb[k] = (int32_t)w_blocks[k].ld;
    }
    pr.args.out = y.ptr; pr.args.ldo = y.ld; pr.args.out_f32 = y.dtype == TP_F32;
    pr.args.pre = preact.ptr; pr.args.ldp = preact.ld;
    pr.args.bias = epi == TP_EPI_NONE ? nullptr : bias;
    pr.args.gelu = epi == TP_EPI_BIAS_GELU;
    plan_product(o, pr);
    if (use_static_scratch) {
        if (pr.plan.need > kStaticScratchBytes) return TP_ERR_SCRATCH;
    } else if (!ws_ok(pr.plan.need, workspace, workspace_bytes)) {
        return TP_ERR_WORKSPACE;
    }
    if (int e = check_device()) return e;
    if (use_static_scratch) {
        if (int e = static_scratch(&workspace)) return e;
    }
    return run_product(o, pr, workspace, static_cast<hipStream_t>(hip_stream));
}

}  // namespace

extern "C" {

int tp_block_map(const tp_grid_t* grid, const tp_dims_t* dims, int pass, int* n_steps, int64_t* m, int64_t* n,
                 int64_t* k_per_step, int* a_row, int* a_col, int* b_row, int* b_col, int* out_row, int* out_col,
                 int* is_partial) {
    Share s;
    if (int e = build_share(grid, dims, pass, &s)) return e;
    if (n_steps) *n_steps = s.n_steps;
    if (m) *m = s.m;
    if (n) *n = s.n;
    if (k_per_step) *k_per_step = s.k;
    for (int i = 0; i < TP_MAX_STEPS; ++i) {
        if (a_row) a_row[i] = s.a_row[i];
        if (a_col) a_col[i] = s.a_col[i];
        if (b_row) b_row[i] = s.b_row[i];
        if (b_col) b_col[i] = s.b_col[i];
    }
    if (out_row) *out_row = s.out_row;
    if (out_col) *out_col = s.out_col;
    if (is_partial) *is_partial = s.partial;
    return TP_OK;
}

size_t tp_linear_workspace_size_ex(const tp_grid_t* grid, const tp_dims_t* dims, int pass, const tp_plan_opts_t* opts) {
    Opts o;
    if (resolve_opts(opts, &o) != TP_OK) return 0;
    if (pass == TP_PASS_DX_PARTIALS || pass == TP_PASS_DW_PARTIALS) {
        PartialsShare ps;
        if (build_partials(grid, dims, pass, &ps) != TP_OK) return 0;
        size_t worst = 0;               // any number of products 1 .. n_steps may be asked for
        for (int groups = 1; groups <= ps.n_steps; ++groups)
            worst = std::max(worst, query_plan(o, ps.m, ps.n, ps.k, 1, groups).need);
        return worst;
    }
    Share s;
    if (build_share(grid, dims, pass, &s) != TP_OK) return 0;
    size_t worst = 0;                   // any prefix 1 .. n_steps of the steps may be asked for
    for (int steps = 1; steps <= s.n_steps; ++steps)
        worst = std::max(worst, query_plan(o, s.m, s.n, s.k, steps).need);
    Share sf;                           // the bias gradient of tp_linear_bwd sums the forward block's columns in two passes
    if (pass != TP_PASS_FWD && build_share(grid, dims, TP_PASS_FWD, &sf) == TP_OK)
        worst = std::max(worst, colsum_ws_bytes(sf.m, sf.n));
    return worst;
}

size_t tp_linear_workspace_size(const tp_grid_t* grid, const tp_dims_t* dims, int pass) {
    return tp_linear_workspace_size_ex(grid, dims, pass, nullptr);
}

int tp_linear_fwd_ex(const tp_grid_t* grid, const tp_dims_t* dims, int n_steps, const tp_cblk_t* x_blocks,
                     const tp_cblk_t* w_blocks, const void* bias, int epi, tp_oblk_t y, tp_oblk_t preact,
                     void* workspace, size_t workspace_bytes, void* hip_stream, const tp_plan_opts_t* opts) {
    return linear_fwd(grid, dims, n_steps, x_blocks, w_blocks, bias, epi, y, preact, workspace, workspace_bytes, hip_stream,
                      opts, false);
}

int tp_linear_fwd_static(const tp_grid_t* grid, const tp_dims_t* dims, int n_steps, const tp_cblk_t* x_blocks,
                         const tp_cblk_t* w_blocks, const void* bias, int epi, tp_oblk_t y, tp_oblk_t preact,
                         void* hip_stream) {
    return linear_fwd(grid, dims, n_steps, x_blocks, w_blocks, bias, epi, y, preact, nullptr, 0, hip_stream, nullptr, true);
}

size_t tp_static_scratch_bytes(void) { return kStaticScratchBytes; }

int tp_linear_fwd(const tp_grid_t* grid, const tp_dims_t* dims, int n_steps, const tp_cblk_t* x_blocks,
                  const tp_cblk_t* w_blocks, const void* bias, int epi, tp_oblk_t y, tp_oblk_t preact,
                  void* workspace, size_t workspace_bytes, void* hip_stream) {
    return tp_linear_fwd_ex(grid, dims, n_steps, x_blocks, w_blocks, bias, epi, y, preact, workspace, workspace_bytes,
                            hip_stream, nullptr);
}

int tp_linear_bwd_ex(const tp_grid_t* grid, const tp_dims_t* dims, int n_steps_dx, int n_steps_dw,
                     const tp_cblk_t* dy_own, const tp_cblk_t* preact_own, const tp_cblk_t* da_row_blocks,
                     const tp_cblk_t* w_blocks_dx, const tp_cblk_t* x_blocks_dw, const tp_cblk_t* da_col_blocks,
                     int own_slot_dx, int own_slot_dw, const tp_cblk_t* dgelu_preact, tp_oblk_t dx, tp_oblk_t dw,
                     tp_oblk_t da_own_out, void* db_f32, void* workspace, size_t workspace_bytes, void* hip_stream,
                     const tp_plan_opts_t* opts) {
    Opts o;
    if (int e = resolve_opts(opts, &o)) return e;
    Share sf, sx, sw;
    if (int e = build_share(grid, dims, TP_PASS_FWD, &sf)) return e;
    if (int e = build_share(grid, dims, TP_PASS_DX, &sx)) return e;
    if (int e = build_share(grid, dims, TP_PASS_DW, &sw)) return e;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (sf.m > INT32_MAX || sf.n > INT32_MAX || sf.k > INT32_MAX) return TP_ERR_SHAPE;

    // ---- (1) own dA
    const bool want_da = da_own_out.ptr != nullptr;
    if (want_da) {
        if (!dy_own || !preact_own) return TP_ERR_NULL;
        if (int e = check_cblk(*dy_own, sf.n)) return e;
        if (int e = check_cblk(*preact_own, sf.n)) return e;
        if (int e = check_oblk(da_own_out, sf.n, false)) return e;
        if (da_own_out.dtype != TP_BF16) return TP_ERR_DTYPE;
        if (da_own_out.ld > kMaxLd) return TP_ERR_SHAPE;
    } else if (db_f32 || own_slot_dx >= 0 || own_slot_dw >= 0) {
        return TP_ERR_NULL;                      // both need the dA that only part (1) produces
    }
    if (db_f32 && !aligned16(db_f32)) return TP_ERR_ALIGN;
    const tp_cblk_t own_blk{da_own_out.ptr, da_own_out.ld};

    // ---- (2) dX
    Product px{}; px.active = dx.ptr != nullptr;
    if (px.active) {
        if (!da_row_blocks || !w_blocks_dx) return TP_ERR_NULL;
        if (n_steps_dx < 1 || n_steps_dx > sx.n_steps) return TP_ERR_SHAPE;
        if (own_slot_dx >= n_steps_dx) return TP_ERR_SHAPE;
        if (sx.partial) {               // a summand of a reduction: fp32, and GeLU' belongs after the sum
            if (dgelu_preact) return TP_ERR_MODE;
            if (dx.dtype != TP_F32) return TP_ERR_DTYPE;
        }
        fill_common(o, px.args, sx.m, sx.n, sx.k, n_steps_dx);
        for (int k = 0; k < n_steps_dx; ++k) {
            const tp_cblk_t& a = (k == own_slot_dx) ? own_blk : da_row_blocks[k];
            if (int e = check_cblk(a, sx.k)) return e;
            if (int e = check_cblk(w_blocks_dx[k], sx.k)) return e;       // W block is [n = H_blk][k = F_blk]
            px.args.a[k] = a.ptr; px.args.lda[k] = (int32_t)a.ld;
            px.args.b[k] = w_blocks_dx[k].ptr; px.args.ldb[k] = (int32_t)w_blocks_dx[k].ld;
        }
        if (int e = check_oblk(dx, sx.n, false)) return e;
        if (dgelu_preact) {
            if (int e = check_cblk(*dgelu_preact, sx.n)) return e;
            px.args.dg = dgelu_preact->ptr; px.args.lddg = dgelu_preact->ld;
        }
        px.args.out = dx.ptr; px.args.ldo = dx.ld; px.args.out_f32 = dx.dtype == TP_F32;
        px.form = FORM_NT;
        plan_product(o, px);
    }
    // ---- (3) dW
    Product pw{}; pw.active = dw.ptr != nullptr;
    if (pw.active) {
        if (!x_blocks_dw || !da_col_blocks) return TP_ERR_NULL;
        if (n_steps_dw < 1 || n_steps_dw > sw.n_steps) return TP_ERR_SHAPE;
        if (own_slot_dw >= n_steps_dw) return TP_ERR_SHAPE;
        fill_common(o, pw.args, sw.m, sw.n, sw.k, n_steps_dw);
        for (int k = 0; k < n_steps_dw; ++k) {
            const tp_cblk_t& b = (k == own_slot_dw) ? own_blk : da_col_blocks[k];
            if (int e = check_cblk(x_blocks_dw[k], sw.m)) return e;       // X block is [k = tokens][m = H_blk]
            if (int e = check_cblk(b, sw.n)) return e;
            pw.args.a[k] = x_blocks_dw[k].ptr; pw.args.lda[k] = (int32_t)x_blocks_dw[k].ld;
            pw.args.b[k] = b.ptr; pw.args.ldb[k] = (int32_t)b.ld;
        }
        if (int e = check_oblk(dw, sw.n, true)) return e;
        pw.args.out = dw.ptr; pw.args.ldo = dw.ld; pw.args.out_f32 = 1;
        pw.form = FORM_TN;
        plan_product(o, pw);
    }
    size_t need = 0;
    if (px.active) need = std::max(need, px.plan.need);
    if (pw.active) need = std::max(need, pw.plan.need);
    if (!ws_ok(need, workspace, workspace_bytes)) return TP_ERR_WORKSPACE;
    if (want_da || px.active || pw.active)
        if (int e = check_device()) return e;

    // ---- launches (stream order: dA, db, dX, dW)
    if (want_da) {
        // (the column sums take two passes over row slabs when the workspace holds the slab sums, else one)
        float* const cws = (workspace && aligned16(workspace) && workspace_bytes >= colsum_ws_bytes(sf.m, sf.n))
                               ? static_cast<float*>(workspace) : nullptr;
        const hipError_t e = db_f32 ? launch_dgelu_colsum(dy_own->ptr, dy_own->ld, preact_own->ptr, preact_own->ld, da_own_out.ptr,
                                                          da_own_out.ld, sf.m, sf.n, static_cast<float*>(db_f32), cws, stream)
                                    : launch_dgelu(dy_own->ptr, dy_own->ld, preact_own->ptr, preact_own->ld, da_own_out.ptr,
                                                   da_own_out.ld, sf.m, sf.n, stream);
        if (e != hipSuccess) return TP_ERR_HIP;
    }
    return run_backward(o, px, pw, workspace, stream);
}

int tp_linear_bwd(const tp_grid_t* grid, const tp_dims_t* dims, int n_steps_dx, int n_steps_dw,
                  const tp_cblk_t* dy_own, const tp_cblk_t* preact_own, const tp_cblk_t* da_row_blocks,
                  const tp_cblk_t* w_blocks_dx, const tp_cblk_t* x_blocks_dw, const tp_cblk_t* da_col_blocks,
                  int own_slot_dx, int own_slot_dw, const tp_cblk_t* dgelu_preact, tp_oblk_t dx, tp_oblk_t dw,
                  tp_oblk_t da_own_out, void* db_f32, void* workspace, size_t workspace_bytes, void* hip_stream) {
    return tp_linear_bwd_ex(grid, dims, n_steps_dx, n_steps_dw, dy_own, preact_own, da_row_blocks, w_blocks_dx,
                            x_blocks_dw, da_col_blocks, own_slot_dx, own_slot_dw, dgelu_preact, dx, dw, da_own_out,
                            db_f32, workspace, workspace_bytes, hip_stream, nullptr);
}

int tp_partials_map(const tp_grid_t* grid, const tp_dims_t* dims, int pass, int* n_steps, int64_t* m, int64_t* n,
                    int64_t* k, int* own_row, int* own_col, int* other_row, int* other_col, int* out_row, int* out_col) {
    PartialsShare s;
    if (int e = build_partials(grid, dims, pass, &s)) return e;
    if (n_steps) *n_steps = s.n_steps;
    if (m) *m = s.m;
    if (n) *n = s.n;
    if (k) *k = s.k;
    if (own_row) *own_row = s.own_row;
    if (own_col) *own_col = s.own_col;
    for (int i = 0; i < TP_MAX_STEPS; ++i) {
        if (other_row) other_row[i] = s.other_row[i];
        if (other_col) other_col[i] = s.other_col[i];
        if (out_row) out_row[i] = s.out_row[i];
        if (out_col) out_col[i] = s.out_col[i];
    }
    return TP_OK;
}

int tp_linear_bwd_partials_ex(const tp_grid_t* grid, const tp_dims_t* dims, int n_dx, int n_dw, const tp_cblk_t* da_own,
                              const tp_cblk_t* w_blocks_dx, const tp_oblk_t* dx_partials, const tp_cblk_t* x_blocks_dw,
                              const tp_oblk_t* dw_partials, void* workspace, size_t workspace_bytes, void* hip_stream,
                              const tp_plan_opts_t* opts) {
    Opts o;
    if (int e = resolve_opts(opts, &o)) return e;
    PartialsShare sx, sw;
    if (int e = build_partials(grid, dims, TP_PASS_DX_PARTIALS, &sx)) return e;
    if (int e = build_partials(grid, dims, TP_PASS_DW_PARTIALS, &sw)) return e;
    if (n_dx < 0 || n_dx > sx.n_steps || n_dw < 0 || n_dw > sw.n_steps) return TP_ERR_SHAPE;
    if (sx.m > INT32_MAX || sx.n > INT32_MAX || sx.k > INT32_MAX) return TP_ERR_SHAPE;
    if (n_dx == 0 && n_dw == 0) return TP_OK;
    if (!da_own) return TP_ERR_NULL;
    if (int e = check_cblk(*da_own, sx.k)) return e;                  // [M_blk, F_blk]
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);

    Range ranges[2 * TP_MAX_STEPS];
    int n_ranges = 0;
    Product px{}; px.active = n_dx > 0;
    if (px.active) {
        if (!w_blocks_dx || !dx_partials) return TP_ERR_NULL;
        fill_common(o, px.args, sx.m, sx.n, sx.k, 1);
        for (int k = 0; k < n_dx; ++k) {
            if (int e = check_cblk(w_blocks_dx[k], sx.k)) return e;    // W block [H_blk][F_blk]: n x k
            if (int e = check_oblk(dx_partials[k], sx.n, true)) return e;
            ranges[n_ranges++] = span(dx_partials[k].ptr, dx_partials[k].ld, sx.m, sx.n, 4);
            px.args.a[k] = da_own->ptr; px.args.lda[k] = (int32_t)da_own->ld;
            px.args.b[k] = w_blocks_dx[k].ptr; px.args.ldb[k] = (int32_t)w_blocks_dx[k].ld;
            px.args.outs[k] = dx_partials[k].ptr; px.args.ldos[k] = dx_partials[k].ld;
        }
        px.args.out = dx_partials[0].ptr; px.args.ldo = dx_partials[0].ld; px.args.out_f32 = 1;
        px.args.n_groups = n_dx; px.args.group_along_n = 1;            // the products side by side along N
        px.form = FORM_NT;
        plan_product(o, px);
    }
    Product pw{}; pw.active = n_dw > 0;
    if (pw.active) {
        if (!x_blocks_dw || !dw_partials) return TP_ERR_NULL;
        fill_common(o, pw.args, sw.m, sw.n, sw.k, 1);
        for (int k = 0; k < n_dw; ++k) {
            if (int e = check_cblk(x_blocks_dw[k], sw.m)) return e;    // X block [M_blk][H_blk]: k x m
            if (int e = check_oblk(dw_partials[k], sw.n, true)) return e;
            ranges[n_ranges++] = span(dw_partials[k].ptr, dw_partials[k].ld, sw.m, sw.n, 4);
            pw.args.a[k] = x_blocks_dw[k].ptr; pw.args.lda[k] = (int32_t)x_blocks_dw[k].ld;
            pw.args.b[k] = da_own->ptr; pw.args.ldb[k] = (int32_t)da_own->ld;
            pw.args.outs[k] = dw_partials[k].ptr; pw.args.ldos[k] = dw_partials[k].ld;
        }
        pw.args.out = dw_partials[0].ptr; pw.args.ldo = dw_partials[0].ld; pw.args.out_f32 = 1;
        pw.args.n_groups = n_dw; pw.args.group_along_n = 0;            // the products stacked along M
        pw.form = FORM_TN;
        plan_product(o, pw);
    }
    for (int i = 0; i < n_ranges; ++i)
        for (int j = i + 1; j < n_ranges; ++j)
            if (overlap(ranges[i], ranges[j])) return TP_ERR_SHAPE;
    size_t need = 0;
    if (px.active) need = std::max(need, px.plan.need);
    if (pw.active) need = std::max(need, pw.plan.need);
    if (!ws_ok(need, workspace, workspace_bytes)) return TP_ERR_WORKSPACE;
    if (int e = check_device()) return e;
    return run_backward(o, px, pw, workspace, stream);
}

int tp_linear_bwd_partials(const tp_grid_t* grid, const tp_dims_t* dims, int n_dx, int n_dw, const tp_cblk_t* da_own,
                           const tp_cblk_t* w_blocks_dx, const tp_oblk_t* dx_partials, const tp_cblk_t* x_blocks_dw,
                           const tp_oblk_t* dw_partials, void* workspace, size_t workspace_bytes, void* hip_stream) {
    return tp_linear_bwd_partials_ex(grid, dims, n_dx, n_dw, da_own, w_blocks_dx, dx_partials, x_blocks_dw, dw_partials,
                                     workspace, workspace_bytes, hip_stream, nullptr);
}

int tp_bias_act(const void* c, int64_t ld_c, const void* bias, int epi, tp_oblk_t y, tp_oblk_t preact, int64_t rows,
                int64_t cols, void* hip_stream) {
    if (!c || !y.ptr) return TP_ERR_NULL;
    if (epi != TP_EPI_NONE && epi != TP_EPI_BIAS && epi != TP_EPI_BIAS_GELU) return TP_ERR_MODE;
    if (epi != TP_EPI_NONE && !bias) return TP_ERR_NULL;
    if (rows < 0 || cols < 0) return TP_ERR_SHAPE;
    if (!aligned16(c) || (bias && !aligned16(bias)) || (ld_c & 7)) return TP_ERR_ALIGN;
    if (ld_c < cols) return TP_ERR_SHAPE;
    if (int e = check_oblk(y, cols, false)) return e;
    if (preact.ptr) {
        if (int e = check_oblk(preact, cols, false)) return e;
        if (preact.dtype != TP_BF16) return TP_ERR_DTYPE;
    }
    if (launch_bias_act(static_cast<const float*>(c), ld_c, epi == TP_EPI_NONE ? nullptr : bias, epi == TP_EPI_BIAS_GELU,
                        y.ptr, y.ld, y.dtype == TP_F32, preact.ptr, preact.ld, rows, cols,
                        static_cast<hipStream_t>(hip_stream)) != hipSuccess)
        return TP_ERR_HIP;
    return TP_OK;
}

int tp_dgelu(const void* dy, int64_t ld_dy, const void* preact, int64_t ld_pre, void* da, int64_t ld_da,
             int64_t rows, int64_t cols, void* hip_stream) {
    if (!dy || !preact || !da) return TP_ERR_NULL;
    if (rows < 0 || cols < 0) return TP_ERR_SHAPE;
    if (!aligned16(dy) || !aligned16(preact) || !aligned16(da) || (cols & 7) || (ld_dy & 7) || (ld_pre & 7) || (ld_da & 7))
        return TP_ERR_ALIGN;
    if (ld_dy < cols || ld_pre < cols || ld_da < cols) return TP_ERR_SHAPE;
    if (launch_dgelu(dy, ld_dy, preact, ld_pre, da, ld_da, rows, cols, static_cast<hipStream_t>(hip_stream)) != hipSuccess)
        return TP_ERR_HIP;
    return TP_OK;
}

size_t tp_bias_grad_workspace_size(int64_t rows, int64_t cols) {
    return rows > 0 && cols > 0 ? colsum_ws_bytes(rows, cols) : 0;
}

int tp_bias_grad(const void* da, int64_t ld_da, int64_t rows, int64_t cols, void* db_f32, void* workspace,
                 size_t workspace_bytes, void* hip_stream) {
    if (!da || !db_f32) return TP_ERR_NULL;
    if (rows < 0 || cols < 0) return TP_ERR_SHAPE;
    if (!aligned16(da) || !aligned16(db_f32) || (cols & 7) || (ld_da & 7)) return TP_ERR_ALIGN;
    if (ld_da < cols) return TP_ERR_SHAPE;
    if (workspace && (!aligned16(workspace) || workspace_bytes < colsum_ws_bytes(rows, cols))) return TP_ERR_WORKSPACE;
    if (cols == 0) return TP_OK;
    if (launch_colsum(da, ld_da, rows, cols, static_cast<float*>(db_f32), static_cast<float*>(workspace),
                      static_cast<hipStream_t>(hip_stream)) != hipSuccess)
        return TP_ERR_HIP;
    return TP_OK;
}

const char* tp_strerror(int status) {
    switch (status) {
        case TP_OK: return "ok";
        case TP_ERR_NULL: return "a required pointer is NULL";
        case TP_ERR_MODE: return "unknown mode, pass, epilogue or option, or an epilogue asked of an additive partial";
        case TP_ERR_GRID: return "grid size or rank coordinate out of range";
        case TP_ERR_SHAPE: return "layer dimensions, leading dimension or step count do not fit the grid, or outputs overlap";
        case TP_ERR_ALIGN: return "pointer not 16-byte aligned, or a column extent / leading dimension not a multiple of 8";
        case TP_ERR_DTYPE: return "output dtype not supported here";
        case TP_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
        case TP_ERR_HIP: return "a HIP call failed, or the device is not a 256-CU MI355X";
        case TP_ERR_SCRATCH: return "the product needs more than the library's built-in scratch: call tp_linear_fwd with a workspace";
        default: return "unknown status";
    }
}

}  // extern "C"
