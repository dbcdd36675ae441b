// The choice among the batched kernels, by estimates of their times.
//
// Five ways serve a batch: the few-token kernels (tsvd_few.hip, groups of 16 tokens side by side), thin token panels (both stages in one
// launch, 16 or 32 tokens per workgroup), planes of x with tiles of tsvd_fp6_split.hip per stage (128 x 16 to 256 x 64, the contraction split over groups of wavefronts), the same with the tiles of
// tsvd_fp6.hip (many rows and tokens), and the ring and large-tile kernels of tsvd_gemm.hip on 16-bit operands.  No single quantity
// separates them: a launch with few workgroups is bound by its serial chain (steps of a workgroup's loop), one with many by
// matrix instructions, a thin panel by the code words it streams.  So each gets an estimate in microseconds, a sum of
// the quantities that bound it: the launch, rounds of workgroups over the compute units, loop steps, records of x made, code bytes.
// The factors are fits (non-negative least squares on relative errors) to measurements on MI355X of calls of random shapes (17 to
// 16384 tokens, factors of 1 KB to 64 MB).  Checked on 220 other calls (profiles/batch_choice.csv: each of the ways timed, and what
// the rule took): the estimates' root mean square error is 10 to 15 % for bf16, 8 to 20 % for fp32 and 10 to 13 % for
// convolutions; the time of the way taken is 4.9 % above the best way's on the average for bf16 (one call in ten more than 18 %), 2.6 % for fp32, 1.4 %
// for convolutions, and 1.20, 1.84 and 1.23 times the speed of always taking the older ones.
#include "tsvd_batch.h"

#include <algorithm>
#include <initializer_list>

#include "tsvd_few.h"
#include "tsvd_gemm_common.h"
#include "tsvd_kernels.h"
#include "tsvd_thin.h"

namespace {

long long up(long long a, long long b) { return (a + b - 1) / b; }

struct sizes {
    long long M, N, B, cus, nvb, nub, sets;       // blocks of 128 of N and of K; sets of three planes (two for fp32)
};

// ---- the plane path: x to planes, stage V with shape v, stage U with shape u (0: tsvd_fp6.hip) -------------------
double planes_cost(const sizes& s, int v) {
    if (tsvd_fp6_split_makes_x(v, (int)std::min<long long>(s.sets * s.nvb, 1 << 20))) return 0;      // stage V makes them
    return 4.9 + 8.4 * (double)(s.nvb * up(s.B, 16) * s.sets) / 4096;
}
// (Fitted to kernels with a barrier for each step of 16 records.  All four shapes are faster since: tsvd_fp6_own_kernel for 9 and 10, tsvd_fp6_pair_kernel for 18 and 20.
// On 136 calls the shapes that these factors take are 1.2 % slower than the best of all 16 pairs of them, those of new factors for 9 and 10 1.1 %; and lower estimates
// would take calls from kernels that hold x exactly.)
struct split_factors {
    int shape;
    double v0, v_round, v_step, v_x, u0, u_round, u_step;
};
constexpr split_factors split_table[] = {
    {9, 1.3, 2.1, 2.9, 2.2, 0.7, 1.3, 3.0},
    {10, 0.3, 4.4, 1.9, 2.2, 0.4, 2.5, 2.1},
    {18, 0.0, 4.1, 3.0, 2.4, 0.3, 2.8, 3.4},
    {20, 0.0, 5.7, 2.3, 2.4, 0.0, 5.8, 2.4},
};
// rounds of workgroups and loop steps (16 records each) of a stage
double rounds(const sizes& s, int shape, long long row_blocks) { return (double)up(up(row_blocks, shape >> 3) * up(s.B, 16 * (shape & 7)), s.cus); }
double steps(int shape, long long blocks) { return (double)up(blocks, 16 / (shape & 7)); }

double split_v_cost(const sizes& s, const split_factors* f) {
    if (!f) {       // 256 x 128 or 512 x 64 tiles, two workgroups per compute unit
        const bool small = up(s.nub, 2) * up(s.B, 128) < s.cus;
        const double w = (double)(s.nub % 4 || small ? up(s.nub, 2) * up(s.B, 128) : up(s.nub, 4) * up(s.B, 64));
        const double r = (double)up((long long)w, 2 * s.cus), fill = w > (double)s.cus ? std::min(1.0, std::max(0.5, w / (2.0 * (double)s.cus * r))) : 0.55;
        return planes_cost(s, 0) + r * fill * (12.5 + 2.4 * (double)(s.sets * s.nvb));
    }
    const double r = rounds(s, f->shape, s.nub), x = planes_cost(s, f->shape);
    // records of x per wavefront where the stage makes them
    const double made = x > 0 ? 0 : r * (double)(up(s.nvb * (f->shape & 7), 8) * s.sets) * f->v_x;
    return x + f->v0 + r * f->v_round + r * steps(f->shape, s.sets * s.nvb) * f->v_step + made;
}
double split_u_cost(const sizes& s, const split_factors* f) {
    if (!f) {       // 128 x 64 (four per compute unit), 256 x 64 (three), 512 x 64 or 256 x 128 (two)
        const long long t256 = up(s.M, 256), c64 = up(s.B, 64), c128 = up(s.B, 128);
        const bool small = t256 * c128 < s.cus;
        double w, slots, size;
        if (small && 4 * t256 * c64 < 3 * s.cus) { w = (double)(up(s.M, 128) * c64); slots = 4; size = 1; }
        else if (small) { w = (double)(t256 * c64); slots = 3; size = 2; }
        else if (t256 % 2 == 0) { w = (double)(up(s.M, 512) * c64); slots = 2; size = 4; }
        else { w = (double)(t256 * c128); slots = 2; size = 4; }
        const double all = slots * (double)s.cus, fill = w <= all ? std::max(1 / slots, w / all) : w / all, n = (double)(s.sets * s.nub);
        return 2.7 + fill * size * (4.2 + 0.51 * n) + 0.4 * n;
    }
    const double r = rounds(s, f->shape, up(s.M, 128));
    return f->u0 + r * f->u_round + r * steps(f->shape, s.sets * s.nub) * f->u_step;
}

// ---- thin panels ----------------------------------------------------------------------------------
// (Fitted to one workgroup for each panel and to loads by element: several workgroups where panels are few, and rows of three taps in one load, are faster
// since and not in these numbers.)
double thin_cost(const tsvd_batch_call& c, int tiles) {
    const long long nvb = up(c.N, 128), nub = up(c.K, 128), panels = up(c.B, 16 * tiles);
    const double r = (double)up(panels, c.cus), busy = (double)std::min(panels, c.cus) / (double)c.cus;
    long long passes = 1ll << 60, units = 0;         // 16-row blocks of stage U per wavefront, and the units they come in
    for (int utm : {8, 4, 2}) {
        const long long u = up(up(c.M, 16 * utm), 8);
        if (u * utm < passes) passes = u * utm, units = u;
    }
    const double Kp = (double)tsvd_round_up(c.K, 256), mb_u = Kp * (double)tsvd_round_up(c.M, 256) / 4e6, mb_v = Kp * (double)tsvd_round_up(c.N, 256) / 4e6;
    if (c.x_token_major) {      // (a pass of stage U takes its blocks of K, or its part of y: the stores of all panels share the memory)
        auto total = [&](double t, double round, double record, double v1, double block, double store, double pass, double unit, double code) {
            return t + r * (round + (double)up(nvb * tiles, 8) * record + v1 * (double)(up(nub, 8) * nvb) + unit * (double)units + code * busy * (mb_u + mb_v) +
                            (double)passes * std::max(block * (double)nub, store * busy * (c.out_bf16 ? 0.5 : 1) + pass));
        };
        return tiles == 1 ? total(2.2, 2.07, 0.60, 0.473, 0.085, 0.096, 0.195, 0.483, 4.28) : total(3.0, 1.54, 0.66, 0.84, 0.165, 0.196, 0.386, 0.45, 11.6);
    }
    const double gather = c.conv ? r * (double)up(nvb * tiles, 8) : 0, v = r * (double)(up(nub, 8) * nvb), u = r * (double)(passes * nub) / 8,
                 y = r * (double)passes * (c.out_bf16 ? 0.5 : 1) * (c.y_token_major ? 2.6 : 1);
    if (tiles == 1) return 1.2 + 3.2 * r + 1.6 * gather + 0.57 * v + 0.29 * u + 0.35 * r * (double)units + 11.2 * r * mb_u + 8.1 * busy * r * (mb_u + mb_v) + 0.08 * y;
    return 1.4 + 3.7 * r + 0.92 * gather + 0.92 * v + 0.45 * u + 0.34 * r * (double)units + 25.1 * r * mb_u + 13.3 * busy * r * (mb_u + mb_v) + 0.10 * y;
}

// A copy of x for the kernels that read aligned feature-major rows: a transposition, or rows moved to aligned ones.
double copy_cost(const tsvd_batch_call& c) {
    const double m = (double)c.N * (double)c.B / 1e6;
    return c.copies ? 3.3 + 1.9 * m : 0;
}

// ---- ring and large-tile kernels ----------------------------------------------------------------
double older_cost(const tsvd_batch_call& c) {
    double t = 7.3;
    if (c.conv) t += 6.0 + 1.3 * (double)c.N * (double)c.B / 1e6;               // columns written first
    else t += copy_cost(c);
    auto stage = [&](long long rows, long long rows_p, long long blocks, double ring64, double ring128_0, double ring128, double large_0, double large) {
        const int shape = tsvd_gemm_tile_shape(rows_p, c.B, c.cus, true);
        const long long tr = shape < 2 ? 256 : shape == 15 ? 128 : shape == 17 ? 96 : 64, tt = shape == 0 ? 256 : shape == 1 ? 128 : 64;
        const double work = std::max(1.0, (double)(up(rows, tr) * up(c.B, tt)) / (double)c.cus) * (double)(tr * tt) / 4096 * (double)blocks / 8;
        t += shape < 2 ? large_0 + large * work : shape == 15 ? ring128_0 + ring128 * work : ring64 * work;
    };
    stage(128 * up(c.K, 128), tsvd_round_up(c.K, 256), up(c.N, 128), 3.45, 2.0, 3.2, 5.0, 1.87);
    stage(c.M, tsvd_round_up(c.M, 256), up(c.K, 128), 3.76, 4.3, 3.6, 18.3, 2.0);
    return t;
}

// 64-token panels, for the calls that their rule gives them (288 such calls measured)
double panel_cost(const tsvd_batch_call& c) {
    const long long nvb = up(c.N, 128), nub = up(c.K, 128), strips = up(c.M, 128);
    const double r = (double)up(up(c.B, 64), c.cus);
    if (c.x_token_major) return r * (6.3 + 2.2 * (double)nvb + 1.3 * (double)(up(strips, 8) * nub) + (double)strips * (c.y_token_major ? 0.95 : 0.61));
    return 0.95 * r * (7.5 + 2.3 * (double)nvb + 1.8 * (double)(up(strips, 8) * nub) + (double)strips * (c.y_token_major ? 1.9 : 0.83));
}

// fp32 activations run on planes whatever the shapes, so theirs are chosen by factors of their own up to 1024 tokens, fitted to the kernels as they are (kernel traces of 180 calls, 90 of them
// fp32, each with all shapes: 10 to 17 % rms; the shapes taken are 0.6 % slower than the best of each stage, those of the factors above 5 %: those know neither that wavefronts take blocks of
// their own nor what y costs).  Beyond, where rounds of many workgroups follow each other, they take split tiles too often (3520 x 2156 x 6144 at 6540 tokens 631 -> 758 us, 768 x 911 x 512 at 10040
// 69 -> 74).  1898 x 1344 x 1120 at 211 tokens 22.4 -> 17.2 us, 4655 x 1408 x 114 at 23 17.4 -> 12.2, 455 x 1052 x 263 at 896 19.6 -> 13.5;
// 172 calls of 17 to 1024 tokens 0.96 of the time on the average, one of them longer (3072 x 768 x 1536 at 333, between two tiles' lines, 21.3 -> 22.0).
struct own_factors {
    int shape;
    double v0, v_round, v_step, v_made, planes, planes_each, u0, u_round, u_step, u_mb;
};
constexpr own_factors f32_table[] = {
    {9, 2.06, 1.18, 1.09, 1.21, 5.4, 6.3, 1.33, 1.02, 1.19, 0.086},
    {10, 0.88, 3.70, 0.83, 1.13, 3.7, 7.2, 1.11, 1.08, 0.94, 0.183},
    {18, 0.0, 4.19, 2.24, 1.30, 5.1, 7.8, 1.80, 1.44, 2.64, 0.259},
    {20, 0.0, 5.59, 1.79, 1.41, 5.3, 7.9, 1.07, 4.41, 2.03, 0.194},
};
// rounds of workgroups, and what the slowest wavefront of one multiplies: blocks of its own times token tiles (128 rows), steps of four records (256 rows)
double own_v_cost(const sizes& s, const own_factors& f) {
    const long long n = s.sets * s.nvb, tiles = f.shape & 7;
    const double r = rounds(s, f.shape, s.nub), steps = f.shape < 16 ? (double)(up(n, 8) * tiles) : (double)up(up(n * tiles, 4), 4);
    const bool makes = tsvd_fp6_split_makes_x(f.shape, (int)std::min<long long>(n, 1 << 20));
    return f.v0 + r * (f.v_round + f.v_step * steps) +
           (makes ? r * f.v_made * (double)(up(s.nvb * tiles, 8) * s.sets) : f.planes + f.planes_each * (double)(s.nvb * up(s.B, 16) * s.sets) / 4096);
}
double own_u_cost(const sizes& s, const own_factors& f, bool out_bf16) {
    const long long n = s.sets * s.nub, tiles = f.shape & 7;
    const double r = rounds(s, f.shape, up(s.M, 128)), steps = f.shape < 16 ? (double)(up(n, 8) * tiles) : (double)up(up(n * tiles, 4), 4);
    return f.u0 + r * (f.u_round + f.u_step * steps) + f.u_mb * (double)s.M * (double)s.B * (out_bf16 ? 2e-6 : 4e-6);
}

// The shapes of the plane path's stages, 0 each for the tiles of tsvd_fp6.hip.
struct tiles_choice {
    int v, u;
    double time, fp6_tiles;         // with these shapes; with 0 and 0
};
tiles_choice choose_tiles(const tsvd_batch_call& c) {
    const sizes s = {c.M, c.N, c.B, c.cus, up(c.N, 128), up(c.K, 128), c.f32 ? 2 : 1};
    double best_v = split_v_cost(s, nullptr), best_u = split_u_cost(s, nullptr);
    tiles_choice t = {0, 0, 0, best_v + best_u};
    if (c.f32 && c.B <= 1024) {
        for (const own_factors& f : f32_table) {
            const double cv = own_v_cost(s, f), cu = own_u_cost(s, f, c.out_bf16);
            if (cv < best_v) best_v = cv, t.v = f.shape;
            if (cu < best_u) best_u = cu, t.u = f.shape;
        }
        t.time = best_v + best_u;
        return t;
    }
    for (const split_factors& f : split_table) {
        const double cv = split_v_cost(s, &f), cu = split_u_cost(s, &f);
        if (cv < best_v) best_v = cv, t.v = f.shape;
        if (cu < best_u) best_u = cu, t.u = f.shape;
    }
    t.time = best_v + best_u;
    return t;
}
// The columns of a convolution, written first.
double columns_cost(const tsvd_batch_call& c) { return c.conv ? 6.0 + 1.3 * (double)c.N * (double)c.B / 1e6 : 0; }
bool takes_panel(const tsvd_batch_call& c) {
    return c.whole && tsvd_gemm_use_panel(tsvd_round_up(c.M, 256), tsvd_round_up(c.K, 256), tsvd_round_up(c.N, 256), c.B, c.cus, true);
}
// Another way replaces the older one only where its estimate is below this: a tenth less, the estimates' own error (a twentieth for rows of tokens: on 150
// such calls of 513 to 16384 tokens that the factors are not fitted to, 0.97 of the time of the choices made by the factors from before
// rows were read and written at any alignment; feature-major calls gain nothing by a new fit).  Where an older call runs on planes of x
// too, its estimate is that of the same tiles; where stage V is on 16-bit operands it has a pass over z, and x copied.
double to_beat(const tsvd_batch_call& c, double fp6_tiles, bool panel) {
    const long long Mp = tsvd_round_up(c.M, 256), Kp = tsvd_round_up(c.K, 256), Np = tsvd_round_up(c.N, 256);
    return (c.conv || panel ? 1.0 : c.x_token_major ? 0.95 : 0.9) *
           (panel ? panel_cost(c) + columns_cost(c)
            : !tsvd_gemm_use_fp6(Mp, Kp, Np, c.B, c.cus, true) ? older_cost(c)
            : c.x_token_major && !tsvd_gemm_reads_in_place(Mp, Kp, Np, c.B, c.cus) ? 1.15 * fp6_tiles + copy_cost(c) : fp6_tiles + columns_cost(c));
}
bool splits(const tsvd_batch_call& c, const tiles_choice& t, bool panel, double beat) {
    return !panel && (t.v || t.u) && t.time + columns_cost(c) < beat && tsvd_gemm_split_bytes(c.K, c.N, c.B, false) < (1ull << 31);
}

}  // namespace

size_t tsvd_gemm_split_bytes(long long K, long long N, long long B, bool f32) {
    const long long sets = f32 ? 2 : 1, Bp = tsvd_round_up(B, f32 ? 256 : 128);
    auto part = [&](long long len) { return (tsvd_gemm_fp6_bytes(128 * sets * up(len, 128), Bp) + 255) & ~(size_t)255; };
    return part(N) + part(K);
}

bool tsvd_batch_may_split(tsvd_batch_call c) {
    const bool panel = takes_panel(c);
    const tiles_choice t = choose_tiles(c);
    for (const bool tokens : {false, true}) {
        c.x_token_major = tokens;
        if (tsvd_tuning_any() ? tsvd_plan_batch(c).split : splits(c, t, panel, to_beat(c, t.fp6_tiles, panel))) return true;
    }
    return false;
}

tsvd_batch_plan tsvd_plan_batch(const tsvd_batch_call& c) {
    tsvd_batch_plan plan = {false, 0, c.f32, 0, 0};
    if (tsvd_tuning_any()) {        // a diagnostic that sets switches means the kernels that they select
        const int thin = tsvd_tune("TSVD_THIN", 0), v = tsvd_tune("TSVD_SPLIT_V", 0), u = tsvd_tune("TSVD_SPLIT_U", 0);
        if (thin > 0 && !c.f32 && c.whole) plan.thin = thin;
        plan.few = c.few && c.B <= tsvd_tune("TSVD_FEW", 0);
        if (v > 0 || u > 0) plan = {false, plan.thin, true, v, u};
        return plan;
    }
    const tiles_choice t = choose_tiles(c);
    if (c.f32) {
        plan.split_v = t.v;
        plan.split_u = t.u;
        return plan;
    }
    const bool panel = takes_panel(c);
    double best = to_beat(c, t.fp6_tiles, panel);
    if (splits(c, t, panel, best)) {
        best = t.time + columns_cost(c);
        plan = {false, 0, true, t.v, t.u};
    }
    // (every panel streams both factors: measured for code words that one XCD's L2 holds)
    if (c.whole && c.K * (c.M + c.N) <= (16ll << 20))
        for (int tiles : {1, 2})
            if (tsvd_thin_chunk(c.K, c.N, tiles, c.conv) > 0) {
                const double t = thin_cost(c, tiles);
                if (t < best) best = t, plan.thin = tiles;
            }
    // Few tokens: each group of 16 reads both factors again, measured up to 600 tokens.  A twentieth and 0.7 us less than the best of the others (what
    // either estimate is off by where a call is hardly more than its launches).  On 200 calls of 17 to 128 tokens 0.67
    // of the time without them on the average (the worst 1.04), 0.3 to 0.4 for thousands of rows at 17 to 30 tokens; on 160 of 129 to 1024 tokens 0.83.
    // (The best of both ways would have been 0.6 and 0.9 % faster.)
    if (c.few && c.whole && c.B <= 1024) {
        const double t = tsvd_few_cost({c.M, c.N, c.K, c.B, c.cus, c.x_token_major, c.x_aligned, c.out_bf16});
        plan.few = t < 0.95 * best && t < best - 0.7;
    }
    return plan;
}
