// Host-side planning of the sequence-length GEMMs: which tile, how many splits of the reduction, how two GEMMs share a
// launch.  Sizes and the chip's width in, plans out; the buffer sizes and the launches both ask here.
#pragma once

#include <string.h>

#include "flurka_fast.h"
#include "flurka_gemm.h"

namespace flurka {

// A plan depends on sizes alone, and a call asks for it three or four times (buffer sizes, layout, launch): each thread
// keeps its last few, so that neither the call's own questions nor a few alternating shapes work it out again.
template <class Plan>
struct KeptPlans {
    static constexpr int PLANS = 8, SIZES = 6;
    long key[PLANS][SIZES] = {};       // no plan has sizes of 0
    Plan plan[PLANS] = {};
    int next = 0;
    template <class Make>
    const Plan& get(const long (&sizes)[SIZES], Make&& make) {
        for (int i = 0; i < PLANS; ++i)
            if (memcmp(key[i], sizes, sizeof(sizes)) == 0) return plan[i];
        const int i = next;
        next = (next + 1) % PLANS;
        plan[i] = make();
        memcpy(key[i], sizes, sizeof(sizes));
        return plan[i];
    }
};

// ===========================================================================
// Products that leave fp32 split partials: the projection, and the two products of the paper-order path
// ===========================================================================
struct SplitGemmPlan {
    int kind;              // index into SPLIT_GEMM_KINDS
    PartialTile t;         // output tile
    int tilesM, tilesN, splits, steps_per_split, total_steps;
    size_t partial_bytes() const { return (size_t)2 * splits * tilesM * tilesN * t.tm * t.tn * 4; }
};

// Output tiles of the products that leave fp32 split partials, and the time of one 64-deep reduction step of a
// workgroup that has a compute unit to itself: with all compute units at work, and with three quarters of them or fewer.
// Measured with operands from HBM: the 256 x 256 tile is bound by its matrix instructions, which run faster where some of
// the chip idles (1.51 - 1.55 us per step with 144 to 192 workgroups, 1.8 - 1.9 with 256); the others by how fast a
// compute unit takes its operands in (50 - 57 GB/s).
struct SplitGemmKind { PartialTile t; double step_us, step_us_part; };
constexpr SplitGemmKind SPLIT_GEMM_KINDS[] = {{{256, 256, 128, 128}, 1.78, 1.55}, {{128, 256, 64, 64}, 0.95, 0.95},
                                              {{128, 128, 64, 64}, 0.6, 0.6}, {{64, 128, 32, 64}, 0.45, 0.45}};

// Tile and split of two products of k rows, `batches` times `cols` columns (no tile crosses a batch) and `total_steps`
// steps whose operands are `bytes` long.
// The partial results are the price of a split (written at the end, when nothing is left to read beside it, and
// read again by the second stage, both at about 4.5 TB/s): 64 MiB with a 256 x 256 tile on every compute unit,
// whatever the size of the problem.  Short reductions want the smaller tiles and few splits, long ones the large
// tile.  Measured, projection + second stage, 256 x 256 with one split per compute unit against this rule's choice:
//   k 256, n 4096, 64 heads of 64:   29.2 + 17.2 -> 24.7 + 11.8 us (128 x 128)
//   k 256, n 16384, 64 heads of 64:  92 + 14.8 -> 86.8 + 11.8 (128 x 256)
//   k 256, n 8192, 48 heads of 64:   35.2 + 14.8 -> 30.7 + 13.0 (128 x 256; devices differ: 30.7 - 38 for the same tile)
//   k 64, n 512, 4 heads of 64:      11.1 + 7.3 -> 6.3 + 6.5 (64 x 128)
//   k 512, n 65536, 16 heads of 128: 229 + 21 (stays)
//   k 768 - 1129, n 8192 - 13280, 24 to 48 heads (stay, 192 to 240 workgroups): 104 - 177 + 22 - 31, with 128 x 256
//   tiles 110 - 197 + 20
inline SplitGemmPlan make_split_gemm_plan(int k, int batches, int cols, int total_steps, double bytes, int cus) {
    SplitGemmPlan best{};
    double best_t = -1.0;
    for (int kind = 0; kind < 4; ++kind) {
        SplitGemmPlan q;
        q.kind = kind;
        q.t = SPLIT_GEMM_KINDS[kind].t;
        q.tilesM = (k + q.t.tm - 1) / q.t.tm;
        q.tilesN = batches * ((cols + q.t.tn - 1) / q.t.tn);
        q.total_steps = total_steps;
        const int tiles = q.tilesM * q.tilesN * 2;
        const int most = tiles < cus ? (cus / tiles < total_steps ? cus / tiles : total_steps) : 1;
        for (int want = 1; want <= most; want += want < 8 ? 1 : 8) {
            q.steps_per_split = (total_steps + want - 1) / want;
            q.splits = (total_steps + q.steps_per_split - 1) / q.steps_per_split;
            const double read = bytes / 4.8e6;
            // rounds of workgroups: the smaller tiles hand out ids padded to a multiple of 8 per row tile
            const long ids = kind == 0 ? (long)tiles * q.splits : 8L * q.tilesM * ((2L * q.splits * q.tilesN + 7) / 8);
            const long rounds = (ids + cus - 1) / cus;
            // share of the chip at work in a round, from three quarters (0) to all of it (1)
            double full = 4.0 * (double)tiles * q.splits / (double)(rounds * cus) - 3.0;
            if (full < 0.0) full = 0.0;
            const SplitGemmKind& g = SPLIT_GEMM_KINDS[kind];
            double t = (double)q.steps_per_split * (double)rounds * (g.step_us_part + full * (g.step_us - g.step_us_part));
            if (t < read) t = read;
            t += 2.0 * (double)q.partial_bytes() / 4.5e6 + 0.1 * q.splits;
            if (best_t < 0.0 || t < best_t) { best_t = t; best = q; }
        }
    }
    return best;
}

inline SplitGemmPlan split_gemm_plan(int k, int batches, int cols, int total_steps, double bytes) {
    static thread_local KeptPlans<SplitGemmPlan> kept;
    const int cus = chip_cus();
    const long sizes[] = {k, batches, cols, total_steps, (long)bytes, cus};
    return kept.get(sizes, [&]() { return make_split_gemm_plan(k, batches, cols, total_steps, bytes, cus); });
}

inline SplitGemmPlan proj_plan(const Problem& p) {
    return split_gemm_plan(p.k, 1, p.BH * p.d, (p.n + GBK - 1) / GBK, 4.0 * p.n * ((double)p.BH * p.d + p.k));
}

struct FusedWPlan {
    int tpb1, tpb2;                // column tiles per batch of the two products
    SplitGemmPlan s1, s2;
};

inline FusedWPlan fusedw_plan(const Problem& p, int dm) {
    FusedWPlan q;
    q.s1 = split_gemm_plan(p.k, p.B, dm, (p.n + GBK - 1) / GBK, 4.0 * p.n * ((double)p.B * dm + p.k));
    q.tpb1 = q.s1.tilesN / p.B;
    const double terms = 3.0 * dm * 2.0;
    q.s2 = split_gemm_plan(p.k, p.B, p.H * p.d, 3 * dm / GBK, 2.0 * terms * p.B * p.k + 4.0 * p.H * p.d * dm);
    q.tpb2 = q.s2.tilesN / p.B;
    return q;
}

// ===========================================================================
// Gradient products: dE, dF and dK, dV in one launch
// ===========================================================================
// Split of one resident round of `resident` workgroups between two GEMMs of items_a items of ta us each
// (items_a a multiple of 8) and items_b items of tb us; `us` receives the time the model expects.
// Measured on MI355X with operands from HBM, 256 x 256 tiles: 1.8 us per reduction step of a
// workgroup that has a compute unit to itself, about 3 us for an epilogue that stores its accumulators
// as they are, 4.4 us for the transposing epilogue of dK, dV.
constexpr double G_STEP_US = 1.8, G_EPILOGUE_US = 3.0, G_EPILOGUE_T_US = 4.4;

inline PairPlan plan_pair(int items_a, double ta, int items_b, double tb, int resident, double* us) {
    PairPlan best{};
    double best_t = -1.0;
    // as few starters as run their first-part items in `rounds` rounds
    for (int rounds = 1; rounds <= 16; ++rounds) {
        int ba = ((items_a + rounds - 1) / rounds + 7) / 8 * 8;
        if (ba > resident - 8) ba = resident - 8;
        const int bb = resident - ba;
        const double t_first = ((items_a + ba - 1) / ba) * ta;
        // items per workgroup of the second kind near the point where both kinds finish together
        const int x0 = (int)((t_first / tb * ba + items_b) / resident);
        for (int xb = x0 > 0 ? x0 : 1; xb <= x0 + 1; ++xb) {
            long main_b = (long)bb * xb / 8 * 8;
            if (main_b > items_b) main_b = items_b;
            const int xa = (int)((items_b - main_b + ba - 1) / ba);
            const double t_a = t_first + xa * tb, t_b = (double)((main_b + bb - 1) / bb) * tb;
            const double t = t_a > t_b ? t_a : t_b;
            if (best_t < 0.0 || t < best_t) {
                best_t = t;
                best.blocks_a = ba; best.main_b = (int)main_b; best.items_a = items_a; best.items_b = items_b;
            }
        }
        if (ba <= 8) break;
    }
    if (us) *us = best_t;
    return best;
}

struct GradEPlan {
    bool fine;             // 128 x 128 tiles (two workgroups per compute unit) instead of 256 x 256
    int tilesM, tilesN;    // of the dE/dF GEMM: slots x positions, fine: positions x slots
    int total_steps, splits, steps_per_split;
    int resident;          // workgroups of the launch dE/dF share with dK/dV
    PairPlan pair;
    size_t partial_bytes() const {
        return splits == 1 ? 0 : (size_t)2 * splits * tilesM * tilesN * (fine ? 128 * 128 : G_TILE_ELEMS) * 4;
    }
};

// dE/dF (few items with a reduction over all B*H*d/64 steps) share their launch with dK/dV (many items of
// kp/64 steps).  Unsplit, the long items are the critical path whenever there are fewer of them than
// compute units (64 at the headline size with 256 x 256 tiles: 89 us, the short items done after 46); split s
// ways they finish sooner, their workgroups go on with short items, and a second pass sums the s partial
// results.  The tile and the split that the cost model (plan_pair, plus the traffic of the second pass) expects
// to finish first win.  128 x 128 tiles: 1.15 us per step with two workgroups to a compute unit, 2.0 and 2.2 us
// for the epilogues.  They take twice the operand traffic, so long reductions on both sides stay with 256 x 256;
// elsewhere they need no or fewer partial results and fill the chip.  Both products and the second pass, 256 x 256 ->
// this rule: 48 heads of 64, n 8192, k 256: 74 + 9.7 -> 76.8 us (no second pass); 16 heads of 128, n 6016, k 300:
// 62.6 -> 49.9; 128 heads of 64, n 512, k 64: 27.9 + 6.6 -> 13.6 + 7.1; training step of 64 heads of 128, n 65536, k 512
// (stays): 1810, with 128 x 128 1905.
constexpr double T_PAIR_STEP_US = 1.15, T_PAIR_EPILOGUE_E_US = 2.0, T_PAIR_EPILOGUE_X_US = 2.2;

inline GradEPlan make_grad_e_plan(const Problem& p, int cus) {
    GradEPlan best{};
    double best_t = -1.0;
    const int kp = (p.k + 63) / 64 * 64, steps_b = kp / GBK, rows_b = p.BH * p.d;
    for (int fine = 0; fine < 2; ++fine) {
        // no shape needs more scratch than with 256 x 256 tiles alone: a buffer that a caller keeps stays large enough
        const size_t coarse_bytes = fine ? best.partial_bytes() : 0;
        GradEPlan q{};
        const int tile = fine ? 128 : GBM;
        const int slots = (p.k + tile - 1) / tile, positions = (p.n + tile - 1) / tile;
        q.fine = fine != 0;
        q.tilesM = fine ? positions : slots;
        q.tilesN = fine ? slots : positions;
        q.total_steps = p.BH * p.d / GBK;
        q.resident = fine ? 2 * cus / 8 * 8 : cus / 8 * 8;
        const int items_b = 8 * ((rows_b + tile - 1) / tile) * ((positions * 2 + 7) / 8);
        const double tb = fine ? steps_b * T_PAIR_STEP_US + T_PAIR_EPILOGUE_X_US : ((steps_b + 1) & ~1) * G_STEP_US + G_EPILOGUE_T_US;
        for (int want = 1; want <= (fine ? 32 : 8) && want <= q.total_steps; want += want < 8 ? 1 : 8) {
            const int sps = (q.total_steps + want - 1) / want;
            const int splits = (q.total_steps + sps - 1) / sps;
            if (want <= 8 && splits != want) continue;
            const int items_a = 8 * slots * ((splits * positions * 2 + 7) / 8);
            q.splits = splits; q.steps_per_split = sps;
            if (fine && q.partial_bytes() > coarse_bytes) continue;
            double t = 0.0;
            q.pair = plan_pair(items_a, fine ? sps * T_PAIR_STEP_US + T_PAIR_EPILOGUE_E_US : ((sps + 1) & ~1) * G_STEP_US + G_EPILOGUE_US,
                               items_b, tb, q.resident, &t);
            // second pass: reads the fp32 partials, writes bf16; about 4 TB/s plus a launch
            if (splits > 1) t += 4.0 + ((double)q.partial_bytes() + 4.0 * p.k * (double)p.n) / 4.0e6;
            if (best_t < 0.0 || t < best_t) { best_t = t; best = q; }
        }
    }
    return best;
}

inline GradEPlan grad_e_plan(const Problem& p) {
    static thread_local KeptPlans<GradEPlan> kept;
    const int cus = chip_cus();
    const long sizes[] = {p.BH, p.n, p.d, p.k, cus, 1};
    return kept.get(sizes, [&]() { return make_grad_e_plan(p, cus); });
}

}  // namespace flurka
