// Sizes of k_rows_run (several iterations on stored features in one launch): how its workgroups share a problem and what they
// keep in LDS, shared with the host-only check program (sanitizer build).
#pragma once

#include <algorithm>

#include "gpga_internal.hpp"

constexpr int kRowsRunWaves = 12;                    // of a workgroup: three a SIMD, 168 registers each
constexpr int kRowsRunThreads = kRowsRunWaves * kWave;
constexpr int kRowWaves = 10;                        // those that may hold rows; the others exchange
constexpr int kFixedSlots = 12;                      // ... in double precision: four conversions a row and use cost as much as the sums
constexpr int kAheadSlots = 20;                      // ... with registers for half of the next iteration's rows besides
constexpr int kRowsRunMaxSlots = 32;                 // rows a thread holds

inline int log2_ceil(int v) {
    int l = 0;
    while ((1 << l) < v) ++l;
    return l;
}

// How the workgroups of a launch share nodes, columns and rows, and what an iteration is then expected to take.
struct RunPlan {
    int P = 0, w = 0, QW = 0, RG = 0, slots = 0;
    double us = 0.0;
};

// More slices are fewer rows and columns a workgroup but more words of margins to exchange.  Measured, us an iteration
// (ring or one-peer graph): 20 x 1001 with 16 samples P = 1 / 2 / 4 / 8 5.9 / 6.0 / 4.9 / 5.3; 8 x 845 with 50 15.7 / 7.4 / 5.6 /
// 6.3; 9 x 222 with 32 4.1 / 4.7 / 4.8 / 5.0; 8 x 1000 full batches of 100 - / 9.2 / 7.0 / 7.8; 6 x 5164 with 16 P = 4 / 8 / 12 / 24
// 9.7 / 7.5 / 7.0 / 7.3.  The terms: 3.5 us for barriers, update and y; a row of a wavefront, by how many of them share a SIMD;
// the words of the margins a thread has to look at; half of the time the rows take from memory.  They rank plans and no more: there
// is nothing for an average's share and little for more slices, so that P = 9 is taken on 20 x 1001 and 21 on 6 x 5164, some 8 and 4 %
// off the best of these; what a run takes in all is run_us.
inline RunPlan plan_run(int n, int64_t d, int num_cus, int32_t B, bool batches) {
    RunPlan best;
    const int64_t d4 = (d + 3) / 4;
    for (int P = 1; P <= kWave && (int64_t)P * n <= num_cus; ++P) {
        const int64_t w = (d4 + P - 1) / P;
        if (w > kRowWaves * kWave || (d4 + w - 1) / w != P) continue;
        RunPlan p;
        p.P = P;
        p.w = (int)w;
        p.QW = (p.w + kWave - 1) / kWave;
        for (int rg = 1; rg * p.QW <= kRowWaves && rg <= B; ++rg) {
            const int slots = (B + rg - 1) / rg, waves = p.QW * rg, threads = kWave * std::min(kRowsRunWaves - waves, 4);
            if (slots > (batches ? kAheadSlots : kRowsRunMaxSlots)) continue;
            const double row = batches ? 0.22 : slots <= kFixedSlots ? 0.08 : 0.2;
            double us = 3.5 + row * slots * ((waves + 3) / 4);  // wavefronts are dealt to the four SIMDs in turn
            if (P > 1) us += 1.2 + 0.5 * (((B << log2_ceil(P)) + threads - 1) / threads) + 0.02 * P;
            if (batches) us += 0.5 * B * p.w * 16.0 / 25e3;  // 25 bytes a ns and compute unit
            if (!p.RG || us <= p.us) p.RG = rg, p.slots = slots, p.us = us;
        }
        if (p.RG && (!best.P || p.us < best.us)) best = p;
    }
    return best;
}

// What a gpga_run is expected to take, us, in this form and in the two it stands for.  Each is a sum of terms fitted to 2362 measured
// runs (4 to 128 nodes, 64 to 12 000 columns, 1 to 100 samples, 3 to 16 iterations, with and without an average in every one, W of 0 to
// 64 entries a row; 10 % off at one sigma).
struct RunWork {
    int n;
    int64_t d;
    int32_t B;
    bool batches;
    int entries;        // of W a node reads besides its own: 0, 1 (one peer), 2 (ring), or those of a sparse W's row
    bool sparse;
    int64_t T, averages;
    bool adaptive;      // the host reads back: in the other forms at every average, here once a launch
    double mb() const { return (double)n * (double)d * 4e-6; }
};

inline int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// This form.  A launch costs what loads and stores the state; an iteration the update, a thread's columns, the rows by how many
// wavefronts share a SIMD, the words of the margins, and a trip for the y of one or a few nodes and columns at a time: 5000 columns
// on 64 nodes with 64 entries of W a row are 1269 us in 16 iterations, 258 with two launches each.  An average gathers a share of the
// columns over all nodes, forms their means and hands them on (104 x 5000 with one sample, 3 averages in 3 iterations: 62.5 and 44.6).
inline double run_us(const RunWork& r, const RunPlan& p, int most) {
    const int waves = p.QW * p.RG, threads = kWave * std::min(kRowsRunWaves - waves, 4), simd = (waves + 3) / 4;
    const int cols = (int)std::min<int64_t>(4 * p.w, r.d), passes = ceil_div(cols, threads), share = ceil_div(4 * p.w, r.n);
    double one = 2.5 + 0.09 * passes + (r.batches || p.slots <= kFixedSlots ? 0.02 : 0.06) * p.slots * simd + 0.08 * r.mb();
    if (r.batches) one += 0.3e-3 * r.B * p.w;
    if (p.P > 1) one += 0.94 + 0.46 * ceil_div((int64_t)r.B << log2_ceil(p.P), threads);
    const int trips = r.entries == 0   ? 0
                      : r.entries == 1 ? ceil_div(cols, (cols <= 2 * threads ? 2 : 10) * threads)
                      : r.entries == 2 ? ceil_div(cols, (cols <= threads ? 1 : 5) * threads)
                      : cols <= threads ? ceil_div(r.entries, 8)
                                        : ceil_div(cols, 4 * threads) * ceil_div(r.entries, 4);
    const double gossip = 1.04 * trips + 0.045 * r.entries * passes;
    const double average = 0.34 + 0.035 * r.n + 0.19 * r.mb() + 0.89 * ceil_div(share, threads) + 0.62 * ceil_div((int64_t)r.n * share, 5 * threads) +
                           0.34 * ceil_div(cols, (cols <= 2 * threads ? 2 : 10) * threads) + 0.13 * passes;
    return ceil_div(r.T, most) * (8.7 + 1.6 * r.mb() + (r.adaptive ? 10.0 : 0.0)) + (double)r.T * one + (double)(r.T - r.averages) * gossip + (double)r.averages * average;
}

// k_rows_margin and k_rows_step in turn; where that does not take the problem the separate passes, at least twice that.
inline double two_launches_us(const RunWork& r, bool step_fits) {
    const double one = 7.7 + 0.256 * r.mb() * r.B + 1.2 * r.mb() + 1.74e-3 * r.n * r.B;
    const double gossip = r.sparse ? 0.38 + 0.04 * r.entries + 0.0375 * r.entries * r.mb() : 0.0, average = 0.75 + 0.1 * r.mb() + (r.adaptive ? 13.0 : 0.0);
    const double all = 2.0 + (double)r.T * one + (double)(r.T - r.averages) * gossip + (double)r.averages * average;
    return step_fits ? all : 2.0 * all;
}

// k_small_run.
inline double one_workgroup_us(const RunWork& r) {
    const double nd = (double)r.n * (double)r.d;
    const double one = 1.85 + 250e-6 * nd * r.B + 540e-6 * nd + 0.035 * r.n * r.B;
    const double gossip = r.sparse ? 88e-6 * nd * r.entries : 0.0, average = 0.5 + 0.017 * (double)r.d;
    return 2.0 + (double)r.T * one + (double)(r.T - r.averages) * gossip + (double)r.averages * average;
}

// This form is to be the faster one by some of what the terms are off, so that few runs lose by it: 404 of the measured ones are
// slower with it, down to a fifth of the speed, 34 of those that are to take it, down to 0.82; 112 that are not would gain 9 % at the median.
constexpr double kRowsRunMargin = 1.03;
inline bool rows_run_pays(const RunWork& r, const RunPlan& p, int most, double other_us) { return kRowsRunMargin * run_us(r, p, most) <= other_us; }

// What the launches of one gpga_run have in common.
struct RowsRun {
    int32_t most = 0;     // iterations a launch, 0: none of this kind
    int32_t B = 0;        // samples a node
    int splitters = 0;    // of an average
    bool mean64 = false;
    RunPlan plan;
};
// Several iterations on stored features in one launch, for `wanted` iterations on this context and batch.  Under an adaptive
// period the launch decides itself which iterations average and leaves the period's state in host memory.
RowsRun rows_run_for(const gpga_ctx* c, int64_t wanted, const int32_t* idx, int32_t B);
// T <= run.most; false if it cannot be made now, and then nothing was launched and no error is left behind.
bool launch_rows_run(gpga_ctx* c, const RowsRun& run, int32_t T, const int32_t* idx, bool want_g);

// Rows a thread has room for.
inline int slots_for(int rows, bool fixed) {
    if (rows <= 8) return rows <= 4 ? 4 : 8;
    if (fixed) return rows <= kFixedSlots ? kFixedSlots : kRowsRunMaxSlots;
    return rows <= 12 ? 12 : rows <= 16 ? 16 : kAheadSlots;
}

// A workgroup's arrays in LDS, in bytes from its start.  x is read four columns at a time: behind an even number of doubles.
struct RunLds {
    int z, sum;         // after [RG][held] sums at 0: [QW][B] shares of the margins, [B] whole margins
    int x, m;           // [held] columns of the slice
    int y;              // [n][share] what a mean is formed of
    int coef;           // [RG slots] zeros behind B
    int tgt, row;       // [staged]
    int off, val;       // [K] this node's entries of a sparse W
    int bytes;
    __host__ __device__ RunLds(int n, int B, int w, int QW, int RG, int slots, int staged, int K) {
        const int held = 4 * kWave * QW, share = (4 * w + n - 1) / n;
        z = 8 * RG * held;
        sum = z + 8 * QW * B;
        x = (sum + 8 * B + 15) & ~15;
        m = x + 4 * held;
        y = m + 4 * held;
        coef = y + 4 * n * share;
        tgt = coef + 4 * RG * slots;
        row = tgt + 4 * staged;
        off = row + 4 * staged;
        val = off + 4 * K;
        bytes = val + 4 * K;
    }
};
