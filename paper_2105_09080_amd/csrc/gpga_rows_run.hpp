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
// the words of the margins a thread has to look at; half of the time the rows take from memory.
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
