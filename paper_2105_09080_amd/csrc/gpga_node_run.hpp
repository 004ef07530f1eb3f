// Sizes of k_node_run (small trajectories with four lanes a node): which problems it takes and the LDS a launch asks for,
// shared with the host-only check program (sanitizer build).
#pragma once

#include "gpga_internal.hpp"

constexpr int kNodeLanes = 4, kNodeSamples = 4, kNodeMaxNodes = 128, kNodeMaxCols = 20;
constexpr int64_t kNodeMaxEntries = 20 * kNodeMaxNodes;  // of W
constexpr size_t kNodeMaxLds = 64 * 1024;                // what a launch may have unless the kernel's attribute says otherwise

constexpr int node_trace_waves(int samples) { return samples == 1 ? 8 : 4; }  // at most; fewer leave the registers that several samples take
constexpr int kNodeTraceRows = 4;                                                // of a lane read at a time
constexpr int node_columns(int64_t d) { return d <= 4 ? 1 : d <= 12 ? 3 : 5; }  // of a lane; never more than d
constexpr int node_samples(int B) { return B <= 2 ? B : kNodeSamples; }       // rows a node's lanes hold

// Column means, two sets of trace sums per trace wavefront, two copies of x^(k+1/2) and x, W.
constexpr size_t node_run_lds(int n, int columns, int samples, int64_t entries) {
    const size_t row = (size_t)kNodeLanes * columns;
    return (row + 4 * (size_t)node_trace_waves(samples) * row) * sizeof(double) + 4 * (size_t)n * row * sizeof(float) +
           2 * (size_t)entries * sizeof(int32_t);
}

// Rows and batches that fit the registers, nodes that fit 512 threads, state and W in 64 KiB of LDS (128 nodes of 13 to 20
// columns, one sample each: W of up to 2412 entries).
constexpr bool node_run_takes(int n, int64_t d, int B, int64_t entries) {
    return n <= kNodeMaxNodes && d <= kNodeMaxCols && B <= kNodeSamples && entries <= kNodeMaxEntries &&
           node_run_lds(n, node_columns(d), node_samples(B), entries) <= kNodeMaxLds;
}
