// How k_rows_step deals the lane groups of a workgroup to nodes and samples, in one place so that the kernel and the
// host-only check program (sanitizer build) run the same arithmetic.
#pragma once

#include "gpga_internal.hpp"

constexpr int kRowsThreads = 1024;

// `groups` lane groups: `split` neighbouring ones share the samples of a node, at least eight each, `nodes` nodes at a
// time.  Where `split` does not divide `groups`, the groups behind the last whole share are idle: they own no node, and
// no sums of theirs may be taken (the groups such a share would need lie past the end of the partial sums).
struct RowsDeal {
    int groups, split, nodes;
    __host__ __device__ __forceinline__ RowsDeal(int lanes, int n, int B) : groups(kRowsThreads / lanes) {
        const int most = groups > n ? groups / n : 1, want = (B + 7) / 8;
        split = want < most ? want : most;
        nodes = groups / split;
    }
    __host__ __device__ __forceinline__ int node(int group) const { return group / split; }
    __host__ __device__ __forceinline__ int part(int group) const { return group % split; }
    __host__ __device__ __forceinline__ bool dealt(int group) const { return node(group) < nodes; }
    // The group that adds up its share's partial sums: groups group .. group + split - 1.
    __host__ __device__ __forceinline__ bool adds(int group) const { return dealt(group) && part(group) == 0; }
};
