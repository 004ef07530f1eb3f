// The order in which k_step_global adds the rows of a column, for kernels that hold x^(k+1/2) of a column unit in LDS
// and are to leave the same bits: the rows are dealt to RL x wpb splitters, each adds batches of U rows, and the
// splitters' sums meet in a binary tree (a butterfly over lanes, then a tree over wavefronts).
#pragma once

#include "gpga_internal.hpp"

// Sum of splitter r0 over n rows of one column unit, `step` units apart.  `whole`: the unit lies in a whole 64-lane tile
// of the step kernel, which, unsplit, keeps a sum of the even and one of the odd batches and adds the rows behind the last
// full batch one by one.
// The odd batches go first and their sum waits in the place of their first row, which costs no registers.
__device__ __forceinline__ v4f splitter_sum(const GlobalOrder& o, int r0, int n, bool whole, v4f* __restrict__ y, int step) {
    const int RS = o.RL * o.wpb;
    const bool by_parity = RS == 1 && whole;
    const int batched = by_parity ? n - n % o.U : n;
    const int stride = by_parity ? 2 * o.U : RS * o.U;
    v4f sum = v4f(0.f);
#pragma unroll 1
    for (int base = by_parity ? o.U : r0;;) {
#pragma unroll 1
        for (; base < batched; base += stride) {
            v4f part = v4f(0.f);
#pragma unroll 1
            for (int u = 0; u < o.U && base + u * RS < n; ++u) part += y[(base + u * RS) * step];
            sum += part;
        }
        if (!by_parity || (base / o.U) % 2 == 0) break;
        if (o.U < batched) y[o.U * step] = sum;  // the odd batches are done; now the even ones
        sum = v4f(0.f);
        base = 0;
    }
    if (!by_parity) return sum;
#pragma unroll 1
    for (int base = batched; base < n; ++base) sum += y[base * step];
    return o.U < batched ? sum + y[o.U * step] : sum;
}

// The tree as a binary counter: splitters' sums go in in order, after the last of a power of two `sum` is the total.
struct SplitterTree {
    v4f level[5], sum;
    __device__ __forceinline__ SplitterTree() {
        sum = v4f(0.f);
#pragma unroll
        for (int l = 0; l < 5; ++l) level[l] = v4f(0.f);
    }
    __device__ __forceinline__ void add(int r0, const v4f& leaf) {
        sum = leaf;
        bool carry = true;
#pragma unroll
        for (int l = 0; l < 5; ++l) {
            if (carry && (r0 >> l) & 1) {
                sum = level[l] + sum;
            } else if (carry) {
                level[l] = sum;
                carry = false;
            }
        }
    }
};
