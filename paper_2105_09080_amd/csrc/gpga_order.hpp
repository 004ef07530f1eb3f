// The order in which k_step_global adds the rows of a column, for kernels that hold x^(k+1/2) of a column unit in LDS
// and are to leave the same bits: the rows are dealt to RL x wpb splitters, each adds batches of U rows, and the
// splitters' sums meet in a binary tree (a butterfly over lanes, then a tree over wavefronts).
#pragma once

#include <type_traits>

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

// The same sum of one column, rows `step` floats apart, for many columns at a time: a chain of LDS reads that a few lanes run
// while the others wait, so eight rows are read ahead of the additions.
__device__ __forceinline__ float splitter_column_sum(const GlobalOrder& o, int r0, int n, bool whole, const float* __restrict__ y, int step) {
    const int RS = o.RL * o.wpb;
    const bool by_parity = RS == 1 && whole;
    const int batched = by_parity ? n - n % o.U : n;
    const int stride = by_parity ? 2 * o.U : RS * o.U;
    auto batches = [&](int base, auto batch_rows) {  // base, base + stride, ...
        constexpr int U = decltype(batch_rows)::value, per = 8 / U;
        float sum = 0.f;
#pragma unroll 1
        for (; base < batched; base += per * stride) {
            float v[per][U];
#pragma unroll
            for (int b = 0; b < per; ++b)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int row = base + b * stride + u * RS;
                    v[b][u] = y[(row < n ? row : n - 1) * step];
                }
#pragma unroll
            for (int b = 0; b < per; ++b) {
                float part = 0.f;
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (base + b * stride + u * RS < n) part += v[b][u];
                if (base + b * stride < batched) sum += part;
            }
        }
        return sum;
    };
    auto from = [&](int base) {  // batches of 1 or 4 rows (global_order, four nodes and more)
        return o.U == 1 ? batches(base, std::integral_constant<int, 1>{}) : batches(base, std::integral_constant<int, 4>{});
    };
    if (!by_parity) return from(r0);
    const float odd = from(o.U);
    float sum = from(0);
#pragma unroll 1
    for (int base = batched; base < n; ++base) sum += y[base * step];
    return sum + odd;
}

// The tree as a binary counter: splitters' sums go in in order, after the last of a power of two `sum` is the total.
template <typename T>
struct SplitterTree {
    T level[5], sum;
    __device__ __forceinline__ SplitterTree() {
        sum = T(0);
#pragma unroll
        for (int l = 0; l < 5; ++l) level[l] = T(0);
    }
    __device__ __forceinline__ void add(int r0, const T& leaf) {
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
