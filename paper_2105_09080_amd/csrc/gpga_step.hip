// Fused Gossip-PGA step kernels for gfx950 (Algorithm 1, lines 2-6 of the
// paper's listing in Sec. 3; matrix form in App. A):
//
//     m_i <- mu*m_i + g_i ;  y_i = x_i - gamma*m_i              (local update)
//     Nesterov momentum (App. F.1):  y_i = x_i - gamma*(g_i + mu*m_i)
//     gossip :  x_new_i = sum_j w_ij y_j                         (W_k sparse)
//     global :  x_new_i = (1/n) sum_j y_j                        (every H-th step)
//
// The node axis (rows) is the only axis along which elements interact, so a
// lane owns one 128-bit column group (4 fp32 columns) and *walks down rows*.
// Lanes of a wavefront sit on consecutive column groups: every access of a wave
// is one fully coalesced 1 KiB row segment.  Each element of x, m, g is read
// from HBM exactly once per step and each element of m, x_new written once.
//
// Gossip ("walk") kernel.  Both graphs are stencils along cycles of the row
// permutation i -> (i + S) mod n:
//   ring      S = 1      one cycle of length n, taps (prev, cur, next)/3
//   one-peer  S = 2^s    gcd(S,n) cycles of length n/gcd, taps (cur, next)/2
//   W = I     -          n cycles of length 1, tap cur (also used, writing y over the old
//                        iterate, as the first pass of sparse-W steps with many rows)
// A "walker" is one wavefront walking a contiguous segment of one cycle with
// the last two y values kept in registers.  When a cycle is split over Q
// wavefronts of a workgroup (few columns, many rows) the first/last y of every
// segment are staged through LDS, so neighbour rows are never re-read from HBM.
// Large problems run as persistent launches paced against the chip's clock (see
// gpga_pace.hpp): every wavefront is then at the same row at the same time, a
// paced one-peer work item takes all cycles of its column tile in turn, and
// one-peer cycles of two rows have a kernel of their own whose batches are whole
// cycles (k_step_cycles).  A tracing variant also sums the squared deviations of
// what it stores from the column means (the consensus distance of the new X).
//
// Global-average kernel.  Small problems: rows are spread over (row lanes of a
// wave) x (waves of the workgroup); partial column sums are combined with a
// wavefront shuffle (xor butterfly) and then an LDS tree across waves.  Large
// problems: one lane sums its whole column while walking it, and the n copies
// of the mean are stored row by row while the wavefront already reads its next
// tile.  Every row gets the same bits of the mean, so the rows are bit-identical
// afterwards.
#include <type_traits>

#include "gpga_internal.hpp"
#include "gpga_pace.hpp"
#include "gpga_spread.hpp"
#include "gpga_unit.hpp"

namespace {

__device__ __forceinline__ float shfl_xor_t(float v, int off) { return __shfl_xor(v, off, kWave); }
__device__ __forceinline__ v4f shfl_xor_t(v4f v, int off) {
    v4f r;
    r.x = __shfl_xor(v.x, off, kWave);
    r.y = __shfl_xor(v.y, off, kWave);
    r.z = __shfl_xor(v.z, off, kWave);
    r.w = __shfl_xor(v.w, off, kWave);
    return r;
}

// x^(k+1/2) from x, the gradient and the NEW momentum value (mom = g when there is no buffer).
template <int MOM, typename T>
__device__ __forceinline__ T half_step(const T& xv, const T& gv, const T& mom, float lr, float mu) {
    if (MOM == 2) return xv - lr * (gv + mu * mom);
    return xv - lr * mom;
}

// Running consensus sums of the values a lane stores into its column group of
// x_new (all n rows of it): shifted by a reference close to them (the old iterate of
// the first row, set by the caller before the first add), deviations
// formed in fp32 (exact or nearly so while rows are close), sums in fp64, so
// that sum_i (x_i - xbar)^2 = S2 - S1^2 / n keeps the small quantity.
constexpr int kMaxWaves = 8;
constexpr int kDefaultUnroll = 2;  // rows per batch; two batches are in flight (software pipeline)

struct WalkArgs {
    StepGeom ge;
    int32_t S;    // row stride of the permutation
    int32_t C;    // number of cycles
    int32_t L;    // cycle length
    int32_t Q;    // segments (wavefronts) per cycle
    int32_t tpb;  // column tiles per workgroup
    int32_t xcd;  // remap tile groups so that an XCD sees contiguous tiles
    int64_t gx;   // tile groups
    int64_t gy;   // walker groups; work items = gx * gy, tile group fastest
    int32_t cpi;  // cycles per work item (1, or all C cycles when the consensus sums ride along)
    double* spread_partials;  // TRACE kernels: one sum of squared deviations per workgroup
    PaceArgs pace;
};

// blockIdx.x -> logical tile-group index.  Hardware hands consecutive workgroup
// ids to the 8 XCDs round-robin; with the remap each XCD walks a contiguous
// range of column tiles (its own L2 and the fabric then see sequential
// streams).
__device__ __forceinline__ int64_t logical_block(int64_t bid, int64_t gx, int xcd) {
    if (!xcd) return bid;
    const int64_t per = gx >> 3;          // groups per XCD (floor)
    const int64_t main_part = per << 3;   // blocks covered by the regular part
    if (bid >= main_part) return bid;     // ragged tail keeps its identity
    return (bid & 7) * per + (bid >> 3);
}


// MOM: 0 = no momentum buffer, 1 = heavy-ball, 2 = Nesterov.
// TRACE: also sum (x_new - column mean)^2 over everything stored; requires that one
// walker covers whole columns (one cycle, one segment), which the launcher checks.
template <typename T, int MODE, int MOM, int U, bool TRACE = false>
__global__ void __launch_bounds__(kWave* kMaxWaves) k_step_walk(const WalkArgs a) {
    __shared__ T s_first[kMaxWaves][kWave];
    __shared__ T s_last[kMaxWaves][kWave];
    __shared__ double s_spread[kMaxWaves];
    ColumnSpread<T> spread;
    double spread_acc = 0.0;

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform -> SGPR
    const int waves = blockDim.x >> 6;
    const int wpb = waves / a.tpb;  // walkers per workgroup
    const int tile_l = wave / wpb;
    const int walk_l = wave - tile_l * wpb;
    const int n = a.ge.n;
    const int S = a.S;
    const int64_t ld = a.ge.ld;
    const float lr = a.ge.lr, mu = a.ge.mu;
    const float third = 1.0f / 3.0f;
    constexpr uint32_t kRowUnits = MOM ? 5u : 3u;  // 4-byte streams touched per row

    const PaceRun run = pace_begin(a.pace, lane);
    uint32_t units_done = 0;

    // Grid-stride over work items (walker group, tile group), tile group
    // fastest.  With a grid sized to the resident workgroups of the chip
    // (persistent launch) all wavefronts start the same rows together and,
    // paced, stay in step: at any moment the whole chip streams a few rows of
    // x, m, g over a wide contiguous column window instead of touching all n
    // rows of every array at once.
    const int64_t work = a.gx * a.gy;
    for (int64_t w = blockIdx.x; w < work; w += gridDim.x) {
        const int by = (int)(w / a.gx);
        const int64_t bx = w - (int64_t)by * a.gx;
        // cpi > 1 (tracing one-peer steps): this work item takes all cycles of its column tile one
        // after the other, so that the lane stores - and sums - whole columns
        for (int cc = 0; cc < a.cpi; ++cc) {
        const int walker = (by * a.cpi + cc) * wpb + walk_l;
        const bool walker_on = walker < a.C * a.Q;
        const int cyc = walker / a.Q;
        const int seg = walker - cyc * a.Q;
        const int p0 = (int)(((int64_t)seg * a.L) / a.Q);
        const int p1 = (int)(((int64_t)(seg + 1) * a.L) / a.Q);
        const int len = p1 - p0;
        const int row_first = (int)(((int64_t)cyc + (int64_t)p0 * S) % n);

        const int64_t tile = logical_block(bx, a.gx, a.xcd) * a.tpb + tile_l;
        const bool on = walker_on && unit_on(a.ge, tile, kWave, lane);
        const int64_t col = unit_column<T>(a.ge, tile, kWave, lane);

        const float* __restrict__ xp = a.ge.x + col;
        const float* __restrict__ gp = a.ge.g + col;
        float* __restrict__ mp = MOM ? a.ge.m + col : nullptr;
        float* __restrict__ xnp = a.ge.x_new + col;
        auto put = [&](int rw, const T& v) {
            st_unit<T>(xnp + (int64_t)rw * ld, v);
            if (TRACE) spread.add(v);
        };

        T yf = T(0), ys = T(0), pp = T(0), pc = T(0);
        int row = row_first;
        int row_prev = row;

        // One row: issue its three loads / turn loaded values into y (and store m).
        auto load_row = [&](T& xv, T& mv, T& gv, int& rw) {
            rw = row;
            const int64_t off = (int64_t)row * ld;
            xv = ld_unit<T>(xp + off);
            if (MOM) mv = ld_unit<T>(mp + off);
            gv = ld_unit<T>(gp + off);
            row += S;
            if (row >= n) row -= n;
        };
        auto y_of = [&](const T& xv, const T& mv, const T& gv, int rw) -> T {
            T mom = gv;
            if (MOM) {
                mom = mu * mv + gv;
                st_unit<T>(mp + (int64_t)rw * ld, mom);
            }
            return half_step<MOM>(xv, gv, mom, lr, mu);
        };
        // Steady state (third row of the segment onwards): the new y completes the
        // stencil of the previous row.
        auto emit = [&](const T& y, int rw) {
            if (MODE == MODE_RING) put(row_prev, (pp + pc + y) * third);
            if (MODE == MODE_PEER) put(row_prev, (pc + y) * 0.5f);
            pp = pc;
            pc = y;
            row_prev = rw;
        };
        struct Batch {
            T xv[U], mv[U], gv[U];
            int rw[U];
        };
        auto load_full = [&](Batch& b) {
            pace_wait(run, units_done);
            units_done += U * kRowUnits;
#pragma unroll
            for (int u = 0; u < U; ++u) load_row(b.xv[u], b.mv[u], b.gv[u], b.rw[u]);
        };
        auto process_full = [&](const Batch& b) {
#pragma unroll
            for (int u = 0; u < U; ++u) emit(y_of(b.xv[u], b.mv[u], b.gv[u], b.rw[u]), b.rw[u]);
        };

        if (on) {
            // First two rows of the segment: they only start the stencil window.
            {
                T x0, m0, g0, x1, m1, g1;
                int r0 = 0, r1 = 0;
                pace_wait(run, units_done);
                units_done += (len >= 2 ? 2u : 1u) * kRowUnits;
                load_row(x0, m0, g0, r0);
                if (len >= 2) load_row(x1, m1, g1, r1);
                if (TRACE && cc == 0) spread.reset(x0);
                yf = y_of(x0, m0, g0, r0);
                if (MODE == MODE_SELF) st_unit<T>(xnp + (int64_t)r0 * ld, yf);
                // in place: over the old iterate, through a pointer derived from the one it was read with
                if (MODE == MODE_INPLACE) st_unit<T>(const_cast<float*>(xp) + (int64_t)r0 * ld, yf);
                pc = yf;
                row_prev = r0;
                if (len >= 2) {
                    ys = y_of(x1, m1, g1, r1);
                    if (MODE == MODE_PEER) put(r0, (yf + ys) * 0.5f);
                    if (MODE == MODE_SELF) st_unit<T>(xnp + (int64_t)r1 * ld, ys);
                    if (MODE == MODE_INPLACE) st_unit<T>(const_cast<float*>(xp) + (int64_t)r1 * ld, ys);
                    pp = yf;
                    pc = ys;
                    row_prev = r1;
                }
            }
            // Software-pipelined steady state over full batches of U rows.  The
            // loads of the next batch are issued BEFORE the stores of the current
            // one: a wavefront's memory operations retire in order, so a wait for
            // those loads never includes the slower write acknowledgements of the
            // stores behind them.  The hot loop is branch-free so that the wait
            // counts stay exact.
            const int rem = len > 2 ? len - 2 : 0;
            const int nfull = rem / U;
            const int tail = rem - nfull * U;
            Batch A, B;
            if (nfull >= 1) {
                load_full(A);
                int b = 0;
                for (; b + 3 <= nfull; b += 2) {
                    load_full(B);
                    __builtin_amdgcn_sched_barrier(0);  // keep the issue order: loads, then stores
                    process_full(A);
                    __builtin_amdgcn_sched_barrier(0);
                    load_full(A);
                    __builtin_amdgcn_sched_barrier(0);
                    process_full(B);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (nfull - b == 2) {
                    load_full(B);
                    __builtin_amdgcn_sched_barrier(0);
                    process_full(A);
                    process_full(B);
                } else {
                    process_full(A);
                }
            }
            for (int t = 0; t < tail; ++t) {
                T xv, mv, gv;
                int rw;
                units_done += kRowUnits;
                load_row(xv, mv, gv, rw);
                emit(y_of(xv, mv, gv, rw), rw);
            }
        }
        if (MODE == MODE_SELF || MODE == MODE_INPLACE) continue;

        // Close the stencil at the two ends of the segment.  One walker per
        // cycle: the cycle closes on itself.  Q walkers per cycle: neighbours'
        // boundary y values come through LDS.
        T left = pc, right = yf;
        if (a.Q > 1) {
            s_first[wave][lane] = yf;
            s_last[wave][lane] = pc;
            __syncthreads();
            const int w0 = wave - seg;
            left = s_last[w0 + (seg + a.Q - 1) % a.Q][lane];
            right = s_first[w0 + (seg + 1) % a.Q][lane];
            __syncthreads();  // LDS is rewritten by the next tile group
        }
        if (on) {
            if (MODE == MODE_RING) {
                if (len == 1) {
                    put(row_first, (left + yf + right) * third);
                } else {
                    put(row_first, (left + yf + ys) * third);
                    put(row_prev, (pp + pc + right) * third);
                }
            } else {  // MODE_PEER: last row of the segment pairs with the next segment's first
                put(row_prev, (pc + right) * 0.5f);
            }
            if (TRACE && cc == a.cpi - 1) spread_acc += spread.sum_sq(1.0 / (double)n);
        }
        }  // cycles of this work item
    }
    const unsigned long long t_done = pace_now(a.pace);
    if (TRACE) {
        // one partial per workgroup, summed in a fixed order
        double v = spread_acc;
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_down(v, off, kWave);
        if (lane == 0) s_spread[wave] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int w = 0; w < waves; ++w) t += s_spread[w];
            a.spread_partials[blockIdx.x] = t;
        }
    }
    pace_end(a.pace, run, units_done, lane, t_done);
}

// One-peer steps whose cycles are short (instantiated for L = 2, 4, 8 and 16 rows: offsets n/2 ... n/16).
// A lane streams the rows of its column group cycle after cycle - rows c, c+S, ..., c+(L-1)S of
// cycle c, then cycle c+1 - as ONE software pipeline: one row per batch, the loads of the next row
// (which may belong to the next cycle) issued ahead of this row's stores, two rows in flight
// throughout.  Only the stencil restarts at a cycle boundary: the first y of a cycle is kept to
// close it, (y_{L-1} + y_0) / 2, when its last row arrives.  The general walk kernel drains its
// pipeline at the end of every cycle; with 4-row cycles that exposed one memory latency per four
// rows and its wavefronts fell behind the pacing clock 5 % earlier than on long cycles.
// The body is unrolled over the L rows of a cycle, so the loop over cycles is branch-free.
struct CycleArgs {
    StepGeom ge;
    int32_t S;   // row offset of the peer
    int32_t C;   // number of cycles
    int64_t gx;  // tile groups (one column tile per wavefront)
    double* spread_partials;  // TRACE kernels: one sum of squared deviations per workgroup
    PaceArgs pace;
};

template <int MOM, int L, bool TRACE = false>
__global__ void __launch_bounds__(kWave* kMaxWaves) k_step_cycles(const CycleArgs a) {
    static_assert(L >= 2 && L % 2 == 0, "two row buffers alternate: a cycle has an even number of rows");
    typedef v4f T;
    __shared__ double s_spread[kMaxWaves];
    ColumnSpread<T> spread;
    double spread_acc = 0.0;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    const int n = a.ge.n;
    const int S = a.S;
    const int64_t ld = a.ge.ld;
    const float lr = a.ge.lr, mu = a.ge.mu;
    constexpr uint32_t kRowUnits = MOM ? 5u : 3u;
    const PaceRun run = pace_begin(a.pace, lane);
    uint32_t units_done = 0;

    for (int64_t w = blockIdx.x; w < a.gx; w += gridDim.x) {
        if (!unit_on(a.ge, w * waves + wave, kWave, lane)) continue;
        const int64_t col = unit_column<T>(a.ge, w * waves + wave, kWave, lane);
        if (TRACE) spread.reset(ld_unit_cached<T>(a.ge.x + col));  // row 0 of the old iterate
        const float* __restrict__ xp = a.ge.x + col;
        const float* __restrict__ gp = a.ge.g + col;
        float* __restrict__ mp = MOM ? a.ge.m + col : nullptr;
        float* __restrict__ xnp = a.ge.x_new + col;

        struct Row {
            T xv, mv, gv;
            int rw;
        };
        int next_row = 0;  // row the next load takes: walks cycle 0, then cycle 1, ...
        int next_pos = 0, next_cyc = 0;
        auto load_row = [&](Row& b) {
            pace_wait(run, units_done);
            units_done += kRowUnits;
            b.rw = next_row;
            const int64_t off = (int64_t)next_row * ld;
            b.xv = ld_unit<T>(xp + off);
            if (MOM) b.mv = ld_unit<T>(mp + off);
            b.gv = ld_unit<T>(gp + off);
            if (++next_pos == L) {  // on to the first row of the next cycle
                next_pos = 0;
                next_row = ++next_cyc;
            } else {
                next_row += S;
                if (next_row >= n) next_row -= n;
            }
        };
        T yf = T(0), pc = T(0);
        int row_prev = 0;
        auto process = [&](const Row& b, int pos) {  // pos is a compile-time constant at every call
            T mom = b.gv;
            if (MOM) {
                mom = mu * b.mv + b.gv;
                st_unit<T>(mp + (int64_t)b.rw * ld, mom);
            }
            const T y = half_step<MOM>(b.xv, b.gv, mom, lr, mu);
            if (pos == 0) {
                yf = y;
            } else {
                const T v = (pc + y) * 0.5f;
                st_unit<T>(xnp + (int64_t)row_prev * ld, v);
                if (TRACE) spread.add(v);
            }
            if (pos == L - 1) {
                const T v = (y + yf) * 0.5f;
                st_unit<T>(xnp + (int64_t)b.rw * ld, v);
                if (TRACE) spread.add(v);
            }
            pc = y;
            row_prev = b.rw;
        };
        Row A, B;
        load_row(A);
        for (int c = 0; c + 1 < a.C; ++c) {  // every cycle but the last: the load after its last row opens the next cycle
#pragma unroll
            for (int pos = 0; pos < L; pos += 2) {
                load_row(B);
                __builtin_amdgcn_sched_barrier(0);  // keep the issue order: loads, then stores
                process(A, pos);
                __builtin_amdgcn_sched_barrier(0);
                load_row(A);
                __builtin_amdgcn_sched_barrier(0);
                process(B, pos + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int pos = 0; pos < L; pos += 2) {  // the last cycle: nothing to load after its last row
            load_row(B);
            __builtin_amdgcn_sched_barrier(0);
            process(A, pos);
            __builtin_amdgcn_sched_barrier(0);
            if (pos + 2 < L) load_row(A);
            __builtin_amdgcn_sched_barrier(0);
            process(B, pos + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (TRACE) spread_acc += spread.sum_sq(1.0 / (double)n);
    }
    const unsigned long long t_done = pace_now(a.pace);
    if (TRACE) {
        double v = spread_acc;
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_down(v, off, kWave);
        if (lane == 0) s_spread[wave] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int w2 = 0; w2 < waves; ++w2) t += s_spread[w2];
            a.spread_partials[blockIdx.x] = t;
        }
    }
    pace_end(a.pace, run, units_done, lane, t_done);
}

struct GlobalArgs {
    StepGeom ge;
    int32_t RL;   // lanes of a wave spread over rows (1, 2, 4)
    int32_t tpb;  // column tiles per workgroup
    int32_t xcd;
    int64_t gx;
    float inv_n;
    PaceArgs pace;
};

template <typename T, int MOM, int U>
__global__ void __launch_bounds__(kWave* kMaxWaves) k_step_global(const GlobalArgs a) {
    __shared__ T s_part[kMaxWaves][kWave];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform -> SGPR
    const int waves = blockDim.x >> 6;
    const int wpb = waves / a.tpb;  // waves sharing one column tile
    const int tile_l = wave / wpb;
    const int wrow = wave - tile_l * wpb;
    const int CL = kWave / a.RL;  // column lanes per wave
    const int lane_c = lane & (CL - 1);
    const int lane_r = lane / CL;
    const int n = a.ge.n;
    const int RS = a.RL * wpb;            // row splitters per column
    const int r0 = wrow * a.RL + lane_r;  // this lane's first row
    const int64_t ld = a.ge.ld;
    const float lr = a.ge.lr, mu = a.ge.mu;
    constexpr uint32_t kReadUnits = MOM ? 4u : 2u;  // 4-byte streams per row in the read phase
    const PaceRun run = pace_begin(a.pace, lane);
    uint32_t units_done = 0;

    // deferred mean of the previous whole tile of this wavefront (see below)
    T prev_mean = T(0);
    float* prev_xnp = nullptr;
    bool have_prev = false;  // wave-uniform
    auto flush_prev = [&]() {
        for (int row = 0; row < n; row += U) {
            pace_wait(run, units_done);
            units_done += U;
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (row + u < n) st_unit<T>(prev_xnp + (int64_t)(row + u) * ld, prev_mean);
        }
    };

    for (int64_t bx = blockIdx.x; bx < a.gx; bx += gridDim.x) {
        const int64_t tile = logical_block(bx, a.gx, a.xcd) * a.tpb + tile_l;
        const bool on = unit_on(a.ge, tile, CL, lane_c);
        const int64_t col = unit_column<T>(a.ge, tile, CL, lane_c);

        const float* __restrict__ xp = a.ge.x + col;
        const float* __restrict__ gp = a.ge.g + col;
        float* __restrict__ mp = MOM ? a.ge.m + col : nullptr;
        float* __restrict__ xnp = a.ge.x_new + col;

        T sum = T(0);
        // One lane walks all n rows of its column group (large problems).  The n copies of
        // a tile's mean are not written in a burst of their own: they are DEFERRED and
        // stored row by row while the next tile of this wavefront is being read, so that
        // the chip sees the same steady 3-read : 2-write mix as in the gossip walk.  Only
        // whole tiles take this path (the ragged last tile falls through to the plain one).
        const bool whole_tile = whole_units(a.ge, tile, CL);  // wave-uniform
        if (RS == 1 && whole_tile) {
            // Same software pipeline as the gossip walk: next batch's loads are issued
            // ahead of this batch's stores; branch-free hot loop.
            struct Batch {
                T xv[U], mv[U], gv[U];
            };
            auto rows_pass = [&](auto with_prev) {
                constexpr bool WP = decltype(with_prev)::value;
                constexpr uint32_t kUnits = kReadUnits + (WP ? 1u : 0u);
                int row = 0;
                auto load_full = [&](Batch& b) {
                    pace_wait(run, units_done);
                    units_done += U * kUnits;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int64_t off = (int64_t)(row + u) * ld;
                        b.xv[u] = ld_unit<T>(xp + off);
                        if (MOM) b.mv[u] = ld_unit<T>(mp + off);
                        b.gv[u] = ld_unit<T>(gp + off);
                    }
                    row += U;
                };
                auto process_full = [&](const Batch& b, int first_row, T& into) {
                    T part = T(0);
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        T mom = b.gv[u];
                        if (MOM) {
                            mom = mu * b.mv[u] + b.gv[u];
                            st_unit<T>(mp + (int64_t)(first_row + u) * ld, mom);
                        }
                        if (WP) st_unit<T>(prev_xnp + (int64_t)(first_row + u) * ld, prev_mean);
                        part += half_step<MOM>(b.xv[u], b.gv[u], mom, lr, mu);
                    }
                    into += part;
                };
                const int nfull = n / U;
                // even and odd batches have a sum each: half the length of either chain of roundings
                T odd = T(0);
                Batch A, B;
                int done = 0;
                if (nfull >= 1) {
                    load_full(A);
                    int b = 0;
                    for (; b + 3 <= nfull; b += 2) {
                        load_full(B);
                        __builtin_amdgcn_sched_barrier(0);
                        process_full(A, done, sum);
                        __builtin_amdgcn_sched_barrier(0);
                        load_full(A);
                        __builtin_amdgcn_sched_barrier(0);
                        process_full(B, done + U, odd);
                        __builtin_amdgcn_sched_barrier(0);
                        done += 2 * U;
                    }
                    if (nfull - b == 2) {
                        load_full(B);
                        __builtin_amdgcn_sched_barrier(0);
                        process_full(A, done, sum);
                        process_full(B, done + U, odd);
                        done += 2 * U;
                    } else {
                        process_full(A, done, sum);
                        done += U;
                    }
                }
                for (; done < n; ++done) {
                    const int64_t off = (int64_t)done * ld;
                    const T xv = ld_unit<T>(xp + off);
                    const T gv = ld_unit<T>(gp + off);
                    T mom = gv;
                    if (MOM) {
                        mom = mu * ld_unit<T>(mp + off) + gv;
                        st_unit<T>(mp + off, mom);
                    }
                    if (WP) st_unit<T>(prev_xnp + off, prev_mean);
                    units_done += kUnits;
                    sum += half_step<MOM>(xv, gv, mom, lr, mu);
                }
                sum += odd;
            };
            if (have_prev) rows_pass(std::true_type{}); else rows_pass(std::false_type{});
            prev_mean = sum * a.inv_n;
            prev_xnp = xnp;
            have_prev = true;
            continue;
        }
        if (have_prev) {  // a tile that writes at once follows: nothing may stay deferred behind it
            flush_prev();
            have_prev = false;
        }
        if (on) {
            for (int base = r0; base < n; base += RS * U) {
                T xv[U], mv[U], gv[U];
                pace_wait(run, units_done);
                units_done += U * kReadUnits;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int row = base + u * RS;
                    if (row < n) {
                        const int64_t off = (int64_t)row * ld;
                        xv[u] = ld_unit<T>(xp + off);
                        if (MOM) mv[u] = ld_unit<T>(mp + off);
                        gv[u] = ld_unit<T>(gp + off);
                    }
                }
                T part = T(0);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int row = base + u * RS;
                    if (row < n) {
                        T mom = gv[u];
                        if (MOM) {
                            mom = mu * mv[u] + gv[u];
                            st_unit<T>(mp + (int64_t)row * ld, mom);
                        }
                        part += half_step<MOM>(xv[u], gv[u], mom, lr, mu);
                    }
                }
                sum += part;
            }
        }
        // wavefront shuffle across the row lanes (xor butterfly: all lanes end equal)
        for (int off = CL; off < kWave; off <<= 1) sum += shfl_xor_t(sum, off);
        // LDS tree across the waves that share this column tile
        if (wpb > 1) {
            if (lane_r == 0) s_part[wave][lane_c] = sum;
            __syncthreads();
            const int w0 = tile_l * wpb;
            for (int stride = 1; stride < wpb; stride <<= 1) {
                if (lane_r == 0 && (wrow & (2 * stride - 1)) == 0 && wrow + stride < wpb)
                    s_part[wave][lane_c] += s_part[wave + stride][lane_c];
                __syncthreads();
            }
            sum = s_part[w0][lane_c];
            __syncthreads();  // LDS is rewritten by the next tile group
        }
        const T mean = sum * a.inv_n;
        if (on) {
            for (int base = r0; base < n; base += RS * U) {
                pace_wait(run, units_done);
                units_done += U;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int row = base + u * RS;
                    if (row < n) st_unit<T>(xnp + (int64_t)row * ld, mean);
                }
            }
        }
    }
    if (have_prev) flush_prev();
    pace_end(a.pace, run, units_done, lane, pace_now(a.pace));
}

int gcd_i(int a, int b) {
    while (b) {
        int t = a % b;
        a = b;
        b = t;
    }
    return a;
}
int pow2_floor(int v) {
    int p = 1;
    while (p * 2 <= v) p *= 2;
    return p;
}
int pow2_ceil(int v) {
    int p = 1;
    while (p < v) p *= 2;
    return p;
}

// Launch plan shared by both kernels: `work` work items; persistent launches
// use at most blocks_per_cu resident workgroups per compute unit (never more
// than the kernel's occupancy allows, so that every workgroup is resident and
// the paced wavefronts really run side by side).
struct LaunchPlan {
    int64_t work = 0;        // work items of a one-shot launch
    int bpc = 0;             // requested resident workgroups per CU (0 = one-shot launch)
    int num_cus = 0;
    int waves = 0;           // wavefronts per workgroup
    double pace_gbs = 0.0;   // 0 = free running, > 0 = paced at this rate, < 0 = paced at the rate the controller finds
    int pace_key = 0;        // which controller state the launch shares (PaceKey)
    double clock_hz = 1e8;
    int vec = 4;
    const gpga_ctx* ctx = nullptr;
    int64_t* blocks_out = nullptr;  // receives the number of workgroups launched
};

template <typename Args, typename Kernel>
hipError_t launch_planned(Kernel kernel, LaunchPlan plan, Args a, hipStream_t st) {
    const int threads = kWave * plan.waves;
    int64_t blocks = plan.work;
    pace_setup(nullptr, 0.0, 0, 0.0, 0, &a.pace);
    if (plan.bpc > 0) {
        int occ = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel, threads, 0) != hipSuccess || occ < 1) occ = 1;
        const int bpc = plan.bpc < occ ? plan.bpc : occ;
        const int64_t resident = (int64_t)plan.num_cus * bpc;
        if (resident < blocks) blocks = balanced_blocks(plan.work, resident);  // persistent: each workgroup strides over the work items
        // Pacing needs every workgroup of the launch to be resident at once, which
        // holds here: blocks <= CUs x workgroups per CU that fit.
        pace_setup(const_cast<gpga_ctx*>(plan.ctx), plan.pace_gbs, plan.pace_key, (double)blocks * plan.waves, plan.vec * 4, &a.pace);
    }
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    if (plan.blocks_out) *plan.blocks_out = blocks;
    if (plan.ctx->plan_only) return hipSuccess;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(threads), 0, st, a);
    return hipGetLastError();
}

template <int MOM, int L>
hipError_t launch_cycles_traced(bool traced, const LaunchPlan& plan, const CycleArgs& a, hipStream_t st) {
    return traced ? launch_planned(k_step_cycles<MOM, L, true>, plan, a, st)
                  : launch_planned(k_step_cycles<MOM, L, false>, plan, a, st);
}
template <int MOM>
hipError_t launch_cycles_len(int L, bool traced, const LaunchPlan& plan, const CycleArgs& a, hipStream_t st) {
    if (L == 2) return launch_cycles_traced<MOM, 2>(traced, plan, a, st);
    if (L == 4) return launch_cycles_traced<MOM, 4>(traced, plan, a, st);
    if (L == 8) return launch_cycles_traced<MOM, 8>(traced, plan, a, st);
    return launch_cycles_traced<MOM, 16>(traced, plan, a, st);
}
hipError_t launch_cycles(int L, int mom, bool traced, const LaunchPlan& plan, const CycleArgs& a, hipStream_t st) {
    if (mom == 2) return launch_cycles_len<2>(L, traced, plan, a, st);
    return mom ? launch_cycles_len<1>(L, traced, plan, a, st) : launch_cycles_len<0>(L, traced, plan, a, st);
}

template <typename T, int MODE, int MOM>
hipError_t launch_walk_u(int U, const LaunchPlan& plan, hipStream_t st, const WalkArgs& a) {
    switch (U) {
        case 1: return launch_planned(k_step_walk<T, MODE, MOM, 1>, plan, a, st);
        case 2: return launch_planned(k_step_walk<T, MODE, MOM, 2>, plan, a, st);
        case 8: return launch_planned(k_step_walk<T, MODE, MOM, 8>, plan, a, st);
        default: return launch_planned(k_step_walk<T, MODE, MOM, 4>, plan, a, st);
    }
}

// Tracing variants exist for the default geometry only (128-bit lanes, 1 or 2 rows per batch).
template <int MOM>
hipError_t launch_walk_trace(int mode, int U, const LaunchPlan& plan, hipStream_t st, const WalkArgs& a) {
    if (mode == MODE_RING) {
        return U == 1 ? launch_planned(k_step_walk<v4f, MODE_RING, MOM, 1, true>, plan, a, st)
                      : launch_planned(k_step_walk<v4f, MODE_RING, MOM, 2, true>, plan, a, st);
    }
    return U == 1 ? launch_planned(k_step_walk<v4f, MODE_PEER, MOM, 1, true>, plan, a, st)
                  : launch_planned(k_step_walk<v4f, MODE_PEER, MOM, 2, true>, plan, a, st);
}

template <typename T, int MOM>
hipError_t launch_walk_mode(int mode, int U, const LaunchPlan& plan, hipStream_t st, const WalkArgs& a) {
    switch (mode) {
        case MODE_RING: return launch_walk_u<T, MODE_RING, MOM>(U, plan, st, a);
        case MODE_PEER: return launch_walk_u<T, MODE_PEER, MOM>(U, plan, st, a);
        case MODE_INPLACE: return launch_walk_u<T, MODE_INPLACE, MOM>(U, plan, st, a);
        default: return launch_walk_u<T, MODE_SELF, MOM>(U, plan, st, a);
    }
}

template <typename T, int MOM>
hipError_t launch_global_u(int U, const LaunchPlan& plan, hipStream_t st, const GlobalArgs& a) {
    switch (U) {
        case 1: return launch_planned(k_step_global<T, MOM, 1>, plan, a, st);
        case 2: return launch_planned(k_step_global<T, MOM, 2>, plan, a, st);
        case 8: return launch_planned(k_step_global<T, MOM, 8>, plan, a, st);
        default: return launch_planned(k_step_global<T, MOM, 4>, plan, a, st);
    }
}

// From this many whole-column walkers on (half of the 256 CUs x 16 resident
// wavefronts) the chip is kept busy with one wavefront per column tile walking
// all its rows, which is the shape the paced launch needs; below it the rows
// are split over lanes / wavefronts of a workgroup instead.
constexpr int64_t kPacedWaves = 2048;
// Walks along cycles of 32 rows and more keep one wavefront per cycle and column tile down to five and three quarters of them
// a compute unit (shorter cycles are as fast either way: n = 16, 1563 tiles 25.4 us split, 25.7 whole), very long ones down to
// five: split rows have every row open at once.  Ring, us split / whole: 1454 tiles n = 64 91 / 94, n = 256 375 / 385; 1504
// tiles n = 32 54.5 / 52, n = 64 108 / 103, n = 256 441 / 428; 1290 tiles n = 256 364 / 376, n = 1000 1445 / 1400.
inline int64_t split_waves(int64_t cycle) { return cycle >= 512 ? 1280 : cycle >= 32 ? 1472 : kPacedWaves; }

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool rows_on_16_bytes(const gpga_ctx* c) {
    return c->ld % 4 == 0 && aligned16(c->x) && aligned16(c->x_new) && aligned16(c->g) && (!c->m || aligned16(c->m));
}

// Default policy: large launches whose wavefronts each walk many rows run
// persistent and paced, at the rate the controller of their kind has found;
// everything else is a one-shot launch.
constexpr int kAutoBlocksPerCu = 4;

// One-shot walks of few rows.  Pacing buys the rate of one open row (6.2 TB/s) and costs some 100 us at the end of the
// launch; a free-running launch of n rows loses 7 % (n = 8) to 16 % (n = 64) of that rate and ends with its last
// tile.  So the fewer rows, the longer a step must be before pacing pays: up to this many bytes of a step free-running
// wins.  Us paced / free, momentum 0.9: 8 x 25.6M full 809 / 753, ring 827 / 706, 8 x 60M 1706 / 1666, 8 x 70M 1939 / 2000;
// 12 x 17M 792 / 742; 16 x 14M 854 / 816, 16 x 20M 1150 / 1170; 20 x 7M 580 / 516; 32 x 5M ring 661 / 624, 32 x 8M 965 / 996;
// 64 x 3M 730 / 750; without momentum 6 x 40M ring 617 / 469, 20 x 8M 438 / 342, 64 x 3M 478 / 432, 64 x 8M 1093 / 1134.
// A caller who sets a rate or the workgroups of a compute unit asks for a persistent launch and gets it.
constexpr double kFreeRowBytes = 80e9;  // divided by the rows, and at least / at most
constexpr double kFreeMinBytes = 3.2e9, kFreeMaxBytes = 10e9;
constexpr int kFreeRows = 64;
bool free_running_pays(const gpga_ctx* c) {
    if (c->n > kFreeRows || c->opt_blocks_per_cu >= 0 || c->opt_pace_gbs >= 0) return false;
    const double most = kFreeRowBytes / c->n, bytes = 4.0 * (c->mu != 0.f ? 5 : 3) * c->n * (double)c->d;
    return bytes <= (most < kFreeMinBytes ? kFreeMinBytes : most > kFreeMaxBytes ? kFreeMaxBytes : most);
}
// A walk: nor were paced cycles or the persistent one-peer kernel asked for.
bool walk_runs_free(const gpga_ctx* c) { return free_running_pays(c) && c->opt_pace_min_cycle <= 0 && c->opt_cycle_kernel != 1; }
// Wavefronts per workgroup.  One where a launch of few rows streams past the caches on 16-byte rows: tiles are then
// handed out one by one, in order, and fewer of them are open at once (8 x 25.6M ring 728 -> 706 us, full 758 -> 753, 16 x 8M
// one-peer 482 -> 461; 8 x 25 600 001, where neighbouring tiles share cache lines, ring 813 -> 900; 16 x 2M, 32 x 2M even;
// 64 x 1.1M without momentum 158 -> 162).
constexpr int64_t kLoneWaveElements = 1 << 26;
int walk_waves(const gpga_ctx* c, int64_t tiles, bool runs_free) {
    if (c->opt_waves) return c->opt_waves;
    const bool lone = runs_free && !c->opt_row_split && (int64_t)c->n * c->d >= (c->n <= 32 ? 1 : 2) * kLoneWaveElements &&
                      tiles >= kPacedWaves && rows_on_16_bytes(c);
    return lone ? 1 : 4;
}
// Rows per batch of a free-running walk along a cycle (us with 2 / 4 / 8, four wavefronts: 8 x 25.6M ring 778 / 762 / 731,
// 16 x 14M without momentum 481 / 483 / 451; 4 x 51.2M 736 / 717 / 725; long columns of few tiles keep 2).  Eight rows of x, m
// and g fill the registers of two wavefronts a SIMD, and on the ring five more spill, 24 bytes of scratch memory a lane.
int walk_unroll(const gpga_ctx* c, int64_t tiles, int64_t cycle, bool runs_free) {
    if (!runs_free || (int64_t)c->n * c->d < kLoneWaveElements || tiles < kPacedWaves) return kDefaultUnroll;
    return cycle >= 8 ? 8 : cycle >= 4 ? 4 : kDefaultUnroll;
}

LaunchPlan make_plan(const gpga_ctx* c, int64_t work, int waves, int vec, bool walks_rows, bool runs_free, int pace_key) {
    LaunchPlan p;
    p.work = work;
    p.num_cus = c->num_cus;
    p.waves = waves;
    p.vec = vec;
    p.ctx = c;
    p.clock_hz = c->clock_hz;
    p.pace_key = pace_key;
    const bool big = walks_rows && vec == 4 && (int64_t)c->n * c->d * 4 >= kPaceMinBytes && !runs_free;
    p.bpc = c->opt_blocks_per_cu < 0 ? (big ? kAutoBlocksPerCu : 0) : c->opt_blocks_per_cu;
    p.pace_gbs = c->opt_pace_gbs < 0 ? (big ? -1.0 : 0.0) : (double)c->opt_pace_gbs;
    if (!walks_rows) p.pace_gbs = 0.0;
    return p;
}

}  // namespace

hipError_t launch_step_walk(const gpga_ctx* c, const StepGeom& geom, int mode, int32_t S, int vec,
                            double* spread_partials, int64_t* spread_count) {
    if (spread_count) *spread_count = 0;
    StepGeom ge = geom;
    set_units(&ge, vec, kWave);
    const int n = ge.n;
    WalkArgs a;
    a.ge = ge;
    if (mode == MODE_SELF || mode == MODE_INPLACE) {
        a.S = 0;
        a.C = n;
        a.L = 1;
    } else {
        a.S = S;
        a.C = gcd_i(S, n);
        a.L = n / a.C;
    }
    const int64_t tiles = unit_tiles(ge, kWave);
    const bool runs_free = walk_runs_free(c);
    // (a ring of two or three rows has nothing to stream: 2 x 60M without momentum 238 us with four wavefronts, 273 with one)
    const int waves = walk_waves(c, tiles, runs_free && vec == 4 && !(mode == MODE_RING && n < 4));

    // One-peer steps over short cycles (2, 4, 8 or 16 rows) on large problems: the row-streaming kernel,
    // persistent where it does not run free, and paced from kPaceMinBytes on (below, us persistent / free: 2 x 30M 222 / 194,
    // 8 x 14M 427 / 393, 16 x 8M 499 / 465, 16 x 2M 115 / 116, 64 x 2M 494 / 498; 128 x 1M even, persistent).
    // Forced ("always"), it takes rows of whole lanes or on 16-byte boundaries.
    const bool takes_rows = c->opt_cycle_kernel != 1 || ge.d % 4 == 0 || rows_on_16_bytes(c);
    if (mode == MODE_PEER && vec == 4 && takes_rows && (a.L == 2 || a.L == 4 || a.L == 8 || a.L == 16) && !c->opt_row_split &&
        c->opt_cycle_kernel != 0 && (tiles >= kPacedWaves || c->opt_cycle_kernel == 1)) {
        CycleArgs ca;
        ca.ge = ge;
        ca.S = S;
        ca.C = a.C;
        ca.gx = (tiles + waves - 1) / waves;
        LaunchPlan plan = make_plan(c, ca.gx, waves, vec, true, runs_free,
                                    a.L == 2 ? PACE_CYCLES : a.L == 4 ? PACE_PEER_4 : a.L == 8 ? PACE_PEER_8 : PACE_PEER_16);
        if (!runs_free && c->opt_blocks_per_cu < 0 && plan.bpc == 0) plan.bpc = kAutoBlocksPerCu;
        const int momk = c->mu != 0.f ? (c->nesterov ? 2 : 1) : 0;
        ca.spread_partials = nullptr;
        const bool traced = spread_partials && spread_count;  // every lane stores whole columns: the consensus sums ride along
        if (traced) {
            ca.spread_partials = spread_partials;
            plan.blocks_out = spread_count;
        }
        c->note_path(PATH_CYCLES, 16);
        return launch_cycles(a.L, momk, traced, plan, ca, c->stream);
    }

    c->note_path(PATH_WALK, vec * 4);
    int Q = 1;
    if (mode != MODE_SELF && mode != MODE_INPLACE) {
        if (c->opt_row_split) {
            Q = c->opt_row_split;
        } else if (tiles * a.C < split_waves(a.L)) {
            // too few column tiles to occupy the chip with one walker per cycle:
            // split each cycle over the wavefronts of a workgroup (LDS exchange)
            Q = pow2_floor(a.L / 4 > 0 ? a.L / 4 : 1);  // keep segments of >= 4 rows
        }
        if (Q > waves) Q = waves;
        if (Q > a.L) Q = pow2_floor(a.L);
    }
    a.Q = Q;
    // Walkers per workgroup.  One walker per cycle and plenty of tiles: give a
    // workgroup adjacent tiles of ONE cycle (wpb = 1), so that a launch works on
    // one cycle group at a time and few rows are open at once.  Otherwise pack
    // the walkers of a tile into one workgroup.
    int wpb = pow2_ceil((int)((int64_t)a.C * Q > waves ? waves : a.C * Q));
    if (wpb > waves) wpb = waves;
    if (Q == 1 && tiles >= kPacedWaves && !c->opt_row_split) wpb = 1;
    if (wpb < Q) wpb = Q;
    a.tpb = waves / wpb;
    const int64_t gx = (tiles + a.tpb - 1) / a.tpb;
    const int64_t gy = ((int64_t)a.C * Q + wpb - 1) / wpb;
    if (gx * gy > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    a.gx = gx;
    a.gy = gy;
    a.xcd = c->opt_xcd_swizzle;
    // pacing assumes every wavefront does the same work: one walker per cycle, equal segments
    const bool uniform = (Q == 1) && (((int64_t)a.C * Q) % wpb == 0);
    // cycles of 4 rows and more are paced (a work item then takes all cycles of its tile, below);
    // shorter ones keep few rows open in a one-shot launch anyway
    const int min_cycle = c->opt_pace_min_cycle > 0 ? c->opt_pace_min_cycle : 4;
    // short cycles sustain lower rates than long walks (measured on n = 64, d = 25.6M: 8 rows 5.97 TB/s,
    // 4 rows 5.78 TB/s, long walks 6.15 TB/s), so each class has a controller of its own
    const int pace_key = mode == MODE_RING ? PACE_RING
                         : mode != MODE_PEER ? PACE_SELF
                         : a.L <= 4 ? PACE_PEER_4 : a.L <= 8 ? PACE_PEER_8 : PACE_PEER_LONG;
    const LaunchPlan plan = make_plan(c, gx * gy, waves, vec, uniform && a.L >= min_cycle, runs_free, pace_key);
    // paced wavefronts advance one row per batch (two rows in flight)
    const int U = c->opt_unroll                                 ? c->opt_unroll
                  : plan.pace_gbs != 0.0                        ? 1
                  : spread_partials || vec != 4 || a.Q > 1      ? kDefaultUnroll
                                                                : walk_unroll(c, tiles, a.L, runs_free);
    const int mom = c->mu != 0.f ? (c->nesterov ? 2 : 1) : 0;
    a.spread_partials = nullptr;
    a.cpi = 1;
    LaunchPlan lp = plan;
    // Paced launches with one cycle per workgroup: a work item takes ALL cycles of its column tile
    // in turn instead of one (measured 3.41 -> 3.33 ms on n = 1024, d = 1M); its lanes then store
    // whole columns, as they do when there is a single cycle.  So do free-running ones that would else be paced, if the
    // trace is to ride along (one-peer steps, us with a reduction pass / without: 20 x 7M 580 / 545, 12 x 27M 1306 / 1254,
    // 20 x 10M without momentum 513 / 441; paced 587, 1274, 520).
    const bool traced_free = runs_free && spread_partials && uniform && a.L >= min_cycle && (int64_t)n * ge.d * 4 >= kPaceMinBytes;
    if (a.C > 1 && Q == 1 && wpb == 1 && ((plan.pace_gbs != 0.0 && plan.bpc > 0) || traced_free) && mode == MODE_PEER) {
        a.cpi = a.C;
        a.gy = 1;
        lp.work = a.gx;
    }
    const bool whole_columns = a.C == 1 || a.cpi == a.C;
    // the consensus sums can ride along when one walker stores whole columns
    if (spread_partials && spread_count && vec == 4 && Q == 1 && whole_columns && (U == 1 || U == 2) &&
        (mode == MODE_RING || mode == MODE_PEER)) {
        lp.blocks_out = spread_count;
        a.spread_partials = spread_partials;
        if (mom == 2) return launch_walk_trace<2>(mode, U, lp, c->stream, a);
        return mom ? launch_walk_trace<1>(mode, U, lp, c->stream, a) : launch_walk_trace<0>(mode, U, lp, c->stream, a);
    }
    if (vec == 4) {
        if (mom == 2) return launch_walk_mode<v4f, 2>(mode, U, lp, c->stream, a);
        return mom ? launch_walk_mode<v4f, 1>(mode, U, lp, c->stream, a)
                   : launch_walk_mode<v4f, 0>(mode, U, lp, c->stream, a);
    }
    if (mom == 2) return launch_walk_mode<float, 2>(mode, U, lp, c->stream, a);
    return mom ? launch_walk_mode<float, 1>(mode, U, lp, c->stream, a)
               : launch_walk_mode<float, 0>(mode, U, lp, c->stream, a);
}

// 16-byte lanes on rows on 16-byte boundaries, and on wide rows whatever their alignment (4-byte lanes there: ring n = 64,
// d = 25 000 001 10.7 -> 5.9 ms, they are not paced; n = 16, d = 1 000 003 85 -> 65 us; grid n = 64, d = 4 100 001 2.60 ->
// 1.23 ms; W = I n = 64, d = 1 000 001 447 -> 219 us).  Narrow rows of another alignment keep 4-byte lanes: their steps are
// bound by the chain of rows of a wavefront, and a quarter of the columns a lane makes four times the wavefronts (16 / 4
// bytes: ring n = 1000, d = 201 79 / 48 us, d = 4001 104 / 58, n = 100, d = 17 001 16.5 / 15.1, n = 20, d = 17 001 6.7 / 6.2;
// n = 230, d = 20 001 even).
constexpr int64_t kWideRagged = 36864;
int step_lane_columns(const gpga_ctx* c) {
    if (c->d < 4) return 1;
    const bool wide = c->d >= kWideRagged || (c->d >= kWideRagged / 2 && (int64_t)c->n * c->d >= 64 * kWideRagged);
    return wide || rows_on_16_bytes(c) ? 4 : 1;
}

GlobalOrder global_order(const gpga_ctx* c) {
    const int n = c->n, waves = c->opt_waves ? c->opt_waves : 4;
    const int vec = step_lane_columns(c);
    // Spread rows over lanes and waves only when columns alone cannot fill the chip.
    const int64_t tiles64 = ((c->d + vec - 1) / vec + kWave - 1) / kWave;
    int RL = 1, wpb = 1;
    if (c->opt_row_lanes) {
        RL = c->opt_row_lanes;
    } else if (tiles64 < kPacedWaves) {
        // Row pieces of 16 lanes, but whole ones on wide rows of another alignment than 16 bytes, where every piece shares its
        // lines with its neighbours (full average, us 4 / 1 row lanes: n = 200, d = 150 001 230 / 144, d = 500 001 702 / 441,
        // n = 64, d = 31 249 26.5 / 12.9, n = 1000, d = 30 001 216 / 147).
        RL = vec == 4 && n >= 8 && !rows_on_16_bytes(c) ? 1 : 4;
    }
    while (RL > 1 && RL > n) RL >>= 1;
    if (c->opt_row_split) {
        wpb = c->opt_row_split;
    } else if (tiles64 < kPacedWaves) {
        wpb = pow2_floor(n / (4 * RL) > 0 ? n / (4 * RL) : 1);
    }
    if (wpb > waves) wpb = waves;
    while (wpb > 1 && RL * wpb > n) wpb >>= 1;
    const LaunchPlan plan = make_plan(c, 1, waves, vec, RL == 1 && wpb == 1 && n >= 8, free_running_pays(c), PACE_GLOBAL);
    // (2 x 60M: 376 us with two rows a batch, 415 with four)
    return {RL, wpb, c->opt_unroll ? c->opt_unroll : (plan.pace_gbs != 0.0 ? 1 : n < 4 ? 2 : 4)};
}

hipError_t launch_step_global(const gpga_ctx* c, const StepGeom& geom, int vec) {
    c->note_path(PATH_GLOBAL, vec * 4);
    GlobalArgs a;
    a.ge = geom;
    const int n = a.ge.n;
    const GlobalOrder go = global_order(c);
    const int CL = kWave / go.RL;
    set_units(&a.ge, vec, CL);
    const bool runs_free = free_running_pays(c);
    const int waves = walk_waves(c, unit_tiles(a.ge, CL), runs_free && go.wpb == 1 && vec == 4);
    a.inv_n = 1.0f / (float)n;
    a.RL = go.RL;
    a.tpb = waves / go.wpb;
    const int64_t tiles = unit_tiles(a.ge, CL);
    const int64_t gx = (tiles + a.tpb - 1) / a.tpb;
    if (gx > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    a.gx = gx;
    a.xcd = c->opt_xcd_swizzle;
    const LaunchPlan plan = make_plan(c, gx, waves, vec, go.RL == 1 && go.wpb == 1 && n >= 8, runs_free, PACE_GLOBAL);
    const int U = go.U;
    const int mom = c->mu != 0.f ? (c->nesterov ? 2 : 1) : 0;
    if (vec == 4) {
        if (mom == 2) return launch_global_u<v4f, 2>(U, plan, c->stream, a);
        return mom ? launch_global_u<v4f, 1>(U, plan, c->stream, a)
                   : launch_global_u<v4f, 0>(U, plan, c->stream, a);
    }
    if (mom == 2) return launch_global_u<float, 2>(U, plan, c->stream, a);
    return mom ? launch_global_u<float, 1>(U, plan, c->stream, a)
               : launch_global_u<float, 0>(U, plan, c->stream, a);
}
