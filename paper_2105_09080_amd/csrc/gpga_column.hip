// Trajectories of synthetic gradients with whole columns on chip (gpga_run).
//
// Synthetic gradients (counter RNG) and mixing both leave columns apart: no value of a column depends on another
// column.  So a workgroup loads x and m of all n rows of a column tile once, runs T iterations of Algorithm 1 on
// them - gradients generated in registers, momentum and x in registers, x^(k+1/2) exchanged between rows through
// LDS - and stores x, m and the last gradient once: 20 bytes per element for the whole trajectory, where one
// iteration at a time takes 24 (g written, then read by the step) per iteration.
//
// Bound: the vector ALUs, some 75 instructions per four elements and iteration (ten Philox rounds, Box-Muller, update, mix);
// memory for very few iterations.  Measured on 64 x 25.6M elements, momentum 0.9: 0.5 ms an iteration on top of 5.9 ms for
// the load and the store (33 GB, 5.6 TB/s); 6 iterations 37.8 -> 8.5 ms, 2 iterations 12.5 -> 7.2 ms.  One iteration would
// take the 6.2 ms that the gradient kernel and a paced step take, so a run of one iteration stays with those.
// A thread owns R consecutive rows of one 16-byte column unit: with R = 2 the state takes 24 registers, and 64 in all let two
// workgroups of 16 wavefronts fit on a compute unit, so that one loads or stores while the other computes.  That cap is
// tight: 33 to 128 nodes spill 10 registers a lane (4 without momentum), up to 32 nodes 5 (none), more than 128 none.
#include "gpga_internal.hpp"
#include "gpga_order.hpp"
#include "gpga_rng.hpp"
#include "gpga_schedule.hpp"
#include "gpga_unit.hpp"

namespace {

struct ColumnArgs {
    StepGeom ge;      // x: iterates before the first iteration; x_new: where they go after the last one (may be x)
    float* g_out;
    uint32_t k0, k1;  // RNG key
    uint32_t kiter;   // counter word of the first iteration
    float sigma;
    int32_t T;
    int32_t mode;     // ColumnMix
    GlobalOrder go;   // the summation order of the global-average kernel on this problem
    int32_t lead64;   // StepGeom::lead of that kernel's 64-lane tiles
    float inv_n;
    const int32_t* wptr;
    const int32_t* wcol;
    const float* wval;
    float lr[kColumnRunMaxIters];
    int32_t shift[kColumnRunMaxIters];  // one-peer offset of the iteration; -1 = global average
};

enum ColumnMix : int { MIX_SELF = 0, MIX_RING = 1, MIX_PEER = 2, MIX_CSR = 3 };

template <int MOM, int R, int QT>
__global__ void __launch_bounds__(1024, R == 2 ? 8 : 4) k_column_run(const ColumnArgs a) {
    extern __shared__ __align__(16) unsigned char s_raw[];
    v4f* __restrict__ sy = reinterpret_cast<v4f*>(s_raw);  // [n][QT]
    const int n = a.ge.n;
    const int q = threadIdx.x % QT;
    int rs = threadIdx.x / QT;
    if (QT == kWave) rs = __builtin_amdgcn_readfirstlane(rs);
    const int row0 = rs * R;
    const int64_t tile = blockIdx.x;
    const bool on = unit_on(a.ge, tile, QT, q);
    const int64_t col = unit_column<v4f>(a.ge, tile, QT, q);
    const uint32_t c4 = (uint32_t)(col >> 2);
    const int skew = (int)(col & 3);  // the last unit of a ragged width starts inside an RNG quad
    const float mu = a.ge.mu;
    const float third = 1.0f / 3.0f;
    // whether the 64-lane tile of the step kernels that unit number u of this tile lies in is a whole one (decides their row order)
    auto whole_tile = [&](int u) {
        const int64_t unit = tile * QT + u - a.ge.lead;
        return (((unit < 0 ? 0 : unit) + a.lead64) / kWave + 1) * kWave - a.lead64 <= a.ge.ncols;
    };

    v4f x[R], m[R], y[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        x[j] = m[j] = v4f(0.f);
        if (on && row0 + j < n) {
            const int64_t o = (int64_t)(row0 + j) * a.ge.ld + col;
            x[j] = ld_unit<v4f>(a.ge.x + o);
            if (MOM) m[j] = ld_unit<v4f>(a.ge.m + o);
        }
    }
    for (int t = 0; t < a.T; ++t) {
        const float lr = a.lr[t];
        const int shift = a.shift[t];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int row = row0 + j;
            v4f g = synth_quad(c4, (uint32_t)row, a.kiter + (uint32_t)t, a.k0, a.k1, a.sigma);
            if (skew) {
                const v4f h = synth_quad(c4 + 1u, (uint32_t)row, a.kiter + (uint32_t)t, a.k0, a.k1, a.sigma);
                g = skew == 1 ? v4f{g.y, g.z, g.w, h.x} : skew == 2 ? v4f{g.z, g.w, h.x, h.y} : v4f{g.w, h.x, h.y, h.z};
            }
            v4f mom = g;
            if (MOM) m[j] = mom = mu * m[j] + g;
            y[j] = MOM == 2 ? x[j] - lr * (g + mu * mom) : x[j] - lr * mom;
            if (row < n) {
                sy[row * QT + q] = y[j];
                if (t == a.T - 1 && on) st_unit<v4f>(a.g_out + (int64_t)row * a.ge.ld + col, g);
            }
        }
        if (n == 1 || (shift >= 0 && a.mode == MIX_SELF)) {
#pragma unroll
            for (int j = 0; j < R; ++j) x[j] = y[j];
            continue;
        }
        __syncthreads();
        if (shift < 0) {
            // Narrow tiles have many rows: a column a thread, of the first ones (with a whole unit a lane, 256 x 2M averaged
            // in every iteration took 4920 us an iteration, 128 x 4M 2705, against 1260 and 892).  Wide tiles, of up to 32
            // rows, leave it to the lanes of one wavefront.
            if (QT < kWave) {
                float* const sf = reinterpret_cast<float*>(sy);
                for (int e = threadIdx.x; e < 4 * QT; e += blockDim.x) {
                    SplitterTree<float> tree;
                    for (int r0 = 0; r0 < a.go.RL * a.go.wpb; ++r0)
                        tree.add(r0, splitter_column_sum(a.go, r0, n, whole_tile(e / 4), sf + e, 4 * QT));
                    sf[e] = tree.sum * a.inv_n;  // nobody else reads this column meanwhile
                }
            } else if (rs == 0) {
                SplitterTree<v4f> tree;
                for (int r0 = 0; r0 < a.go.RL * a.go.wpb; ++r0) tree.add(r0, splitter_sum(a.go, r0, n, whole_tile(q), sy + q, QT));
                sy[q] = tree.sum * a.inv_n;
            }
            __syncthreads();
            const v4f mean = sy[q];
#pragma unroll
            for (int j = 0; j < R; ++j) x[j] = mean;
        } else if (a.mode == MIX_RING) {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int row = row0 + j;
                if (row >= n) break;
                const v4f prev = j > 0 ? y[j > 0 ? j - 1 : 0] : sy[(row == 0 ? n - 1 : row - 1) * QT + q];
                const v4f next = (j + 1 < R && row + 1 < n) ? y[j + 1 < R ? j + 1 : 0] : sy[(row + 1 == n ? 0 : row + 1) * QT + q];
                x[j] = (prev + y[j] + next) * third;
            }
        } else if (a.mode == MIX_PEER) {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int row = row0 + j;
                if (row >= n) break;
                const int peer = row + shift >= n ? row + shift - n : row + shift;
                x[j] = shift ? (y[j] + sy[peer * QT + q]) * 0.5f : y[j];
            }
        } else {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int row = row0 + j;
                if (row >= n) break;
                v4f acc = v4f(0.f);
                const int p1 = a.wptr[row + 1];
                for (int p = a.wptr[row]; p < p1; ++p) acc += a.wval[p] * sy[a.wcol[p] * QT + q];
                x[j] = acc;
            }
        }
        __syncthreads();  // the next iteration overwrites the rows
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if (on && row0 + j < n) {
            const int64_t o = (int64_t)(row0 + j) * a.ge.ld + col;
            st_unit<v4f>(a.ge.x_new + o, x[j]);
            if (MOM) st_unit<v4f>(a.ge.m + o, m[j]);
        }
    }
}

template <int MOM, int R, int QT>
hipError_t launch_column(const gpga_ctx* c, ColumnArgs a) {
    set_units(&a.ge, 4, QT);
    const int threads = ((a.ge.n + R - 1) / R * QT + kWave - 1) / kWave * kWave;
    const size_t lds = (size_t)a.ge.n * QT * sizeof(v4f);
    const int64_t blocks = unit_tiles(a.ge, QT);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((k_column_run<MOM, R, QT>), dim3((unsigned)blocks), dim3(threads), lds, c->stream, a);
    return hipGetLastError();
}

// Tile width: all rows in 1024 threads and 64 KiB of LDS at most.  (n = 64: row pieces of 256 bytes instead of 512 in
// workgroups of half the size ran 2 iterations in 7.35 instead of 7.18 ms and 6 in 9.33 instead of 9.61; a persistent
// launch that loads the next tile while it computes - half the wavefronts for twice the registers - took 8.6 and 11.5.)
template <int MOM>
hipError_t launch_column_rows(const gpga_ctx* c, const ColumnArgs& a) {
    if (a.ge.n <= 32) return launch_column<MOM, 2, 64>(c, a);
    if (a.ge.n <= 64) return launch_column<MOM, 2, 32>(c, a);
    if (a.ge.n <= 128) return launch_column<MOM, 2, 16>(c, a);
    return launch_column<MOM, 4, 16>(c, a);
}

}  // namespace

bool column_run_fits(const gpga_ctx* c, int64_t T) {
    if (c->opt_column_run == 0 || !c->default_geometry() || c->problem != PROB_SYNTH || c->aga || T < 2) return false;
    if (c->n > 256 || c->d < 4) return false;
    if (c->trace && c->k < c->trace_cap) return false;  // the trace wants every iterate
    if ((c->topo == GPGA_TOPO_GRID || c->topo == GPGA_TOPO_EXPO || c->topo == GPGA_TOPO_CUSTOM) && !c->csr_ready) return false;
    // A trajectory that is being captured keeps its launch per step: the paced launches in a graph are what
    // gpga_query counts and what callers tune.
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &st) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return st == hipStreamCaptureStatusNone;
}

hipError_t launch_column_run(const gpga_ctx* c, int32_t T) {
    if (T < 1 || T > kColumnRunMaxIters) return hipErrorInvalidValue;
    ColumnArgs a;
    a.ge.x = c->x;
    a.ge.x_new = (T % 2) ? c->x_new : c->x;  // where T separate steps would leave the live iterates
    a.ge.m = c->m;
    a.ge.g = c->g;
    a.ge.ld = c->ld;
    a.ge.d = c->d;
    a.ge.n = c->n;
    a.ge.lr = 0.f;
    a.ge.mu = c->mu;
    a.g_out = c->g;
    a.k0 = (uint32_t)(c->seed & 0xffffffffu);
    a.k1 = (uint32_t)(c->seed >> 32);
    a.kiter = (uint32_t)(c->k & 0xffffffff);
    a.sigma = c->grad_sigma;
    a.T = T;
    a.mode = c->topo == GPGA_TOPO_RING ? MIX_RING : c->topo == GPGA_TOPO_EXPO1 ? MIX_PEER
             : (c->topo == GPGA_TOPO_NONE || c->topo == GPGA_TOPO_FULL) ? MIX_SELF : MIX_CSR;
    a.go = global_order(c);
    set_units(&a.ge, 4, kWave);
    a.lead64 = a.ge.lead;
    a.inv_n = 1.0f / (float)c->n;
    a.wptr = c->csr_ptr_d;
    a.wcol = c->csr_col_d;
    a.wval = c->csr_val_d;
    for (int32_t t = 0; t < T; ++t) {
        a.lr[t] = scheduled_lr(c, c->k + t);
        a.shift[t] = is_global_iteration(c->topo, c->H, c->k + t) ? -1
                     : a.mode == MIX_PEER ? one_peer_shift(c->n, c->k + t) : 0;
    }
    if (c->mu == 0.f) return launch_column_rows<0>(c, a);
    return c->nesterov ? launch_column_rows<2>(c, a) : launch_column_rows<1>(c, a);
}
