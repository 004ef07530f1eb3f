// Trajectories of synthetic gradients with whole columns on chip (gpga_run).
//
// Synthetic gradients (counter RNG) and mixing both leave columns apart: no value of a column depends on another
// column.  So a workgroup loads x and m of all n rows of a column tile once, runs T iterations of Algorithm 1 on
// them - gradients generated in registers, momentum and x in registers, x^(k+1/2) exchanged between rows through
// LDS - and stores x, m and the last gradient once: 20 bytes per element for the whole trajectory, where one
// iteration at a time takes 24 (g written, then read by the step) per iteration.
//
// Bound: vector issue from about six iterations on, some 85 instructions per four elements and iteration (eight Philox rounds
// and a half, Box-Muller, update, mix); memory for fewer.  Measured on 64 x 25.6M elements, momentum 0.9: 0.85 ms an
// iteration (24 iterations of the ring 29.6 -> 22.4 ms), 5.3 to 6.4 ms for the load, two iterations and the store
// (33 GB), 6 iterations of the one-peer graph 8.9 -> 7.2 - 7.4 ms, of the ring 9.7 -> 7.3, where the two calls an iteration
// take 37.8.  One iteration would take the 6.2 ms that the gradient kernel and a paced step take, so a run of one
// iteration stays with those.
// A thread owns R consecutive rows of one quad: with R = 2 the state takes 24 registers, and 64 in all let two workgroups
// of 16 wavefronts fit on a compute unit, so that one loads or stores while the other computes.  That cap and the 78 scalar
// registers that go with it are tight: addresses, round keys and lane masks kept over the loop end up in scratch memory and in
// vector lanes, 70 moves per two rows (ring, 24 iterations 24.6 ms); formed anew in each iteration they are scalar additions.
#include "gpga_exchange.hpp"
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

// Two exchange buffers are used in turn, so that an exchange has one barrier (an average two): gpga_exchange.hpp.
// QUADS: an average is formed a quad a lane by the first wavefront, else a column a thread.
template <int MIX, int MOM, int R, int QT, bool QUADS>
__global__ void __launch_bounds__(1024, R == 2 ? 8 : 4) k_column_run(const ColumnArgs a) {
    extern __shared__ __align__(16) unsigned char s_raw[];
    const int n = a.ge.n;
    const int q = threadIdx.x % QT;
    int rs = threadIdx.x / QT;
    if (QT == kWave) rs = __builtin_amdgcn_readfirstlane(rs);
    const int row0 = rs * R;
    // Quads of the counter RNG start at multiples of four, whatever the width: the last one of a ragged width is a part.
    const uint32_t c4 = blockIdx.x * QT + q;
    const int64_t col = (int64_t)c4 * 4;
    const bool whole = ((int64_t)blockIdx.x + 1) * QT * 4 <= a.ge.d;  // uniform: every lane has a whole quad
    const int have = whole || col + 4 <= a.ge.d ? 4 : col < a.ge.d ? (int)(a.ge.d - col) : 0;
    const float mu = a.ge.mu;
    const float third = 1.0f / 3.0f;

    // `all`: the lane's four columns are all there, without a look at `have`
    auto load = [&](const float* p, bool all) -> v4f {
        if (all || have == 4) return ld_unit<v4f>(p);
        v4f v = v4f(0.f);
        if (have > 0) v.x = p[0];
        if (have > 1) v.y = p[1];
        if (have > 2) v.z = p[2];
        return v;
    };
    auto store = [&](float* p, const v4f& v, bool all) {
        if (all || have == 4) {
            st_unit<v4f>(p, v);
            return;
        }
        if (have > 0) p[0] = v.x;
        if (have > 1) p[1] = v.y;
        if (have > 2) p[2] = v.z;
    };
    // The same value, but nothing derived from it is kept for the next iteration (see above).
    auto once = [&](int v) {
        if (R == 2 && QT == kWave) asm volatile("" : "+s"(v));
        if (R == 2 && QT < kWave) asm volatile("" : "+v"(v));
        return v;
    };
    v4f x[R], m[R], y[R];
    auto load_state = [&](bool all) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            x[j] = m[j] = v4f(0.f);
            if (row0 + j < n) {
                const int64_t o = (int64_t)(row0 + j) * a.ge.ld + col;
                x[j] = load(a.ge.x + o, all);
                if (MOM) m[j] = load(a.ge.m + o, all);
            }
        }
    };
    if (whole) load_state(true); else load_state(false);
    const SynthQuad quad(c4, a.k1);
    constexpr bool kOwn = MIX == MIX_SELF;
    int exchanges = 0;
    for (int t = 0; t < a.T; ++t) {
        v4f* __restrict__ sy = reinterpret_cast<v4f*>(s_raw) + exchange_buffer<kOwn>(t, exchanges) * n * QT;  // [n][QT]
        const float lr = a.lr[t];
        const int shift = a.shift[t];
        const bool meets = exchanges_rows<kOwn>(n, shift);
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int row = row0 + j;
            // the keys of the ten rounds likewise: twenty scalar registers otherwise, and as many moves out of vector lanes
            uint32_t k0 = a.k0, k1 = a.k1;
            if (R == 2) asm volatile("" : "+s"(k0), "+s"(k1));
            const v4f g = quad.gradient((uint32_t)row, a.kiter + (uint32_t)t, k0, k1, a.sigma);
            v4f mom = g;
            if (MOM) m[j] = mom = mu * m[j] + g;
            y[j] = MOM == 2 ? x[j] - lr * (g + mu * mom) : x[j] - lr * mom;
            if (row < n) {
                if (!kOwn || meets) sy[row * QT + q] = y[j];
                if (t == a.T - 1) {
                    float* const to = a.g_out + (int64_t)(once(row0) + j) * a.ge.ld + col;
                    if (whole) store(to, g, true); else store(to, g, false);
                }
            }
        }
        if (!meets) {
#pragma unroll
            for (int j = 0; j < R; ++j) x[j] = y[j];
            continue;
        }
        ++exchanges;
        __syncthreads();
        if (shift < 0) {
            // whether the 64-lane tile of the step kernels that a unit lies in is a whole one decides their row order
            if (!QUADS) {
                float* const sf = reinterpret_cast<float*>(sy);
                for (int e = threadIdx.x; e < 4 * QT; e += blockDim.x) {
                    const int64_t unit = (int64_t)blockIdx.x * QT + e / 4;
                    const bool whole64 = ((unit + a.lead64) / kWave + 1) * kWave - a.lead64 <= a.ge.ncols;
                    SplitterTree<float> tree;
                    for (int r0 = 0; r0 < a.go.RL * a.go.wpb; ++r0)
                        tree.add(r0, splitter_column_sum(a.go, r0, n, whole64, sf + e, 4 * QT));
                    sf[e] = tree.sum * a.inv_n;  // nobody else reads this column meanwhile
                }
            } else if (rs == 0) {
                const int64_t unit = (int64_t)blockIdx.x * QT + q;
                const bool whole64 = ((unit + a.lead64) / kWave + 1) * kWave - a.lead64 <= a.ge.ncols;
                SplitterTree<v4f> tree;
                for (int r0 = 0; r0 < a.go.RL * a.go.wpb; ++r0) tree.add(r0, splitter_sum(a.go, r0, n, whole64, sy + q, QT));
                sy[q] = tree.sum * a.inv_n;
            }
            __syncthreads();
            const v4f mean = sy[q];
#pragma unroll
            for (int j = 0; j < R; ++j) x[j] = mean;
        } else if (MIX == MIX_RING) {
            const int first = once(row0);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int row = first + j;
                if (row >= n) break;
                const v4f prev = j > 0 ? y[j > 0 ? j - 1 : 0] : sy[(row == 0 ? n - 1 : row - 1) * QT + q];
                const v4f next = (j + 1 < R && row + 1 < n) ? y[j + 1 < R ? j + 1 : 0] : sy[(row + 1 == n ? 0 : row + 1) * QT + q];
                x[j] = (prev + y[j] + next) * third;
            }
        } else if (MIX == MIX_PEER) {
            const int first = once(row0);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int row = first + j;
                if (row >= n) break;
                const int peer = row + shift >= n ? row + shift - n : row + shift;
                x[j] = shift ? (y[j] + sy[peer * QT + q]) * 0.5f : y[j];
            }
        } else if (MIX == MIX_CSR) {
            const int first = once(row0);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int row = first + j;
                if (row >= n) break;
                v4f acc = v4f(0.f);
                const int p1 = a.wptr[row + 1];
                for (int p = a.wptr[row]; p < p1; ++p) acc += a.wval[p] * sy[a.wcol[p] * QT + q];
                x[j] = acc;
            }
        }
    }
    const int row_out = once(row0);
    auto store_state = [&](bool all) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if (row_out + j < n) {
                const int64_t o = (int64_t)(row_out + j) * a.ge.ld + col;
                store(a.ge.x_new + o, x[j], all);
                if (MOM) store(a.ge.m + o, m[j], all);
            }
        }
    };
    if (whole) store_state(true); else store_state(false);
}

size_t column_lds(int n, int lanes) { return (size_t)2 * n * lanes * sizeof(v4f); }  // 64 KiB at most, 128 beyond 128 rows

template <int MIX, int MOM, int R, int QT, bool QUADS = false>
hipError_t launch_column(const gpga_ctx* c, const ColumnArgs& a) {
    const int threads = ((a.ge.n + R - 1) / R * QT + kWave - 1) / kWave * kWave;
    const size_t lds = column_lds(a.ge.n, QT);
    if (lds > 64 * 1024) {  // per instantiation and device: more than the default 64 KiB of dynamic LDS
        static bool attr_set[64] = {false};
        const int dev = c->device >= 0 && c->device < 64 ? c->device : 0;
        if (!attr_set[dev]) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_column_run<MIX, MOM, R, QT, QUADS>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)c->max_lds_block);
            if (e != hipSuccess) return e;
            attr_set[dev] = true;
        }
    }
    const int64_t blocks = (a.ge.ncols + QT - 1) / QT;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((k_column_run<MIX, MOM, R, QT, QUADS>), dim3((unsigned)blocks), dim3(threads), lds, c->stream, a);
    return hipGetLastError();
}

// How averages are formed on 64-lane tiles.  A thread adds a column, eight rows read ahead: where rows are few, and dealt to
// splitters besides, most of what it reads is not used, and the workgroup has fewer threads than columns.  Us of four averages,
// a column a thread / a quad a lane of the first wavefront: n = 2, d = 50 000 19.2 / 9.0, n = 4, d = 291 188 25.2 / 16.1,
// d = 3M 58.7 / 49.3, n = 7, d = 50 000 13.2 / 13.6, d = 1.5M 48.3 / 45.6; n = 8, d = 50 000 13.4 / 14.0, d = 400 000 27.2 / 21.6,
// d = 600 000 25.9 / 28.8; n = 12, d = 100 000 16.9 / 17.9, d = 150 000 20.0 / 19.4, d = 291 188 27.5 / 25.1, d = 600 000
// 37.4 / 44.0; n = 13, d = 291 188 30.7 / 34.7; n = 32, d = 3M 404 / 586.  (Narrow tiles have more rows: a column a thread;
// 256 x 2M averaged in every iteration 4920 us an iteration a quad a lane, 1260 a column a thread, 128 x 4M 2705 and 892.)
bool quad_averages(const gpga_ctx* c) {
    const int64_t tiles = ((c->d + 3) / 4 + kWave - 1) / kWave;
    return c->n < 8 || (c->n <= 12 && tiles >= 512 && tiles < 2048);
}

// Tile width: all rows in 1024 threads, and two workgroups of up to 128 rows in a compute unit's LDS.  (n = 64, before: row
// pieces of 256 bytes instead of 512 in workgroups of half the size ran 2 iterations in 7.35 instead of 7.18 ms and 6 in 9.33
// instead of 9.61; a persistent launch that loads the next tile while it computes - half the wavefronts for twice the
// registers - took 8.6 and 11.5.)
template <int MIX, int MOM>
hipError_t launch_column_rows(const gpga_ctx* c, const ColumnArgs& a) {
    if (a.ge.n <= 32) return quad_averages(c) ? launch_column<MIX, MOM, 2, 64, true>(c, a) : launch_column<MIX, MOM, 2, 64>(c, a);
    if (a.ge.n <= 64) return launch_column<MIX, MOM, 2, 32>(c, a);
    if (a.ge.n <= 128) return launch_column<MIX, MOM, 2, 16>(c, a);
    return launch_column<MIX, MOM, 4, 16>(c, a);
}
template <int MIX>
hipError_t launch_column_mix(const gpga_ctx* c, const ColumnArgs& a) {
    if (c->mu == 0.f) return launch_column_rows<MIX, 0>(c, a);
    return c->nesterov ? launch_column_rows<MIX, 2>(c, a) : launch_column_rows<MIX, 1>(c, a);
}

}  // namespace

bool column_run_fits(const gpga_ctx* c, int64_t T) {
    if (c->opt_column_run == 0 || !c->default_geometry() || c->problem != PROB_SYNTH || c->aga || T < 2) return false;
    if (c->n > 256 || c->d < 4 || (c->n > 128 && column_lds(c->n, 16) > (size_t)c->max_lds_block)) return false;
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
    const int mode = c->topo == GPGA_TOPO_RING ? MIX_RING : c->topo == GPGA_TOPO_EXPO1 ? MIX_PEER
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
                     : mode == MIX_PEER ? one_peer_shift(c->n, c->k + t) : 0;
    }
    switch (mode) {
        case MIX_SELF: return launch_column_mix<MIX_SELF>(c, a);
        case MIX_RING: return launch_column_mix<MIX_RING>(c, a);
        case MIX_PEER: return launch_column_mix<MIX_PEER>(c, a);
        default: return launch_column_mix<MIX_CSR>(c, a);
    }
}
