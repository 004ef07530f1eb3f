// Second half of an iteration on stored features, in one launch (gpga_run): gradient sum, local update and mixing.
//
//     g_i = sum_b coef_b * row_b ;  m_i, y_i from g_i, x_i ;  x_new_i = sum_j w_ij y_j  or the mean of all y_j
//
// The coefficients come from the margin pass.  From there on columns are apart, so a workgroup takes a column tile of
// all n nodes: QT lanes of four columns, the 1024 / QT lane groups share nodes and samples, the groups' fp64 sums and
// then x^(k+1/2) meet in LDS.  Problems of this kind (n <= 128, a few million elements) are bound by the latency of
// dependent launches of 4 - 10 us each; one launch instead of two also leaves g unwritten and unread but for the last
// iteration of a run.
// The whole iteration, margin pass included: 8 x 1000 with full batches of 100 rows 12.9 -> 9.8 us, 20 x 1001 with 16 rows
// under the adaptive period 17.1 -> 11.7, 32 x 10 000 with 32 rows 27.7 -> 25.2, 16 x 39 999 with 50 rows 130 -> 59.
#include "gpga_internal.hpp"
#include "gpga_order.hpp"
#include "gpga_rows_deal.hpp"
#include "gpga_unit.hpp"

namespace {

constexpr int kRowsMaxNodes = 128;
constexpr int64_t kRowsMaxStaged = 4352;       // (node, sample) pairs whose row numbers and coefficients go to LDS first
// Larger states are bound by their rows, which the separate kernels read in longer pieces (64 x 40 000: 1102 us a run
// of 8 iterations here, 1025 there; 50 x 20 000: 660 here, 721 there).
constexpr int64_t kRowsMaxElements = 1 << 21;

struct RowsStepArgs {
    StepGeom ge;
    float* g_out;          // NULL: the gradients of this iteration are not wanted
    const float* feat;     // n x M x d
    const float* coef;     // n x B
    const int32_t* idx;    // n x B, or NULL: rows 0 .. B-1
    int32_t B, M;
    int32_t mode;          // StencilMode, or one of the two below
    int32_t shift;         // one-peer offset
    const int32_t* off;    // sparse W: (signed circular offset, weight) entries, K a node at most
    const float* val;
    const int32_t* wptr;   // node i has wptr[i + 1] - wptr[i] of them
    int32_t K;
    GlobalOrder go;
    int32_t lead64;
    float inv_n;
};
constexpr int kModeSparse = 8, kModeGlobal = 9;

template <int MOM, int QT>
__global__ void __launch_bounds__(kRowsThreads) k_rows_step(const RowsStepArgs a) {
    constexpr int NG = kRowsThreads / QT;
    extern __shared__ __align__(16) unsigned char s_raw[];
    const int n = a.ge.n, B = a.B;
    const bool staged = (int64_t)n * B <= kRowsMaxStaged;
    const int pairs = staged ? n * B : 0, pad = (pairs + 1) & ~1;
    v4f* __restrict__ sy = reinterpret_cast<v4f*>(s_raw);                      // [n][QT]
    int32_t* __restrict__ sRow = reinterpret_cast<int32_t*>(sy + n * QT);      // [n][B]
    float* __restrict__ sCoef = reinterpret_cast<float*>(sRow + pad);          // [n][B]
    double* __restrict__ sPart = reinterpret_cast<double*>(sRow + 2 * pad);    // [4][1024] groups' sums, if SG > 1; then the leaves
    const int tid = threadIdx.x, q = tid % QT, grp = tid / QT;
    const int64_t tile = blockIdx.x;
    const bool on = unit_on(a.ge, tile, QT, q);
    const int64_t col = unit_column<v4f>(a.ge, tile, QT, q);
    const float lr = a.ge.lr, mu = a.ge.mu;
    for (int p = tid; p < pairs; p += kRowsThreads) {
        const int32_t r = a.idx ? a.idx[p] : p % B;
        sRow[p] = r >= 0 && r < a.M ? r : 0;  // outside [0, M): its coefficient is NaN, row 0 is only a safe address
        sCoef[p] = a.coef[p];
    }
    __syncthreads();

    const RowsDeal deal(QT, n, B);
    const int SG = deal.split, per = deal.nodes, part = deal.part(grp);
    for (int i0 = 0; i0 < n; i0 += per) {
        const int i = i0 + deal.node(grp);
        const bool mine = deal.dealt(grp) && i < n && on;
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        v4f xv = v4f(0.f), mv = v4f(0.f);
        const int64_t o = (int64_t)i * a.ge.ld + col;
        if (mine) {
            if (part == 0) {
                xv = ld_unit_cached<v4f>(a.ge.x + o);
                if (MOM) mv = ld_unit_cached<v4f>(a.ge.m + o);
            }
            const float* __restrict__ f = a.feat + (int64_t)i * a.M * a.ge.d + col;
            auto sample = [&](int b, float* cb) -> int32_t {
                if (staged) {
                    *cb = sCoef[i * B + b];
                    return sRow[i * B + b];
                }
                *cb = a.coef[(int64_t)i * B + b];
                const int32_t r = a.idx ? a.idx[(int64_t)i * B + b] : b;
                return r >= 0 && r < a.M ? r : 0;
            };
            for (int b = part; b < B; b += 8 * SG) {  // eight rows in flight
                v4f v[8];
                float cf[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int bu = b + u * SG < B ? b + u * SG : b;
                    v[u] = ld_unit_cached<v4f>(f + (int64_t)sample(bu, &cf[u]) * a.ge.d);
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (b + u * SG < B) {
                        const double cb = cf[u];
                        acc[0] += cb * v[u].x;
                        acc[1] += cb * v[u].y;
                        acc[2] += cb * v[u].z;
                        acc[3] += cb * v[u].w;
                    }
                }
            }
        }
        if (SG > 1) {
#pragma unroll
            for (int c = 0; c < 4; ++c) sPart[c * kRowsThreads + tid] = acc[c];
            __syncthreads();
            if (deal.adds(grp)) {
#pragma unroll 4
                for (int w = 1; w < SG; ++w)
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[c] += sPart[c * kRowsThreads + tid + w * QT];
            }
            if (i0 + per < n) __syncthreads();  // the next nodes' sums overwrite these
        }
        if (mine && part == 0) {
            const v4f g = {(float)acc[0], (float)acc[1], (float)acc[2], (float)acc[3]};
            v4f mom = g;
            if (MOM) {
                mom = mu * mv + g;
                *reinterpret_cast<v4u*>(a.ge.m + o) = mom;
            }
            if (a.g_out) st_unit<v4f>(a.g_out + o, g);
            sy[i * QT + q] = MOM == 2 ? xv - lr * (g + mu * mom) : xv - lr * mom;
        }
    }
    __syncthreads();

    if (a.mode == kModeGlobal) {  // a splitter's rows per lane group, then the tree
        v4f* __restrict__ leaf = reinterpret_cast<v4f*>(sPart);
        const int64_t unit = tile * QT + q - a.ge.lead;
        const bool whole = (((unit < 0 ? 0 : unit) + a.lead64) / kWave + 1) * kWave - a.lead64 <= a.ge.ncols;
        const int RS = a.go.RL * a.go.wpb;
        for (int r0 = grp; r0 < RS; r0 += NG)
            if (on) leaf[r0 * QT + q] = splitter_sum(a.go, r0, n, whole, sy + q, QT);
        __syncthreads();
        if (!on) return;
        SplitterTree<v4f> tree;
        for (int r0 = 0; r0 < RS; ++r0) tree.add(r0, leaf[r0 * QT + q]);
        const v4f mean = tree.sum * a.inv_n;
        for (int i = grp; i < n; i += NG) *reinterpret_cast<v4u*>(a.ge.x_new + (int64_t)i * a.ge.ld + col) = mean;
        return;
    }
    if (!on) return;
    for (int i = grp; i < n; i += NG) {
        const v4f y = sy[i * QT + q];
        v4f v = y;
        if (a.mode == MODE_RING) {
            v = (sy[(i == 0 ? n - 1 : i - 1) * QT + q] + y + sy[(i == n - 1 ? 0 : i + 1) * QT + q]) * (1.0f / 3.0f);
        } else if (a.mode == MODE_PEER) {
            v = (y + sy[(i + a.shift >= n ? i + a.shift - n : i + a.shift) * QT + q]) * 0.5f;
        } else if (a.mode == kModeSparse) {
            v = v4f(0.f);
            const int entries = a.wptr[i + 1] - a.wptr[i];
            for (int p = 0; p < entries; ++p) {
                int j = i + a.off[i * a.K + p];
                j = j < 0 ? j + n : j >= n ? j - n : j;
                v += a.val[i * a.K + p] * sy[j * QT + q];
            }
        }
        *reinterpret_cast<v4u*>(a.ge.x_new + (int64_t)i * a.ge.ld + col) = v;
    }
}

template <int MOM, int QT>
hipError_t launch_rows_tile(const gpga_ctx* c, RowsStepArgs a) {
    set_units(&a.ge, 4, QT);
    const size_t part = RowsDeal(QT, a.ge.n, a.B).split > 1 ? 4 * kRowsThreads * sizeof(double) : 0;
    const size_t leaves = a.mode == kModeGlobal ? (size_t)a.go.RL * a.go.wpb * QT * sizeof(v4f) : 0;
    const size_t staged = (int64_t)a.ge.n * a.B <= kRowsMaxStaged ? (size_t)a.ge.n * a.B : 0;
    const size_t lds = (size_t)a.ge.n * QT * sizeof(v4f) + 2 * ((staged + 1) & ~(size_t)1) * sizeof(int32_t) +
                       (part > leaves ? part : leaves);
    static bool attr_set[64] = {false};  // per instantiation and device: more than the default 64 KiB of dynamic LDS
    const int dev = c->device >= 0 && c->device < 64 ? c->device : 0;
    if (!attr_set[dev]) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_rows_step<MOM, QT>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)c->max_lds_block);
        if (e != hipSuccess) return e;
        attr_set[dev] = true;
    }
    hipLaunchKernelGGL((k_rows_step<MOM, QT>), dim3((unsigned)unit_tiles(a.ge, QT)), dim3(kRowsThreads), lds, c->stream, a);
    return hipGetLastError();
}

template <int MOM>
hipError_t launch_rows_mom(const gpga_ctx* c, const RowsStepArgs& a) {
    // Row pieces: wide ones touch fewer pages of the feature array, narrow ones give more workgroups.  Measured a run of
    // 8 - 16 iterations with pieces of 64 / 128 / 256 / 512 / 1024 bytes, us: 8 x 1000 78 / 82 / 91 / 107 / 144;
    // 30 x 3000 132 / 125 / 132 / 167 / 260; 32 x 10 000 552 / 486 / 405 / 431 / 555; 50 x 20 000 941 / 707 / 709 /
    // 660 / 821; 16 x 39 999 880 / 663 / 549 / 526 / 469.
    if (a.ge.d > 32768 && a.ge.n <= 64) return launch_rows_tile<MOM, 64>(c, a);
    if (a.ge.d > 16384) return launch_rows_tile<MOM, 32>(c, a);
    if (a.ge.d > 4096) return launch_rows_tile<MOM, 16>(c, a);
    return a.ge.d > 2048 ? launch_rows_tile<MOM, 8>(c, a) : launch_rows_tile<MOM, 4>(c, a);
}

}  // namespace

bool rows_step_fits(const gpga_ctx* c, int32_t Beff) {
    if (!c->default_geometry() || (c->problem != PROB_LSQ && c->problem != PROB_LOGREG)) return false;
    const bool sparse = c->topo == GPGA_TOPO_GRID || c->topo == GPGA_TOPO_EXPO || c->topo == GPGA_TOPO_CUSTOM;
    if (sparse && (!c->csr_ready || !c->csr_off_d)) return false;
    // at most 64 KiB of x^(k+1/2), 32 KiB of sums and 34 KiB of samples in LDS
    if (c->d < 4 || c->n > kRowsMaxNodes || (int64_t)c->n * c->d > kRowsMaxElements || c->max_lds_block < 130 * 1024) return false;
    // Batches: a workgroup here takes the samples of all nodes for its columns, the separate accumulate pass has a workgroup
    // per node and 256 columns.  Up to as many samples as are staged this form wins or is even (n = 128, 32 samples: d = 64
    // 19.7 -> 13.8 us an iteration, d = 2000 30.7 -> 23.9; n = 32, 128 samples, d = 20 000 121 -> 115, d = 3000 27.3 -> 28.3;
    // with 160 samples d = 1500 24.8 -> 27.5); beyond them only where the separate pass leaves most of the chip idle (n = 8,
    // d = 1000, 1000 samples 55.5 -> 34.0; n = 16, d = 1000, 2000 samples 104 -> 99; against n = 16, d = 2500 75 -> 92; n = 32,
    // d = 256, 4000 samples 238 -> 309; n = 100, d = 10, 8000 samples 281 -> 1740).
    return (int64_t)c->n * Beff <= kRowsMaxStaged || (c->n <= 16 && (int64_t)c->n * ((c->d + 255) / 256) <= 128);
}

hipError_t launch_rows_step(const gpga_ctx* c, const StepGeom& geom, const int32_t* idx, int32_t Beff, bool global, int mode,
                            int32_t shift, bool csr, bool want_g) {
    RowsStepArgs a;
    a.ge = geom;
    a.g_out = want_g ? c->g : nullptr;
    a.feat = c->feat;
    a.coef = c->coef;
    a.idx = idx;
    a.B = Beff;
    a.M = c->M;
    a.mode = global ? (c->n > 1 ? kModeGlobal : (int)MODE_SELF) : csr ? kModeSparse : mode;
    a.shift = shift;
    a.off = c->csr_off_d;
    a.val = c->csr_ellval_d;
    a.wptr = c->csr_ptr_d;
    a.K = c->csr_max_row;
    a.go = global_order(c);
    set_units(&a.ge, 4, kWave);
    a.lead64 = a.ge.lead;
    a.inv_n = 1.0f / (float)c->n;
    c->note_path(PATH_ROWS_STEP, 16);
    if (c->mu == 0.f) return launch_rows_mom<0>(c, a);
    return c->nesterov ? launch_rows_mom<2>(c, a) : launch_rows_mom<1>(c, a);
}
