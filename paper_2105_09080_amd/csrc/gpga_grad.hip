// Local stochastic gradients g_i = grad F_i(x_i; xi_i) for all n simulated nodes
// (Algorithm 1, line 1 of the loop).  Three families:
//
//  * synthetic    G[i][c] = sigma * N(seed, TAG_GRAD, i, k, c): a counter-addressed
//                 normal (Philox4x32-10 + Box-Muller) standing in for a network's
//                 backward pass.  Integer/ALU bound; one 128-bit store per lane.
//  * stored rows  least squares and logistic regression (Sec. 5.1 loss) on a
//                 materialised n x M x d array: a batched GEMV pair per node,
//                 (1) margins z_b = <row_b, x_i> -> per-sample coefficient,
//                 (2) g_i = sum_b coef_b * row_b.  Plain FMA, no matrix cores: each
//                 node has its own x_i, so there is no shared operand to tile.
//  * virtual rows logistic regression whose feature rows are regenerated from
//                 the counter RNG inside both passes (the array would not fit).
#include "gpga_internal.hpp"
#include "gpga_node_run.hpp"
#include "gpga_rng.hpp"
#include "gpga_samples.hpp"
#include "gpga_schedule.hpp"
#include "gpga_unit.hpp"

namespace {

// ---------------------------------------------------------------- synthetic

__global__ void __launch_bounds__(256) k_synth_grad(float* __restrict__ g, int64_t ld, int64_t d,
                                                    uint32_t k0, uint32_t k1, uint32_t kiter,
                                                    float sigma, int vec_ok) {
    const int64_t c4 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t c = c4 * 4;
    if (c >= d) return;
    const uint32_t i = blockIdx.y;
    const v4f z = synth_quad((uint32_t)c4, i, kiter, k0, k1, sigma);
    float* row = g + (int64_t)i * ld;
    if (vec_ok && c + 3 < d) {
        __builtin_nontemporal_store(z, reinterpret_cast<v4f*>(row + c));
    } else {
        row[c] = z.x;
        if (c + 1 < d) row[c + 1] = z.y;
        if (c + 2 < d) row[c + 2] = z.z;
        if (c + 3 < d) row[c + 3] = z.w;
    }
}

// ---------------------------------------------------------------- reductions

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_down(v, off, kWave);
    return v;
}

// Sum over the workgroup; result valid in thread 0.
__device__ __forceinline__ double block_sum(double v, double* s_buf) {
    v = wave_sum(v);
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    if (lane == 0) s_buf[wave] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += s_buf[w];
    return t;
}

// Sum over each aligned group of G lanes, G = 16, 32 or 64 (uniform); complete in the group's
// last lane.  Every lane of the wavefront must be active.
__device__ __forceinline__ double group_sum_last(double v, int G) {
    v = row16_sum_last(v);
    if (G == 16) return v;
    const double r0 = readlane_f64(v, 15), r1 = readlane_f64(v, 31), r2 = readlane_f64(v, 47), r3 = readlane_f64(v, 63);
    if (G == 32) return (threadIdx.x & 32) ? r2 + r3 : r0 + r1;
    return (r0 + r1) + (r2 + r3);
}

// ---------------------------------------------------------------- stored rows

// Pass 1: one workgroup per (sample slot b, node i): z = <row, x_i> in fp64.  16-byte lanes at any alignment, the last
// d % 4 columns on lanes of their own.  Bound by latency (sample index, then the row) on the sizes of a minibatch, so
// rows_margin_threads gives a row lanes enough to have it in flight at once.
template <int KIND>
__global__ void __launch_bounds__(1024) k_rows_margin(const float* __restrict__ feat,
                                                     const float* __restrict__ tgt,
                                                     const float* __restrict__ x, int64_t ld,
                                                     const int32_t* __restrict__ idx, int32_t B,
                                                     int32_t M, int64_t d,
                                                     float* __restrict__ coef,
                                                     float* __restrict__ lossterm) {
    __shared__ double s_buf[16];
    const int b = blockIdx.x, i = blockIdx.y;
    const int32_t r = idx ? idx[(int64_t)i * B + b] : b;
    if (r < 0 || r >= M) {  // a sample index outside [0, M): no access, the node's gradient and loss become NaN
        if (threadIdx.x == 0) {
            coef[(int64_t)i * B + b] = __builtin_nanf("");
            lossterm[(int64_t)i * B + b] = __builtin_nanf("");
        }
        return;
    }
    const float* __restrict__ f = feat + ((int64_t)i * M + r) * d;
    const float* __restrict__ xi = x + (int64_t)i * ld;
    const float target = tgt[(int64_t)i * M + r];  // fetched with the row, not after the reduction
    double acc = 0.0;
    const int64_t d4 = d >> 2;
#pragma unroll 4
    for (int64_t c = threadIdx.x; c < d4; c += blockDim.x) {
        const v4f fv = ld_unit_cached<v4f>(f + 4 * c), xv = ld_unit_cached<v4f>(xi + 4 * c);
        acc += (double)fv.x * xv.x + (double)fv.y * xv.y + (double)fv.z * xv.z +
               (double)fv.w * xv.w;
    }
    if ((int64_t)threadIdx.x < d - 4 * d4) acc += (double)f[4 * d4 + threadIdx.x] * xi[4 * d4 + threadIdx.x];
    const double z = block_sum(acc, s_buf);
    if (threadIdx.x == 0) {
        float cf, ls;
        sample_terms<KIND>(z, target, 1.0f / (float)B, &cf, &ls);
        coef[(int64_t)i * B + b] = cf;
        lossterm[(int64_t)i * B + b] = ls;
    }
}

// Pass 1 for short rows (d <= 32): one thread per (node, sample slot); neighbouring threads
// read neighbouring rows, so a full-batch evaluation over many samples streams the
// feature array instead of spending a workgroup on every ten-element dot product.
template <int KIND>
__global__ void __launch_bounds__(256) k_rows_margin_short(const float* __restrict__ feat,
                                                           const float* __restrict__ tgt,
                                                           const float* __restrict__ x, int64_t ld,
                                                           const int32_t* __restrict__ idx, int32_t B,
                                                           int32_t M, int32_t d, int64_t pairs,
                                                           float* __restrict__ coef,
                                                           float* __restrict__ lossterm) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // i * B + b
    if (p >= pairs) return;
    const int64_t i = p / B;
    const int32_t r = idx ? idx[p] : (int32_t)(p - i * B);
    float cf = __builtin_nanf(""), ls = __builtin_nanf("");  // index outside [0, M): no access, NaN
    if (r >= 0 && r < M) {
        const float* __restrict__ f = feat + (i * M + r) * d;
        const float* __restrict__ xi = x + i * ld;
        double acc = 0.0;
        for (int c = 0; c < d; ++c) acc += (double)f[c] * xi[c];
        sample_terms<KIND>(acc, tgt[i * M + r], 1.0f / (float)B, &cf, &ls);
    }
    coef[p] = cf;
    lossterm[p] = ls;
}

// Pass 2: g = sum_b coef_b * row_b[c] for node i.  A workgroup of W wavefronts owns 64 column quads;
// the wavefronts share the samples (b = wave, wave + W, ...) and their fp64 partial sums meet in LDS in
// wavefront order, so a minibatch of 32 rows is four chains of eight dependent loads instead of one of 32
// and a small problem still fills the chip (cfg2: 1280 -> 5120 wavefronts, 15 -> 9 us).  W = 4
// wavefronts per workgroup, 16 for minibatches of 64 rows and more.
// Rows of up to 256 columns that are no whole quads keep one column a lane: such rows are bound by the chain of samples of
// a wavefront, and a quad brings four chains of fp64 sums to a lane and fewer workgroups (gradient over 8000 rows of 10 on
// 8 nodes 226 us with quads, 156 without, on 100 nodes 311 / 195; over 4000 rows of 255 on 8 nodes 154 / 103).
__host__ __device__ __forceinline__ bool accum_quads(int64_t d) { return d > 256 || (d >= 4 && d % 4 == 0); }
template <int W>
__global__ void __launch_bounds__(kWave* W) k_rows_accum(const float* __restrict__ feat,
                                                    const float* __restrict__ coef,
                                                    const int32_t* __restrict__ idx, int32_t B,
                                                    int32_t M, int64_t d,
                                                    float* __restrict__ g, int64_t ld) {
    __shared__ double s_part[W - 1][4][kWave];
    const int i = blockIdx.y;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float* __restrict__ fi = feat + (int64_t)i * M * d;
    const float* __restrict__ ci = coef + (int64_t)i * B;
    const int32_t* __restrict__ ii = idx ? idx + (int64_t)i * B : nullptr;
    float* __restrict__ gi = g + (int64_t)i * ld;
    // column quad; the last one of a ragged width is moved left and overlaps its neighbour (both store the same sums).
    const int64_t t = (int64_t)blockIdx.x * kWave + lane;
    const bool quads = accum_quads(d), on = quads ? t * 4 < d : t < d;
    const int64_t col = !quads ? t : t * 4 > d - 4 ? d - 4 : t * 4;
    double a0 = 0, a1 = 0, a2 = 0, a3 = 0;
    if (on) {
        for (int b = wave; b < B; b += W) {
            int32_t r = ii ? ii[b] : b;
            if (r < 0 || r >= M) r = 0;  // its coefficient is NaN (set by the margin pass): row 0 is only a safe address
            const double cb = ci[b];
            if (quads) {
                const v4f fv = ld_unit_cached<v4f>(fi + (int64_t)r * d + col);
                a0 += cb * fv.x;
                a1 += cb * fv.y;
                a2 += cb * fv.z;
                a3 += cb * fv.w;
            } else {
                a0 += cb * fi[(int64_t)r * d + col];
            }
        }
    }
    if (wave > 0) {
        s_part[wave - 1][0][lane] = a0;
        s_part[wave - 1][1][lane] = a1;
        s_part[wave - 1][2][lane] = a2;
        s_part[wave - 1][3][lane] = a3;
    }
    __syncthreads();
    if (wave == 0 && on) {
#pragma unroll
        for (int w = 0; w < W - 1; ++w) {
            a0 += s_part[w][0][lane];
            a1 += s_part[w][1][lane];
            a2 += s_part[w][2][lane];
            a3 += s_part[w][3][lane];
        }
        if (quads) {
            v4f out;
            out.x = (float)a0;
            out.y = (float)a1;
            out.z = (float)a2;
            out.w = (float)a3;
            st_unit<v4f>(gi + col, out);
        } else {
            gi[col] = (float)a0;
        }
    }
}

// loss[i] = sum_b lossterm[i][b]  (terms already carry the 1/B)
__global__ void __launch_bounds__(256) k_loss_sum(const float* __restrict__ lossterm, int32_t B,
                                                  float* __restrict__ loss) {
    __shared__ double s_buf[4];
    const int i = blockIdx.x;
    double acc = 0.0;
    for (int b = threadIdx.x; b < B; b += blockDim.x) acc += lossterm[(int64_t)i * B + b];
    const double t = block_sum(acc, s_buf);
    if (threadIdx.x == 0) loss[i] = (float)t;
}

// Losses alone on short rows (d <= 32): one thread per sample, the 256 rows of a workgroup staged through LDS with
// coalesced loads when they are consecutive (full batch) and read back V columns at a time; one fp64 partial sum per
// workgroup, and the node's last workgroup to end adds them in their order (many workgroups: k_loss_chunks).
// Bound: reading the rows, and an exponential and a logarithm in fp64 a sample.  Us, two launches and a column at a time
// -> this form: 100 x 8000 x 10 13.5 -> 13.0, 20 x 8000 x 10 7.2 -> 5.6, 100 x 4000 x 16 14.1 -> 8.7, 64 x 2000 x 20 8.2 -> 5.6, 50 x
// 4000 x 32 23.4 -> 8.8 (rows of 32 columns: every lane on the same LDS bank), 10 x 200 x 10 6.3 -> 3.9, 120 x 16 000 x 10 23.6 both
// (26.8 with x in LDS too).  Workgroups of several times 256 rows, the next ones loaded ahead, took 13.3 - 16 on the first.
// Columns are unrolled twofold and the form whose sums are a launch of their own knows nothing of counts: with eight columns and
// both in one kernel narrow rows lost to the start of their workgroups (540 x 33 000 x 1, 69 660 workgroups, 73.8 -> 80.4, now 74.8).
template <int KIND, int V, bool ALONG>
__global__ void __launch_bounds__(256) k_rows_loss_short(const float* __restrict__ feat, const float* __restrict__ tgt,
                                                         const float* __restrict__ x, int64_t ld,
                                                         const int32_t* __restrict__ idx, int32_t B, int32_t M,
                                                         int32_t d, int cached, double* __restrict__ partials,
                                                         uint32_t* __restrict__ left, float* __restrict__ loss) {
    extern __shared__ __align__(16) unsigned char s_raw[];  // 256 rows (full batch)
    float* __restrict__ s_rows = reinterpret_cast<float*>(s_raw);
    __shared__ double s_buf[4];
    __shared__ int s_last;
    const int64_t i = blockIdx.y;
    const int32_t b0 = blockIdx.x * 256, b = b0 + (int32_t)threadIdx.x;
    const int32_t r = idx ? (b < B ? idx[i * B + b] : 0) : b;
    const bool ok = b < B && r >= 0 && r < M;
    const float target = ok ? tgt[i * M + r] : 0.f;
    const float* __restrict__ xi = x + i * ld;
    if (!idx) {
        const float* __restrict__ rows = feat + (i * M + b0) * d;
        const int32_t count = (B - b0 < 256 ? B - b0 : 256) * d;
        if (cached) {
            for (int32_t e = threadIdx.x * 4; e + 4 <= count; e += 1024)
                *reinterpret_cast<v4f*>(s_rows + e) = ld_unit_cached<v4f>(rows + e);
        } else {
            for (int32_t e = threadIdx.x * 4; e + 4 <= count; e += 1024)
                *reinterpret_cast<v4f*>(s_rows + e) = ld_unit<v4f>(rows + e);
        }
        for (int32_t e = (count & ~3) + (int32_t)threadIdx.x; e < count; e += 256) s_rows[e] = rows[e];
        __syncthreads();
    }
    double term = 0.0;
    if (ok) {
        double z = 0.0;
        if (idx) {
            const float* __restrict__ f = feat + (i * M + r) * d;
            for (int c = 0; c < d; ++c) z += (double)f[c] * xi[c];
        } else {
            typedef float vec __attribute__((ext_vector_type(V)));
            const float* __restrict__ f = s_rows + threadIdx.x * d;
#pragma unroll 2
            for (int c = 0; c < d; c += V) {
                const vec v = *reinterpret_cast<const vec*>(f + c);
#pragma unroll
                for (int u = 0; u < V; ++u) z += (double)v[u] * xi[c + u];
            }
        }
        term = sample_loss<KIND>(z, target, 1.0f / (float)B);
    } else if (b < B) {
        term = __builtin_nan("");  // a sample index outside [0, M): no access, the node's loss becomes NaN
    }
    const double t = block_sum(term, s_buf);
    if (!ALONG) {
        if (threadIdx.x == 0) partials[i * gridDim.x + blockIdx.x] = t;  // for k_loss_chunks
        return;
    }
    if (gridDim.x == 1) {
        if (threadIdx.x == 0) loss[i] = (float)t;
        return;
    }
    if (threadIdx.x == 0) {
        // The sum past the caches that are not shared, waited for, and only then the count: a release would write back the
        // whole L2, once a workgroup (44 us instead of 11 at 100 x 8000 x 10).
        __hip_atomic_store(partials + i * gridDim.x + blockIdx.x, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        s_last = __hip_atomic_fetch_add(left + i * kLossLeftStride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    }
    __syncthreads();
    if (!s_last || threadIdx.x >= kWave) return;
    double v = 0.0;
    for (uint32_t ch = threadIdx.x; ch < gridDim.x; ch += kWave)
        v += __hip_atomic_load(partials + i * gridDim.x + ch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    v = wave_sum(v);
    if (threadIdx.x == 0) {
        loss[i] = (float)v;
        __hip_atomic_store(left + i * kLossLeftStride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // for the next launch
    }
}

__global__ void __launch_bounds__(kWave) k_loss_chunks(const double* __restrict__ partials, int32_t chunks,
                                                       float* __restrict__ loss) {
    double v = 0.0;
    for (int32_t ch = threadIdx.x; ch < chunks; ch += kWave) v += partials[(int64_t)blockIdx.x * chunks + ch];
    v = wave_sum(v);
    if (threadIdx.x == 0) loss[blockIdx.x] = (float)v;
}

// ---------------------------------------------------------------- virtual rows

// Virtual features are bound by vector issue.  Splitting off what the first two Philox rounds share between draws of a
// quad and between quads of a draw: n = 1024, d = 1M, B = 16 a new state's iteration 19.5 -> 18.2 ms (gradient and step).

// Pass 1: grid (column chunks, node).  Each lane owns column quads and keeps B
// partial margins; the node shift mu_i is generated once per quad and reused for
// all B samples.  Partial margins are combined per workgroup and stored as
// zpart[i][b][chunk]; the coefficient kernel adds the chunks in a fixed order, so the
// result does not depend on the order in which workgroups finish.
template <int BMAX>
__global__ void __launch_bounds__(256) k_virtual_margin(const float* __restrict__ x, int64_t ld,
                                                        int64_t d, const int32_t* __restrict__ idx,
                                                        int32_t B, uint32_t k0, uint32_t k1,
                                                        float mu_sigma, int64_t quads_per_block,
                                                        double* __restrict__ zpart) {
    __shared__ double s_buf[4];
    const uint32_t i = blockIdx.y;
    const int64_t d4 = (d + 3) >> 2;
    const int64_t q_begin = (int64_t)blockIdx.x * quads_per_block;
    const int64_t q_end = (q_begin + quads_per_block < d4) ? q_begin + quads_per_block : d4;
    const float* __restrict__ xi = x + (int64_t)i * ld;
    double acc[BMAX];
#pragma unroll
    for (int b = 0; b < BMAX; ++b) acc[b] = 0.0;
    for (int64_t q = q_begin + threadIdx.x; q < q_end; q += blockDim.x) {
        const int64_t c = q * 4;
        v4f xv;
        xv.x = xi[c];
        xv.y = (c + 1 < d) ? xi[c + 1] : 0.f;
        xv.z = (c + 2 < d) ? xi[c + 2] : 0.f;
        xv.w = (c + 3 < d) ? xi[c + 3] : 0.f;
        const v4f mu = mu_sigma * normals4((uint32_t)q, i, 0u, TAG_MU, k0, k1);
        const PhiloxQuad quad((uint32_t)q, TAG_FEAT, k1);
#pragma unroll
        for (int b = 0; b < BMAX; ++b) {
            if (b < B) {
                const v4f h = virtual_quad(mu, quad, i, (uint32_t)idx[(int64_t)i * B + b], k0, k1);
                // the four products of a quad are summed in fp32 (three roundings of ~6e-8 relative to
                // the quad's own terms, random in sign over the d/4 quads of a margin), the quads in fp64:
                // 6 issue slots per sample where four conversions and four fp64 operations took 12
                const float t = h.x * xv.x + h.y * xv.y + h.z * xv.z + h.w * xv.w;
                acc[b] += (double)t;
            }
        }
    }
#pragma unroll
    for (int b = 0; b < BMAX; ++b) {
        if (b < B) {
            const double t = block_sum(acc[b], s_buf);
            if (threadIdx.x == 0) zpart[((int64_t)i * B + b) * gridDim.x + blockIdx.x] = t;
            __syncthreads();
        }
    }
}

__global__ void k_virtual_coef(const double* __restrict__ zpart, int32_t chunks, const float* __restrict__ y,
                               const int32_t* __restrict__ idx, int32_t B, int32_t M, int32_t n,
                               float* __restrict__ coef, float* __restrict__ lossterm) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)n * B) return;
    double z = 0.0;
    for (int32_t ch = 0; ch < chunks; ++ch) z += zpart[t * chunks + ch];
    const int i = (int)(t / B);
    float cf, ls;
    const int32_t r = idx[t];
    if (r < 0 || r >= M) {  // label index outside [0, M): no access, NaN marks the node's gradient and loss
        coef[t] = __builtin_nanf("");
        lossterm[t] = __builtin_nanf("");
        return;
    }
    sample_terms<PROB_LOGREG>(z, y[(int64_t)i * M + r], 1.0f / (float)B, &cf, &ls);
    coef[t] = cf;
    lossterm[t] = ls;
}

// Pass 2: one lane per column quad of node i, features regenerated.
template <int BMAX>
__global__ void __launch_bounds__(256) k_virtual_accum(const float* __restrict__ coef,
                                                       const int32_t* __restrict__ idx, int32_t B,
                                                       int64_t d, uint32_t k0, uint32_t k1,
                                                       float mu_sigma, int vec_ok,
                                                       float* __restrict__ g, int64_t ld) {
    const uint32_t i = blockIdx.y;
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t c = q * 4;
    if (c >= d) return;
    const v4f mu = mu_sigma * normals4((uint32_t)q, i, 0u, TAG_MU, k0, k1);
    const PhiloxQuad quad((uint32_t)q, TAG_FEAT, k1);
    // g = sum_b coef_b h_b over at most 32 samples of similar size: fp32 fused multiply-adds (error
    // <= 32 x 6e-8 of sum |coef_b h_b|, far inside 1e-5 of the row's scale).  A sample whose
    // coefficient is exactly zero adds exactly nothing and its features are not regenerated:
    // once the margins of a logistic problem are large, sigma(-y z) underflows to 0 for every
    // correctly classified sample.  (NaN coefficients, which mark invalid sample indices, are
    // not zero and poison the row as before.)  The coefficient is the same for the whole
    // workgroup, so the test is a scalar branch.
    v4f a = v4f(0.f);
#pragma unroll
    for (int b = 0; b < BMAX; ++b) {
        if (b < B) {
            const float cb = coef[(int64_t)i * B + b];
            if (cb != 0.f) {
                const v4f h = virtual_quad(mu, quad, i, (uint32_t)idx[(int64_t)i * B + b], k0, k1);
                a += cb * h;
            }
        }
    }
    const float a0 = a.x, a1 = a.y, a2 = a.z, a3 = a.w;
    float* row = g + (int64_t)i * ld;
    if (vec_ok && c + 3 < d) {
        v4f out;
        out.x = (float)a0;
        out.y = (float)a1;
        out.z = (float)a2;
        out.w = (float)a3;
        // streamed past the caches: the fused step that follows reads g once, and dirty lines left behind
        // here would be written back while that step is already being timed against its pacing clock
        __builtin_nontemporal_store(out, reinterpret_cast<v4f*>(row + c));
    } else {
        row[c] = (float)a0;
        if (c + 1 < d) row[c + 1] = (float)a1;
        if (c + 2 < d) row[c + 2] = (float)a2;
        if (c + 3 < d) row[c + 3] = (float)a3;
    }
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }


// ---------------------------------------------------------------- small problems: whole iterations in one workgroup

// When the n x d state and one minibatch of work fit in a single workgroup, T whole
// iterations of Algorithm 1 - stochastic gradients at the current rows, momentum and local
// update, gossip step or global average, and the consensus distance - run inside ONE launch
// with X, M and x^(k+1/2) held in LDS.  Such problems (the logistic simulation of Sec. 5.1:
// n <= 100 nodes, d = 10) are otherwise bound by the latency of three to five dependent
// kernel launches per iteration; here an iteration costs a few workgroup barriers and one
// dependent pair of global reads (sample index, then feature row).
// The arithmetic follows the large kernels: margins and gradient sums accumulate in fp64,
// state and x^(k+1/2) are fp32, the mean of a global average is one value broadcast to
// all rows.
struct SmallArgs {
    const float* x;  // n x ld, the iterates before the first iteration of this launch
    float* x_out;    // n x ld, receives the iterates after the last one (may be the same array)
    float* m;  // n x ld momentum buffers (unused when mu = 0)
    float* g;  // n x ld, receives the gradients of the last iteration
    int64_t ld;
    int32_t n, d;
    const float* feat;  // n x M x d
    const float* tgt;   // n x M
    int32_t M;
    const int32_t* idx;  // T x n x B sample indices, or NULL = every node's whole data set (B = M)
    int32_t B;
    int32_t topo;
    int64_t H, k0;
    int32_t T;
    float mu;
    const int32_t* wptr;  // W in compressed-row form for the sparse-W topologies
    const int32_t* wcol;
    const float* wval;
    double* trace;  // trace[k] = consensus distance after iteration k, for k < trace_cap
    int64_t trace_cap;
    int32_t nnz;          // entries of W
    int32_t worker_waves;  // k_node_run: wavefronts that hold nodes (the others take the trace)
    float lr[kSmallRunMaxIters];  // step size of each iteration of this launch
    int32_t shift[kSmallRunMaxIters];  // its one-peer offset; -1 = it ends in a global average
};

template <int KIND, int MOM>
__global__ void __launch_bounds__(kSmallRunThreads) k_small_run(const SmallArgs a) {
    extern __shared__ __align__(16) unsigned char s_raw[];
    const int n = a.n, d = a.d, nd = n * d, B = a.B;
    double* __restrict__ sMean = reinterpret_cast<double*>(s_raw);  // d column means
    double* __restrict__ sRed = sMean + d;                          // two sets of one slot per wavefront
    double* __restrict__ sZ = sRed + 2 * (kSmallRunThreads / kWave);  // n x B margins
    float* __restrict__ sX = reinterpret_cast<float*>(sZ + n * a.B);
    float* __restrict__ sY = sX + nd;
    float* __restrict__ sM = sY + nd;               // MOM only
    float* __restrict__ sC = sM + (MOM ? nd : 0);   // n x B per-sample coefficients
    int32_t* __restrict__ sIdx = reinterpret_cast<int32_t*>(sC + n * B);  // n x B sample rows of the iteration
    const int G = d <= 16 ? 16 : d <= 32 ? 32 : kWave;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6, nw = blockDim.x >> 6;
    const float invB = 1.0f / (float)B;
    const float third = 1.0f / 3.0f;
    const double inv_n = 1.0 / (double)n;
    int tau = 0;
    while ((1LL << tau) < n) ++tau;
    if (tau < 1) tau = 1;

    for (int e = tid; e < nd; e += blockDim.x) {
        const int i = e / d, c = e - i * d;
        sX[e] = a.x[(int64_t)i * a.ld + c];
        if (MOM) sM[e] = a.m[(int64_t)i * a.ld + c];
    }
    __syncthreads();

    // column means of src (n x d in LDS) into sMean: one wavefront per column, lanes over rows
    auto column_means = [&](const float* src) {
        for (int c = wave; c < d; c += nw) {
            double s = 0.0;
            for (int i = lane; i < n; i += kWave) s += (double)src[i * d + c];
            s = group_sum_last(s, kWave);
            if (lane == 0) sMean[c] = s * inv_n;
        }
        __syncthreads();
    };

    // Short rows (d <= G) whose pairs fit a few passes are software-pipelined across iterations:
    // lane lg of group tid / G keeps, for pair p = tid / G + j * PP, the sample row, the label and
    // feature value number lg of the NEXT iteration in registers.
    const int npairs = n * B, PP = blockDim.x / G, lg = tid & (G - 1);
    const bool piped = d <= G && npairs <= kSmallRunPasses * PP;
    auto fetch_row = [&](int tt, int j) -> int32_t {  // validated sample row of pair j in iteration tt, or -1
        const int p = tid / G + j * PP;
        if (tt >= a.T || p >= npairs) return -1;
        const int32_t r = a.idx ? a.idx[(int64_t)tt * npairs + p] : p % B;
        return (r >= 0 && r < a.M) ? r : -1;
    };
    auto fetch_sample = [&](int j, int32_t r, float& f, float& y) {
        f = 0.f;
        y = 0.f;
        if (r >= 0) {
            const int i = (tid / G + j * PP) / B;
            if (lg < d) f = a.feat[((int64_t)i * a.M + r) * d + lg];
            y = a.tgt[(int64_t)i * a.M + r];
        }
    };
    // The coefficient of a sample needs a double-precision exponential: with one pass of lane
    // groups the group's last lane computes it on the spot; with several passes the margins
    // go to LDS first and one thread per pair computes them all at once.
    const bool one_pass = npairs <= PP;
    auto coefficient = [&](double z, float y, int32_t r) -> float {
        float cf = __builtin_nanf(""), ls;  // no valid sample: the node's gradient becomes NaN
        if (r >= 0) sample_terms<KIND>(z, y, invB, &cf, &ls);
        return cf;
    };
    auto coefficients_from_margins = [&]() {
        for (int p = tid; p < npairs; p += blockDim.x) sC[p] = coefficient(sZ[p], sC[p], sIdx[p]);
        __syncthreads();
    };
    int32_t rcur[kSmallRunPasses], rnext[kSmallRunPasses];
    float fcur[kSmallRunPasses], ycur[kSmallRunPasses];
    if (piped) {
#pragma unroll
        for (int j = 0; j < kSmallRunPasses; ++j) {
            rcur[j] = rnext[j] = -1;
            fcur[j] = ycur[j] = 0.f;
            if (j * PP >= npairs) continue;
            rcur[j] = fetch_row(0, j);
            fetch_sample(j, rcur[j], fcur[j], ycur[j]);
            rnext[j] = fetch_row(1, j);
        }
    }

    for (int t = 0; t < a.T; ++t) {
        const int64_t k = a.k0 + t;
        const float lr = a.lr[t];
        const int32_t* __restrict__ idx_t = a.idx ? a.idx + (int64_t)t * npairs : nullptr;

        if (piped) {
            // The rows, labels and feature values of this iteration were fetched during the one
            // before (they do not depend on x); only the products with the current x are left.
#pragma unroll
            for (int j = 0; j < kSmallRunPasses; ++j) {
                if (j * PP >= npairs) break;  // uniform: no pair left for this pass
                const int p = tid / G + j * PP;
                const bool have = p < npairs;
                const int i = have ? p / B : 0;
                double acc = (have && rcur[j] >= 0 && lg < d) ? (double)fcur[j] * sX[i * d + lg] : 0.0;
                acc = group_sum_last(acc, G);
                if (have && lg == G - 1) {
                    sIdx[p] = rcur[j];
                    if (one_pass) {
                        sC[p] = coefficient(acc, ycur[j], rcur[j]);
                    } else {  // margin and label now, the coefficient from one thread per pair below
                        sZ[p] = acc;
                        sC[p] = ycur[j];
                    }
                }
            }
            // fetch for the next iteration and the sample rows of the one after it
#pragma unroll
            for (int j = 0; j < kSmallRunPasses; ++j) {
                if (j * PP >= npairs) break;
                rcur[j] = rnext[j];
                fetch_sample(j, rcur[j], fcur[j], ycur[j]);
                rnext[j] = fetch_row(t + 2, j);
            }
            __syncthreads();
            if (!one_pass) coefficients_from_margins();
        } else {
            // sample rows of this iteration into LDS (-1 = index outside [0, M))
            for (int p = tid; p < npairs; p += blockDim.x) {
                const int32_t r = idx_t ? idx_t[p] : p % B;
                sIdx[p] = (r >= 0 && r < a.M) ? r : -1;
            }
            __syncthreads();

            // per-sample coefficients from the margins <h, x_i>: a group of G lanes per (node,
            // sample slot), G the power of two that covers d (16..64)
            for (int p0 = 0; p0 < npairs; p0 += PP) {
                const int p = p0 + tid / G;
                const bool have = p < npairs;
                const int i = have ? p / B : 0;
                const int32_t r = have ? sIdx[p] : -1;
                double acc = 0.0;
                if (r >= 0) {
                    const float* __restrict__ f = a.feat + ((int64_t)i * a.M + r) * d;
                    int c = lg;
                    for (; c + 3 * G < d; c += 4 * G) {  // four loads in flight
                        const float f0 = f[c], f1 = f[c + G], f2 = f[c + 2 * G], f3 = f[c + 3 * G];
                        acc += (double)f0 * sX[i * d + c] + (double)f1 * sX[i * d + c + G] +
                               (double)f2 * sX[i * d + c + 2 * G] + (double)f3 * sX[i * d + c + 3 * G];
                    }
                    for (; c < d; c += G) acc += (double)f[c] * sX[i * d + c];
                }
                acc = group_sum_last(acc, G);
                if (have && lg == G - 1) {
                    const float y = r >= 0 ? a.tgt[(int64_t)i * a.M + r] : 0.f;
                    if (one_pass) {
                        sC[p] = coefficient(acc, y, r);
                    } else {
                        sZ[p] = acc;
                        sC[p] = y;
                    }
                }
            }
            __syncthreads();
            if (!one_pass) coefficients_from_margins();
        }

        // gradient, momentum and local update, one element per thread and pass
        for (int e = tid; e < nd; e += blockDim.x) {
            const int i = e / d, c = e - i * d;
            double acc = 0.0;
            for (int b = 0; b < B; ++b) {
                int32_t r = sIdx[i * B + b];
                if (r < 0) r = 0;  // its coefficient is NaN: row 0 is only a safe address
                acc += (double)sC[i * B + b] * a.feat[((int64_t)i * a.M + r) * d + c];
            }
            const float gv = (float)acc;
            float mom = gv;
            if (MOM) {
                mom = a.mu * sM[e] + gv;
                sM[e] = mom;
            }
            sY[e] = MOM == 2 ? sX[e] - lr * (gv + a.mu * mom) : sX[e] - lr * mom;
            if (t == a.T - 1) a.g[(int64_t)i * a.ld + c] = gv;
        }
        __syncthreads();

        // gossip step or global average (Algorithm 1: the mean iff mod(k+1, H) = 0)
        const bool global = a.topo == GPGA_TOPO_FULL || (a.H > 0 && (k + 1) % a.H == 0);
        if (n > 1 && global) column_means(sY);
        const int S = (int)((1LL << (int)(k % tau)) % n);  // one-peer offset of this iteration
        for (int e = tid; e < nd; e += blockDim.x) {
            const int i = e / d, c = e - i * d;
            float v = sY[e];
            if (n > 1) {
                if (global) {
                    v = (float)sMean[c];
                } else if (a.topo == GPGA_TOPO_RING) {
                    const int im = i == 0 ? n - 1 : i - 1, ip = i == n - 1 ? 0 : i + 1;
                    v = (sY[im * d + c] + v + sY[ip * d + c]) * third;
                } else if (a.topo == GPGA_TOPO_EXPO1) {
                    if (S) v = (v + sY[((i + S) % n) * d + c]) * 0.5f;
                } else if (a.topo != GPGA_TOPO_NONE) {
                    float acc = 0.f;
                    for (int p = a.wptr[i]; p < a.wptr[i + 1]; ++p) acc += a.wval[p] * sY[a.wcol[p] * d + c];
                    v = acc;
                }
            }
            sX[e] = v;
        }
        __syncthreads();

        // consensus distance ||X - 1 xbar^T||_F of the new iterates (exactly 0 after an average):
        // a wavefront takes whole columns, lanes over the rows, so the column mean and the
        // squared deviations from it need no exchange with other wavefronts
        if (a.trace && k < a.trace_cap) {
            double part = 0.0;
            if (n > 1 && !global) {
                for (int c = wave; c < d; c += nw) {
                    double s1 = 0.0;
                    for (int i = lane; i < n; i += kWave) s1 += (double)sX[i * d + c];
                    const double mean = group_sum_last(s1, kWave) * inv_n;
                    for (int i = lane; i < n; i += kWave) {
                        const double dv = (double)sX[i * d + c] - mean;
                        part += dv * dv;
                    }
                }
            }
            part = group_sum_last(part, kWave);
            double* __restrict__ slots = sRed + (t & 1) * (kSmallRunThreads / kWave);  // the other half next time
            if (lane == 0) slots[wave] = part;
            __syncthreads();
            if (tid == 0) {
                double tot = 0.0;
                for (int w = 0; w < nw; ++w) tot += slots[w];
                a.trace[k] = sqrt(tot);
            }
        }
    }

    for (int e = tid; e < nd; e += blockDim.x) {
        const int i = e / d, c = e - i * d;
        a.x_out[(int64_t)i * a.ld + c] = sX[e];
        if (MOM) a.m[(int64_t)i * a.ld + c] = sM[e];
    }
}

// The same trajectories for short rows (d <= 20), up to four samples a node and iteration and up to 128 nodes - the
// shapes of Sec. 5.1.  Bound: the latency of one iteration's dependent chain (margin, double-precision sigmoid,
// update, exchange), so everything off that chain is taken off it:
//  * four neighbouring lanes own a node, C columns each; x, m and the sample's row stay in registers, the margin is C
//    multiply-adds and two lane exchanges within the quad, lane b of the quad evaluates the sigmoid of sample b;
//  * rows and labels are fetched three iterations ahead, two with several samples a node, and their row numbers as
//    many again (both lie in HBM: about 1 us away, more than an iteration takes), and the gradient uses the registers the margin used;
//  * a lane's columns are neighbours in its row and come in one wide load (the last lanes' overlap the one before): the loads
//    are scattered, some 20 lines each, and a compute unit takes one line a clock.  50 iterations and the five launches of a
//    loss evaluation (16 us), 100 nodes, us with a load a column -> wide: d = 10, one sample 63.4 -> 63.0, two 82 -> 67, four
//    133 -> 76; d = 20 75 -> 70, 117 -> 90, 209 -> 109.  Two lanes a node (half the wavefronts, one sigmoid less a SIMD, but
//    registers for the double) took 66, 74, 93 and 74, 94, 123;
//  * x^(k+1/2) is exchanged through two LDS arrays in turn, so an iteration has ONE barrier;
//  * the consensus distance of iteration t is formed by wavefronts of its own while the nodes do iteration
//    t + 1: shifted sums per column (row 0 is the shift), then the columns one iteration later.  They share the SIMDs with the
//    nodes, so their reads go ahead four rows at a time and rows of lanes are added by exchanges of registers (one row at a
//    time and through LDS 100 x 10 63.4 -> 56.2 us, 64 x 20 65.3 -> 54.9; one, two or all rows by a runtime count 58 - 66).
// Measured with the trace, 50 iterations, one sample a node: n = 100, d = 10 231 us in k_small_run -> 50.5 us here
// (71 us with loads the compiler could not count).  Rows of 13 to 20 columns with three or four samples spill 10 to 51 registers
// a lane, logistic ones with momentum and one sample 1 to 3; the former still take a seventh of k_small_run's time (n = 128, d = 20
// 18.9 us an iteration, 2.3 here).
__device__ __forceinline__ double quad_sum(double v) {
    v += dpp_f64<0xB1>(v);  // quad_perm [1,0,3,2]
    v += dpp_f64<0x4E>(v);  // quad_perm [2,3,0,1]
    return v;
}
template <int B>
__device__ __forceinline__ float quad_bcast(float v) {  // the value of lane B of the quad
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), B * 0x55, 0xf, 0xf, true));
}

template <int KIND, int MOM, int C, int NB, int TW>
__global__ void __launch_bounds__(kNodeMaxNodes * kNodeLanes + kWave * node_trace_waves(NB)) k_node_run(const SmallArgs a) {
    constexpr int DP = kNodeLanes * C;            // padded row
    constexpr int LG = DP <= 16 ? 16 : 32;        // lanes over columns in the trace wavefronts
    constexpr int kNodeTraceWaves = TW;
    constexpr int kNodeDepth = NB == 1 ? 3 : 2;   // iterations the samples are fetched ahead
    extern __shared__ __align__(16) unsigned char s_raw[];
    const int n = a.n, d = a.d, B = a.B;
    double* __restrict__ sMean = reinterpret_cast<double*>(s_raw);      // [DP]
    double* __restrict__ sP = sMean + DP;                               // [2][trace waves][2][DP]
    float* __restrict__ sY = reinterpret_cast<float*>(sP + 2 * kNodeTraceWaves * 2 * DP);  // [2][n][DP]
    float* __restrict__ sX = sY + 2 * n * DP;                           // [2][n][DP]
    int32_t* __restrict__ sCol = reinterpret_cast<int32_t*>(sX + 2 * n * DP);  // W: [nnz] columns, [nnz] weights
    float* __restrict__ sVal = reinterpret_cast<float*>(sCol + a.nnz);
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
    const bool worker = wave < a.worker_waves;
    const int tw = wave - a.worker_waves;         // trace wavefront
    const int i = tid / kNodeLanes, l = tid & (kNodeLanes - 1);
    const bool have = worker && i < n;
    const float invB = 1.0f / (float)B, third = 1.0f / 3.0f, mu = a.mu;
    const double inv_n = 1.0 / (double)n;
    const bool sparse = a.topo == GPGA_TOPO_GRID || a.topo == GPGA_TOPO_EXPO || a.topo == GPGA_TOPO_CUSTOM;

    // Columns of a lane: C neighbouring ones from `first` on, one wide load; those that the lane before has too are padding.
    const int first = l * C + C <= d ? l * C : d - C;
    float x[C], m[C];
    bool real[C];                                 // the padding stays 0
    int w0 = 0, w1 = 0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        real[c] = have && first + c >= l * C;
        x[c] = real[c] ? a.x[(int64_t)i * a.ld + first + c] : 0.f;
        m[c] = MOM && real[c] ? a.m[(int64_t)i * a.ld + first + c] : 0.f;
    }
    if (sparse) {
        for (int p = tid; p < a.nnz; p += blockDim.x) {
            sCol[p] = a.wcol[p];
            sVal[p] = a.wval[p];
        }
        if (have) {
            w0 = a.wptr[i];
            w1 = a.wptr[i + 1];
        }
    }

    // All loads of the pipeline are unconditional (clamped addresses, values checked when used): a load under a
    // condition would make every later wait one for all loads in flight.
    struct Slot {
        float f[NB][C];
        float y;          // label of this lane's sample (sample l of the node)
        int32_t r;        // its row as given
        int32_t rows[NB]; // row numbers, kNodeDepth iterations ahead of f
    };
    Slot slots[kNodeDepth];
    const int in = i < n ? i : n - 1;
    const char* __restrict__ feat_i = reinterpret_cast<const char*>(a.feat + (int64_t)in * a.M * d + first);
    const uint32_t row_bytes = 4u * (uint32_t)d;
    const float* __restrict__ tgt_i = a.tgt + (int64_t)in * a.M;
    const int32_t* __restrict__ idx = a.idx ? a.idx : reinterpret_cast<const int32_t*>(a.tgt);  // full batch: not used
    auto valid = [&](int32_t r) { return (uint32_t)r < (uint32_t)a.M; };
    const int64_t idx_bytes = a.idx ? 4ll * n * B : 0;
    uint32_t pick[NB];                            // a lane's offsets in a table of row numbers
#pragma unroll
    for (int b = 0; b < NB; ++b) pick[b] = a.idx ? 4u * (uint32_t)(in * B + (b < B ? b : 0)) : 0u;
    auto fetch_rows = [&](Slot& s, int t) {
        const char* __restrict__ p = reinterpret_cast<const char*>(idx) + (t < a.T ? t : a.T - 1) * idx_bytes;
#pragma unroll
        for (int b = 0; b < NB; ++b) s.rows[b] = *reinterpret_cast<const int32_t*>(p + pick[b]);
    };
    auto fetch = [&](Slot& s) {
        if (!a.idx) {
#pragma unroll
            for (int b = 0; b < NB; ++b) s.rows[b] = b < B ? b : 0;
        }
        s.r = s.rows[0];
#pragma unroll
        for (int b = 1; b < NB; ++b) s.r = l == b ? s.rows[b] : s.r;
        s.y = tgt_i[valid(s.r) ? (uint32_t)s.r : 0u];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const uint32_t r = valid(s.rows[b]) ? (uint32_t)s.rows[b] : 0u;
            const float* __restrict__ f = reinterpret_cast<const float*>(feat_i + (uint64_t)r * row_bytes);
#pragma unroll
            for (int c = 0; c < C; ++c) s.f[b][c] = f[c];
        }
    };
    if (worker) {
#pragma unroll
        for (int s = 0; s < kNodeDepth; ++s) fetch_rows(slots[s], s);
#pragma unroll
        for (int s = 0; s < kNodeDepth; ++s) fetch(slots[s]);
#pragma unroll
        for (int s = 0; s < kNodeDepth; ++s) fetch_rows(slots[s], kNodeDepth + s);
    }

    auto traced = [&](int t) { return a.trace && t >= 0 && t < a.T && a.k0 + t < a.trace_cap; };
    // shifted sums of iteration t's rows, this wavefront's share of them; after an average all rows have the same bits,
    // whatever they are, and none is looked at
    auto trace_columns = [&](int t, bool average) {
        const int c = lane & (LG - 1), group = tw * (kWave / LG) + lane / LG;
        double s1 = 0.0, s2 = 0.0;
        if (c < DP) {
            const float* __restrict__ X = sX + (t & 1) * n * DP + c;
            const double ref = X[0];
            constexpr int step = kNodeTraceWaves * (kWave / LG);
            for (int r = group; r < (average ? 0 : n); r += kNodeTraceRows * step) {
                float v[kNodeTraceRows];
#pragma unroll
                for (int u = 0; u < kNodeTraceRows; ++u) v[u] = X[(r + u * step < n ? r + u * step : 0) * DP];  // row 0 adds nothing
#pragma unroll
                for (int u = 0; u < kNodeTraceRows; ++u) {
                    const double dv = (double)v[u] - ref;
                    s1 += dv;
                    s2 += dv * dv;
                }
            }
        }
        if (LG == 16) {
            s1 = swap_add(s1, s1, false);
            s2 = swap_add(s2, s2, false);
        }
        s1 = swap_add(s1, s2, true);
        if ((lane & 31) < DP) sP[((t & 1) * kNodeTraceWaves + tw) * 2 * DP + (lane >> 5) * DP + (lane & 31)] = s1;
    };
    auto trace_entry = [&](int t) {
        double ss = 0.0;
        if (lane < DP) {
            double s1 = 0.0, s2 = 0.0;
            const double* __restrict__ p = sP + (t & 1) * kNodeTraceWaves * 2 * DP + lane;
#pragma unroll
            for (int w = 0; w < kNodeTraceWaves; ++w) {
                s1 += p[w * 2 * DP];
                s2 += p[w * 2 * DP + DP];
            }
            const double v = s2 - s1 * s1 * inv_n;
            ss = (v > 0.0 ? v : 0.0) + 0.0 * s1;  // the last term: a state that is not finite has no distance
        }
        ss = group_sum_last(ss, kWave);
        if (lane == 0) a.trace[a.k0 + t] = sqrt(ss);
    };

    // Every wavefront takes columns, lanes over rows; a lane with fewer than C of its own has them behind its padding.
    const int whole = d - d % C, gap = C - d % C;
    auto column_means = [&](int t) {
        const float* __restrict__ Y = sY + (t & 1) * n * DP;
        for (int k = wave; k < d; k += nw) {
            const int c = k < whole ? k : k + gap;
            double v = 0.0;
            for (int r = lane; r < n; r += kWave) v += (double)Y[r * DP + c];
            v = group_sum_last(v, kWave);
            if (lane == 0) sMean[c] = v * inv_n;
        }
        __syncthreads();
    };
    float g[C];                                   // gradient of the latest iteration
#pragma unroll
    for (int c = 0; c < C; ++c) g[c] = 0.f;
    float lr = a.lr[0];                           // of the coming iteration, read ahead of its use
    int shift_of = a.shift[0];
    auto iteration = [&](int t, Slot& s) {
        const int shift = shift_of;
        const int tn = t + 1 < a.T ? t + 1 : t;
        float lr_next = a.lr[tn];
        int shift_next = a.shift[tn];
        float y[C];
        float* __restrict__ Y = sY + (t & 1) * n * DP;
        double z = 0.0;                           // margin of this lane's sample
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            double acc = 0.0;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                // padding: an infinite column of another lane times x = 0 would be no number
                const float f = real[c] ? s.f[b][c] : 0.f;
                acc += (double)f * (double)x[c];
            }
            acc = quad_sum(acc);
            if (b == 0 || l == b) z = acc;
        }
        float cf = __builtin_nanf(""), ls;        // no valid sample: the node's gradient becomes NaN
        if (valid(s.r)) sample_terms<KIND>(z, s.y, invB, &cf, &ls);
        asm volatile("" : "+s"(lr_next), "+s"(shift_next));
        const float cb[4] = {quad_bcast<0>(cf), quad_bcast<1>(cf), quad_bcast<2>(cf), quad_bcast<3>(cf)};
#pragma unroll
        for (int c = 0; c < C; ++c) {
            double acc = 0.0;
#pragma unroll
            for (int b = 0; b < NB; ++b)
                if (b < B) acc += (double)cb[b] * (double)s.f[b][c];
            g[c] = real[c] ? (float)acc : 0.f;
            float mom = g[c];
            if (MOM) m[c] = mom = mu * m[c] + g[c];
            y[c] = MOM == 2 ? x[c] - lr * (g[c] + mu * mom) : x[c] - lr * mom;
        }
        if (have) {
#pragma unroll
            for (int c = 0; c < C; ++c) Y[i * DP + l * C + c] = y[c];
        }
        fetch(s);                                 // for iteration t + kNodeDepth
        fetch_rows(s, t + 2 * kNodeDepth);
        lr = lr_next;
        shift_of = shift_next;
        __syncthreads();
        if (shift < 0) column_means(t);
        if (!have) return;
        const float* __restrict__ Yl = Y + l * C;
        if (n == 1) {
#pragma unroll
            for (int c = 0; c < C; ++c) x[c] = y[c];
        } else if (shift < 0) {
#pragma unroll
            for (int c = 0; c < C; ++c) x[c] = real[c] ? (float)sMean[l * C + c] : 0.f;
        } else if (a.topo == GPGA_TOPO_RING) {
            const float* __restrict__ lo = Yl + (i == 0 ? n - 1 : i - 1) * DP;
            const float* __restrict__ hi = Yl + (i == n - 1 ? 0 : i + 1) * DP;
#pragma unroll
            for (int c = 0; c < C; ++c) x[c] = (lo[c] + y[c] + hi[c]) * third;
        } else if (a.topo == GPGA_TOPO_EXPO1) {
            const float* __restrict__ peer = Yl + (i + shift >= n ? i + shift - n : i + shift) * DP;
#pragma unroll
            for (int c = 0; c < C; ++c) x[c] = shift ? (y[c] + peer[c]) * 0.5f : y[c];
        } else if (sparse) {
#pragma unroll
            for (int c = 0; c < C; ++c) x[c] = 0.f;
            for (int p = w0; p < w1; ++p) {
                const float* __restrict__ row = Yl + sCol[p] * DP;
                const float wt = sVal[p];
#pragma unroll
                for (int c = 0; c < C; ++c) x[c] += wt * row[c];
            }
        } else {
#pragma unroll
            for (int c = 0; c < C; ++c) x[c] = y[c];
        }
        if (a.trace) {
            float* __restrict__ X = sX + (t & 1) * n * DP + i * DP + l * C;
#pragma unroll
            for (int c = 0; c < C; ++c) X[c] = x[c];
        }
    };
    bool average = false;                         // trace wavefronts: whether the latest iteration ended in one
    // The two kinds of wavefront run loops of their own that meet at the same barriers: one loop with both roles in
    // it, or one that leaves in the middle of a round, blurs the count of loads in flight.
    if (worker) {
        int t = 0;
        for (; t + kNodeDepth <= a.T; t += kNodeDepth) {
#pragma unroll
            for (int s = 0; s < kNodeDepth; ++s) iteration(t + s, slots[s]);
        }
#pragma unroll
        for (int s = 0; s < kNodeDepth - 1; ++s)
            if (t + s < a.T) iteration(t + s, slots[s]);
    } else {
        for (int t = 0; t < a.T; ++t) {
            __syncthreads();
            const bool now = a.shift[t] < 0;
            if (now) column_means(t);
            if (traced(t - 1)) trace_columns(t - 1, average);
            average = now || n == 1;
            if (tw == 0 && traced(t - 2)) trace_entry(t - 2);
        }
    }
    __syncthreads();
    if (!worker) {
        if (traced(a.T - 1)) trace_columns(a.T - 1, average);
        if (tw == 0 && traced(a.T - 2)) trace_entry(a.T - 2);
    }
    __syncthreads();
    if (!worker && tw == 0 && traced(a.T - 1)) trace_entry(a.T - 1);
#pragma unroll
    for (int c = 0; c < C; ++c) {
        if (real[c]) {
            a.x_out[(int64_t)i * a.ld + first + c] = x[c];
            a.g[(int64_t)i * a.ld + first + c] = g[c];
            if (MOM) a.m[(int64_t)i * a.ld + first + c] = m[c];
        }
    }
}

size_t small_run_lds(const gpga_ctx* c, int32_t Beff) {
    const size_t nd = (size_t)c->n * (size_t)c->d;
    return ((size_t)c->d + 2 * (kSmallRunThreads / kWave) + (size_t)c->n * (size_t)Beff) * sizeof(double) +
           ((c->mu != 0.f ? 3 : 2) * nd + 2 * (size_t)c->n * (size_t)Beff) * sizeof(float);
}

}  // namespace

hipError_t launch_synth_grad(const gpga_ctx* c) {
    const int64_t d4 = (c->d + 3) / 4;
    dim3 grid((unsigned)((d4 + 255) / 256), (unsigned)c->n), block(256);
    const int vec_ok = aligned16(c->g) && (c->ld % 4 == 0);
    hipLaunchKernelGGL(k_synth_grad, grid, block, 0, c->stream, c->g, c->ld, c->d,
                       (uint32_t)(c->seed & 0xffffffffu), (uint32_t)(c->seed >> 32),
                       (uint32_t)(c->k & 0xffffffff), c->grad_sigma, vec_ok);
    return hipGetLastError();
}

// Lanes a row of the margin pass: one quad each up to 256 lanes; more, of five quads each, where there are too few rows
// to fill the chip (1024 rows of 10 000: 14.0 us with 256 lanes, 12.7 with 512).
static int rows_margin_threads(int64_t d, int64_t rows) {
    int t = kWave;
    while (t < 256 && d / 4 > t) t *= 2;
    while (t < 1024 && d / 4 > (int64_t)5 * t && rows * t < 256 * 2048) t *= 2;
    return t;
}

// Pass 1: coefficients and loss terms of every sample, and the losses if they are wanted.
hipError_t launch_rows_margin(const gpga_ctx* c, const int32_t* idx, int32_t B, float* loss_out) {
    const int32_t Beff = idx ? B : c->M;
    float* coef = c->coef;
    float* lossterm = c->coef + (size_t)c->n * Beff;
    dim3 grid1((unsigned)Beff, (unsigned)c->n), block(256), block1(rows_margin_threads(c->d, (int64_t)c->n * Beff));
    const int64_t pairs = (int64_t)c->n * Beff;
    if (c->d <= 32 && (pairs + 255) / 256 <= 0x7fffffffLL) {
        const dim3 grid_short((unsigned)((pairs + 255) / 256));
        if (c->problem == PROB_LSQ) {
            hipLaunchKernelGGL((k_rows_margin_short<PROB_LSQ>), grid_short, block, 0, c->stream, c->feat, c->tgt,
                               c->x, c->ld, idx, Beff, c->M, (int32_t)c->d, pairs, coef, lossterm);
        } else {
            hipLaunchKernelGGL((k_rows_margin_short<PROB_LOGREG>), grid_short, block, 0, c->stream, c->feat, c->tgt,
                               c->x, c->ld, idx, Beff, c->M, (int32_t)c->d, pairs, coef, lossterm);
        }
    } else if (c->problem == PROB_LSQ) {
        hipLaunchKernelGGL((k_rows_margin<PROB_LSQ>), grid1, block1, 0, c->stream, c->feat, c->tgt,
                           c->x, c->ld, idx, Beff, c->M, c->d, coef, lossterm);
    } else {
        hipLaunchKernelGGL((k_rows_margin<PROB_LOGREG>), grid1, block1, 0, c->stream, c->feat,
                           c->tgt, c->x, c->ld, idx, Beff, c->M, c->d, coef, lossterm);
    }
    if (loss_out) {
        hipLaunchKernelGGL(k_loss_sum, dim3((unsigned)c->n), block, 0, c->stream, lossterm, Beff, loss_out);
    }
    return hipGetLastError();
}

// Data that the L2s hold is read through them (100 x 8000 x 10, 32 MB, 13.3 us, past them 13.8; 64 x 2000 x 20 6.7 / 8.4; 120 x
// 8000 x 20, 77 MB, 23.0 / 22.2).
constexpr int64_t kLossCachedBytes = 32 << 20;
// The sums of a node's workgroups ride along (a launch less, 3 us) while their counts on one word, some 15 ns each, take less
// time, and while most workgroups are resident at once, since each stays until its sum has arrived (us along / apart: 235
// workgroups a node, 8 x 60 000 x 30 21.9 / 19.6; 3840, 120 x 8000 x 20 21.4 / 22.0).
constexpr unsigned kLossLastMost = 64;
template <int KIND, int V>
static void launch_loss_kind(const gpga_ctx* c, const int32_t* idx, int32_t Beff, float* loss_out) {
    // the partial sums (one double per 256 samples) take the place of the per-sample terms
    double* partials = reinterpret_cast<double*>(c->coef);
    const dim3 grid((unsigned)((Beff + 255) / 256), (unsigned)c->n), block(256);
    const size_t lds = idx ? 0 : (size_t)256 * c->d * sizeof(float);
    const int cached = (int64_t)c->n * c->M * c->d * 4 <= kLossCachedBytes;
    if (grid.x == 1 || (c->loss_left && grid.x <= kLossLastMost && (int64_t)grid.x * grid.y <= 16 * c->num_cus)) {
        hipLaunchKernelGGL((k_rows_loss_short<KIND, V, true>), grid, block, lds, c->stream, c->feat, c->tgt, c->x, c->ld, idx, Beff,
                           c->M, (int32_t)c->d, cached, partials, c->loss_left, loss_out);
        return;
    }
    hipLaunchKernelGGL((k_rows_loss_short<KIND, V, false>), grid, block, lds, c->stream, c->feat, c->tgt, c->x, c->ld, idx, Beff, c->M,
                       (int32_t)c->d, cached, partials, nullptr, nullptr);
    hipLaunchKernelGGL(k_loss_chunks, dim3((unsigned)c->n), dim3(kWave), 0, c->stream, partials, (int32_t)grid.x, loss_out);
}
template <int V>
static void launch_loss_short(const gpga_ctx* c, const int32_t* idx, int32_t Beff, float* loss_out) {
    if (c->problem == PROB_LSQ) launch_loss_kind<PROB_LSQ, V>(c, idx, Beff, loss_out);
    else launch_loss_kind<PROB_LOGREG, V>(c, idx, Beff, loss_out);
}
static hipError_t launch_rows_loss_short(const gpga_ctx* c, const int32_t* idx, int32_t Beff, float* loss_out) {
    if (c->d % 4 == 0) launch_loss_short<4>(c, idx, Beff, loss_out);
    else if (c->d % 2 == 0) launch_loss_short<2>(c, idx, Beff, loss_out);
    else launch_loss_short<1>(c, idx, Beff, loss_out);
    return hipGetLastError();
}

hipError_t launch_rows_grad(const gpga_ctx* c, const int32_t* idx, int32_t B, float* loss_out, bool grad) {
    const int32_t Beff = idx ? B : c->M;
    if (!grad && c->d <= 32) return launch_rows_loss_short(c, idx, Beff, loss_out);
    const hipError_t e = launch_rows_margin(c, idx, B, loss_out);
    if (e != hipSuccess || !grad) return e;
    const int64_t cols = accum_quads(c->d) ? (c->d + 3) / 4 : c->d;
    dim3 grid2((unsigned)((cols + kWave - 1) / kWave), (unsigned)c->n);
    if (Beff >= 64) {
        hipLaunchKernelGGL(k_rows_accum<16>, grid2, dim3(kWave * 16), 0, c->stream, c->feat, c->coef, idx, Beff, c->M,
                           c->d, c->g, c->ld);
    } else {
        hipLaunchKernelGGL(k_rows_accum<4>, grid2, dim3(256), 0, c->stream, c->feat, c->coef, idx, Beff, c->M,
                           c->d, c->g, c->ld);
    }
    return hipGetLastError();
}

// Column chunks per node of the margin pass: enough workgroups per node to fill the chip, at least
// 256 quads each, every chunk non-empty.
int64_t virtual_margin_chunks(const gpga_ctx* c) {
    const int64_t d4 = (c->d + 3) / 4;
    int64_t chunks = (4096 + c->n - 1) / c->n;
    const int64_t max_chunks = (d4 + 255) / 256;
    if (chunks > max_chunks) chunks = max_chunks;
    if (chunks < 1) chunks = 1;
    const int64_t qpb = (d4 + chunks - 1) / chunks;
    return (d4 + qpb - 1) / qpb;
}

hipError_t launch_virtual_grad(const gpga_ctx* c, const int32_t* idx, int32_t B, float* loss_out, bool grad) {
    constexpr int BMAX = 32;
    if (B > BMAX) return hipErrorInvalidValue;
    float* coef = c->coef;
    float* lossterm = c->coef + (size_t)c->n * B;
    double* zpart = c->partials;  // n*B*chunks doubles, sized by the caller (n * B * virtual_margin_chunks)
    const uint32_t k0 = (uint32_t)(c->seed & 0xffffffffu), k1 = (uint32_t)(c->seed >> 32);
    const int64_t nb = (int64_t)c->n * B;
    const int64_t d4 = (c->d + 3) / 4;
    const int64_t chunks = virtual_margin_chunks(c);
    const int64_t qpb = (d4 + chunks - 1) / chunks;
    dim3 grid1((unsigned)chunks, (unsigned)c->n), block(256);
    hipLaunchKernelGGL((k_virtual_margin<BMAX>), grid1, block, 0, c->stream, c->x, c->ld, c->d, idx,
                       B, k0, k1, c->mu_sigma, qpb, zpart);
    hipLaunchKernelGGL(k_virtual_coef, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, c->stream,
                       zpart, (int32_t)chunks, c->tgt, idx, B, c->M, c->n, coef, lossterm);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (loss_out) {
        hipLaunchKernelGGL(k_loss_sum, dim3((unsigned)c->n), block, 0, c->stream, lossterm, B,
                           loss_out);
    }
    if (!grad) return hipGetLastError();
    const int vec_ok = aligned16(c->g) && (c->ld % 4 == 0);
    dim3 grid2((unsigned)((d4 + 255) / 256), (unsigned)c->n);
    hipLaunchKernelGGL((k_virtual_accum<BMAX>), grid2, block, 0, c->stream, coef, idx, B, c->d, k0,
                       k1, c->mu_sigma, vec_ok, c->g, c->ld);
    return hipGetLastError();
}

bool small_run_fits(const gpga_ctx* c, const int32_t* idx, int32_t B) {
    if (c->opt_small_run == 0 || c->aga) return false;
    if (c->problem != PROB_LSQ && c->problem != PROB_LOGREG) return false;
    if ((c->topo == GPGA_TOPO_GRID || c->topo == GPGA_TOPO_EXPO || c->topo == GPGA_TOPO_CUSTOM) && !c->csr_ready)
        return false;
    const int64_t Beff = idx ? B : c->M;
    if (Beff < 1 || Beff > 32 || c->d > 512 || c->n > 4096) return false;  // a thread walks a row / a batch: keep both short
    const int64_t nd = (int64_t)c->n * c->d, nb = (int64_t)c->n * Beff;
    // one workgroup does all the work of an iteration: keep it to a few hundred operations per thread
    if (nd > 8192 || nb > 4096 || nb * c->d > (1 << 17)) return false;
    return small_run_lds(c, (int32_t)Beff) <= 100 * 1024 && small_run_lds(c, (int32_t)Beff) <= (size_t)c->max_lds_block;
}

template <int KIND, int MOM, int C, int NB, int TW>
static hipError_t launch_node(const gpga_ctx* c, SmallArgs a) {
    a.worker_waves = (a.n * kNodeLanes + kWave - 1) / kWave;
    const int threads = kWave * (a.worker_waves + (a.trace ? TW : 0));
    const size_t lds = node_run_lds(a.n, C, NB, a.nnz);
    if (lds > kNodeMaxLds) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((k_node_run<KIND, MOM, C, NB, TW>), dim3(1), dim3(threads), lds, c->stream, a);
    return hipGetLastError();
}

template <int KIND, int MOM, int C>
static hipError_t launch_node_samples(const gpga_ctx* c, const SmallArgs& a) {
    switch (node_samples(a.B)) {
        case 1:
            // Four wavefronts where they have all rows at once, eight where they would need a second batch (us a pass with the
            // trace, four / eight: 20 x 10 43.7 / 47.1, 64 x 10 51.0 / 54.5, 100 x 10 58.1 / 56.2, 64 x 20 59.2 / 54.9).
            return a.n <= 4 * kNodeTraceRows * (kNodeLanes * C <= 16 ? 4 : 2) ? launch_node<KIND, MOM, C, 1, 4>(c, a)
                                                                            : launch_node<KIND, MOM, C, 1, node_trace_waves(1)>(c, a);
        case 2: return launch_node<KIND, MOM, C, 2, node_trace_waves(2)>(c, a);
        default: return launch_node<KIND, MOM, C, kNodeSamples, node_trace_waves(kNodeSamples)>(c, a);
    }
}

template <int KIND, int MOM>
static hipError_t launch_node_cols(const gpga_ctx* c, const SmallArgs& a) {
    switch (node_columns(a.d)) {
        case 1: return launch_node_samples<KIND, MOM, 1>(c, a);
        case 3: return launch_node_samples<KIND, MOM, 3>(c, a);
        default: return launch_node_samples<KIND, MOM, 5>(c, a);
    }
}

template <int KIND>
static hipError_t launch_node_kind(const gpga_ctx* c, const SmallArgs& a) {
    if (c->mu == 0.f) return launch_node_cols<KIND, 0>(c, a);
    return c->nesterov ? launch_node_cols<KIND, 2>(c, a) : launch_node_cols<KIND, 1>(c, a);
}

template <int KIND>
static hipError_t launch_small_kind(const gpga_ctx* c, const SmallArgs& a, size_t lds) {
    const dim3 grid(1), block(kSmallRunThreads);
    if (c->mu == 0.f) {
        hipLaunchKernelGGL((k_small_run<KIND, 0>), grid, block, lds, c->stream, a);
    } else if (!c->nesterov) {
        hipLaunchKernelGGL((k_small_run<KIND, 1>), grid, block, lds, c->stream, a);
    } else {
        hipLaunchKernelGGL((k_small_run<KIND, 2>), grid, block, lds, c->stream, a);
    }
    return hipGetLastError();
}

hipError_t launch_small_run(const gpga_ctx* c, int32_t T, const int32_t* idx, int32_t B, const float* lr) {
    if (T < 1 || T > kSmallRunMaxIters) return hipErrorInvalidValue;
    SmallArgs a;
    a.x = c->x;
    a.x_out = (T % 2) ? c->x_new : c->x;  // where T separate steps would leave the live iterates
    a.m = c->m;
    a.g = c->g;
    a.ld = c->ld;
    a.n = c->n;
    a.d = (int32_t)c->d;
    a.feat = c->feat;
    a.tgt = c->tgt;
    a.M = c->M;
    a.idx = idx;
    a.B = idx ? B : c->M;
    a.topo = c->topo;
    a.H = c->H;
    a.k0 = c->k;
    a.T = T;
    a.mu = c->mu;
    a.wptr = c->csr_ptr_d;
    a.wcol = c->csr_col_d;
    a.wval = c->csr_val_d;
    a.trace = c->trace;
    a.trace_cap = c->trace_cap;
    a.nnz = a.wptr ? (int32_t)c->csr.col.size() : 0;
    a.worker_waves = 0;
    for (int t = 0; t < T; ++t) {
        a.lr[t] = lr[t];
        a.shift[t] = is_global_iteration(c->topo, c->H, c->k + t) ? -1 : one_peer_shift(c->n, c->k + t);
    }
    if (node_run_takes(a.n, a.d, a.B, a.nnz)) {
        return c->problem == PROB_LSQ ? launch_node_kind<PROB_LSQ>(c, a) : launch_node_kind<PROB_LOGREG>(c, a);
    }
    const size_t lds = small_run_lds(c, a.B);
    return c->problem == PROB_LSQ ? launch_small_kind<PROB_LSQ>(c, a, lds) : launch_small_kind<PROB_LOGREG>(c, a, lds);
}
