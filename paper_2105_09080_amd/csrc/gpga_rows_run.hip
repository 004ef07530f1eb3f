// Several iterations on stored features in one launch (gpga_run): margins, gradient sums, update and mixing.
//
// A workgroup owns (node, slice of columns) for the whole launch; P of them share a node.  Up to ten of its twelve wavefronts hold
// the features of the samples in registers, from the margins to the gradient sums (full batches: for the whole launch); the
// others exchange, a thread a column, with x and m in LDS.  What workgroups owe each other goes as words that carry their
// launch's number (gpga_gang.hpp): the slices' shares of the margins within a node, then y = x^(k+1/2) between nodes; at a
// global average every workgroup adds one n-th of its slice's columns over all nodes and hands the mean on.  Under an adaptive
// period every workgroup takes the same decisions from the same losses, and the host reads the period once a launch that averages.
//
// An iteration is two trips through memory of 0.7 - 1.2 us (one where P = 1) in the place of two dependent launches of 4 - 5.
// What bounds it then is code: the instructions between arrival and the next store (3 us an iteration on the smallest problems),
// fp64 conversions and sums (0.2 us a row and wavefront), and, with 40 MB of rows an iteration, that a workgroup's memory
// operations are served in order, so that the exchange waits behind rows on their way (32 x 10 000 with 32 samples: 12.5 us an
// iteration, 6.4 of them the rows from memory).  Hence roles for wavefronts: one that has rows under way cannot look at a word
// before they have arrived.
// Whole calls of gpga_run, us, two launches an iteration -> this: 8 iterations on 8 x 1000 with full batches of 100 75.8 -> 58; 50 x 400
// 158 -> 63; 16 iterations on 32 x 10 000 with 32 samples 389 -> 219; 8 on 35 x 3160 124 -> 57.6, 64 x 3000 with 50 216 -> 113; 12 on
// 20 x 1001 under the adaptive period 143.5 -> 77.3; from a single workgroup: 8 on 9 x 222 with 32 277 -> 37, 28 x 201 142 -> 35.
// Which runs it takes: rows_run_pays.  Registers: full batches of 13 to 32 slots spill 5 a lane, minibatches of 17 to 20 two, the
// others none.
#include <algorithm>
#include <type_traits>

#include "gpga_gang.hpp"
#include "gpga_internal.hpp"
#include "gpga_order.hpp"
#include "gpga_rows_run.hpp"
#include "gpga_samples.hpp"
#include "gpga_schedule.hpp"
#include "gpga_unit.hpp"

namespace {

constexpr int kRowsRunFewest = 3;                    // iterations that are worth a launch of this kind
constexpr int64_t kRowsRunStaged = 2048;             // (iteration, sample) pairs whose row numbers and targets go to LDS first
constexpr int64_t kRowsRunMaxWords = 8ll << 20;      // of x^(k+1/2) a launch may exchange (64 MiB)

struct RowsRunArgs {
    const float* x;
    float* x_other;      // the array x is not in
    float* m;
    float* g;            // NULL: the last iteration's gradients are not wanted
    uint64_t* m_keep;    // words: n x d
    const float* feat;   // n x M x d
    const float* tgt;    // n x M
    const int32_t* idx;  // T x n x B, or NULL: rows 0 .. B-1
    RowsRunAga* aga;     // adaptive averaging period: state before and after, or NULL
    RowsRunAga begin;
    uint64_t* wz;        // words: [T][n][B][P][2] shares of the margins
    uint64_t* wy;        // [T][n][d] x^(k+1/2)
    uint64_t* wmean;     // [T][d] means
    uint64_t* wloss;     // [T][n] minibatch losses, in iterations that end in an average under an adaptive period
    GangArgs gang;
    int64_t ld, d;
    int32_t n, B, M, T;
    int32_t P, LP;       // slices of a node; 2^LP lanes add their shares
    int32_t w;           // quads of a slice
    int32_t threads;
    int32_t QW, RG;      // wavefronts across a slice, wavefronts across the rows: QW x RG hold rows
    int32_t problem;     // PROB_LSQ or PROB_LOGREG
    int32_t mom;         // 0: no momentum, 1: heavy ball, 2: Nesterov
    int32_t mode;        // StencilMode of the gossip iterations, or kRunSparse
    const int32_t* off;  // sparse W: (signed circular offset, weight) entries, K a node at most
    const float* val;
    const int32_t* wptr;
    int32_t K;
    int32_t splitters;   // of an average
    float inv_n, mu;
    int32_t gives_up;    // workgroup that does not store what it has, or -1
    int32_t mean64;      // averages are formed in double precision
    float lr[kRowsRunMaxIters];
    int32_t shift[kRowsRunMaxIters];  // one-peer offset; -1: the iteration ends in a global average (fixed period)
};
constexpr int kRunSparse = 8, kRunMean = 9;

// Sums over the 64 lanes of four values; the lanes 15, 31, 47 and 63 hold those of v0, v2, v1 and v3.
__device__ __forceinline__ double four_sums(double v0, double v1, double v2, double v3) {
    return row16_sum_last(swap_add(swap_add(v0, v1, true), swap_add(v2, v3, true), false));
}

__device__ __forceinline__ float local_update(int mom_kind, float x, float g, float lr, float mu, float* m) {
    if (mom_kind == 0) return x - lr * g;
    const float mom = mu * *m + g;
    *m = mom;
    return mom_kind == 2 ? x - lr * (g + mu * mom) : x - lr * mom;
}

__device__ __forceinline__ float run_coefficient(const RowsRunArgs& a, double z, float target, float invB) {
    return a.problem == PROB_LSQ ? sample_coefficient<PROB_LSQ>(z, target, invB) : sample_coefficient<PROB_LOGREG>(z, target, invB);
}
__device__ __forceinline__ float run_loss(const RowsRunArgs& a, double z, float target, float invB) {
    return a.problem == PROB_LSQ ? sample_loss<PROB_LSQ>(z, target, invB) : sample_loss<PROB_LOGREG>(z, target, invB);
}

// Barrier of the workgroup, reached by its two kinds of wavefront from different places.
__device__ __forceinline__ void run_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Sum over each aligned group of 2^lanes_log2 lanes, in all of them.
__device__ __forceinline__ double slices_sum(double z, int lanes_log2) {
    const int lanes = 1 << lanes_log2;
    if (lanes >= 2) z += dpp_f64<0xB1>(z);    // neighbours
    if (lanes >= 4) z += dpp_f64<0x4E>(z);    // pairs of a quad
    if (lanes >= 8) z += dpp_f64<0x141>(z);   // quads of eight (mirrored: a quad's lanes are equal by now)
    if (lanes >= 16) z += dpp_f64<0x140>(z);  // eights of sixteen
    if (lanes >= 32) z += __shfl_xor(z, 16, kWave);
    if (lanes >= 64) z += __shfl_xor(z, 32, kWave);
    return z;
}

// Algorithm 2 after the global average of iteration t of the launch: the period that follows from the sum of the n losses.
__device__ __forceinline__ void aga_next(RowsRunAga* s, double loss_sum, int n, int t) {
    s->since = 0;
    s->step(s->k0 + t, loss_sum / (double)n);
}
__device__ __forceinline__ void aga_store(RowsRunAga* to, const RowsRunAga& s) {  // host memory
    __hip_atomic_store(&to->since, s.since, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&to->period, s.period, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&to->first_loss, s.first_loss, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The mean of one column, rows `step` floats apart, added as k_step_global adds them (gpga_order.hpp) with batches of four rows
// dealt to two splitters or more; in double precision on the problems that k_small_run, which adds so, takes in launches of
// other lengths.
__device__ __forceinline__ float column_mean(const RowsRunArgs& a, const float* y, int step) {
    const int n = a.n, splitters = a.splitters;
    if (a.mean64) {
        double sum = 0.0;
#pragma unroll 4
        for (int i = 0; i < n; ++i) sum += (double)y[i * step];
        return (float)(sum * (1.0 / (double)n));
    }
    SplitterTree<float> tree;
#pragma unroll 1
    for (int s = 0; s < splitters; ++s) {
        float sum = 0.f;
#pragma unroll 1
        for (int base = s; base < n; base += 4 * splitters) {
            float v[4], part = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = y[(base + k * splitters < n ? base + k * splitters : n - 1) * step];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (base + k * splitters < n) part += v[k];
            sum += part;
        }
        tree.add(s, sum);
    }
    return tree.sum * a.inv_n;
}

enum RowsHeld : int {
    ROWS_FIXED = 0,    // full batches: the same rows in every iteration, held in double precision up to kFixedSlots of them
    ROWS_AHEAD = 1     // minibatches: the next iteration's rows are fetched ahead, half of them as soon as the margins are formed, into
                       // registers of their own
};

template <int S, int HELD>
__global__ void __launch_bounds__(kRowsRunThreads) k_rows_run(const RowsRunArgs a) {
    extern __shared__ __align__(16) unsigned char s_raw[];
    __shared__ int s_gone_z, s_gone_y, s_last, s_average;
    const int n = a.n, B = a.B, P = a.P, RG = a.RG, nthr = a.threads;
    const int wcols = 4 * a.w, held = 4 * kWave * a.QW;  // columns of a slice; of its lanes
    const int share = (wcols + n - 1) / n;               // columns whose mean this workgroup forms
    const int staged = HELD != ROWS_FIXED ? a.T * B : B;
    const RunLds lds(n, B, a.w, a.QW, RG, S, staged, a.mode == kRunSparse ? a.K : 0);
    double* __restrict__ sAcc = reinterpret_cast<double*>(s_raw);                 // [RG][held]
    double* __restrict__ sZ = reinterpret_cast<double*>(s_raw + lds.z);           // [QW][B]
    double* __restrict__ sSum = reinterpret_cast<double*>(s_raw + lds.sum);       // [B] whole margins
    float* __restrict__ sX = reinterpret_cast<float*>(s_raw + lds.x);             // [held]
    float* __restrict__ sM = reinterpret_cast<float*>(s_raw + lds.m);             // [held]
    float* __restrict__ sY = reinterpret_cast<float*>(s_raw + lds.y);             // [n][share]
    float* __restrict__ sCoef = reinterpret_cast<float*>(s_raw + lds.coef);       // [RG S], zeros behind B
    float* __restrict__ sTgt = reinterpret_cast<float*>(s_raw + lds.tgt);         // [staged]
    int32_t* __restrict__ sRow = reinterpret_cast<int32_t*>(s_raw + lds.row);     // [staged]
    int32_t* __restrict__ sOff = reinterpret_cast<int32_t*>(s_raw + lds.off);     // [K] this node's entries of a sparse W
    float* __restrict__ sVal = reinterpret_cast<float*>(s_raw + lds.val);

    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int node = blockIdx.x / P, slice = blockIdx.x - node * P;
    const int64_t d = a.d, c0 = (int64_t)slice * wcols;
    const int ncol = d - c0 < wcols ? (int)(d - c0) : wcols;
    const float invB = 1.0f / (float)B;
    float* const x_out = a.T % 2 ? a.x_other : const_cast<float*>(a.x);

    if (tid == 0) {
        s_gone_z = s_gone_y = 0;
        s_average = a.aga ? a.begin.since + 1 == a.begin.period : a.shift[0] < 0;
    }
    if (a.mode == kRunSparse) {
        for (int e = tid; e < a.wptr[node + 1] - a.wptr[node]; e += nthr) {
            sOff[e] = a.off[node * a.K + e];
            sVal[e] = a.val[node * a.K + e];
        }
    }
    for (int e = tid; e < staged; e += nthr) {
        const int t = e / B, b = e - t * B;
        const int32_t r = HELD != ROWS_FIXED ? a.idx[((int64_t)t * n + node) * B + b] : b;
        const bool ok = r >= 0 && r < a.M;  // outside [0, M): no access; the coefficient becomes NaN
        sRow[e] = ok ? r : -1;
        sTgt[e] = ok ? a.tgt[(int64_t)node * a.M + r] : 0.f;
    }
    for (int e = tid; e < RG * S; e += nthr) sCoef[e] = 0.f;
    for (int cc = tid; cc < held; cc += nthr) {
        float x = 0.f, m = 0.f;
        if (cc < ncol) {
            const int64_t o = (int64_t)node * a.ld + c0 + cc;
            x = a.x[o];
            if (a.mom) m = a.m[o];
            // kept for a launch that has to be done again
            if (a.T % 2 == 0) gang_put32(reinterpret_cast<uint32_t*>(a.x_other + o), __float_as_uint(x));
            if (a.mom) gang_put(a.m_keep + (int64_t)node * d + c0 + cc, a.gang.number, __float_as_uint(m));
        }
        sX[cc] = x;
        sM[cc] = m;
    }
    run_barrier();

    // Gradient, momentum and x^(k+1/2) of iteration t, two columns a thread at a time.
    auto update_columns = [&](int t) {
        const bool last = t == a.T - 1;
        uint64_t* const wy = a.wy + ((int64_t)t * n + node) * d + c0;
        const float lr = a.lr[t];
#pragma unroll 1
        for (int c = tid; c < ncol; c += 2 * nthr) {
            const int cc[2] = {c, c + nthr < ncol ? c + nthr : c};
            double s[2] = {sAcc[cc[0]], sAcc[cc[1]]};
            const float x[2] = {sX[cc[0]], sX[cc[1]]};
            float m[2] = {sM[cc[0]], sM[cc[1]]};
#pragma unroll 4
            for (int v = 1; v < RG; ++v)
#pragma unroll
                for (int k = 0; k < 2; ++k) s[k] += sAcc[v * held + cc[k]];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                if (k == 1 && c + nthr >= ncol) break;
                const float g = (float)s[k];
                const float y = local_update(a.mom, x[k], g, lr, a.mu, &m[k]);
                gang_put(wy + cc[k], a.gang.number, __float_as_uint(y));
                sX[cc[k]] = y;
                if (a.mom) sM[cc[k]] = m[k];
                if (last && a.g) gang_put32(reinterpret_cast<uint32_t*>(a.g + (int64_t)node * a.ld + c0 + cc[k]), __float_as_uint(g));
            }
        }
    };

    bool gone = false;
    if (wave < a.QW * RG) {
        // ---- wavefronts that hold rows
        const int wq = wave % a.QW, rg = wave / a.QW;
        const int q = wq * kWave + lane;  // this lane's quad of the slice
        const int have = ncol - 4 * q < 4 ? ncol - 4 * q : 4;  // columns of it that are there; the others stay zeros
        const float* __restrict__ feat = a.feat + (int64_t)node * a.M * d + c0;
        const uint32_t lane_bytes = 16u * (uint32_t)q;
        typedef double v4d __attribute__((ext_vector_type(4)));
        using Row = std::conditional_t<HELD == ROWS_FIXED && S <= kFixedSlots, v4d, v4f>;
        constexpr int kAhead = HELD == ROWS_AHEAD ? S / 2 : 0;
        Row f[S], ahead[kAhead ? kAhead : 1];
        // Rows of the slots [U0, U1) of iteration t into to[slot].  A workgroup's memory operations are served in order, so a wavefront
        // has two rows in flight: 20 KB a workgroup are what the memory's latency needs, and what the exchange may have to wait
        // behind (32 x 10 000: all at once 300 us, four in flight 247, two 217; two or three make no difference elsewhere).
        auto load_rows = [&](auto& to, int t, auto from, auto until) {
            constexpr int U0 = decltype(from)::value, U1 = decltype(until)::value;
            const int b0 = rg + lane * RG;  // slot `lane`
            const int32_t r0 = lane < S && b0 < B ? sRow[(HELD != ROWS_FIXED ? t * B : 0) + b0] : 0;
            const int32_t rows = r0 < 0 ? 0 : r0;
            auto row = [&](int u) {
                return reinterpret_cast<const float*>(reinterpret_cast<const char*>(feat + (int64_t)__builtin_amdgcn_readlane(rows, u) * d) + lane_bytes);
            };
            if (have == 4) {
#pragma unroll
                for (int u = U0; u < U1; ++u) {
                    if (rg + u * RG >= B) break;
                    to[u] = __builtin_convertvector(ld_unit_cached<v4f>(row(u)), Row);
                    if (HELD == ROWS_AHEAD && u > U0) __builtin_amdgcn_s_waitcnt(0x0F71);  // vmcnt(1)
                }
            } else if (have > 0) {  // the last quad of a ragged width
#pragma unroll
                for (int u = U0; u < U1; ++u) {
                    if (rg + u * RG >= B) break;
                    const float* const p = row(u);
                    to[u].x = p[0];
                    if (have > 1) to[u].y = p[1];
                    if (have > 2) to[u].z = p[2];
                }
            }
        };
        constexpr std::integral_constant<int, 0> slot_0{};
        constexpr std::integral_constant<int, S> slot_S{};
#pragma unroll
        for (int u = 0; u < S; ++u) f[u] = Row(0);
#pragma unroll
        for (int u = 0; u < kAhead; ++u) ahead[u] = Row(0);
        load_rows(f, 0, slot_0, slot_S);
        for (int t = 0; t < a.T; ++t) {
            const bool more = HELD != ROWS_FIXED && t + 1 < a.T;
            const bool average = __builtin_amdgcn_readfirstlane(s_average) != 0;
            const v4f xq = *reinterpret_cast<const v4f*>(sX + 4 * q);  // columns past the slice are zeros there
            const double x0 = xq.x, x1 = xq.y, x2 = xq.z, x3 = xq.w;
#pragma unroll
            for (int u = 0; u < S; u += 4) {
                if (rg + u * RG >= B) break;
                double z[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    z[j] = u + j < S ? (double)f[u + j].x * x0 + (double)f[u + j].y * x1 + (double)f[u + j].z * x2 + (double)f[u + j].w * x3 : 0.0;
                const double sum = four_sums(z[0], z[1], z[2], z[3]);
                const int part = lane >> 4, j = part == 1 ? 2 : part == 2 ? 1 : part, b = rg + (u + j) * RG;
                if ((lane & 15) == 15 && u + j < S && b < B) sZ[wq * B + b] = sum;
                __builtin_amdgcn_sched_barrier(0);
            }
            // The rows stay in 32 bits between their two uses, and all of them are here before the next are asked for: waits
            // count loads in order.
#pragma unroll
            for (int u = 0; u < S && std::is_same<Row, v4f>::value; ++u) asm volatile("" : "+v"(f[u]));
            run_barrier();
            if (kAhead && more) load_rows(ahead, t + 1, slot_0, std::integral_constant<int, kAhead>{});
            run_barrier();
            gone = s_gone_z != 0;
            if (gone) break;
            double g0 = 0.0, g1 = 0.0, g2 = 0.0, g3 = 0.0;
            const float coefs = sCoef[rg + (lane < S ? lane : 0) * RG];
#pragma unroll
            for (int u = 0; u < S; ++u) {
                if (u % 4 == 0 && rg + u * RG >= B) break;
                const double cf = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(coefs), u));
                g0 += cf * (double)f[u].x;
                g1 += cf * (double)f[u].y;
                g2 += cf * (double)f[u].z;
                g3 += cf * (double)f[u].w;
                if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
            }
            double* const to = sAcc + rg * held + 4 * q;
            to[0] = g0, to[1] = g1, to[2] = g2, to[3] = g3;
            run_barrier();
            update_columns(t);
            run_barrier();
            if (more) {
#pragma unroll
                for (int u = 0; u < kAhead; ++u) f[u] = ahead[u];
                load_rows(f, t + 1, std::integral_constant<int, kAhead>{}, slot_S);
            }
            if (average) run_barrier();
            run_barrier();
            gone = s_gone_y != 0;
            if (gone) break;
        }
    } else {
        // ---- wavefronts that exchange: margins and coefficients, then update and mixing, a thread a column
        const int ct = tid - a.QW * RG * kWave, NT = nthr - a.QW * RG * kWave;
        constexpr int U = 5;  // words of a thread in flight, where a mean's share is collected
        RowsRunAga aga = a.begin;
        const int gossip_entries = a.mode == MODE_SELF ? 0 : a.mode == kRunSparse ? __builtin_amdgcn_readfirstlane(a.wptr[node + 1] - a.wptr[node])
                                                       : a.mode == MODE_RING ? 2 : 1;
        const uint64_t none = (uint64_t)a.gang.number << 32;  // stands for a word that is not wanted
        for (int t = 0; t < a.T; ++t) {
            const bool last = t == a.T - 1;
            const int st = HELD != ROWS_FIXED ? t * B : 0;
            const bool average = __builtin_amdgcn_readfirstlane(s_average) != 0;
            run_barrier();  // margins are in sZ
            uint64_t* const wz = a.wz + ((int64_t)t * n + node) * B * P * 2;
            auto own_share = [&](int b) {
                double z = sZ[b];
                for (int v = 1; v < a.QW; ++v) z += sZ[v * B + b];
                return z;
            };
            if (P > 1) {
                for (int b = ct; b < B; b += NT) {
                    const uint64_t z = (uint64_t)__double_as_longlong(own_share(b));
                    uint64_t* const to = wz + ((int64_t)b * P + slice) * 2;
                    gang_put(to, a.gang.number, (uint32_t)z);
                    gang_put(to + 1, a.gang.number, (uint32_t)(z >> 32));
                }
            }
            // E (sample, slice) pairs of a thread in flight
            auto margins = [&](auto in_flight) {
                constexpr int E = decltype(in_flight)::value;
                const int p = ct & ((1 << a.LP) - 1), per = kWave >> a.LP;
#pragma unroll 1
                for (int e0 = 0; e0 < B << a.LP; e0 += E * NT) {
                    double z[E];
                    if (P == 1) {
#pragma unroll
                        for (int k = 0; k < E; ++k) z[k] = own_share(e0 + k * NT + ct < B ? e0 + k * NT + ct : 0);
                    } else {
                        uint32_t half[2 * E], at[E];
                        bool on[E];
#pragma unroll
                        for (int k = 0; k < E; ++k) {  // pairs that are not there look at the workgroup's own share of sample 0
                            const int b = (e0 + k * NT + ct) >> a.LP;
                            on[k] = b < B && p < P;
                            at[k] = 2 * (on[k] ? b * P + p : slice);
                        }
                        gang_wait<2 * E>(a.gang, &s_gone_z, [&](uint64_t (&v)[2 * E]) {
#pragma unroll
                            for (int k = 0; k < E; ++k) v[2 * k] = gang_peek_at(wz, at[k]), v[2 * k + 1] = gang_peek_at(wz, at[k] + 1);
                        }, half);
#pragma unroll
                        for (int k = 0; k < E; ++k)
                            z[k] = slices_sum(on[k] ? __longlong_as_double((long long)(((uint64_t)half[2 * k + 1] << 32) | half[2 * k])) : 0.0, a.LP);
                    }
                    // The wavefront's samples, a lane each: the coefficient's double-precision exponential once.
#pragma unroll
                    for (int k = 0; k < E; ++k)
                        if (p == 0 && (e0 + k * NT + ct) >> a.LP < B) sSum[(e0 + k * NT + ct) >> a.LP] = z[k];
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    __builtin_amdgcn_wave_barrier();
                    const int lane_k = lane >> (6 - a.LP);
                    const int b = ((e0 + lane_k * NT + (ct & ~(kWave - 1))) >> a.LP) + (lane & (per - 1));
                    for (int k = lane_k, bb = b; k < E; k += 1 << a.LP, bb += NT)
                        if (bb < B)
                            sCoef[bb] = sRow[st + bb] >= 0 ? run_coefficient(a, sSum[bb], sTgt[st + bb], invB) : __builtin_nanf("");
                }
            };
            if (B << a.LP <= NT) margins(std::integral_constant<int, 1>{}); else margins(std::integral_constant<int, 4>{});
            run_barrier();  // coefficients are in sCoef
            gone = s_gone_z != 0;
            if (gone) break;
            run_barrier();  // gradient sums are in sAcc
            uint64_t* const wy = a.wy + (int64_t)t * n * d + c0;
            update_columns(t);
            run_barrier();  // x^(k+1/2) is in sX
            if (a.aga && average && slice == 0 && ct < kWave) {
                double l = 0.0;
#pragma unroll 1
                for (int b = ct; b < B; b += kWave)
                    l += sRow[st + b] >= 0 ? run_loss(a, sSum[b], sTgt[st + b], invB) : __builtin_nanf("");
                for (int off = kWave / 2; off > 0; off >>= 1) l += __shfl_down(l, off, kWave);
                if (ct == 0) gang_put(a.wloss + t * n + node, a.gang.number, __float_as_uint((float)l));
            }
            if (average) {
                const int first = node * share, count = ncol - first < share ? (ncol > first ? ncol - first : 0) : share;
                for (int eu = 0; eu < n * count; eu += U * NT) {
                    const int e0 = eu + ct;
                    uint32_t at[U], v[U];
#pragma unroll
                    for (int k = 0; k < U; ++k) {
                        const int e = e0 + k * NT < n * count ? e0 + k * NT : 0, j = e / count;
                        at[k] = (uint32_t)(j * (int)d + first + (e - j * count));
                    }
                    gang_wait<U>(a.gang, &s_gone_y, [&](uint64_t (&w)[U]) {
#pragma unroll
                        for (int k = 0; k < U; ++k) w[k] = eu + k * NT < n * count ? gang_peek_at(wy, at[k]) : none;
                    }, v);
#pragma unroll
                    for (int k = 0; k < U; ++k)
                        if (e0 + k * NT < n * count) sY[e0 + k * NT] = __uint_as_float(v[k]);
                }
                run_barrier();
                uint64_t* const wm = a.wmean + (int64_t)t * d + c0;
                for (int e = ct; e < count; e += NT)
                    gang_put(wm + first + e, a.gang.number, __float_as_uint(column_mean(a, sY + e, count)));
            }
            // What comes from other workgroups: the means, or the y of one or more other nodes, two at a time.
            const int mode = average ? kRunMean : a.mode, shift = a.shift[t];
            const int entries = average ? 1 : gossip_entries;
            auto source = [&](int e) -> const uint64_t* {
                if (mode == kRunMean) return a.wmean + (int64_t)t * d + c0;
                const int j = node + (mode == kRunSparse ? __builtin_amdgcn_readfirstlane(sOff[e]) : mode == MODE_RING ? 2 * e - 1 : shift);
                return wy + (int64_t)(j < 0 ? j + n : j >= n ? j - n : j) * d;
            };
            // A thread looks at U columns of N sources at a time.
            auto mix = [&](auto columns, auto sources) {
                constexpr int U = decltype(columns)::value, N = decltype(sources)::value;
#pragma unroll 1
                for (int cu = 0; cu < ncol; cu += U * NT) {
                    uint32_t at[U], v[U * N];
                    float sum[U];
#pragma unroll
                    for (int k = 0; k < U; ++k) {
                        const int cc = cu + ct + k * NT;
                        at[k] = cc < ncol ? cc : 0;  // columns that are not there look at the first
                        sum[k] = mode == kRunSparse ? 0.f : sX[at[k]];
                    }
#pragma unroll 1
                    for (int e = 0; e < entries; e += N) {
                        const uint64_t* y[N];
#pragma unroll
                        for (int s = 0; s < N; ++s) y[s] = s == 0 || e + s < entries ? source(e + s) : nullptr;
                        gang_wait<U * N>(a.gang, &s_gone_y, [&](uint64_t (&w)[U * N]) {
#pragma unroll
                            for (int s = 0; s < N; ++s)
#pragma unroll
                                for (int k = 0; k < U; ++k) {
                                    w[s * U + k] = none;
                                    if ((k == 0 || cu + k * NT < ncol) && (s == 0 || e + s < entries)) w[s * U + k] = gang_peek_at(y[s], at[k]);
                                }
                        }, v);
                        float p[N][U];
#pragma unroll
                        for (int s = 0; s < N; ++s)
#pragma unroll
                            for (int k = 0; k < U; ++k) p[s][k] = __uint_as_float(v[s * U + k]);
                        if (mode == kRunSparse) {
#pragma unroll
                            for (int s = 0; s < N; ++s) {
                                if (s > 0 && e + s >= entries) break;
                                const float weight = sVal[e + s];
#pragma unroll
                                for (int k = 0; k < U; ++k) sum[k] += weight * p[s][k];
                            }
                        } else {
#pragma unroll
                            for (int k = 0; k < U; ++k)
                                sum[k] = mode == kRunMean ? p[0][k] : mode == MODE_PEER ? (sum[k] + p[0][k]) * 0.5f : (p[0][k] + sum[k] + p[N - 1][k]) * (1.0f / 3.0f);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < U; ++k)
                        if (cu + ct + k * NT < ncol) sX[at[k]] = sum[k];
                }
            };
            constexpr std::integral_constant<int, 1> c1{};
            constexpr std::integral_constant<int, 2> c2{};
            constexpr std::integral_constant<int, 4> c4{};
            constexpr std::integral_constant<int, 5> c5{};
            constexpr std::integral_constant<int, 8> c8{};
            constexpr std::integral_constant<int, 10> c10{};
            if (entries == 1) {
                if (ncol <= 2 * NT) mix(c2, c1); else mix(c10, c1);
            } else if (entries == 2) {
                if (ncol <= NT) mix(c1, c2); else mix(c5, c2);
            } else if (entries > 2) {
                if (ncol <= NT) mix(c1, c8); else mix(c4, c4);
            }
            if (a.aga && ct < kWave) {
                ++aga.since;
                if (average) {
                    uint32_t l[2];
                    const bool on0 = lane < n, on1 = lane + kWave < n;
                    gang_wait<2>(a.gang, &s_gone_y, [&](uint64_t (&w)[2]) {
                        w[0] = on0 ? gang_peek_at(a.wloss, t * n + lane) : none;
                        w[1] = on1 ? gang_peek_at(a.wloss, t * n + lane + kWave) : none;
                    }, l);
                    double l0 = on0 ? __uint_as_float(l[0]) : 0.f, l1 = on1 ? __uint_as_float(l[1]) : 0.f;
                    for (int off = kWave / 2; off > 0; off >>= 1) {
                        l0 += __shfl_down(l0, off, kWave);
                        l1 += __shfl_down(l1, off, kWave);
                    }
                    aga_next(&aga, readlane_f64(l0, 0) + readlane_f64(l1, 0), n, t);
                }
            }
            if (ct == 0 && !last) s_average = a.aga ? aga.since + 1 == aga.period : a.shift[t + 1] < 0;
            run_barrier();  // the iterates are in sX
            gone = s_gone_y != 0;
            if (gone) break;
        }
        if ((int)blockIdx.x == a.gives_up) {
            if (ct == 0) gang_put32(&a.gang.words->given_up, a.gang.number);
            gone = true;
        }
        if (!gone && a.aga && blockIdx.x == 0 && ct == 0) aga_store(a.aga, aga);
        if (!gone) {
            for (int cc = ct; cc < ncol; cc += NT) {
                const int64_t o = (int64_t)node * a.ld + c0 + cc;
                gang_put32(reinterpret_cast<uint32_t*>(x_out + o), __float_as_uint(sX[cc]));
                if (a.mom) gang_put32(reinterpret_cast<uint32_t*>(a.m + o), __float_as_uint(sM[cc]));
            }
            if (ct == 0) gang_put32(a.gang.finished + blockIdx.x, a.gang.number);
        }
    }
    // All of this workgroup's stores are through before it says that it leaves.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
        s_last = 0;
        if (__hip_atomic_fetch_add(&a.gang.words->left, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1) {
            gang_put32(&a.gang.words->left, 0u);
            s_last = gang_get32(&a.gang.words->given_up) == a.gang.number;
            if (!s_last) gang_ended(a.gang);
        }
    }
    __syncthreads();
    if (!s_last) return;

    // A launch that was given up: its last workgroup does it alone, from the state the launch began with.
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    float* const x = const_cast<float*>(a.x);
    float* const y = a.x_other;
    for (int w = 0; w < (int)gridDim.x; ++w) {
        if (gang_get32(a.gang.finished + w) != a.gang.number) continue;
        const int i = w / P;
        const int64_t from = (int64_t)(w - i * P) * wcols;
        for (int cc = tid; cc < wcols && from + cc < d; cc += nthr) {
            const int64_t o = (int64_t)i * a.ld + from + cc;
            if (a.T % 2 == 0) x[o] = y[o];
            if (a.mom) a.m[o] = __uint_as_float((uint32_t)gang_peek(a.m_keep + (int64_t)i * d + from + cc));
        }
    }
    __syncthreads();
    RowsRunAga aga = a.begin;
    for (int t = 0; t < a.T; ++t) {
        const bool last = t == a.T - 1;
        const bool average = a.aga ? aga.since + 1 == aga.period : a.shift[t] < 0;
        const float lr = a.lr[t];
        for (int i = 0; i < n; ++i) {
            auto row_of = [&](int b) { return a.idx ? a.idx[((int64_t)t * n + i) * B + b] : b; };
            const float* const fi = a.feat + (int64_t)i * a.M * d;
            for (int b = wave; b < B; b += nthr / kWave) {
                const int32_t r = row_of(b);
                const bool ok = r >= 0 && r < a.M;
                double z = 0.0;
                if (ok)
                    for (int64_t c = lane; c < d; c += kWave) z += (double)fi[(int64_t)r * d + c] * x[(int64_t)i * a.ld + c];
                for (int off = kWave / 2; off > 0; off >>= 1) z += __shfl_down(z, off, kWave);
                if (lane == 0) {
                    const float target = ok ? a.tgt[(int64_t)i * a.M + r] : 0.f;
                    sCoef[b] = ok ? run_coefficient(a, z, target, invB) : __builtin_nanf("");
                    if (a.aga && average) sSum[b] = ok ? run_loss(a, z, target, invB) : __builtin_nan("");
                }
            }
            __syncthreads();
            if (tid == 0 && a.aga && average) {
                double l = 0.0;
                for (int b = 0; b < B; ++b) l += sSum[b];
                sX[i] = (float)l;
            }
            for (int64_t c = tid; c < d; c += nthr) {
                double s = 0.0;
                for (int b = 0; b < B; ++b) {
                    const int32_t r = row_of(b);
                    s += (double)sCoef[b] * fi[(int64_t)(r >= 0 && r < a.M ? r : 0) * d + c];
                }
                const int64_t o = (int64_t)i * a.ld + c;
                if (last && a.g) a.g[o] = (float)s;
                float mv = a.mom ? a.m[o] : 0.f;
                y[o] = local_update(a.mom, x[o], (float)s, lr, a.mu, &mv);
                if (a.mom) a.m[o] = mv;
            }
            __syncthreads();
        }
        if (a.aga) {
            ++aga.since;
            if (average) {
                double l = 0.0;
                for (int i = 0; i < n; ++i) l += sX[i];
                aga_next(&aga, l, n, t);
            }
        }
        const int shift = a.shift[t];
        for (int64_t c = tid; c < d; c += nthr) {
            const float* const yc = y + c;
            auto at = [&](int i) { return yc[(int64_t)i * a.ld]; };
            const float mean = average ? column_mean(a, yc, (int)a.ld) : 0.f;
            for (int i = 0; i < n; ++i) {
                float v = at(i);
                if (average) {
                    v = mean;
                } else if (a.mode == MODE_RING) {
                    v = (at(i == 0 ? n - 1 : i - 1) + v + at(i == n - 1 ? 0 : i + 1)) * (1.0f / 3.0f);
                } else if (a.mode == MODE_PEER) {
                    v = (v + at(i + shift >= n ? i + shift - n : i + shift)) * 0.5f;
                } else if (a.mode == kRunSparse) {
                    v = 0.f;
                    for (int e = 0; e < a.wptr[i + 1] - a.wptr[i]; ++e) {
                        int j = i + a.off[i * a.K + e];
                        j = j < 0 ? j + n : j >= n ? j - n : j;
                        v += a.val[i * a.K + e] * at(j);
                    }
                }
                x[(int64_t)i * a.ld + c] = v;
            }
        }
        __syncthreads();
    }
    if (a.aga && tid == 0) aga_store(a.aga, aga);
    if (a.T % 2)
        for (int i = 0; i < n; ++i)
            for (int64_t c = tid; c < d; c += nthr) y[(int64_t)i * a.ld + c] = x[(int64_t)i * a.ld + c];
    if (tid == 0) {
        gang_done_alone(a.gang);
        gang_ended(a.gang);
    }
}

// Success is what the launch itself returns: hipGetLastError may tell of an older call's failure, and who is told that nothing was
// launched takes the iterations another way.
template <int S, int HELD>
hipError_t launch_slots(const gpga_ctx* c, const RowsRunArgs& a, int threads, size_t lds) {
    static bool attr_set[64] = {false};  // per instantiation and device: more than the default 64 KiB of dynamic LDS
    const int dev = c->device >= 0 && c->device < 64 ? c->device : 0;
    if (!attr_set[dev]) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_rows_run<S, HELD>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, c->max_lds_block - 1024);
        if (e != hipSuccess) return e;
        attr_set[dev] = true;
    }
    RowsRunArgs args = a;
    void* const packed[] = {&args};
    return hipLaunchKernel(reinterpret_cast<const void*>(&k_rows_run<S, HELD>), dim3((unsigned)(a.n * a.P)), dim3((unsigned)threads),
                           const_cast<void**>(packed), lds, c->stream);
}

hipError_t launch_run(const gpga_ctx* c, const RowsRunArgs& a, int slots, int threads, size_t lds) {
    if (!a.idx) {
        if (slots == 4) return launch_slots<4, ROWS_FIXED>(c, a, threads, lds);
        if (slots == 8) return launch_slots<8, ROWS_FIXED>(c, a, threads, lds);
        if (slots == kFixedSlots) return launch_slots<kFixedSlots, ROWS_FIXED>(c, a, threads, lds);
        return launch_slots<kRowsRunMaxSlots, ROWS_FIXED>(c, a, threads, lds);
    }
    if (slots == 4) return launch_slots<4, ROWS_AHEAD>(c, a, threads, lds);
    if (slots == 8) return launch_slots<8, ROWS_AHEAD>(c, a, threads, lds);
    if (slots == 12) return launch_slots<12, ROWS_AHEAD>(c, a, threads, lds);
    if (slots == 16) return launch_slots<16, ROWS_AHEAD>(c, a, threads, lds);
    return launch_slots<kAheadSlots, ROWS_AHEAD>(c, a, threads, lds);
}

size_t round64(size_t bytes) { return (bytes + 63) & ~(size_t)63; }

struct RunSpace {  // of the exchange memory, in bytes; the device's launches agree on what is not words
    size_t words, finished, keep, wz, wy, wmean, wloss, total;
    RunSpace(const gpga_ctx* c, const RunPlan& p, int32_t B, int64_t T) {
        words = 0;
        finished = 64;
        keep = finished + round64((size_t)c->num_cus * sizeof(uint32_t));
        wz = keep + (c->mu != 0.f ? round64((size_t)c->n * c->d * 8) : 0);
        wy = wz + round64((size_t)T * c->n * B * p.P * 16);
        wmean = wy + round64((size_t)T * c->n * c->d * 8);
        wloss = wmean + round64((size_t)T * c->d * 8);
        total = wloss + round64((size_t)T * c->n * 8);
    }
};

}  // namespace

RowsRun rows_run_for(const gpga_ctx* c, int64_t wanted, const int32_t* idx, int32_t B) {
    const RowsRun no;
    if (wanted < kRowsRunFewest || !c->default_geometry() || !c->opt_rows_run || (c->problem != PROB_LSQ && c->problem != PROB_LOGREG)) return no;
    if (c->trace && c->k < c->trace_cap) return no;  // the trace wants every iterate
    const bool sparse = c->topo == GPGA_TOPO_GRID || c->topo == GPGA_TOPO_EXPO || c->topo == GPGA_TOPO_CUSTOM;
    if (sparse && (!c->csr_ready || !c->csr_off_d)) return no;
    if (c->n < 4 || c->n > 128 || c->d < 32 || c->max_lds_block < 130 * 1024 || (int64_t)c->n * c->ld > 0x7fffffff) return no;
    const GlobalOrder order = global_order(c);
    if (order.U != 4 || order.RL * order.wpb < 2) return no;  // not on these sizes: column_mean adds in no other way
    const int32_t Beff = idx ? B : c->M;
    if (Beff < 1 || Beff > kRowWaves * kRowsRunMaxSlots) return no;
    RowsRun run;
    run.B = Beff;
    run.splitters = order.RL * order.wpb;
    run.mean64 = small_run_fits(c, idx, B);
    if (run.mean64 && (wanted < 4 || (int64_t)c->n * Beff * c->d < 1280)) return no;
    run.plan = plan_run(c->n, c->d, c->num_cus, Beff, idx != nullptr);
    if (!run.plan.P) return no;
    int64_t T = kRowsRunMaxWords / ((int64_t)c->n * c->d);
    if (T > kRowsRunMaxIters) T = kRowsRunMaxIters;
    if (idx && T > kRowsRunStaged / Beff) T = kRowsRunStaged / Beff;
    if (T < kRowsRunFewest) return no;
    RunWork work{c->n, c->d, Beff, idx != nullptr, sparse ? c->csr_max_row : c->topo == GPGA_TOPO_RING ? 2 : c->topo == GPGA_TOPO_EXPO1 ? 1 : 0, sparse, wanted, 0, c->aga};
    if (c->aga) work.averages = wanted / c->H;
    else if (c->topo == GPGA_TOPO_FULL) work.averages = wanted;
    else if (c->H > 0) work.averages = (c->k + wanted) / c->H - c->k / c->H;
    // (16 iterations, us, one workgroup / this: 4 x 32 with one sample 38 / 52, 10 x 40 44 / 52, 20 x 33 with two 68 / 55,
    // 12 x 100 with 8 151 / 61, 9 x 222 with 32 531 / 65; 8 x 100 with 4, 4 iterations 21.9 / 21.7).
    const double other = run.mean64 ? one_workgroup_us(work) : two_launches_us(work, rows_step_fits(c, Beff));
    if (!rows_run_pays(work, run.plan, (int)T, other)) return no;
    // A stream that is being captured keeps its launches per iteration: the number of a launch is the host's.
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &st) != hipSuccess) {
        (void)hipGetLastError();
        return no;
    }
    if (st != hipStreamCaptureStatusNone) return no;
    run.most = (int32_t)T;
    return run;
}

bool launch_rows_run(gpga_ctx* c, const RowsRun& run, int32_t T, const int32_t* idx, bool want_g) {
    const int32_t Beff = run.B;
    const RunPlan& p = run.plan;
    if (T < 1 || T > run.most) return false;
    const RunSpace at(c, p, Beff, T);
    RowsRunArgs a;
    unsigned char* base = nullptr;
    if (!gang_begin(c, at.total, &a.gang, &base)) return false;
    a.x = c->x;
    a.x_other = c->x_new;
    a.m = c->m;
    a.g = want_g ? c->g : nullptr;
    a.m_keep = reinterpret_cast<uint64_t*>(base + at.keep);
    a.feat = c->feat;
    a.tgt = c->tgt;
    a.idx = idx;
    a.aga = c->aga ? &c->host->aga : nullptr;
    if (c->aga) a.begin = aga_begin(c);
    a.wz = reinterpret_cast<uint64_t*>(base + at.wz);
    a.wy = reinterpret_cast<uint64_t*>(base + at.wy);
    a.wmean = reinterpret_cast<uint64_t*>(base + at.wmean);
    a.wloss = reinterpret_cast<uint64_t*>(base + at.wloss);
    a.gang.words = reinterpret_cast<GangWords*>(base);
    a.gang.finished = reinterpret_cast<uint32_t*>(base + at.finished);
    a.gang.count = &c->host->given_up;
    a.gives_up = c->opt_run_give_up < 0 ? -1 : c->opt_run_give_up % (c->n * p.P);
    a.gang.limit = (uint32_t)(c->opt_run_wait_us * 1e-6 * c->clock_hz);
    a.ld = c->ld;
    a.d = c->d;
    a.n = c->n;
    a.B = Beff;
    a.M = c->M;
    a.T = T;
    a.P = p.P;
    a.LP = log2_ceil(p.P);
    a.threads = kWave * (p.QW * p.RG + std::min(kRowsRunWaves - p.QW * p.RG, 4));
    a.w = p.w;
    a.QW = p.QW;
    a.RG = p.RG;
    const bool sparse = c->topo == GPGA_TOPO_GRID || c->topo == GPGA_TOPO_EXPO || c->topo == GPGA_TOPO_CUSTOM;
    a.mode = sparse ? kRunSparse : c->topo == GPGA_TOPO_RING ? MODE_RING : c->topo == GPGA_TOPO_EXPO1 ? MODE_PEER : MODE_SELF;
    a.off = c->csr_off_d;
    a.val = c->csr_ellval_d;
    a.wptr = c->csr_ptr_d;
    a.K = c->csr_max_row;
    a.splitters = run.splitters;
    a.inv_n = 1.0f / (float)c->n;
    a.mu = c->mu;
    a.mean64 = run.mean64;
    a.problem = c->problem;
    a.mom = c->mu == 0.f ? 0 : c->nesterov ? 2 : 1;
    for (int t = 0; t < T; ++t) {
        a.lr[t] = scheduled_lr(c, c->k + t);
        a.shift[t] = !c->aga && is_global_iteration(c->topo, c->H, c->k + t) ? -1 : one_peer_shift(c->n, c->k + t);
    }
    const int slots = slots_for(p.slots, !idx);
    const RunLds lds(c->n, Beff, p.w, p.QW, p.RG, slots, idx ? T * Beff : Beff, sparse ? c->csr_max_row : 0);
    const hipError_t e = launch_run(c, a, slots, a.threads, (size_t)lds.bytes);
    gang_end(c, e == hipSuccess);
    if (e != hipSuccess) (void)hipGetLastError();
    return e == hipSuccess;
}
