// Column reductions over the node axis and row fills.
//
//  * node mean       xbar = (1/n) sum_i x_i                       (App. A notation)
//  * consensus error ||X - 1 xbar^T||_F^2 = sum_c sum_i (x_ic - xbar_c)^2
//                    (the consensus distance of Sec. 4 / App. B)
//  * fill            every row <- one d-vector (Algorithm 1: all x_i^(0) equal)
//
// Both reductions read X exactly once (4 B per element).  The consensus error
// uses the shifted one-pass form with row 0 as the shift:
//     d_i = x_i - x_0 ;  sum_i (x_i - xbar)^2 = sum_i d_i^2 - (sum_i d_i)^2 / n
// with d_i formed in fp32 (exact or nearly so when rows are close) and both
// sums carried in fp64, so the subtraction never loses the small quantity the
// method is about.  Column results are reduced with a wavefront shuffle, an LDS
// step across waves and one partial per workgroup; a last single-workgroup
// kernel adds the partials in a fixed order (bitwise reproducible).
#include "gpga_internal.hpp"
#include "gpga_unit.hpp"

namespace {

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_down(v, off, kWave);
    return v;
}

__device__ __forceinline__ v4f ld_stream(const v4f* p) {
    return __builtin_nontemporal_load(p);
}

struct d4 {
    double x, y, z, w;
};
__device__ __forceinline__ void acc_add(double& a, float v) { a += (double)v; }
__device__ __forceinline__ void acc_add(d4& a, v4f v) {
    a.x += (double)v.x;
    a.y += (double)v.y;
    a.z += (double)v.z;
    a.w += (double)v.w;
}
__device__ __forceinline__ void acc_sq(double& a, float v) { a += (double)v * (double)v; }
__device__ __forceinline__ void acc_sq(d4& a, v4f v) {
    a.x += (double)v.x * v.x;
    a.y += (double)v.y * v.y;
    a.z += (double)v.z * v.z;
    a.w += (double)v.w * v.w;
}
__device__ __forceinline__ float to_mean(double a, double inv_n) { return (float)(a * inv_n); }
__device__ __forceinline__ v4f to_mean(const d4& a, double inv_n) {
    v4f r;
    r.x = (float)(a.x * inv_n);
    r.y = (float)(a.y * inv_n);
    r.z = (float)(a.z * inv_n);
    r.w = (float)(a.w * inv_n);
    return r;
}
// Squared deviations of a unit's columns; the first `dup` of them are counted with the unit before.
__device__ __forceinline__ double col_ss(double s1, double s2, double inv_n, int) {
    const double v = s2 - s1 * s1 * inv_n;
    return v > 0.0 ? v : 0.0;
}
__device__ __forceinline__ double col_ss(const d4& s1, const d4& s2, double inv_n, int dup) {
    return (dup > 0 ? 0.0 : col_ss(s1.x, s2.x, inv_n, 0)) + (dup > 1 ? 0.0 : col_ss(s1.y, s2.y, inv_n, 0)) +
           (dup > 2 ? 0.0 : col_ss(s1.z, s2.z, inv_n, 0)) + col_ss(s1.w, s2.w, inv_n, 0);
}

template <typename T>
struct AccOf;
template <>
struct AccOf<float> {
    typedef double type;
    __device__ static double zero() { return 0.0; }
};
template <>
struct AccOf<v4f> {
    typedef d4 type;
    __device__ static d4 zero() { return {0.0, 0.0, 0.0, 0.0}; }
};

constexpr int U = 4;

// Column unit number u of a reduction: its first column, moved left at a ragged end (reads only, so overlapping units
// need not share a wavefront), and how many of its columns belong to the unit before.
template <typename T>
__device__ __forceinline__ int64_t reduce_column(int64_t u, int64_t d, int* dup) {
    constexpr int V = sizeof(T) / sizeof(float);
    const int64_t c = u * V > d - V ? d - V : u * V;
    *dup = (int)(u * V - c);
    return c;
}

__device__ __forceinline__ void acc_add(double& a, const double& b) { a += b; }
__device__ __forceinline__ void acc_add(d4& a, const d4& b) {
    a.x += b.x;
    a.y += b.y;
    a.z += b.z;
    a.w += b.w;
}

// Both reductions: a workgroup shares the rows of its column units among RS groups of lanes (rows group, group + RS,
// ...), whose fp64 sums meet in LDS in group order.  RS = 1 (256 units a workgroup) streams wide arrays at the memory's
// rate; narrow ones would leave most of the chip idle and a few lanes with all the rows, so they get 4 or 16 groups of
// a wavefront each (64 units a workgroup).  Consensus distance + mean,
// against one lane a column throughout: n = 256, d = 1172 62.5 -> 26.5 us, n = 100, d = 50 000 56.7 -> 27.7, n = 64,
// d = 100 000 44.9 -> 29.1; rows without 16-byte alignment (n = 64, d = 5 000 001) 517 -> 466.
// CL column units a workgroup: 64 with shared rows, else 256, or 1024 on arrays that keep every compute unit at it to the end
// (wide_reduce): the 16 KiB of a row that such a workgroup reads at a time keep fewer memory pages open (64 x 25.6M
// distance and mean 2113 -> 2065 us, 16 x 30M 666 -> 642, 256 x 1M 349 -> 337; 64 x 400 000 52 -> 65).
template <typename T, int RS, int CL>
__global__ void __launch_bounds__(CL * RS) k_col_mean(const float* __restrict__ x, int64_t ld, int64_t d, int64_t units,
                                                  int32_t n, float* __restrict__ xbar) {
    typedef typename AccOf<T>::type Acc;
    __shared__ Acc s_acc[RS > 1 ? RS - 1 : 1][CL];
    const int lane = threadIdx.x % CL, grp = threadIdx.x / CL;
    const int64_t u = (int64_t)blockIdx.x * CL + lane;
    const bool on = u < units;
    int dup;
    const int64_t c = reduce_column<T>(on ? u : 0, d, &dup);
    const float* __restrict__ xp = x + c;
    Acc acc = AccOf<T>::zero();
    for (int base = grp; base < n; base += U * RS) {
        T v[U];
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (base + k * RS < n) v[k] = ld_unit<T>(xp + (int64_t)(base + k * RS) * ld);
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (base + k * RS < n) acc_add(acc, v[k]);
    }
    if (RS > 1) {
        if (grp > 0) s_acc[grp - 1][lane] = acc;
        __syncthreads();
        if (grp > 0) return;
#pragma unroll
        for (int k = 0; k < RS - 1; ++k) acc_add(acc, s_acc[k][lane]);
    }
    if (on) *reinterpret_cast<typename Unit<T>::mem*>(xbar + c) = to_mean(acc, 1.0 / (double)n);
}

template <typename T, int RS, int CL>
__global__ void __launch_bounds__(CL * RS) k_consensus(const float* __restrict__ x, int64_t ld, int64_t d, int64_t units,
                                                   int32_t n, double* __restrict__ partials) {
    typedef typename AccOf<T>::type Acc;
    __shared__ Acc s_acc[2][RS > 1 ? RS - 1 : 1][CL];
    __shared__ double s_buf[CL / kWave];
    const int lane = threadIdx.x % CL, grp = threadIdx.x / CL;
    const int64_t u = (int64_t)blockIdx.x * CL + lane;
    const bool on = u < units;
    int dup;
    const float* __restrict__ xp = x + reduce_column<T>(on ? u : 0, d, &dup);
    const T x0 = ld_unit_cached<T>(xp);
    Acc s1 = AccOf<T>::zero(), s2 = AccOf<T>::zero();
    for (int base = RS == 1 ? 1 : grp; base < n; base += U * RS) {
        T v[U];
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (base + k * RS < n) v[k] = ld_unit<T>(xp + (int64_t)(base + k * RS) * ld);
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (base + k * RS < n) {
                const T dlt = v[k] - x0;
                acc_add(s1, dlt);
                acc_sq(s2, dlt);
            }
    }
    if (RS > 1) {
        if (grp > 0) {
            s_acc[0][grp - 1][lane] = s1;
            s_acc[1][grp - 1][lane] = s2;
        }
        __syncthreads();
        if (grp == 0) {
#pragma unroll
            for (int k = 0; k < RS - 1; ++k) {
                acc_add(s1, s_acc[0][k][lane]);
                acc_add(s2, s_acc[1][k][lane]);
            }
        }
    }
    double ss = on && grp == 0 ? col_ss(s1, s2, 1.0 / (double)n, dup) : 0.0;
    ss = wave_sum(ss);
    if (RS > 1) {  // the first wavefront has all the columns
        if (threadIdx.x == 0) partials[blockIdx.x] = ss;
        return;
    }
    const int wl = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    if (wl == 0) s_buf[wave] = ss;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < CL / kWave; ++w) t += s_buf[w];
        partials[blockIdx.x] = t;
    }
}

// out[0] = sum of `count` partials, one workgroup, fixed order.
__global__ void __launch_bounds__(256) k_final_sum(const double* __restrict__ partials,
                                                   int64_t count, double* __restrict__ out) {
    __shared__ double s_buf[4];
    double acc = 0.0;
    for (int64_t t = threadIdx.x; t < count; t += blockDim.x) acc += partials[t];
    acc = wave_sum(acc);
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    if (lane == 0) s_buf[wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = (s_buf[0] + s_buf[1]) + (s_buf[2] + s_buf[3]);
}

// slot[0] = sqrt(sum of `count` partials), one workgroup, fixed order: with 256 threads that of k_final_sum, so that a reduction
// pass gives the same bits whichever entry point asks.  One-shot steps leave a partial a workgroup, and lone
// wavefronts one for every 256 columns: 1024 threads with eight loads in flight from 1025 partials on (a traced step of
// 8 x 25.6M on the ring 824 -> 748 us, 4 x 100M 1677 -> 1340, 2 x 200M one-peer 2345 -> 1455).
template <int TH>
__global__ void __launch_bounds__(TH) k_trace_store(const double* __restrict__ partials, int64_t count, double* __restrict__ slot) {
    __shared__ double s_buf[TH / kWave];
    constexpr int kAhead = TH > 256 ? 8 : 1;
    double acc = 0.0;
    for (int64_t t = threadIdx.x; t < count; t += TH * kAhead) {
        double v[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) v[u] = t + u * TH < count ? partials[t + u * TH] : 0.0;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) acc += v[u];
    }
    acc = wave_sum(acc);
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    if (lane == 0) s_buf[wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double sum = 0.0;
#pragma unroll
        for (int w = 0; w < TH / kWave; w += 4) sum += (s_buf[w] + s_buf[w + 1]) + (s_buf[w + 2] + s_buf[w + 3]);
        slot[0] = sqrt(sum);
    }
}

// out[0] = (1/count) sum v[i], one workgroup, fixed order.
__global__ void __launch_bounds__(256) k_mean_f32(const float* __restrict__ v, int64_t count,
                                                  double* __restrict__ out) {
    __shared__ double s_buf[4];
    double acc = 0.0;
    for (int64_t t = threadIdx.x; t < count; t += blockDim.x) acc += (double)v[t];
    acc = wave_sum(acc);
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    if (lane == 0) s_buf[wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = ((s_buf[0] + s_buf[1]) + (s_buf[2] + s_buf[3])) / (double)count;
}

constexpr int kFillRows = 16;  // rows a lane fills: short chains of stores, and a grid that narrow arrays fill too
template <typename T>
__global__ void __launch_bounds__(256) k_fill_rows(float* __restrict__ dst, int64_t ld, int64_t d, int64_t units,
                                                   int32_t n, const float* __restrict__ src) {
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= units) return;
    int dup;
    const int64_t c = reduce_column<T>(u, d, &dup);
    const T v = src ? ld_unit_cached<T>(src + c) : T(0);
    const int32_t r0 = blockIdx.y * kFillRows, r1 = r0 + kFillRows < n ? r0 + kFillRows : n;
    for (int32_t row = r0; row < r1; ++row) *reinterpret_cast<typename Unit<T>::mem*>(dst + c + (int64_t)row * ld) = v;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Plain streaming kernels used to measure what this chip's memory system delivers
// for reads, writes and copies (the context in which the fused step's rate is read).
// kind 0: read only (the sum keeps the loads alive), kind 1: write only, kind 2: copy
// src -> dst, kind 3: the fused step's arithmetic on flat arrays (read src, src2,
// inout; write inout, dst).  128-bit non-temporal accesses, consecutive lanes on
// consecutive 16-byte words; one word per lane, or grid-stride when the grid is capped.
template <int KIND>
__global__ void __launch_bounds__(256) k_probe_stream(const v4f* __restrict__ src, v4f* __restrict__ dst,
                                                      const v4f* __restrict__ src2, v4f* __restrict__ inout,
                                                      int64_t count, float* __restrict__ sink) {
    v4f acc = v4f(0);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
#pragma unroll 4
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < count; t += stride) {
        if (KIND == 0) acc += ld_stream(src + t);
        if (KIND == 1) __builtin_nontemporal_store(v4f(1.0f), dst + t);
        if (KIND == 2) __builtin_nontemporal_store(ld_stream(src + t), dst + t);
        if (KIND == 3) {  // the fused step's mix without any row structure: 3 reads, 2 writes
            const v4f xv = ld_stream(src + t), mv = ld_stream(inout + t), gv = ld_stream(src2 + t);
            const v4f mom = 0.9f * mv + gv;
            __builtin_nontemporal_store(mom, inout + t);
            __builtin_nontemporal_store(xv - 0.1f * mom, dst + t);
        }
    }
    if (KIND == 0) {
        float v = acc.x + acc.y + acc.z + acc.w;
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_down(v, off, kWave);
        if ((threadIdx.x & (kWave - 1)) == 0 && v == 12345.678f) atomicAdd(sink, v);  // practically never taken
    }
}

}  // namespace

hipError_t launch_probe_stream(int kind, const float* src, float* dst, const float* src2, float* inout,
                               int64_t count16, float* sink, int64_t blocks, hipStream_t st) {
    const v4f* s = reinterpret_cast<const v4f*>(src);
    v4f* d = reinterpret_cast<v4f*>(dst);
    const v4f* s2 = reinterpret_cast<const v4f*>(src2);
    v4f* io = reinterpret_cast<v4f*>(inout);
    const dim3 grid((unsigned)blocks), block(256);
    if (kind == 0) hipLaunchKernelGGL((k_probe_stream<0>), grid, block, 0, st, s, d, s2, io, count16, sink);
    else if (kind == 1) hipLaunchKernelGGL((k_probe_stream<1>), grid, block, 0, st, s, d, s2, io, count16, sink);
    else if (kind == 2) hipLaunchKernelGGL((k_probe_stream<2>), grid, block, 0, st, s, d, s2, io, count16, sink);
    else hipLaunchKernelGGL((k_probe_stream<3>), grid, block, 0, st, s, d, s2, io, count16, sink);
    return hipGetLastError();
}

// Row groups per workgroup of the two reductions over `units` column units: as few as give the chip lanes enough, for the sum
// of the partials follows in one workgroup, and rows enough for every group to keep its loads in flight.  Consensus distance
// with 1 / 4 groups: 4 x 900 000 8.9 / 11.5 us, 16 x 520 000 8.1 / 9.5, 256 x 400 000 (mean) 60 / 64; with 4 / 16 groups:
// 33 x 150 000 8.0 / 10.0; with 1 / 16: 64 x 250 000 18.9 / 15.8, 64 x 50 000 11.8 / 7.2.
static int reduce_split(int64_t units, int32_t n) {
    return units >= 98304 ? 1 : n <= 32 || units >= (n <= 48 ? 24576 : 49152) ? 4 : 16;
}

// Whether unsplit reductions take workgroups of 1024 units.  Large ones end in a round of their own, so the last round of a
// workgroup a compute unit is to be half full, unless it is one of many: three on up to 24 rows, ten on more.  Distance and
// mean, us with 256 / 1024, by workgroups of 1024: 263 64 rows 116 / 134, 8 rows 28 / 31, 16 rows 385 49.1 / 50.6; 64 rows 451
// 172 / 161, 521 213 / 223, 701 255 / 250, 801 299 / 311, 941 344 / 338, 1046 392 / 406, 3101 1209 / 1149; 8 rows 801 56 / 54,
// 1046 71 / 65.
static bool wide_reduce(const gpga_ctx* c, int64_t units) {
    if (units < 245760) return false;
    const int64_t blocks = (units + 1023) / 1024, cus = c->num_cus, rounds = blocks / cus, last = blocks % cus;
    return last == 0 || last * 100 >= cus * 52 || rounds >= (c->n <= 24 ? 3 : 10);
}

// One per 256 units on wide arrays although the launch may write a quarter of that: the width that
// gpga_consensus_error_static refuses does not move with the launch shape.
size_t consensus_partials_used(const gpga_ctx* c) {
    const int64_t units = c->d < 4 ? c->d : (c->d + 3) / 4;
    const int lanes = (c->d < 4 ? 16 : reduce_split(units, c->n)) > 1 ? kWave : 256;
    return (size_t)((units + lanes - 1) / lanes);
}

size_t consensus_partials_needed(const gpga_ctx* c) {
    // at most one per 256 columns (64 units) and a narrow last one, + 1 result slot
    return (size_t)((c->d / 4 + 255) / 256) + (size_t)((c->d + 255) / 256) + 2;
}

template <typename T>
static hipError_t launch_fill(const gpga_ctx* c, float* dst, const float* src) {
    constexpr int V = sizeof(T) / sizeof(float);
    const int64_t units = (c->d + V - 1) / V;
    for (int64_t row = 0; row < c->n; row += (int64_t)kFillRows * 65535) {
        const int64_t rows = c->n - row < (int64_t)kFillRows * 65535 ? c->n - row : (int64_t)kFillRows * 65535;
        hipLaunchKernelGGL((k_fill_rows<T>), dim3((unsigned)((units + 255) / 256), (unsigned)((rows + kFillRows - 1) / kFillRows)),
                           dim3(256), 0, c->stream, dst + row * c->ld, c->ld, c->d, units, (int32_t)rows, src);
    }
    return hipGetLastError();
}

hipError_t launch_fill_rows(const gpga_ctx* c, float* dst, const float* src) {
    return c->d >= 4 ? launch_fill<v4f>(c, dst, src) : launch_fill<float>(c, dst, src);
}

template <typename T, int RS, int CL>
static hipError_t launch_mean_split(const gpga_ctx* c, int64_t units, float* xbar) {
    const int64_t blocks = (units + CL - 1) / CL;
    hipLaunchKernelGGL((k_col_mean<T, RS, CL>), dim3((unsigned)blocks), dim3(CL * RS), 0, c->stream, c->x, c->ld, c->d, units,
                       c->n, xbar);
    return hipGetLastError();
}

hipError_t launch_col_mean(const gpga_ctx* c, float* xbar) {
    if (c->d < 4) return launch_mean_split<float, 16, kWave>(c, c->d, xbar);
    const int64_t units = (c->d + 3) / 4;
    const int split = reduce_split(units, c->n);
    if (split == 1 && wide_reduce(c, units)) return launch_mean_split<v4f, 1, 1024>(c, units, xbar);
    if (split == 1) return launch_mean_split<v4f, 1, 256>(c, units, xbar);
    return split == 4 ? launch_mean_split<v4f, 4, kWave>(c, units, xbar) : launch_mean_split<v4f, 16, kWave>(c, units, xbar);
}

template <typename T, int RS, int CL>
static hipError_t launch_consensus_split(const gpga_ctx* c, int64_t units, double* parts, size_t cap, int64_t* count) {
    const int64_t blocks = (units + CL - 1) / CL;
    if ((size_t)blocks > cap) return hipErrorOutOfMemory;
    hipLaunchKernelGGL((k_consensus<T, RS, CL>), dim3((unsigned)blocks), dim3(CL * RS), 0, c->stream, c->x, c->ld, c->d, units,
                       c->n, parts);
    *count = blocks;
    return hipGetLastError();
}

// Per-workgroup partial sums of squared deviations of the live X into parts[0 ..] (room for
// `cap` doubles); *count receives their number.
static hipError_t launch_consensus_partials(const gpga_ctx* c, double* parts, size_t cap, int64_t* count) {
    *count = 0;
    if (c->d < 4) return launch_consensus_split<float, 16, kWave>(c, c->d, parts, cap, count);
    const int64_t units = (c->d + 3) / 4;
    const int split = reduce_split(units, c->n);
    if (split == 1 && wide_reduce(c, units)) return launch_consensus_split<v4f, 1, 1024>(c, units, parts, cap, count);
    if (split == 1) return launch_consensus_split<v4f, 1, 256>(c, units, parts, cap, count);
    return split == 4 ? launch_consensus_split<v4f, 4, kWave>(c, units, parts, cap, count)
                      : launch_consensus_split<v4f, 16, kWave>(c, units, parts, cap, count);
}

hipError_t launch_consensus_sq(gpga_ctx* c, size_t* partials_needed) {
    *partials_needed = consensus_partials_needed(c);
    int64_t count = 0;
    // slot 0 of the context's scratch holds the result of the synchronous entry point
    const hipError_t e = launch_consensus_partials(c, c->partials + 1, c->partials_cap - 1, &count);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_final_sum, dim3(1), dim3(256), 0, c->stream, c->partials + 1, count, c->partials);
    return hipGetLastError();
}

hipError_t launch_consensus_trace(gpga_ctx* c, double* slot) {
    return launch_consensus_distance(c, c->partials + 1, c->partials_cap - 1, slot);
}

hipError_t launch_consensus_distance(const gpga_ctx* c, double* scratch, size_t scratch_cap, double* slot) {
    int64_t count = 0;
    const hipError_t e = launch_consensus_partials(c, scratch, scratch_cap, &count);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_trace_store<256>, dim3(1), dim3(256), 0, c->stream, scratch, count, slot);
    return hipGetLastError();
}

// The partial sums that a step kernel left.
hipError_t launch_trace_store(const gpga_ctx* c, const double* partials, int64_t count, double* slot) {
    if (count > 1024) hipLaunchKernelGGL(k_trace_store<1024>, dim3(1), dim3(1024), 0, c->stream, partials, count, slot);
    else hipLaunchKernelGGL(k_trace_store<256>, dim3(1), dim3(256), 0, c->stream, partials, count, slot);
    return hipGetLastError();
}

hipError_t launch_mean_f32(const gpga_ctx* c, const float* v, int64_t count, double* out) {
    hipLaunchKernelGGL(k_mean_f32, dim3(1), dim3(256), 0, c->stream, v, count, out);
    return hipGetLastError();
}
