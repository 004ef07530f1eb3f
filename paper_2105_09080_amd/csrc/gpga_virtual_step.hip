// Second half of an iteration on virtual features, in one launch (gpga_run): gradient sum, local update and gossip step.
//
//     g_i = sum_b coef_b * h_ib ;  m_i, y_i from g_i, x_i ;  x_new_i = stencil of y along the cycles of i -> (i + S) mod n
//
// The coefficients come from the margin pass; from there on columns are apart.  Regenerating the features is bound by vector
// issue, the step by memory, and as launches of their own each leaves the other unit idle and g travels to memory and
// back.  Here a wavefront walks down the rows of 64 column quads as the walk kernel does: the loads of the next row are under
// way while the features of this one are regenerated, and g is stored only if the caller wants it left.  Up to 16 wavefronts
// share the rows of a tile where tiles are few; their boundary values meet in LDS.
// A row's coefficients sit in the lanes of the wavefront, and only samples whose coefficient is not exactly zero are
// regenerated (see k_virtual_accum), two at a time: two independent Philox chains keep the units busy with four wavefronts a SIMD.
// An iteration of 1024 x 1M with 16 samples, margin pass included, ring / one-peer graph: all coefficients in use 17.8 / 17.9
// -> 17.3 / 17.2 ms (this kernel 9.6: 73 vector instructions a quad and sample, 86 % of the issue slots; 3906 tiles are 3.8
// wavefronts a SIMD, and one more row ahead changes nothing), most of them zero 14.7 -> 13.5; 100 x 1M with 32 samples 3160 ->
// 3220 us (ring) and even (one-peer), 8 x 1M with 8 samples 175 -> 164.
#include <numeric>
#include <type_traits>

#include "gpga_internal.hpp"
#include "gpga_rng.hpp"
#include "gpga_spread.hpp"
#include "gpga_unit.hpp"

namespace {

struct VirtualStepArgs {
    StepGeom ge;
    float* g_out;         // NULL: the gradients of this iteration are not wanted
    const float* coef;    // n x B
    const int32_t* idx;   // n x B
    int32_t B;
    uint32_t k0, k1;
    float mu_sigma;
    int32_t S, C, L;      // C cycles of L rows, stride S (W = I: one of n rows, never closed)
    int32_t Qc, Qs;       // wavefronts of a tile: Qc share the cycles (C is a multiple), Qs the rows of a cycle
    double* spread_partials;  // TRACE: one sum of squared deviations a tile
};
constexpr int kVirtualStepWaves = 16;

template <int MODE, int MOM, bool TRACE>
__global__ void __launch_bounds__(kWave* kVirtualStepWaves) k_virtual_step(const VirtualStepArgs a) {
    extern __shared__ __align__(16) unsigned char s_raw[];  // Qs > 1: first and last y of every wavefront
    v4f(*__restrict__ s_first)[kWave] = reinterpret_cast<v4f(*)[kWave]>(s_raw);
    v4f(*__restrict__ s_last)[kWave] = s_first + blockDim.x / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per_tile = a.Qc * a.Qs, tile_l = wave / per_tile;
    const int cw = (wave - tile_l * per_tile) / a.Qs, seg = wave % a.Qs;
    const int tiles_wg = blockDim.x / kWave / per_tile;
    const int64_t tile_i = (int64_t)blockIdx.x * tiles_wg + tile_l;
    const int n = a.ge.n;
    const int64_t ld = a.ge.ld, d = a.ge.d;
    const float lr = a.ge.lr, mu = a.ge.mu;
    const float third = 1.0f / 3.0f;
    // Quads of the counter RNG start at multiples of four, whatever the width: the last one of a ragged width is a part.
    const uint32_t q = (uint32_t)tile_i * kWave + lane;
    const int64_t col = (int64_t)q * 4;
    // Every lane of the workgroup has a whole quad: one answer for all its tiles, since their wavefronts meet at the barriers of
    // the body that it chooses.
    const bool whole = ((int64_t)blockIdx.x + 1) * tiles_wg * kWave * 4 <= d;
    const int have = whole || col + 4 <= d ? 4 : col < d ? (int)(d - col) : 0;
    const PhiloxQuad quad(q, TAG_FEAT, a.k1);
    ColumnSpread<v4f> spread;
    if (TRACE) spread.reset(whole || have == 4 ? ld_unit_cached<v4f>(a.ge.x + col) : v4f(0.f));

    auto tile = [&](auto all) {  // a body of its own for workgroups of whole quads: no branches around its loads and stores
    constexpr bool kAll = decltype(all)::value;
    auto load = [&](const float* p) -> v4f {
        if (kAll || have == 4) return ld_unit<v4f>(p);
        v4f v = v4f(0.f);
        if (have > 0) v.x = p[0];
        if (have > 1) v.y = p[1];
        if (have > 2) v.z = p[2];
        return v;
    };
    auto store = [&](float* p, const v4f& v) {
        if (kAll || have == 4) {
            st_unit<v4f>(p, v);
            return;
        }
        if (have > 0) p[0] = v.x;
        if (have > 1) p[1] = v.y;
        if (have > 2) p[2] = v.z;
    };
    struct Row {
        v4f x, m;
        float cf;    // coefficient and row number of sample `lane`
        int32_t id;
    };
    auto fetch = [&](Row& r, int row) {
        const int64_t o = (int64_t)row * ld + col;
        const int64_t b = (int64_t)row * a.B + (lane < a.B ? lane : 0);
        r.cf = a.coef[b];
        r.id = a.idx[b];
        r.x = load(a.ge.x + o);
        if (MOM) r.m = load(a.ge.m + o);
    };
    auto gradient = [&](const Row& r, int row) -> v4f {
        v4f g = v4f(0.f);
        uint64_t left = __ballot(lane < a.B && r.cf != 0.f);  // NaN, the mark of a sample index out of range, counts
        if (!left) return g;
        const v4f shift = a.mu_sigma * normals4(q, (uint32_t)row, 0u, TAG_MU, a.k0, a.k1);
        auto take = [&](float* cf) -> uint32_t {
            const int b = __builtin_ctzll(left);
            left &= left - 1;
            *cf = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r.cf), b));
            return (uint32_t)__builtin_amdgcn_readlane(r.id, b);
        };
        while (left) {
            float c0, c1;
            const uint32_t m0 = take(&c0);
            if (left) {
                const uint32_t m1 = take(&c1);
                const v4f h0 = virtual_quad(shift, quad, (uint32_t)row, m0, a.k0, a.k1);
                const v4f h1 = virtual_quad(shift, quad, (uint32_t)row, m1, a.k0, a.k1);
                g += c0 * h0;
                g += c1 * h1;
            } else {
                g += c0 * virtual_quad(shift, quad, (uint32_t)row, m0, a.k0, a.k1);
            }
        }
        return g;
    };

    const int cycles = a.C / a.Qc;  // every wavefront of the workgroup has as many: they meet at the barriers below
    const int p0 = (int)((int64_t)seg * a.L / a.Qs), p1 = (int)((int64_t)(seg + 1) * a.L / a.Qs);
    for (int cc = 0; cc < cycles; ++cc) {
        const int row_first = (int)((cw * cycles + cc + (int64_t)p0 * a.S) % n);
        auto put = [&](int row, const v4f& v) {
            store(a.ge.x_new + (int64_t)row * ld + col, v);
            if (TRACE) spread.add(v);
        };
        v4f yf = v4f(0.f), ys = v4f(0.f), pp = v4f(0.f), pc = v4f(0.f);
        int row = row_first, row_prev = row_first;
        Row next;
        next.m = v4f(0.f);
        fetch(next, row);
        for (int p = p0; p < p1; ++p) {
            const Row cur = next;
            const int row_next = row + a.S >= n ? row + a.S - n : row + a.S;
            if (p + 1 < p1) fetch(next, row_next);
            const v4f g = gradient(cur, row);
            // The next row's loads have had the gradient's time; waited for here, ahead of this row's stores, they are not
            // waited for together with those stores' acknowledgements.
            asm volatile("" : "+v"(next.x), "+v"(next.m), "+v"(next.cf), "+v"(next.id));
            const int64_t o = (int64_t)row * ld + col;
            if (a.g_out) store(a.g_out + o, g);
            v4f mom = g;
            if (MOM) {
                mom = mu * cur.m + g;
                store(a.ge.m + o, mom);
            }
            const v4f y = MOM == 2 ? cur.x - lr * (g + mu * mom) : cur.x - lr * mom;
            if (MODE == MODE_SELF) put(row, y);
            if (MODE == MODE_PEER && p > p0) put(row_prev, (pc + y) * 0.5f);
            if (MODE == MODE_RING && p > p0 + 1) put(row_prev, (pp + pc + y) * third);
            if (p == p0) yf = y;
            if (p == p0 + 1) ys = y;
            pp = pc;
            pc = y;
            row_prev = row;
            row = row_next;
        }
        if (MODE == MODE_SELF) continue;
        // both ends of the segment: the cycle closes on itself, or on the neighbouring segments
        v4f before = pc, after = yf;
        if (a.Qs > 1) {
            s_first[wave][lane] = yf;
            s_last[wave][lane] = pc;
            __syncthreads();
            const int w0 = wave - seg;
            before = s_last[w0 + (seg + a.Qs - 1) % a.Qs][lane];
            after = s_first[w0 + (seg + 1) % a.Qs][lane];
            __syncthreads();  // the next cycle overwrites them
        }
        if (MODE == MODE_PEER) {
            put(row_prev, (pc + after) * 0.5f);
        } else if (p1 - p0 == 1) {
            put(row_first, (before + yf + after) * third);
        } else {
            put(row_first, (before + yf + ys) * third);
            put(row_prev, (pp + pc + after) * third);
        }
    }
    };
    if (whole) tile(std::true_type{}); else tile(std::false_type{});
    if (TRACE) {  // one wavefront a tile, whole quads
        double v = have == 4 ? spread.sum_sq(1.0 / (double)n) : 0.0;
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_down(v, off, kWave);
        if (lane == 0 && tile_i * kWave * 4 < d) a.spread_partials[tile_i] = v;
    }
}

// Wavefronts of a tile: as few as fill the chip with two a SIMD (kVirtualStepFill), eight rows each at least.
constexpr int64_t kVirtualStepFill = 2048;
int64_t virtual_tiles(const gpga_ctx* c) { return ((c->d + 3) / 4 + kWave - 1) / kWave; }
int virtual_step_waves(const gpga_ctx* c) {
    int q = 1;
    while (q < kVirtualStepWaves && virtual_tiles(c) * q < kVirtualStepFill && 2 * q * 8 <= c->n) q *= 2;
    return q;
}

template <int MODE, int MOM>
hipError_t launch_virtual_mode(const gpga_ctx* c, VirtualStepArgs a, double* spread_partials, int64_t* spread_count) {
    // Four wavefronts a workgroup at least, one for each SIMD: lone ones are packed, five to a SIMD while others idle.
    const int waves = a.Qc * a.Qs < 4 ? 4 : a.Qc * a.Qs, tiles = waves / (a.Qc * a.Qs);
    const dim3 grid((unsigned)((virtual_tiles(c) + tiles - 1) / tiles)), block(kWave * waves);
    const size_t lds = a.Qs > 1 ? 2 * sizeof(v4f) * block.x : 0;
    a.spread_partials = spread_partials;
    // the consensus sums ride along where a wavefront stores whole columns and there is a slot for every tile
    if (spread_partials && spread_count && a.Qc * a.Qs == 1 && c->d % 4 == 0 && virtual_tiles(c) < (int64_t)c->partials_cap) {
        *spread_count = virtual_tiles(c);
        hipLaunchKernelGGL((k_virtual_step<MODE, MOM, true>), grid, block, lds, c->stream, a);
    } else {
        hipLaunchKernelGGL((k_virtual_step<MODE, MOM, false>), grid, block, lds, c->stream, a);
    }
    return hipGetLastError();
}

template <int MOM>
hipError_t launch_virtual_mom(const gpga_ctx* c, int mode, const VirtualStepArgs& a, double* spread_partials, int64_t* spread_count) {
    if (mode == MODE_RING) return launch_virtual_mode<MODE_RING, MOM>(c, a, spread_partials, spread_count);
    if (mode == MODE_PEER) return launch_virtual_mode<MODE_PEER, MOM>(c, a, spread_partials, spread_count);
    return launch_virtual_mode<MODE_SELF, MOM>(c, a, spread_partials, spread_count);
}

}  // namespace

// The accumulate pass deals its work to the SIMDs evenly and eight wavefronts at a time; here they have whole wavefronts of long
// walks, four at a time.  So this form pays where the step's memory time is a good part and few SIMDs have one less:
// up to 8 samples if they are busy for three quarters of the time (64 x 300 000 with 8 270 -> 264 us, 1024 x 40 000
// with 4 373 -> 349), up to 16 for nine tenths (32 x 999 997 with 16 643 -> 610, against 32 x 600 000, where they
// are busy for 76 %, 406 -> 437; 500 x 300 002 2953 -> 3061; 100 x 1M with 32 3138 -> 3238).
bool virtual_step_fits(const gpga_ctx* c, int32_t B) {
    if (!c->default_geometry() || c->problem != PROB_LOGREG_VIRTUAL || B > 16) return false;
    if (c->n > 1 && c->topo != GPGA_TOPO_RING && c->topo != GPGA_TOPO_EXPO1 && c->topo != GPGA_TOPO_NONE) return false;
    const int64_t waves = virtual_tiles(c) * virtual_step_waves(c), simds = 4 * (int64_t)c->num_cus;
    const int64_t slots = (waves + simds - 1) / simds * simds;
    return waves >= kVirtualStepFill && waves * 100 >= slots * (B <= 8 ? 75 : 90);
}

hipError_t launch_virtual_step(const gpga_ctx* c, const StepGeom& geom, const int32_t* idx, int32_t B, int mode, int32_t S, bool want_g,
                               double* spread_partials, int64_t* spread_count) {
    VirtualStepArgs a;
    a.ge = geom;
    a.g_out = want_g ? c->g : nullptr;
    a.coef = c->coef;
    a.idx = idx;
    a.B = B;
    a.k0 = (uint32_t)(c->seed & 0xffffffffu);
    a.k1 = (uint32_t)(c->seed >> 32);
    a.mu_sigma = c->mu_sigma;
    const bool walk = mode == MODE_RING || mode == MODE_PEER;
    a.S = walk ? S : 1;
    a.C = walk ? std::gcd(S, c->n) : 1;
    a.L = c->n / a.C;
    const int waves = virtual_step_waves(c);
    a.Qc = 1;
    while (2 * a.Qc <= waves && a.C % (2 * a.Qc) == 0) a.Qc *= 2;
    a.Qs = waves / a.Qc;
    c->note_path(PATH_VIRTUAL_STEP, 16);
    if (c->mu == 0.f) return launch_virtual_mom<0>(c, mode, a, spread_partials, spread_count);
    return c->nesterov ? launch_virtual_mom<2>(c, mode, a, spread_partials, spread_count)
                       : launch_virtual_mom<1>(c, mode, a, spread_partials, spread_count);
}
