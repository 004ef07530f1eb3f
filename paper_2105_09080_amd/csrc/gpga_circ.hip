// Gossip step with a circulant sparse W (node i mixes nodes i + o_0, ..., i + o_{K-1} mod n with the same weights at every
// node: the static exponential graph), for more nodes than the tile kernel takes with wide lanes.
//
// Two passes move 28 bytes an element and fetch eleven neighbours from the L2s.  Here the column tile of ALL n rows lies
// in LDS - LN lanes of 16 bytes: 128-byte row pieces for n <= 1024, one cache line each - and every element of x, m, g
// is read and of m, x_new written once (20 bytes).  Such a tile fills LDS (128 KiB), so one workgroup has the compute
// unit, and what keeps memory busy is a pipeline over tiles: while the workgroup mixes rows of one tile out of LDS, it
// loads the same rows of its next tile, updates them and keeps their x^(k+1/2) in registers (8 x 16 bytes a thread);
// between two tiles they move to LDS.  Being circulant is what makes the mixing cheap: offsets and weights are scalars,
// a neighbour's address is one add and one wrap.
// (y and two rows of x, m and g in flight fill 108 of 128 registers.  Row addresses of all passes kept over the tiles put 32 a
// lane into scratch memory, 300 x 1M 1267 us against 994; four rows in flight, 16 of them again, are no faster.)
// Bound: memory with n rows open at once.  Static exponential graph, momentum 0.9: n = 1024, d = 1M 6.20 -> 3.6 - 4.1 ms
// (5.0 to 5.7 TB/s of 20 bytes an element), n = 700, d = 500k 2.23 -> 1.39 ms; against the tile kernel with 4-byte lanes n = 512,
// d = 2M 5.68 -> 3.95 ms, n = 256, d = 4M 4.77 -> 3.4 - 3.9 ms, n = 300, d = 1M without momentum 1.18 -> 0.71 ms.
#include "gpga_internal.hpp"
#include "gpga_pace.hpp"
#include "gpga_unit.hpp"

namespace {

constexpr int kCircThreads = 1024;
constexpr int kCircPasses = 8;      // rows a thread takes of a tile
constexpr int kCircAhead = 2;       // row passes in flight

struct CircArgs {
    StepGeom ge;
    int64_t tiles;
    int32_t passes;
    int32_t K;
    int32_t off[kMaxCirculant];     // in [0, n)
    float val[kMaxCirculant];
};

template <int MOM, int LN>
__global__ void __launch_bounds__(kCircThreads) k_step_circ(const CircArgs a) {
    const int RP = blockDim.x / LN;         // rows a pass
    extern __shared__ __align__(16) unsigned char s_raw[];
    v4f* __restrict__ sy = reinterpret_cast<v4f*>(s_raw);  // [n][LN]
    const int n = a.ge.n, total = n * LN;
    const int q = threadIdx.x % LN, first = threadIdx.x / LN;
    const float lr = a.ge.lr, mu = a.ge.mu;
    const int64_t ld = a.ge.ld;
    struct Row {
        v4f x, m, g;
    };
    Row rows[kCircAhead];
    v4f y[kCircPasses];
    // Addresses are formed anew at every use: those of all passes, kept, would not fit the registers beside y and the rows.
    auto row_of = [&](int p) -> int {
        int r = first;
        asm volatile("" : "+v"(r));
        return p * RP + r;
    };
    // Rows behind the last one are loaded as that row and dropped; whole passes behind it are skipped.
    const int passes = a.passes;
    auto load = [&](Row& w, int64_t tile, int p) {
        const int row = row_of(p);
        const int64_t o = (int64_t)(row < n ? row : n - 1) * ld + unit_column<v4f>(a.ge, tile, LN, q);
        w.x = ld_unit<v4f>(a.ge.x + o);
        if (MOM) w.m = ld_unit<v4f>(a.ge.m + o);
        w.g = ld_unit<v4f>(a.ge.g + o);
    };
    auto update = [&](const Row& w, int64_t tile, int p) -> v4f {
        const int row = row_of(p);
        v4f mom = w.g;
        if (MOM) {
            mom = mu * w.m + w.g;
            if (row < n && unit_on(a.ge, tile, LN, q)) st_unit<v4f>(a.ge.m + (int64_t)row * ld + unit_column<v4f>(a.ge, tile, LN, q), mom);
        }
        return MOM == 2 ? w.x - lr * (w.g + mu * mom) : w.x - lr * mom;
    };
    auto mix = [&](int64_t tile, int p) {
        const int row = row_of(p);
        const uint32_t at = (uint32_t)(row * LN + q);
        if (row >= n) return;
        v4f acc = v4f(0.f);
        auto tap = [&](int k) {
            const uint32_t j = at + (uint32_t)(a.off[k] * LN);
            acc += a.val[k] * sy[min(j, j - (uint32_t)total)];  // j - total wraps to a huge number unless j is past the end
        };
        int k = 0;
        for (; k + 4 <= a.K; k += 4) {
#pragma unroll
            for (int t = 0; t < 4; ++t) tap(k + t);
        }
        for (; k < a.K; ++k) tap(k);
        if (unit_on(a.ge, tile, LN, q)) st_unit<v4f>(a.ge.x_new + (int64_t)row * ld + unit_column<v4f>(a.ge, tile, LN, q), acc);
    };
    auto to_lds = [&]() {
        __syncthreads();  // the tile before has been mixed
#pragma unroll
        for (int p = 0; p < kCircPasses; ++p) {
            const int row = row_of(p);
            if (row < n) sy[row * LN + q] = y[p];
        }
        __syncthreads();
    };
    int64_t tile = blockIdx.x;
    const int64_t step = gridDim.x, last = a.tiles - 1;
    // the first tile's rows, then the first passes of the next tile in flight
#pragma unroll
    for (int p = 0; p < kCircPasses; ++p) {
        if (p < passes) {
            load(rows[0], tile, p);
            y[p] = update(rows[0], tile, p);
        }
    }
    to_lds();
    int64_t next = tile + step;
    if (next <= last) {
#pragma unroll
        for (int s = 0; s < kCircAhead; ++s) load(rows[s], next, s);
    }
    for (; next <= last; tile = next, next += step) {
        const int64_t after = next + step <= last ? next + step : next;
#pragma unroll
        for (int p = 0; p < kCircPasses; ++p) {
            if (p < passes) {
                y[p] = update(rows[p % kCircAhead], next, p);
                const int ahead = p + kCircAhead;
                if (ahead < passes) load(rows[p % kCircAhead], next, ahead);
                else load(rows[p % kCircAhead], after, (ahead - passes));
                mix(tile, p);
            }
        }
        to_lds();
    }
#pragma unroll
    for (int p = 0; p < kCircPasses; ++p)
        if (p < passes) mix(tile, p);
}

// Row passes of a tile: the smallest even number (the rows in flight alternate between two sets of registers) whose
// rows, a whole number of wavefronts, fit 1024 threads; 0 if eight are not enough.
template <int LN>
int circ_passes(int n, int* threads) {
    for (int p = 2; p <= kCircPasses; p += 2) {
        constexpr int per_wave = kWave / LN;
        const int rows = ((n + p - 1) / p + per_wave - 1) / per_wave * per_wave;
        if (rows * LN <= kCircThreads) {
            *threads = rows * LN;
            return p;
        }
    }
    return 0;
}

template <int MOM, int LN>
hipError_t launch_circ_lanes(const gpga_ctx* c, CircArgs a) {
    set_units(&a.ge, 4, LN);
    a.tiles = unit_tiles(a.ge, LN);
    int threads = 0;
    a.passes = circ_passes<LN>(a.ge.n, &threads);
    if (!a.passes) return hipErrorInvalidConfiguration;
    const size_t lds = (size_t)a.ge.n * LN * sizeof(v4f);
    static bool attr_set[64] = {false};  // per instantiation and device: more than the default 64 KiB of dynamic LDS
    const int dev = c->device >= 0 && c->device < 64 ? c->device : 0;
    if (!attr_set[dev]) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_step_circ<MOM, LN>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)c->max_lds_block);
        if (e != hipSuccess) return e;
        attr_set[dev] = true;
    }
    const int64_t blocks = balanced_blocks(a.tiles, (int64_t)c->num_cus * resident_per_cu(c, k_step_circ<MOM, LN>, threads, lds, 2));
    if (c->plan_only) return hipSuccess;
    hipLaunchKernelGGL((k_step_circ<MOM, LN>), dim3((unsigned)blocks), dim3(threads), lds, c->stream, a);
    return hipGetLastError();
}

int circ_lanes(int n) { return n > 512 ? 8 : n > 256 ? 16 : 32; }

template <int MOM>
hipError_t launch_circ_rows(const gpga_ctx* c, const CircArgs& a) {
    // the widest row pieces whose tile is 128 KiB at most (8 rows a thread)
    switch (circ_lanes(a.ge.n)) {
        case 8: return launch_circ_lanes<MOM, 8>(c, a);
        case 16: return launch_circ_lanes<MOM, 16>(c, a);
        default: return launch_circ_lanes<MOM, 32>(c, a);
    }
}

}  // namespace

// Row pieces of 128 bytes (more than 512 nodes) want whole cache lines: a piece that straddles two moves twice the bytes, and
// the two lines of a row are fetched by workgroups far apart.  Us this kernel / the others, n = 700: rows on 128 bytes, 250M
// elements 963 / 1544; on 64 bytes 1419 / 1625, with 6M 54 / 45; on 32 bytes 1642 / 1711 and 526 / 404 (60M), on 16 bytes 2551
// / 1676; other rows 2652 / 1788, but where those have 4-byte lanes 29 / 56 (3M).  (Wider pieces lose less: 512-byte ones win
// at any alignment, 256-byte ones win or are even up to 60M elements and are within a fifth either way beyond.)
static bool pieces_pay(const gpga_ctx* c) {
    if (c->n <= 512) return true;
    const uintptr_t at = reinterpret_cast<uintptr_t>(c->x) | reinterpret_cast<uintptr_t>(c->x_new) | reinterpret_cast<uintptr_t>(c->g) |
                         reinterpret_cast<uintptr_t>(c->m) | (uintptr_t)(c->ld * 4);
    const int64_t elements = (int64_t)c->n * c->d;
    if (at % 16 == 0) return at % 128 == 0 || (at % 64 == 0 && elements >= 1 << 24);
    return elements < (c->n <= 640 ? 1 << 22 : 3 << 22);
}

bool circulant_fits(const gpga_ctx* c) {
    // From 225 nodes on: with fewer the tile kernel's 4-byte lanes are as fast or faster (n = 200, d = 1M 790 us against 836;
    // n = 250 1111 against 1028).
    if (c->csr_circ_k == 0 || c->n <= 224 || c->n > 1024 || c->d < 4 || c->max_lds_block < 128 * 1024 || !pieces_pay(c)) return false;
    // Tiles for half the compute units: below, the kernels that split rows over more workgroups are faster (n = 1024,
    // 38 tiles 26 us against 16, 157 tiles 38.4 against 40.4; n = 600, 188 tiles 22 against 55).
    return (c->d + 3) / 4 >= (int64_t)circ_lanes(c->n) * c->num_cus / 2;
}

hipError_t launch_step_circulant(const gpga_ctx* c, const StepGeom& geom) {
    CircArgs a;
    a.ge = geom;
    a.K = c->csr_circ_k;
    for (int k = 0; k < c->csr_circ_k; ++k) {
        a.off[k] = c->csr_circ_off[k];
        a.val[k] = c->csr_circ_val[k];
    }
    if (c->mu == 0.f) return launch_circ_rows<0>(c, a);
    return c->nesterov ? launch_circ_rows<2>(c, a) : launch_circ_rows<1>(c, a);
}
