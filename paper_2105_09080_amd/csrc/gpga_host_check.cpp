// Host-only check program for the parts of libgpga that never touch the GPU: the graph
// builders, the validation of a caller's mixing matrix, the connectivity estimate beta
// (Assumption 3), the schedule arithmetic of Algorithm 1 and the controller that sets the
// rate of paced launches (run here against a model of a launch).  It is compiled from the very
// sources the library uses, with AddressSanitizer and UndefinedBehaviorSanitizer on the host
// side, and run by the CPU test suite: the sanitizers abort the run on any bad access, the
// printed values are compared with the oracle by the test.
//
// Output: one line per fact, "key value...".
#include <cinttypes>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "gpga_exchange.hpp"
#include "gpga_gang.hpp"
#include "gpga_internal.hpp"
#include "gpga_node_run.hpp"
#include "gpga_pace.hpp"
#include "gpga_rows_deal.hpp"
#include "gpga_rows_run.hpp"
#include "gpga_schedule.hpp"

namespace {

int failures = 0;
void expect(bool ok, const char* what) {
    if (!ok) {
        std::printf("FAIL %s\n", what);
        ++failures;
    }
}

void row_col_sums(int32_t n, const HostCsr& w, double* worst_row, double* worst_col) {
    std::vector<double> cols((size_t)n, 0.0);
    *worst_row = 0.0;
    for (int32_t i = 0; i < n; ++i) {
        double r = 0.0;
        for (int32_t p = w.ptr[i]; p < w.ptr[i + 1]; ++p) {
            r += w.val[p];
            cols[(size_t)w.col[p]] += w.val[p];
        }
        *worst_row = std::fmax(*worst_row, std::fabs(r - 1.0));
    }
    *worst_col = 0.0;
    for (double c : cols) *worst_col = std::fmax(*worst_col, std::fabs(c - 1.0));
}

void named_graphs() {
    const int32_t sizes[] = {1, 2, 3, 4, 5, 7, 8, 12, 16, 17, 20, 31, 50, 64, 97, 100, 128, 1024};
    for (int32_t n : sizes) {
        for (int topo = 0; topo < 4; ++topo) {
            HostCsr w;
            const char* name = topo == 0 ? "ring" : topo == 1 ? "grid" : topo == 2 ? "expo" : "expo1";
            if (topo == 0) build_ring_csr(n, &w);
            if (topo == 1) build_grid_csr(n, &w);
            if (topo == 2) build_static_expo_csr(n, &w);
            const int kmax = topo == 3 ? (n >= 500 ? 2 : tau_of(n) + 1) : 1;  // every offset, and the wrap of k mod tau
            for (int k = 0; k < kmax; ++k) {
                if (topo == 3) build_one_peer_csr(n, one_peer_shift(n, k), &w);
                const char* why = validate_csr(n, w, 1e-5);
                expect(why == nullptr, why ? why : "");
                double wr, wc;
                row_col_sums(n, w, &wr, &wc);
                expect(wr <= 1e-6 && wc <= 1e-6, "row / column sums of a named graph");
                std::printf("beta %s %d %d %.12f\n", name, n, k, mixing_beta(n, w));
            }
        }
    }
    // a large ring: the builders and the validation at the scale of n itself (no spectrum: O(n) per Lanczos step is fine,
    // but 2^20 nodes are enough to walk every index path)
    HostCsr big;
    build_ring_csr(1 << 20, &big);
    expect(validate_csr(1 << 20, big, 1e-5) == nullptr, "ring of 2^20 nodes");
    std::printf("beta ring %d 0 %.12f\n", 1 << 20, mixing_beta(1 << 20, big));
}

void rejected_matrices() {
    // every way a caller's arrays can be wrong must come back as a message, never as a bad access
    const int32_t n = 6;
    HostCsr good;
    build_ring_csr(n, &good);
    std::vector<int64_t> ptr(good.ptr.begin(), good.ptr.end());
    HostCsr out;
    expect(copy_csr(n, ptr.data(), good.col.data(), good.val.data(), &out) == nullptr, "good ring copies");
    expect(validate_csr(n, out, 1e-5) == nullptr, "good ring validates");
    expect(copy_csr(n, nullptr, good.col.data(), good.val.data(), &out) != nullptr, "NULL row_ptr");
    expect(copy_csr(n, ptr.data(), nullptr, good.val.data(), &out) != nullptr, "NULL col");
    {
        auto p2 = ptr;
        p2[0] = 1;
        expect(copy_csr(n, p2.data(), good.col.data(), good.val.data(), &out) != nullptr, "row_ptr[0] != 0");
        p2 = ptr;
        p2[3] = p2[2] - 1;
        expect(copy_csr(n, p2.data(), good.col.data(), good.val.data(), &out) != nullptr, "decreasing row_ptr");
        p2 = ptr;
        for (auto& v : p2) v = 0;
        expect(copy_csr(n, p2.data(), good.col.data(), good.val.data(), &out) != nullptr, "fewer than n entries");
    }
    auto broken = [&](int which) {
        HostCsr w = good;
        if (which == 0) w.col[4] = n;           // index one past the end
        if (which == 1) w.col[4] = -1;
        if (which == 2) w.val[5] = -0.25f;
        if (which == 3) w.val[5] = NAN;
        if (which == 4) w.val[5] = INFINITY;
        if (which == 5) w.val[0] += 1e-3f;      // row and column sums off
        if (which == 6) w.ptr[n] -= 1;          // shape does not match the arrays
        if (which == 7) w.ptr.pop_back();
        if (which == 8) w.col[2] = 2;           // row 0 mixes node 2 instead of node 5: rows still sum to 1, columns do not
        return validate_csr(n, w, 1e-5);
    };
    for (int which = 0; which < 9; ++which) {
        const char* why = broken(which);
        std::printf("rejected %d %s\n", which, why ? why : "ACCEPTED");
        expect(why != nullptr, "a defective W was accepted");
    }
    // random doubly stochastic matrices (convex combinations of permutations) and random damage
    std::mt19937_64 rng(12345);
    for (int trial = 0; trial < 200; ++trial) {
        const int32_t m = 1 + (int32_t)(rng() % 40);
        std::vector<std::vector<double>> dense((size_t)m, std::vector<double>((size_t)m, 0.0));
        double wsum = 0.0;
        std::vector<double> wts(4);
        for (auto& v : wts) wsum += (v = 0.05 + (double)(rng() % 1000) / 1000.0);
        for (int t = 0; t < 4; ++t) {
            std::vector<int32_t> perm((size_t)m);
            for (int32_t i = 0; i < m; ++i) perm[(size_t)i] = i;
            for (int32_t i = m - 1; i > 0; --i) std::swap(perm[(size_t)i], perm[(size_t)(rng() % (uint64_t)(i + 1))]);
            for (int32_t i = 0; i < m; ++i) dense[(size_t)i][(size_t)perm[(size_t)i]] += wts[(size_t)t] / wsum;
        }
        std::vector<int64_t> rp(1, 0);
        std::vector<int32_t> cl;
        std::vector<float> vl;
        for (int32_t i = 0; i < m; ++i) {
            for (int32_t j = 0; j < m; ++j)
                if (dense[(size_t)i][(size_t)j] > 0.0) {
                    cl.push_back(j);
                    vl.push_back((float)dense[(size_t)i][(size_t)j]);
                }
            rp.push_back((int64_t)cl.size());
        }
        HostCsr w;
        const char* why = copy_csr(m, rp.data(), cl.data(), vl.data(), &w);
        if (!why) why = validate_csr(m, w, 1e-5);
        expect(why == nullptr, "random doubly stochastic W rejected");
        const double beta = mixing_beta(m, w);
        expect(beta >= -1e-9 && beta <= 1.0 + 1e-6, "beta of a doubly stochastic W lies in [0, 1]");
        if (trial < 8) {
            std::printf("random_w %d", m);
            for (int32_t i = 0; i < m; ++i)
                for (int32_t j = 0; j < m; ++j) std::printf(" %.9g", (double)(float)dense[(size_t)i][(size_t)j]);
            std::printf(" beta %.12f\n", beta);
        }
        // damage one entry: an index out of range must be caught by the validation, whatever its value
        if (!cl.empty()) {
            HostCsr bad = w;
            bad.col[(size_t)(rng() % bad.col.size())] = (int32_t)(m + (int32_t)(rng() % 1000));
            expect(validate_csr(m, bad, 1e-5) != nullptr, "out-of-range column accepted");
        }
    }
}

// The pacing controller against a model of what the kernels measure.  A launch at rate r on a
// machine whose memory system sustains E for that kernel: up to E its slowest wavefront ends
// 40-65 us after its last deadline, and one launch in ten is late for no reason (150 us);
// above E it falls behind by 75 us per percent of excess.  The clock runs at 100 MHz; a launch
// moves the 32.768 GB of the 64 x 25.6M fused step.
struct PaceModel {
    std::mt19937 rng;
    double edge_gbs;
    explicit PaceModel(unsigned seed, double e) : rng(seed), edge_gbs(e) {}
    double uniform() { return (double)(rng() >> 8) / 16777216.0; }
    uint32_t lateness(double rate_gbs) {
        double us = 40.0 + 25.0 * uniform();
        if (rate_gbs > edge_gbs) us += (rate_gbs / edge_gbs - 1.0) * 100.0 * 75.0 + 20.0 * uniform();
        else if (uniform() < 0.1) us = 150.0;
        return (uint32_t)(us * 100.0);
    }
};

void pace_controller_model() {
    const double clock_hz = 1e8, bytes = 32.768e9;
    const double fp = 1e9 / clock_hz * 16.0;  // rate units per GB/s
    for (unsigned seed = 1; seed <= 6; ++seed) {
        const double e0 = 6150.0 + 70.0 * seed;  // 6220 .. 6570 GB/s
        PaceModel model(seed, e0);
        PaceState st{};
        PaceArgs p{};
        p.st = &st;
        p.rate_fixed_fp = 0;
        p.rate_init_fp = (uint32_t)(kPaceInitGbs * fp);
        p.rate_min_fp = (uint32_t)(1000.0 * fp);
        p.rate_max_fp = (uint32_t)(kPaceMaxGbs * fp);
        p.late_floor = (uint32_t)(kPaceLateFloorSeconds * clock_hz);
        int settle = -1, drop_recover = -1, rise_recover = -1, over = 0, counted = 0;
        double settled_rate = 0.0, sum_rate = 0.0;
        const int kDrop = 300, kRise = 600, kEnd = 900;
        for (int launch = 0; launch < kEnd; ++launch) {
            if (launch == kDrop) model.edge_gbs = e0 * 0.94;
            if (launch == kRise) model.edge_gbs = e0 * 0.94 * 1.05;
            const uint32_t r = st.rate_fp ? st.rate_fp : p.rate_init_fp;  // what pace_begin would take
            const double gbs = r / fp;
            const uint32_t plan = (uint32_t)(bytes / (gbs * 1e9) * clock_hz);
            pace_controller(p, r, model.lateness(gbs), plan);
            if (!st.rate_fp) st.rate_fp = r;  // a launch whose lateness decided nothing leaves the rate alone
            expect(st.rate_fp >= p.rate_min_fp && st.rate_fp <= p.rate_max_fp, "rate inside its range");
            if (settle < 0 && st.hold > 0) {
                settle = launch + 1;
                settled_rate = st.rate_fp / fp;
            }
            if (launch >= 60 && launch < kDrop) {
                sum_rate += gbs;
                ++counted;
                if (gbs > 1.015 * e0) ++over;
            }
            if (launch >= kDrop && drop_recover < 0 && gbs <= 1.0075 * model.edge_gbs) drop_recover = launch - kDrop;
            if (launch >= kRise && rise_recover < 0 && gbs >= 0.985 * model.edge_gbs) rise_recover = launch - kRise;
        }
        const double mean_rate = sum_rate / counted;
        std::printf("pace_model %u edge %.0f settle %d settled_rate %.0f mean_rate %.0f over %d of %d drop_recover %d rise_recover %d\n",
                    seed, e0, settle, settled_rate, mean_rate, over, counted, drop_recover, rise_recover);
        expect(settle > 0 && settle <= 48, "the controller brackets the edge within 48 launches");
        // two late launches in a row for no reason (one pair in a hundred) can end the first search early:
        // the first hold may start a few percent low, the short first hold and the next search repair it
        expect(settled_rate >= 0.96 * e0 && settled_rate <= 1.012 * e0, "the first held rate is near the edge");
        expect(mean_rate >= 0.985 * e0 && mean_rate <= 1.012 * e0, "the mean rate while holding sits at the edge");
        expect(over * 20 <= counted, "at most one launch in twenty runs more than 1.5 % past the edge");
        expect(drop_recover >= 0 && drop_recover <= 12, "a lower edge is followed within 12 launches");
        expect(rise_recover >= 0 && rise_recover <= 80, "a higher edge is found after the hold runs out");
    }
    // an edge beyond the range: the rate stops at the upper limit
    {
        PaceModel model(99, 9500.0);
        PaceState st{};
        PaceArgs p{};
        p.st = &st;
        p.rate_init_fp = (uint32_t)(kPaceInitGbs * fp);
        p.rate_min_fp = (uint32_t)(1000.0 * fp);
        p.rate_max_fp = (uint32_t)(kPaceMaxGbs * fp);
        p.late_floor = (uint32_t)(kPaceLateFloorSeconds * clock_hz);
        for (int launch = 0; launch < 200; ++launch) {
            const uint32_t r = st.rate_fp ? st.rate_fp : p.rate_init_fp;
            pace_controller(p, r, model.lateness(r / fp), (uint32_t)(bytes / (r / fp * 1e9) * clock_hz));
            if (!st.rate_fp) st.rate_fp = r;
        }
        std::printf("pace_model_limit %.0f\n", st.rate_fp / fp);
        expect(st.rate_fp <= p.rate_max_fp && st.rate_fp >= p.rate_max_fp - p.rate_max_fp / 64, "the rate stops at the upper limit");
    }
}

void schedules() {
    for (int32_t n : {1, 2, 3, 8, 20, 32, 64, 100, 1024, 1 << 24}) {
        std::printf("tau %d %d shifts", n, tau_of(n));
        for (int64_t k = 0; k < 14; ++k) std::printf(" %d", one_peer_shift(n, k));
        std::printf("\n");
    }
    for (int64_t H : {0, 1, 4, 6, 48}) {
        std::printf("global_steps %" PRId64, H);
        for (int64_t k = 0; k < 100; ++k)
            if (is_global_iteration(GPGA_TOPO_RING, H, k)) std::printf(" %" PRId64, k);
        std::printf("\n");
    }
    expect(is_global_iteration(GPGA_TOPO_FULL, 0, 5), "W = J averages at every iteration");
    gpga_ctx c;
    c.lr = 0.3f;
    std::printf("lr none %.9g %.9g\n", (double)scheduled_lr(&c, 0), (double)scheduled_lr(&c, 123456789));
    c.sched = SCHED_STEP;  // Sec. 5.1: 0.2 halved every 1000 iterations
    c.sched_base = 0.2;
    c.sched_factor = 0.5;
    c.sched_period = 1000;
    std::printf("lr step");
    for (int64_t k : {0, 999, 1000, 1999, 2000, 5000, 40000, 2000000}) std::printf(" %.9g", (double)scheduled_lr(&c, k));
    std::printf("\n");
    c.sched = SCHED_MILESTONES;
    c.sched_base = 0.1 * 32;
    c.sched_factor = 0.1;
    c.sched_start = 0.1;
    c.sched_warmup = 500;
    c.sched_count = 3;
    c.sched_milestones[0] = 3000;
    c.sched_milestones[1] = 6000;
    c.sched_milestones[2] = 9000;
    std::printf("lr milestones");
    for (int64_t k : {0, 1, 250, 499, 500, 2999, 3000, 6000, 8999, 9000, 1000000}) std::printf(" %.9g", (double)scheduled_lr(&c, k));
    std::printf("\n");
    c.sched = SCHED_POLY;
    c.sched_base = 4e-3;
    c.sched_warmup = 100;
    c.sched_total = 1000;
    c.sched_power = 0.5;
    std::printf("lr poly");
    for (int64_t k : {0, 50, 100, 550, 999, 1000, 5000}) std::printf(" %.9g", (double)scheduled_lr(&c, k));
    std::printf("\n");
}

// The lane groups of k_rows_step: every node has its share of groups, and whoever adds up partial sums finds all of
// them inside the array (one slot a thread).
void rows_deal() {
    std::vector<double> sums(kRowsThreads);
    int64_t idle = 0;
    for (int lanes : {4, 8, 16, 32, 64}) {
        for (int n = 1; n <= 128; ++n) {
            for (int B : {1, 8, 9, 16, 17, 33, 50, 65, 100, 128, 500, 1000, 100000}) {
                const RowsDeal deal(lanes, n, B);
                expect(deal.split >= 1 && deal.nodes >= 1 && deal.nodes * deal.split <= deal.groups, "shares fit the groups");
                std::vector<int> share((size_t)deal.nodes, 0);
                for (int g = 0; g < deal.groups; ++g) {
                    if (deal.dealt(g)) ++share[(size_t)deal.node(g)];
                    else ++idle;
                    if (!deal.adds(g)) continue;
                    for (int q = 0; q < lanes; ++q)
                        for (int w = 0; w < deal.split; ++w) sums.at((size_t)(g * lanes + q + w * lanes)) += 1.0;
                }
                for (int s : share) expect(s == deal.split, "a node's share is complete");
            }
        }
    }
    expect(idle > 0, "some of these splits leave groups idle");
    double total = 0.0;
    for (double s : sums) total += s;
    std::printf("rows_deal idle %" PRId64 " added %.0f\n", idle, total);
}

// Small trajectories: whatever k_node_run takes fits the LDS a launch gets without an attribute.
void node_run_sizes() {
    size_t most = 0;
    int64_t taken = 0;
    for (int n = 1; n <= kNodeMaxNodes + 1; ++n)
        for (int d = 1; d <= kNodeMaxCols + 1; ++d)
            for (int B = 1; B <= kNodeSamples + 1; ++B)
                for (int64_t entries = 0; entries <= 21 * (int64_t)n; entries += n) {
                    if (!node_run_takes(n, d, B, entries)) continue;
                    const size_t lds = node_run_lds(n, node_columns(d), node_samples(B), entries);
                    expect(lds <= 65536, "LDS of a small trajectory");
                    expect(n <= kNodeMaxNodes && kNodeLanes * node_columns(d) >= d && node_samples(B) >= B, "sizes of a small trajectory");
                    if (lds > most) most = lds;
                    ++taken;
                }
    expect(node_run_takes(128, 20, 1, 18 * 128) && !node_run_takes(128, 20, 1, 20 * 128), "the largest problems, by the entries of W");
    std::printf("node_run taken %" PRId64 " most_lds %zu\n", taken, most);
}

// The arrays of a trajectory on stored features in LDS: in bounds, in order, and on the boundaries that their accesses need.
void rows_run_lds() {
    int64_t plans = 0;
    int most = 0;
    for (int n : {4, 5, 6, 7, 8, 9, 16, 20, 31, 32, 64, 70, 100, 128})
        for (int64_t d : {32, 33, 200, 257, 301, 331, 512, 1000, 1001, 2048, 3003, 5121, 9999, 25000, 163840})
            for (int B : {1, 2, 3, 5, 8, 9, 15, 16, 21, 32, 33, 50, 99, 100, 255, 320})
                for (bool batches : {false, true}) {
                    const RunPlan p = plan_run(n, d, 256, B, batches);
                    if (!p.P) continue;
                    ++plans;
                    expect((int64_t)n * p.P <= 256 && (int64_t)4 * p.w * p.P >= d && p.w <= kWave * p.QW && p.QW * p.RG <= kRowWaves, "sharing of a trajectory");
                    const int slots = slots_for(p.slots, !batches), staged = batches ? std::max(2048 / B, 3) * B : B;
                    expect(slots >= p.slots && slots * p.RG >= B, "rows of a trajectory fit their slots");
                    for (int K : {0, 1, 5, 64}) {
                        const RunLds l(n, B, p.w, p.QW, p.RG, slots, staged, K);
                        expect(l.z % 8 == 0 && l.sum % 8 == 0, "margins of a trajectory lie on 8 bytes");
                        expect(l.x % 16 == 0 && l.m % 16 == 0, "columns of a trajectory lie on 16 bytes");
                        expect(l.x >= l.sum + 8 * B && l.val + 4 * K == l.bytes, "arrays of a trajectory do not overlap");
                        most = std::max(most, l.bytes);
                    }
                }
    expect(most <= 129 * 1024, "LDS of a trajectory");
    std::printf("rows_run plans %" PRId64 " most_lds %d\n", plans, most);
}

// Which form a gpga_run on stored features takes, against measured times (us: several iterations a launch, the other form).
void rows_run_choice() {
    struct Measured {
        int n;
        int64_t d;
        int B;
        bool batches;
        int entries;
        bool sparse;
        int T, averages;
        bool small;      // the other form is one workgroup
        double run, other;
        bool adaptive = false;
    };
    const Measured rows[] = {
        {64, 5000, 2, true, 64, true, 16, 0, false, 1269.2, 258.3},  // many entries of W
        {128, 2000, 2, true, 64, true, 3, 0, false, 168.4, 42.5},
        {32, 2000, 2, true, 32, true, 3, 0, false, 101.0, 31.3},
        {128, 5000, 8, true, 32, true, 16, 0, false, 1012.0, 317.1},
        {104, 5000, 1, true, 2, false, 3, 3, false, 62.5, 44.6},     // averages in every iteration
        {104, 2000, 1, true, 2, false, 4, 4, false, 54.6, 43.3},
        {128, 2000, 1, true, 2, false, 3, 3, false, 44.0, 33.5},
        {4, 2000, 2, true, 2, false, 3, 3, false, 33.4, 26.6},
        {32, 12000, 1, true, 2, false, 3, 0, false, 35.4, 28.5},     // few iterations
        {4, 300, 2, true, 2, false, 16, 0, true, 66.1, 56.1},        // little work in one workgroup
        {8, 1000, 100, false, 2, false, 8, 2, false, 57.9, 76.0},
        {20, 1001, 16, true, 1, false, 12, 1, false, 71.0, 107.0},
        {32, 10000, 32, true, 1, false, 16, 2, false, 212.0, 362.0},
        {32, 801, 8, true, 2, false, 16, 0, false, 76.8, 132.8},
        {128, 801, 8, true, 5, true, 16, 0, false, 104.0, 198.4},
        {9, 222, 32, true, 2, false, 16, 0, true, 65.0, 531.0},
        {6, 2435, 2, true, 0, false, 8, 8, false, 163.0, 205.0, true},
        {118, 771, 4, true, 5, true, 3, 3, false, 56.0, 80.0, true},
        {16, 300, 8, true, 2, false, 16, 0, true, 68.8, 285.2},
    };
    for (const Measured& m : rows) {
        const RunWork work{m.n, m.d, m.B, m.batches, m.entries, m.sparse, m.T, m.averages, m.adaptive};
        const RunPlan p = plan_run(m.n, m.d, 256, m.B, m.batches);
        const bool taken = p.P && rows_run_pays(work, p, 32, m.small ? one_workgroup_us(work) : two_launches_us(work, true));
        expect(taken == (m.run < m.other), "the faster form of a run");
        std::printf("rows_run_choice %d %" PRId64 " %d %d\n", m.n, m.d, m.T, taken ? 1 : 0);
    }
}

// Turns of launches whose workgroups wait for each other: two of them are never under way in two streams.
void gang_turns() {
    const int a = 0, b = 0;
    GangTurn t;
    uint32_t ended = 0;
    expect(t.take(&a, false, ended), "the first launch");
    expect(t.take(&a, false, ended) && t.number == 2, "behind the last one in its stream");
    expect(!t.take(&b, false, ended) && !t.take(&b, false, 1) && t.number == 2, "another stream while one is under way");
    ended = 2;
    expect(t.take(&b, false, ended), "another stream when the last one has ended");
    expect(!t.take(&a, false, ended), "the first stream while the second is at it");
    t.undo(2);
    expect(t.take(&a, false, ended), "a launch that failed holds nobody back");
    expect(!t.take(&a, true, ended), "a stream that every thread has its own of is another one");
    ended = 3;
    expect(t.take(&a, true, ended) && t.take(&a, true, ended), "... and the same in the same thread");
    bool taken = true;
    std::thread([&]() { taken = t.take(&a, true, ended); }).join();
    expect(!taken, "... and another in another thread");
    t = GangTurn();
    t.number = 0xfffffffeu;
    ended = 0xfffffffeu;
    for (int j = 0; j < 4; ++j) {
        expect(t.take(j % 2 ? &a : &b, false, ended), "numbers start again");
        expect(!t.take(j % 2 ? &b : &a, false, ended) && t.number != 0, "numbers start again, another stream");
        ended = t.number;
    }
    GangRest r;
    expect(!r.at_rest(0) && !r.at_rest(1), "one launch given up");
    expect(r.at_rest(2), "two launches given up");
    r.done(4095);
    expect(r.at_rest(2), "the rest is not over");
    r.done(10);
    expect(!r.at_rest(2) && !r.at_rest(3), "the rest is over, and one more launch given up");
    expect(r.at_rest(4), "a second rest");
    r.done(8191);
    expect(r.at_rest(4), "twice as long");
    r.done(1);
    expect(!r.at_rest(4), "over as well");
    for (uint32_t given_up = 6; given_up < 80; given_up += 2) expect(r.at_rest(given_up) && r.left <= (int64_t)4096 << 10, "the longest rest");
    std::printf("gang_turns done\n");
}

// The memory of such launches, of a device that refuses.
struct FakeMemory {
    size_t left = 0;            // bytes the device has
    bool waits = true, clears = true;
    int waited = 0, cleared = 0, held = 0;
    std::vector<std::pair<unsigned char*, size_t>> blocks;
    unsigned char* get(size_t bytes) {
        if (bytes > left) return nullptr;
        left -= bytes;
        ++held;
        blocks.push_back({new unsigned char[bytes], bytes});
        return blocks.back().first;
    }
    void put(unsigned char* p) {
        for (auto& b : blocks)
            if (b.first == p) {
                left += b.second;
                --held;
                b = {nullptr, 0};
                delete[] p;
                return;
            }
        expect(false, "exchange memory given back twice");
    }
    bool wait() { return ++waited, waits; }
    bool clear(unsigned char* p, size_t bytes) {
        for (size_t e = 0; clears && e < bytes; ++e) p[e] = 0;
        return ++cleared, clears;
    }
};
void gang_space() {
    constexpr size_t MB = 1 << 20;
    FakeMemory m;
    GangSpace s;
    expect(!s.room(3 * MB, false, m) && !s.at && m.held == 0, "no memory for the first launch");
    m.left = 100 * MB;
    m.clears = false;
    expect(!s.room(3 * MB, false, m), "memory that cannot be cleared is not used");
    m.clears = true;
    expect(s.room(3 * MB, false, m) && s.cap == 4 * MB && m.cleared == 2 && m.waited == 0, "cleared later, waited for nobody");
    expect(s.room(4 * MB, false, m) && s.room(1, false, m) && m.cleared == 2 && m.held == 1, "neither grown nor cleared again");
    expect(s.room(4 * MB, true, m) && m.cleared == 3, "numbers start again");
    expect(s.room(5 * MB, false, m) && s.cap == 8 * MB && m.waited == 1 && m.held == 1 && m.cleared == 4, "grown twofold, the old block given back");
    m.waits = false;
    expect(!s.room(9 * MB, false, m) && s.cap == 8 * MB && m.held == 1, "the old block may still be in use");
    m.waits = true;
    m.left = 11 * MB;
    expect(s.room(10 * MB, false, m) && s.cap == 10 * MB && m.held == 1, "what is needed where twice as much is not to be had");
    m.left = 0;
    expect(!s.room(11 * MB, false, m) && s.cap == 10 * MB && s.room(10 * MB, false, m), "refused, and smaller launches keep what there is");
    m.put(s.at);
    expect(m.held == 0, "all exchange memory given back");
    std::printf("gang_space done\n");
}

// The exchange buffers of k_column_run.  What wavefronts do between two barriers is in no order, so a buffer must not be read by
// one iteration and written by another there.  Returns how often that happens in T iterations with an average in every
// H-th; `buffer(t, exchanges before)` and `writes(t)` are the rule.
template <bool kOwn, typename Buffer, typename Writes>
int64_t exchange_hazards(int n, int T, int H, Buffer buffer, Writes writes) {
    struct Use {
        int64_t phase;   // barriers passed
        int t, buf;
        bool write;
    };
    std::vector<Use> uses;
    int64_t phase = 0, hazards = 0;
    int exchanges = 0;
    for (int t = 0; t < T; ++t) {
        const int shift = H > 0 && (t + 1) % H == 0 ? -1 : kOwn ? 0 : 1;
        const int b = buffer(t, exchanges);
        expect(b == 0 || b == 1, "two exchange buffers");
        if (writes(t, shift)) uses.push_back({phase, t, b, true});
        if (!exchanges_rows<kOwn>(n, shift)) continue;
        ++exchanges;
        uses.push_back({++phase, t, b, false});
        if (shift < 0) uses.push_back({++phase, t, b, false});  // the mean, behind the second barrier
    }
    for (const Use& u : uses)
        for (const Use& v : uses)
            if (u.write && !v.write && u.t != v.t && u.phase == v.phase && u.buf == v.buf) ++hazards;
    return hazards;
}

template <bool kOwn>
int64_t exchange_rule_hazards(int n, int T, int H) {
    return exchange_hazards<kOwn>(n, T, H, [](int t, int before) { return exchange_buffer<kOwn>(t, before); },
                                  [n](int, int shift) { return !kOwn || exchanges_rows<kOwn>(n, shift); });
}

void exchange_buffers() {
    int64_t schedules = 0, by_iteration = 0;
    for (int n : {1, 2, 3, 40, 256})
        for (int H = 0; H <= 9; ++H) {
            expect(exchange_rule_hazards<true>(n, kColumnRunMaxIters, H) == 0, "exchange buffers, W = I");
            expect(exchange_rule_hazards<false>(n, kColumnRunMaxIters, H) == 0, "exchange buffers, other graphs");
            schedules += 2;
            // buffers in turn by iteration, written whether or not an exchange follows: what the walk has to find
            if (n > 1 && H >= 2)
                by_iteration += exchange_hazards<true>(n, kColumnRunMaxIters, H, [](int t, int) { return t & 1; },
                                                       [](int, int) { return true; }) > 0;
        }
    std::printf("exchange schedules %" PRId64 " found_by_iteration %" PRId64 "\n", schedules, by_iteration);
}

// Recognising circulant matrices: the named graphs that are, whatever the order of a row's entries, and near misses that are not.
void circulant_matrices() {
    int32_t k, off[kMaxCirculant];
    float val[kMaxCirculant];
    std::mt19937 rng(7);
    for (int32_t n : {1, 2, 3, 5, 8, 16, 31, 100, 225, 256, 1000, 1024}) {
        HostCsr w;
        build_static_expo_csr(n, &w);
        expect(circulant_rows(n, w, kMaxCirculant, &k, off, val), "the static exponential graph is circulant");
        expect(k == w.ptr[1], "entries a row");
        std::vector<double> row((size_t)n, 0.0), want((size_t)n, 0.0);
        for (int32_t p = 0; p < k; ++p) {
            expect(off[p] >= 0 && off[p] < n && (p == 0 || off[p] > off[p - 1]), "offsets ascend in [0, n)");
            row[(size_t)off[p]] += val[p];
        }
        for (int32_t p = 0; p < w.ptr[1]; ++p) want[(size_t)w.col[p]] += w.val[p];
        expect(row == want, "offsets and weights are those of row 0");
        std::printf("circulant %d %d\n", n, k);
        if (n < 5) continue;
        HostCsr shuffled = w;
        for (int32_t i = 0; i < n; ++i)
            for (int32_t p = w.ptr[i + 1] - 1; p > w.ptr[i]; --p) {
                const int32_t o = w.ptr[i] + (int32_t)(rng() % (uint32_t)(p - w.ptr[i] + 1));
                std::swap(shuffled.col[(size_t)p], shuffled.col[(size_t)o]);
                std::swap(shuffled.val[(size_t)p], shuffled.val[(size_t)o]);
            }
        expect(circulant_rows(n, shuffled, kMaxCirculant, &k, off, val), "the order of a row's entries does not matter");
        HostCsr other = w;
        other.val[(size_t)w.ptr[n - 1]] += 1e-3f;
        expect(!circulant_rows(n, other, kMaxCirculant, &k, off, val), "another weight in the last row");
        other = w;
        other.col[(size_t)w.ptr[n - 1]] = (w.col[(size_t)w.ptr[n - 1]] + 3) % n;
        expect(!circulant_rows(n, other, kMaxCirculant, &k, off, val), "another neighbour in the last row");
        expect(!circulant_rows(n, w, w.ptr[1] - 1, &k, off, val), "more entries than asked for");
        HostCsr grid;
        build_grid_csr(n, &grid);
        if (n == 100) expect(!circulant_rows(n, grid, kMaxCirculant, &k, off, val), "a torus of 10 x 10 is not circulant");
    }
}

}  // namespace

int main() {
    exchange_buffers();
    circulant_matrices();
    node_run_sizes();
    rows_deal();
    rows_run_lds();
    rows_run_choice();
    gang_turns();
    gang_space();
    named_graphs();
    rejected_matrices();
    schedules();
    pace_controller_model();
    std::printf("failures %d\n", failures);
    return failures ? 1 : 0;
}
