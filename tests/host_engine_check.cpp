// CPU checks of the library's launch decisions on a device made of host memory.
//   host_engine_check NAME
#include <cmath>
#include <memory>
#include <new>

#include "fake_device.h"

// host allocations of at least big_size bytes are counted, and fail if no_big
static size_t big_size = SIZE_MAX;
static int big_count = 0;
static bool no_big = false;
static void *take(size_t n) {
    if (n >= big_size) {
        ++big_count;
        if (no_big) return nullptr;
    }
    return std::malloc(n ? n : 1);
}
void *operator new(size_t n) {
    if (void *p = take(n)) return p;
    throw std::bad_alloc();
}
void *operator new(size_t n, const std::nothrow_t &) noexcept { return take(n); }
void *operator new[](size_t n) { return operator new(n); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
void operator delete(void *p, const std::nothrow_t &) noexcept { std::free(p); }
void operator delete[](void *p) noexcept { std::free(p); }
void operator delete[](void *p, size_t) noexcept { std::free(p); }

using namespace tbpm;

#define CHECK(c)                                                \
    do {                                                        \
        if (!(c)) {                                             \
            std::printf("FAILED %s (line %d)\n", #c, __LINE__); \
            std::exit(1);                                       \
        }                                                       \
    } while (0)

// n rows in a ring, each joined to its neighbours at the given distances
static tbpm_hamiltonian *ring(int64_t n, const std::vector<int64_t> &hops) {
    std::vector<int64_t> rp{0};
    std::vector<int32_t> col;
    for (int64_t r = 0; r < n; ++r) {
        for (int64_t h : hops)
            for (int64_t c : {(r + h) % n, (r + n - h) % n}) col.push_back((int32_t)c);
        rp.push_back((int64_t)col.size());
    }
    std::vector<double> val(2 * col.size(), 0.0), on(n, 0.1);
    for (size_t p = 0; p < col.size(); ++p) val[2 * p] = -1.0;
    tbpm_hamiltonian *H = nullptr;
    CHECK(tbpm_hamiltonian_create(n, rp.data(), col.data(), val.data(), on.data(), 0, &H) == TBPM_OK);
    return H;
}

// device memory of n doubles
struct Dev {
    double *p = nullptr;
    explicit Dev(size_t n) { CHECK(hipMalloc((void **)&p, 8 * n) == hipSuccess); }
    ~Dev() { (void)hipFree(p); }
};

static void config(tbpm_hamiltonian *H, tbpm_precision prec, int fused, int staged = 0) {
    const tbpm_launch_config c{2, 1, 1, 1, staged, 1, fused};
    CHECK(tbpm_set_launch_config(H, prec, &c) == TBPM_OK);
}

static void propagate(tbpm_hamiltonian *H, int S, int n_steps, double z = 3.14159, tbpm_precision prec = TBPM_FP64) {
    const int64_t n = H->csr.n;
    Dev psi(2 * n * S), corr(2 * (size_t)n_steps * S);
    const double f = 5.0;
    CHECK(tbpm_propagate(H, psi.p, S, n_steps, z / f, f, 1e-14, prec, corr.p, nullptr, 0, nullptr, 0, nullptr) == TBPM_OK);
}

// Both runs of a quasi-eigenstate call store the states in one layout, whatever
// the free memory does in between.
static void quasi_layout() {
    for (int first = 0; first < 2; ++first)
        for (tbpm_precision prec : {TBPM_FP64, TBPM_FP32_MIXED})
            for (std::vector<int64_t> hops : {std::vector<int64_t>{1, 50}, std::vector<int64_t>{1, 2, 50}}) {
                tbpm_hamiltonian *H = ring(4000, hops);
                const int S = 6, n_e = 2;
                Dev psi(2 * 4000 * S), states(2 * 4000 * (size_t)S * n_e);
                const double en[2] = {0.3, 0.9};
                int runs = 0, layout[2] = {-1, -1}, fin = -1;
                // memory is short in the first run only, or in the second only
                auto squeeze = [&](int run) { fake::hidden = (run == 0) == (first == 0) ? fake::total : 0; };
                fake::on_init = [&](const InitParams &p) {
                    CHECK(runs < 2);
                    layout[runs++] = p.log2sb;
                    squeeze(1);
                };
                fake::on_qe_finalize = [&](int, int log2sb) { fin = log2sb; };
                squeeze(0);
                const tbpm_status st = tbpm_quasi_eigenstates(H, psi.p, S, 70, 0.5, 5.0, 1e-14, prec, en, n_e,
                                                              TBPM_WIN_HANN, states.p, nullptr, 0, nullptr);
                fake::hidden = 0;
                CHECK(st == TBPM_OK && runs == 2);
                CHECK(layout[0] == layout[1] && fin == layout[1]);
                tbpm_hamiltonian_destroy(H);
                fake::on_init = nullptr;
                fake::on_qe_finalize = nullptr;
            }
}

static void haydock(tbpm_hamiltonian *H, int S, int n_iter) {
    Dev psi(2 * H->csr.n * S), a((size_t)n_iter * S), b((size_t)n_iter * S);
    CHECK(tbpm_haydock(H, psi.p, S, n_iter, a.p, b.p, 0, nullptr) == TBPM_OK);
}

// Timing launches after a propagation, with calls in between that build tables for
// other state counts or take the matrix entries in another precision: the launches
// fit the tables that they are given, and these hold the run's precision.
static void bench_pass() {
    for (tbpm_precision prec : {TBPM_FP64, TBPM_FP32_MIXED})
        for (std::vector<int64_t> hops : {std::vector<int64_t>{1}, std::vector<int64_t>{1, 2, 50}}) {
            const bool fp32 = prec == TBPM_FP32_MIXED, narrow = hops.size() == 1;
            tbpm_hamiltonian *H = ring(8192, hops);
            const int S = narrow ? 1 : 4;
            int values_fp32 = -1, values_tiles = 0, launches = 0, depth = 0;
            fake::on_values = [&](bool p32, int n_tiles) {
                values_fp32 = p32;
                values_tiles = n_tiles;
            };
            auto look = [&](const ChainParams &p, bool p32) {
                ++launches;
                CHECK(p32 == (bool)values_fp32 && p.n_tiles == values_tiles);
                CHECK(p.depth <= p.table_depth || !narrow);
                CHECK(fake::holds(p.x, (fp32 ? 8 : 16) * (size_t)8192 * S));
                depth = p.depth;
            };
            propagate(H, S, 70, 3.14159, prec);
            fake::on_chain = fake::on_wide = look;
            CHECK(tbpm_bench_pass(H, S, prec, 3, nullptr) == TBPM_OK);
            CHECK(launches == 3);
            const int own = depth;
            for (int other = 0; other < 2; ++other) {
                fake::on_chain = fake::on_wide = nullptr;
                if (other == 0)
                    haydock(H, 8, 70);  // tables of larger tiles, entries in FP64
                else {
                    // a propagation in the other precision, then the first one again: what
                    // bench_pass is asked for is what came last
                    propagate(H, S, 70, 3.14159, fp32 ? TBPM_FP64 : TBPM_FP32_MIXED);
                    CHECK(tbpm_bench_pass(H, S, prec, 1, nullptr) == TBPM_E_ARG);
                    propagate(H, S, 70, 3.14159, prec);
                    haydock(H, 2, 70);
                }
                fake::on_chain = fake::on_wide = look;
                launches = 0;
                CHECK(tbpm_bench_pass(H, S, prec, 2, nullptr) == TBPM_OK);
                CHECK(launches == 2 && depth == own);
                CHECK(tbpm_bench_pass(H, S, prec, 2, nullptr) == TBPM_OK);
            }
            fake::on_chain = fake::on_wide = nullptr;
            fake::on_values = nullptr;
            tbpm_hamiltonian_destroy(H);
        }
}

// Every LDS place that a wave of the Haydock step reads lies in the vector that is
// there: u_i of the staged rows in the first product, and u_{i+1} of the evaluated
// rows, one per thread, in the second.
static void haydock_places() {
    int64_t lanes = 0, moved = 0;
    fake::on_hay = [&](int width, int max_eval, int max_stage, const ChainParams &p) {
        const uint32_t nt = (uint32_t)(max_eval + 63) / 64 * 64;
        CHECK(nt <= 1024 && max_stage >= max_eval);
        for (int t = 0; t < p.n_tiles; ++t) {
            const int32_t *c = p.cnt + (int64_t)t * (p.table_depth + 1);
            const int n_own = p.tiles[t].rows, n_eval = c[1];
            CHECK(n_eval <= max_eval && c[2] <= max_stage);
            for (uint32_t tid = 0; tid < nt && (int)(tid & ~63u) < n_own; ++tid) {
                const int lr = std::min((int)tid, n_eval - 1);
                for (int k = 0; k < width; ++k) {
                    const uint32_t na = p.lidx[((int64_t)p.loff[t] + lr) * 4 + k];
                    const uint32_t at = hay_place((int)tid < n_own, na, tid);
                    CHECK((int)na < c[2] && at < nt && ((int)tid >= n_own || ((int)na < n_eval && at == na)));
                    ++lanes;
                    moved += na >= nt;
                }
            }
        }
    };
    for (int64_t n : {100, 210, 777, 1500, 8192})
        for (int S : {1, 8}) {
            tbpm_hamiltonian *H = ring(n, n == 1500 ? std::vector<int64_t>{37, 53} : std::vector<int64_t>{1, 30});
            haydock(H, S, 70);
            tbpm_hamiltonian_destroy(H);
        }
    fake::on_hay = nullptr;
    CHECK(lanes > 0 && moved > 0);
    std::printf("%lld reads, %lld of them past the evaluated rows before\n", (long long)lanes, (long long)moved);
}

// ring (hops {1}, or none) with `matchings` random pairings of its rows on top
static tbpm_hamiltonian *irregular(int64_t n, bool ring, int matchings) {
    std::vector<std::vector<int32_t>> adj(n);
    uint64_t seed = 12345;
    auto rnd = [&](int64_t m) {
        seed = seed * 6364136223846793005ull + 1442695040888963407ull;
        return (int64_t)((seed >> 33) % (uint64_t)m);
    };
    auto bond = [&](int64_t a, int64_t b) {
        adj[a].push_back((int32_t)b);
        adj[b].push_back((int32_t)a);
    };
    for (int64_t r = 0; ring && r < n; ++r) bond(r, (r + 1) % n);
    std::vector<int32_t> p(n);
    for (int m = 0; m < matchings; ++m) {
        for (int64_t r = 0; r < n; ++r) p[r] = (int32_t)r;
        for (int64_t r = n - 1; r > 0; --r) std::swap(p[r], p[rnd(r + 1)]);
        for (int64_t r = 0; r + 1 < n; r += 2) bond(p[r], p[r + 1]);
    }
    std::vector<int64_t> rp{0};
    std::vector<int32_t> col;
    for (int64_t r = 0; r < n; ++r) {
        col.insert(col.end(), adj[r].begin(), adj[r].end());
        rp.push_back((int64_t)col.size());
    }
    std::vector<double> val(2 * col.size(), 0.0), on(n, 0.1);
    for (size_t q = 0; q < col.size(); ++q) val[2 * q] = -1.0;
    tbpm_hamiltonian *H = nullptr;
    CHECK(tbpm_hamiltonian_create(n, rp.data(), col.data(), val.data(), on.data(), 0, &H) == TBPM_OK);
    return H;
}

// Calls that differ in states, orders, precision and method, in turn on one handle:
// the second round finds the tables that the first one made.
static void tables_kept() {
    tbpm_hamiltonian *H = ring(20000, {1, 70});
    int uploads = 0;
    for (int round = 0; round < 3; ++round) {
        propagate(H, 1, 70);
        propagate(H, 8, 70);
        propagate(H, 1, 70, 0.3);
        propagate(H, 8, 70, 3.14159, TBPM_FP32_MIXED);
        haydock(H, 8, 70);
        if (round == 0) uploads = fake::uploads;
        CHECK(fake::uploads == uploads);
    }
    tbpm_hamiltonian_destroy(H);
}

// Operators whose tiles fit no size, or not the first one tried: a second call does
// not look at the rows again (an array of all rows would be allocated).
static void sizes_refused() {
    const int64_t n = 12000;
    for (int kind = 0; kind < 3; ++kind) {
        tbpm_hamiltonian *H = kind == 0 ? irregular(n, true, 1) : (kind == 1 ? irregular(n, true, 2) : irregular(n, false, 24));
        for (int S : {1, 8}) {
            propagate(H, S, 70);
            big_size = 4 * (size_t)n;
            big_count = 0;
            propagate(H, S, 70);
            big_size = SIZE_MAX;
            CHECK(big_count == 0);
        }
        tbpm_hamiltonian_destroy(H);
    }
}

// two sublattices of l^3 rows, four neighbours each
static tbpm_hamiltonian *diamond(int64_t l) {
    const int64_t n = l * l * l;
    std::vector<std::vector<int32_t>> adj(2 * n);
    for (int64_t x = 0; x < l; ++x)
        for (int64_t y = 0; y < l; ++y)
            for (int64_t z = 0; z < l; ++z) {
                const int64_t a = (x * l + y) * l + z, m = l - 1;
                const int64_t b[4] = {a, ((x + m) % l * l + y) * l + z, (x * l + (y + m) % l) * l + z, (x * l + y) * l + (z + m) % l};
                for (int64_t q : b) {
                    adj[a].push_back((int32_t)(q + n));
                    adj[q + n].push_back((int32_t)a);
                }
            }
    std::vector<int64_t> rp{0};
    std::vector<int32_t> col;
    for (const auto &r : adj) {
        col.insert(col.end(), r.begin(), r.end());
        rp.push_back((int64_t)col.size());
    }
    std::vector<double> val(2 * col.size(), 0.0), on(2 * n, 0.1);
    for (size_t q = 0; q < col.size(); ++q) val[2 * q] = -1.0;
    tbpm_hamiltonian *H = nullptr;
    CHECK(tbpm_hamiltonian_create(2 * n, rp.data(), col.data(), val.data(), on.data(), 0, &H) == TBPM_OK);
    return H;
}

// Operators whose shells grow fast keep one order per launch where the overlap of the
// tiles costs more than the launches that it saves; regular ones, and small ones,
// which are bound by launches, take the chain or the wide pass.
static void overlap() {
    int blocked = 0, passes = 0;
    fake::on_chain = fake::on_wide = [&](const ChainParams &, bool) { ++blocked; };
    fake::on_pass = [&](bool) { ++passes; };
    auto takes = [&](tbpm_hamiltonian *H, int S, bool expect) {
        blocked = passes = 0;
        propagate(H, S, 70);
        CHECK((blocked > 0) == expect && (passes > 0) == !expect);
        tbpm_hamiltonian_destroy(H);
    };
    takes(irregular(60000, true, 1), 8, false);
    takes(irregular(6000, true, 1), 1, true);
    takes(ring(60000, {1, 250}), 8, true);
    takes(ring(60000, {1}), 1, true);
    takes(irregular(20000, false, 20), 8, false);
    takes(irregular(20000, false, 6), 16, false);
    takes(ring(20000, {1, 2, 3, 140, 141, 142}), 16, true);
    // a lattice of four neighbours in three dimensions, at the size where it ends
    takes(diamond(16), 1, true);
    takes(diamond(16), 10, false);
    takes(diamond(24), 8, false);
    // and the Haydock recursion
    tbpm_hamiltonian *H = irregular(120000, true, 1);
    blocked = 0;
    haydock(H, 8, 70);
    CHECK(blocked == 0);
    tbpm_hamiltonian_destroy(H);
    H = ring(60000, {1, 250});
    haydock(H, 8, 70);
    CHECK(blocked > 0);
    tbpm_hamiltonian_destroy(H);
    fake::on_chain = fake::on_wide = nullptr;
    fake::on_pass = nullptr;
}

// The wide pass orders its tiles by the size of a vector, not by a configuration that
// was chosen for the staged pass.
static void wide_order() {
    int order = -1;
    fake::on_wide = [&](const ChainParams &p, bool) { order = p.xcd_remap; };
    tbpm_hamiltonian *H = ring(20000, {1, 2, 3, 140, 141, 142});
    for (int remap : {0, 3, 6}) {
        const tbpm_launch_config c{2, remap, 0, 1, 2, 1, 0};
        CHECK(tbpm_set_launch_config(H, TBPM_FP64, &c) == TBPM_OK);
        propagate(H, 4, 5);
        CHECK(order == 1);
    }
    tbpm_hamiltonian_destroy(H);
    H = ring(110000, {1, 2, 3, 330, 331, 332});
    propagate(H, 64, 70);
    CHECK(order == 6);
    Engine::ChainShape cs;
    for (const auto &[n_blk, o] : {std::pair<int32_t, int32_t>{32, 1}, {64, 6}, {192, 6}, {256, 5}, {1024, 5}}) {
        cs.n_blk = n_blk;
        CHECK(H->eng.wide_tile_order(cs) == o);
    }
    tbpm_hamiltonian_destroy(H);
    // the tuner times it in one order (a run twice)
    int runs = 0;
    fake::on_init = [&](const InitParams &p) { runs += p.log2sb == 0; };
    H = ring(20000, {1, 2, 3, 140, 141, 142});
    tbpm_launch_config best;
    double ms = 0.0;
    CHECK(tbpm_autotune(H, 4, TBPM_FP64, &best, &ms, nullptr) == TBPM_OK);
    CHECK(runs == 2);
    tbpm_hamiltonian_destroy(H);
    fake::on_init = nullptr;
    fake::on_wide = nullptr;
}

static std::vector<double> current(const tbpm_hamiltonian *H) {
    std::vector<double> j(2 * (size_t)H->csr.nnz(), 0.0);
    for (int64_t r = 0; r < H->csr.n; ++r)
        for (int64_t p = H->csr.row_ptr[r]; p < H->csr.row_ptr[r + 1]; ++p) j[2 * p + 1] = H->csr.col[p] > r ? 1.0 : -1.0;
    return j;
}

// Without room for the chain's or the wide pass's tables and vectors every call goes
// on with another shape, keeps none of the tables, and does not build them in vain.
static void no_room() {
    int blocked = 0, values = 0;
    fake::on_chain = fake::on_wide = [&](const ChainParams &, bool) { ++blocked; };
    fake::on_values = [&](bool, int) { ++values; };
    for (int cfg = 0; cfg < 3; ++cfg)  // nobody chose a configuration; fused; staged, wide rows
        for (int method = 0; method < (cfg == 2 ? 1 : 5); ++method) {
            tbpm_hamiltonian *H = ring(20000, cfg == 2 ? std::vector<int64_t>{1, 2, 3, 140, 141, 142}
                                                       : std::vector<int64_t>{1, 140});
            const int64_t n = H->csr.n;
            const int S = 4;
            if (cfg == 1) config(H, TBPM_FP64, 2);
            if (cfg == 2) config(H, TBPM_FP64, 0, 2);
            const std::vector<double> j = current(H);
            Dev psi(2 * n * S), mu(2 * 600 * 600), corr(2 * 70 * (size_t)S), gv(2 * j.size()), go(n), ck(2 * n * S * 80);
            auto call = [&]() -> tbpm_status {
                if (method == 0) return propagate(H, S, 70), TBPM_OK;
                if (method == 1) return haydock(H, S, 70), TBPM_OK;
                if (method == 2)
                    return tbpm_kpm_moments(H, j.data(), j.data(), psi.p, S, 600, 5.0, mu.p, nullptr, nullptr);
                if (method == 3)
                    return tbpm_ac_corr(H, j.data(), j.data(), psi.p, S, 70, 0.6, 5.0, 1e-14, 10.0, 0.0, 1e-12, TBPM_FP64,
                                        corr.p, 0, nullptr);
                return tbpm_backward(H, psi.p, S, 70, 0.6, 5.0, 1e-14, corr.p, 10, ck.p, gv.p, go.p, nullptr);
            };
            blocked = values = 0;
            CHECK(call() == TBPM_OK && blocked > 0 && values > 0);
            tbpm_hamiltonian_destroy(H);
            // a new handle
            H = ring(20000, cfg == 2 ? std::vector<int64_t>{1, 2, 3, 140, 141, 142} : std::vector<int64_t>{1, 140});
            if (cfg == 1) config(H, TBPM_FP64, 2);
            if (cfg == 2) config(H, TBPM_FP64, 0, 2);
            // the moments look at the memory for their own vectors: leave them enough, but
            // not the 1 GiB more that the chain asks for
            fake::hidden = fake::total - fake::used - (method == 2 ? (size_t)1900 << 20 : 0);
            blocked = values = 0;
            for (int again = 0; again < 2; ++again) {
                CHECK(call() == TBPM_OK);
                CHECK(blocked == 0 && values == 0);
                CHECK(H->eng.ch_tval.bytes == 0);
            }
            fake::hidden = 0;
            tbpm_hamiltonian_destroy(H);
        }
    fake::on_chain = fake::on_wide = nullptr;
    fake::on_values = nullptr;
}

// The room asked for before a propagation takes the chain is what it then allocates,
// the correlation partials of a graph's steps among it.
static void room_is_what_it_takes() {
    const int64_t n = 40000;
    const int S = 64;
    for (int old = 0; old < 2; ++old) {
        // a new handle, and one that ran with fewer states before
        tbpm_hamiltonian *H = ring(n, {1, 200});
        if (old) propagate(H, 16, 70);
        const size_t used = fake::used;
        propagate(H, S, 70);
        const size_t need = fake::used - used;
        tbpm_hamiltonian_destroy(H);
        for (int more = 0; more < 2; ++more) {
            H = ring(n, {1, 200});
            if (old) propagate(H, 16, 70);
            int blocked = 0;
            fake::on_chain = [&](const ChainParams &, bool) { ++blocked; };
            const int64_t n_el = 2 * n * S + 2 * 70 * S;  // the caller's psi0 and correlation
            fake::hidden = fake::total - fake::used - need - ((size_t)256 << 20) - 8 * (size_t)n_el;
            if (more)
                fake::hidden -= (size_t)1 << 20;
            else
                fake::hidden += (size_t)1 << 20;
            propagate(H, S, 70);
            CHECK((blocked > 0) == (more == 1));
            fake::hidden = 0;
            fake::on_chain = nullptr;
            tbpm_hamiltonian_destroy(H);
        }
    }
}

// The states of several time steps, which the accumulations of quasi-eigenstate and
// optical calls read together, do not stay on the handle where they are large.
static void states_given_back() {
    const int64_t n = 80000;
    for (int S : {4, 64}) {
        const size_t hist = 8 * 16 * (size_t)n * S, keep = (size_t)512 << 20;
        tbpm_hamiltonian *H = ring(n, {1, 250});
        Dev psi(2 * n * S), states(2 * n * (size_t)S), corr(2 * 70 * (size_t)S);
        size_t most = 0;
        fake::on_qe_accum = [&](int64_t, int64_t) { most = std::max(most, H->eng.ch_hist.bytes); };
        const double en = 0.3;
        CHECK(tbpm_quasi_eigenstates(H, psi.p, S, 70, 0.5, 5.0, 1e-14, TBPM_FP64, &en, 1, TBPM_WIN_HANN, states.p, nullptr,
                                     0, nullptr) == TBPM_OK);
        CHECK(most == hist && H->eng.ch_hist.bytes == (hist > keep ? 0 : hist));
        const std::vector<double> j = current(H);
        CHECK(tbpm_ac_corr(H, j.data(), j.data(), psi.p, S / 2, 70, 0.6, 5.0, 1e-14, 10.0, 0.0, 1e-12, TBPM_FP64, corr.p, 0,
                           nullptr) == TBPM_OK);
        CHECK(H->eng.ch_hist.bytes == (hist > keep ? 0 : hist));
        fake::on_qe_accum = nullptr;
        tbpm_hamiltonian_destroy(H);
    }
}

// Without the host memory for tile tables a call goes on with another shape, and a
// later one takes the tiles.
static void no_host_memory() {
    const int64_t n = 20000;
    int blocked = 0;
    fake::on_chain = fake::on_wide = [&](const ChainParams &, bool) { ++blocked; };
    for (bool wide : {false, true}) {
        tbpm_hamiltonian *H = ring(n, wide ? std::vector<int64_t>{1, 2, 3, 140, 141, 142} : std::vector<int64_t>{1, 140});
        for (bool fails : {true, false}) {
            big_size = 4 * (size_t)n;
            no_big = fails;
            blocked = 0;
            propagate(H, 8, 70);
            no_big = false;
            big_size = SIZE_MAX;
            CHECK((blocked > 0) == !fails);
        }
        tbpm_hamiltonian_destroy(H);
    }
    fake::on_chain = fake::on_wide = nullptr;
}

// Square lattices take the chain at any size: tiles of rows that lie apart, where
// a member's order ends, are halved as far as it takes.
static void scattered_tiles() {
    for (int64_t nx : {61, 100, 181}) {
        const int64_t ny = nx == 181 ? 170 : nx, n = nx * ny;
        std::vector<int64_t> rp{0};
        std::vector<int32_t> col;
        for (int64_t y = 0; y < ny; ++y)
            for (int64_t x = 0; x < nx; ++x) {
                if (y > 0) col.push_back((int32_t)((y - 1) * nx + x));
                if (x > 0) col.push_back((int32_t)(y * nx + x - 1));
                if (x + 1 < nx) col.push_back((int32_t)(y * nx + x + 1));
                if (y + 1 < ny) col.push_back((int32_t)((y + 1) * nx + x));
                rp.push_back((int64_t)col.size());
            }
        std::vector<double> val(2 * col.size(), 0.0), on(n, 0.1);
        for (size_t q = 0; q < col.size(); ++q) val[2 * q] = -1.0;
        tbpm_hamiltonian *H = nullptr;
        CHECK(tbpm_hamiltonian_create(n, rp.data(), col.data(), val.data(), on.data(), 0, &H) == TBPM_OK);
        int blocked = 0;
        fake::on_chain = [&](const ChainParams &, bool) { ++blocked; };
        propagate(H, 1, 70);
        CHECK(blocked > 0);
        fake::on_chain = nullptr;
        tbpm_hamiltonian_destroy(H);
    }
}

// Operators whose balls grow so fast that no tiles can pay are not ordered or sampled:
// a first call allocates one array of all rows, for the balls.
static void ruled_out() {
    const int64_t n = 12000;
    for (int kind = 0; kind < 2; ++kind) {
        tbpm_hamiltonian *H = kind == 0 ? irregular(n, false, 24) : irregular(n, true, 2);
        Dev psi(2 * n * 16), corr(2 * 70 * 16);
        big_size = 4 * (size_t)n;
        big_count = 0;
        CHECK(tbpm_propagate(H, psi.p, 16, 70, 0.6, 5.0, 1e-14, TBPM_FP64, corr.p, nullptr, 0, nullptr, 0, nullptr) == TBPM_OK);
        big_size = SIZE_MAX;
        CHECK(big_count == 1 && H->eng.ch_orders.empty());
        tbpm_hamiltonian_destroy(H);
    }
}

// The members of a batch are ordered on several threads, the large ones on several
// each: every member gets the order that it gets alone, whichever comes first.
static void batch_orders() {
    std::vector<tbpm_hamiltonian *> Hs;
    for (int64_t n : {300, 9000, 700, 64, 5000, 40, 2500}) Hs.push_back(ring(n, {1, n / 3}));
    const int S = 4, ni = (int)Hs.size();
    std::vector<std::unique_ptr<Dev>> mem;
    std::vector<const double *> psi;
    std::vector<double *> corr;
    for (tbpm_hamiltonian *H : Hs) {
        mem.push_back(std::make_unique<Dev>(2 * H->csr.n * S));
        psi.push_back(mem.back()->p);
        mem.push_back(std::make_unique<Dev>(2 * 70 * S));
        corr.push_back(mem.back()->p);
    }
    const std::vector<double> dt(ni, 0.6), f(ni, 5.0);
    tbpm_batch *B = nullptr;
    CHECK(tbpm_batch_create(Hs.data(), ni, &B) == TBPM_OK);
    for (int k = 0; k < 2; ++k)
        CHECK(tbpm_propagate_batched(B, psi.data(), S, 70, dt.data(), f.data(), 1e-14, TBPM_FP64, corr.data(), nullptr, 0,
                                     nullptr) == TBPM_OK);
    CHECK((int)B->eng.ch_orders.size() == ni);
    for (int i = 0; i < ni; ++i) {
        const HostCsr &h = Hs[i]->csr;
        std::vector<int64_t> rp{0};
        std::vector<int32_t> cc;
        for (int64_t r = 0; r < h.n; ++r) {
            const int64_t s0 = Hs[i]->eng.h_slice_off[r / 32], w = (Hs[i]->eng.h_slice_off[r / 32 + 1] - s0) / 32;
            for (int64_t e = 0; e < w; ++e) {
                const int32_t g = Hs[i]->eng.h_col[s0 + e * 32 + r % 32];
                if (g != r) cc.push_back(g);
            }
            rp.push_back((int64_t)cc.size());
        }
        CHECK(B->eng.ch_orders[i] == (h.n > 64 ? bisection_order(h.n, rp.data(), cc.data(), 64, 1) : std::vector<int32_t>{}));
    }
    tbpm_batch_destroy(B);
    for (tbpm_hamiltonian *H : Hs) tbpm_hamiltonian_destroy(H);
}

int main(int argc, char **argv) {
    const std::map<std::string, void (*)()> checks = {{"quasi_layout", quasi_layout}, {"bench_pass", bench_pass},
                                                           {"haydock_places", haydock_places},
                                                           {"tables_kept", tables_kept},
                                                           {"sizes_refused", sizes_refused},
                                                           {"overlap", overlap},
                                                           {"wide_order", wide_order},
                                                           {"no_room", no_room},
                                                           {"room_is_what_it_takes", room_is_what_it_takes},
                                                           {"states_given_back", states_given_back},
                                                           {"no_host_memory", no_host_memory},
                                                           {"scattered_tiles", scattered_tiles},
                                                           {"ruled_out", ruled_out},
                                                           {"batch_orders", batch_orders}};
    CHECK(argc == 2 && checks.count(argv[1]));
    checks.at(argv[1])();
    CHECK(fake::blocks.empty());  // every handle gave its memory back
    std::printf("OK\n");
    return 0;
}
