// CPU checks of the library's launch decisions on a device made of host memory.
//   host_engine_check NAME
#include <cmath>

#include "fake_device.h"

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

int main(int argc, char **argv) {
    const std::map<std::string, void (*)()> checks = {{"quasi_layout", quasi_layout}};
    CHECK(argc == 2 && checks.count(argv[1]));
    checks.at(argv[1])();
    CHECK(fake::blocks.empty());  // every handle gave its memory back
    std::printf("OK\n");
    return 0;
}
