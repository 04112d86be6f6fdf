// CPU check of the tile tables of rows of more than four elements (host.cpp): one hop,
// the local indices of a tile stored element by element.  Every row is owned once, a
// tile's other rows are its neighbours, every local index names the row of its element
// (places past a row's end name the row itself), the bounds hold, and a sample of every
// tile says what the tables hold.
//   host_wide_check row_ptr col inst order T width max_eval max_rows
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <fstream>

#include "../paper_2209_00806_amd/csrc/tbpm_internal.h"

extern "C" const char *hipGetErrorString(hipError_t) { return ""; }
using namespace tbpm;

template <typename T>
static std::vector<T> load(const char *p) {
    std::ifstream f(p, std::ios::binary | std::ios::ate);
    std::vector<T> v((size_t)f.tellg() / sizeof(T));
    f.seekg(0);
    f.read((char *)v.data(), (std::streamsize)(v.size() * sizeof(T)));
    return v;
}
#define CHECK(c)                                        \
    do {                                                \
        if (!(c)) {                                     \
            std::printf("FAILED %s (line %d)\n", #c, __LINE__); \
            return 1;                                   \
        }                                               \
    } while (0)

int main(int, char **a) {
    const auto rp = load<int64_t>(a[1]);
    const auto col = load<int32_t>(a[2]);
    const auto inst = load<int64_t>(a[3]);
    const bool order = std::atoi(a[4]) != 0;
    const int64_t T = std::atoll(a[5]), max_eval = std::atoll(a[7]), max_rows = std::atoll(a[8]);
    const int W = std::atoi(a[6]);
    const int64_t n = (int64_t)rp.size() - 1;
    const int ni = (int)inst.size() - 1;
    const HostEll e = build_sliced_ell(n, rp.data(), col.data());
    std::vector<std::vector<int32_t>> orders(ni);
    for (int i = 0; order && i < ni; ++i) {
        std::vector<int64_t> r(1, 0);
        std::vector<int32_t> c;
        for (int64_t q = inst[i]; q < inst[i + 1]; ++q) {
            for (int64_t p = rp[q]; p < rp[q + 1]; ++p) c.push_back(col[p] - (int32_t)inst[i]);
            r.push_back((int64_t)c.size());
        }
        orders[i] = bisection_order(inst[i + 1] - inst[i], r.data(), c.data(), 16, 4);
    }
    ChainTables t;
    chain_tables(e.slice_off, e.col, inst, orders, T, 1, max_eval, max_rows, t, W);
    CHECK(t.depth == 0 || t.depth == 1);
    if (t.depth == 0) return std::printf("NOFIT\n"), 3;
    const size_t nt = t.tiles.size();
    CHECK(t.cnt.size() == 2 * nt && t.toff.size() == nt && t.loff.size() == nt && t.lidx.size() % W == 0);
    CHECK((int)t.inst_tile0.size() == ni + 1 && t.inst_tile0[0] == 0 && (size_t)t.inst_tile0[ni] == nt);
    std::vector<int> owned(n, 0), near(n, -1);
    int64_t eval = 0, rows = 0;
    for (size_t q = 0; q < nt; ++q) {
        const TileDesc &td = t.tiles[q];
        const int32_t *c = &t.cnt[2 * q];
        CHECK((int64_t)q >= t.inst_tile0[td.inst] && (int64_t)q < t.inst_tile0[td.inst + 1]);
        CHECK(c[0] == td.rows && c[0] >= 1 && c[0] <= T && c[0] <= max_eval && c[1] <= max_rows);
        CHECK(c[0] <= t.max_stage[0] && c[1] <= t.max_stage[1]);
        CHECK(t.toff[q] == rows && t.loff[q] == eval);
        rows += c[1];
        eval += c[0];
        CHECK((size_t)rows <= t.rowmap.size() && (size_t)eval * W <= t.lidx.size());
        const uint32_t *rm = &t.rowmap[t.toff[q]];
        for (int l = 0; l < c[1]; ++l) {
            CHECK((int64_t)rm[l] >= inst[td.inst] && (int64_t)rm[l] < inst[td.inst + 1] && near[rm[l]] != (int)q);
            near[rm[l]] = (int)q;
        }
        for (int l = 0; l < c[0]; ++l) {
            CHECK(!t.contiguous || rm[l] == (uint32_t)(td.row0 + l));
            ++owned[rm[l]];
        }
        std::vector<int32_t> want;
        for (int l = 0; l < c[0]; ++l)
            for (int64_t p = rp[rm[l]]; p < rp[rm[l] + 1]; ++p) want.push_back(col[p]);
        want.insert(want.end(), rm, rm + c[0]);
        std::sort(want.begin(), want.end());
        want.erase(std::unique(want.begin(), want.end()), want.end());
        CHECK((int64_t)want.size() == c[1]);
        for (int32_t g : want) CHECK(near[g] == (int)q);
        const uint16_t *li = &t.lidx[(size_t)t.loff[q] * W];
        for (int l = 0; l < c[0]; ++l) {
            const int64_t r = rm[l], s0 = e.slice_off[r / 32], w = (e.slice_off[r / 32 + 1] - s0) / 32;
            CHECK(w <= W);
            for (int k = 0; k < W; ++k) {
                const uint16_t at = li[(size_t)k * c[0] + l];
                CHECK(at < c[1]);
                CHECK((int64_t)rm[at] == (k < w ? e.col[s0 + k * 32 + r % 32] : r));
            }
        }
    }
    CHECK((size_t)rows == t.rowmap.size() && (size_t)eval * W == t.lidx.size() && eval == n);
    for (int64_t r = 0; r < n; ++r) CHECK(owned[r] == 1);
    ChainSample s;
    if (chain_depth(e.slice_off, e.col, inst, orders, T, 1, max_eval, max_rows, &s, 1, 1 << 30) == 1 && s.depth == 1) {
        CHECK(s.tiles == (int64_t)nt);
        CHECK(std::fabs(s.rows[0] - 1.0) < 1e-12 && std::fabs(s.rows[1] * (double)n - (double)rows) < 1e-6 * (double)rows);
        CHECK(s.sectors[1] >= s.rows[1]);
    }
    std::printf("OK tiles %zu\n", nt);
    return 0;
}
