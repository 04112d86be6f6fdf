// CPU check of the tile tables of the several-orders kernel (host.cpp): every row
// is owned once, the shells are the rows at their graph distance, every local
// index names the right row, and the bounds hold.
//   host_chain_check row_ptr col inst order T depth max_eval max_rows
#include <cstdio>
#include <cstdlib>
#include <cstring>
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
    const int order = std::atoi(a[4]);
    const int64_t T = std::atoll(a[5]), max_eval = std::atoll(a[7]), max_rows = std::atoll(a[8]);
    const int cap = std::atoi(a[6]);
    const int64_t n = (int64_t)rp.size() - 1;
    const int ni = (int)inst.size() - 1;
    const HostEll e = build_sliced_ell(n, rp.data(), col.data());
    std::vector<std::vector<int32_t>> orders(ni);
    for (int i = 0; order && i < ni; ++i) {
        std::vector<int64_t> r(inst[i + 1] - inst[i] + 1, 0);
        std::vector<int32_t> c;
        for (int64_t q = inst[i]; q < inst[i + 1]; ++q) {
            for (int64_t p = rp[q]; p < rp[q + 1]; ++p) c.push_back(col[p] - (int32_t)inst[i]);
            r[q - inst[i] + 1] = (int64_t)c.size();
        }
        orders[i] = bisection_order(inst[i + 1] - inst[i], r.data(), c.data(), 16, 1);
    }
    const int D = chain_depth(e.slice_off, e.col, inst, orders, T, cap, max_eval, max_rows);
    CHECK(D >= 0 && D <= cap);
    if (D == 0) return std::printf("NOFIT\n"), 3;
    ChainTables t;
    chain_tables(e.slice_off, e.col, inst, orders, T, D, max_eval, max_rows, t);
    CHECK(t.depth == D);
    const size_t nt = t.tiles.size();
    CHECK(t.cnt.size() == nt * (D + 1) && t.toff.size() == nt && t.loff.size() == nt);
    std::vector<int> owned(n, 0);
    for (int i = 0; i < ni; ++i) CHECK(t.inst_tile0[i] <= t.inst_tile0[i + 1]);
    for (size_t q = 0; q < nt; ++q) {
        const TileDesc &td = t.tiles[q];
        const int32_t *c = &t.cnt[q * (D + 1)];
        CHECK((int64_t)q >= t.inst_tile0[td.inst] && (int64_t)q < t.inst_tile0[td.inst + 1]);
        CHECK(c[0] == td.rows && c[0] <= T && c[D - 1] <= max_eval && c[D] <= max_rows && c[D] <= t.max_stage[D]);
        CHECK((size_t)t.toff[q] + c[D] <= t.rowmap.size() && ((size_t)t.loff[q] + c[D - 1]) * 4 <= t.lidx.size());
        const uint32_t *rm = &t.rowmap[t.toff[q]];
        std::vector<int> dist(n, -1);
        for (int l = 0; l < c[0]; ++l) {
            CHECK(rm[l] < (uint32_t)n && (!t.contiguous || rm[l] == (uint32_t)(td.row0 + l)));
            ++owned[rm[l]];
            dist[rm[l]] = 0;
        }
        std::vector<int64_t> cur(rm, rm + c[0]), nxt;
        for (int h = 1; h <= D; ++h) {
            nxt.clear();
            for (int64_t r : cur)
                for (int64_t p = rp[r]; p < rp[r + 1]; ++p)
                    if (dist[col[p]] < 0) {
                        dist[col[p]] = h;
                        nxt.push_back(col[p]);
                    }
            CHECK((int64_t)nxt.size() == c[h] - c[h - 1]);
            for (int l = c[h - 1]; l < c[h]; ++l) CHECK(rm[l] < (uint32_t)n && dist[rm[l]] == h);
            cur = nxt;
        }
        for (int l = 0; l < c[D - 1]; ++l) {
            const int64_t r = rm[l], s0 = e.slice_off[r / 32], w = (e.slice_off[r / 32 + 1] - s0) / 32;
            CHECK(w <= 4);
            for (int k = 0; k < 4; ++k) {
                const uint16_t li = t.lidx[((size_t)t.loff[q] + l) * 4 + k];
                CHECK(li < c[D]);
                CHECK((int64_t)rm[li] == (k < w ? e.col[s0 + k * 32 + r % 32] : r));
            }
        }
    }
    for (int64_t r = 0; r < n; ++r) CHECK(owned[r] == 1);
    std::printf("OK depth %d tiles %zu\n", D, nt);
    return 0;
}
