// Host side of the chain kernel (several Clenshaw orders per launch): when it
// is taken, the tile tables, and the launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <thread>

#include "tbpm_engine.h"

namespace tbpm {

#define TRY_HIP(expr, what)                              \
    do {                                                 \
        hipError_t e_ = (expr);                          \
        if (e_ != hipSuccess) return hip_fail(e_, what); \
    } while (0)

// Rows of members that keep the caller's order and are too small to be
// renumbered at upload, in a bisection order of their own: tiles take their rows
// from it (the storage order, and with it every sum's order, stays).  keep_local:
// not for members whose tiles in the caller's order reference few rows besides their
// own (the wide pass, one hop: on bilayers in the builder's order a bisection saves
// 5 to 8% of the rows, and takes 12 ms for 14400 of them).
void Engine::chain_orders(bool keep_local) {
    if (!ch_orders.empty()) return;
    const int32_t ni = n_inst();
    std::vector<std::vector<int32_t>> orders(ni);
    // the largest members first, up to 16 threads in all and 8 within a member
    // (14400 rows of 19 elements: 35 ms with one, 12 with eight; a batch of 12
    // members of 5000 to 20000 rows: 13.5 ms one member after another, 3.1 so)
    auto size = [&](int32_t i) { return inst_row0[i + 1] - inst_row0[i]; };
    std::vector<int32_t> todo;
    int64_t rows = 0;
    for (int32_t i = 0; i < ni; ++i) {
        const int64_t n = size(i);
        if (!member_perm[i].empty() || n <= kChainMinTile || n >= kReorderMinRows) continue;
        todo.push_back(i);
        rows += n;
    }
    std::stable_sort(todo.begin(), todo.end(), [&](int32_t i, int32_t j) { return size(i) > size(j); });
    const int64_t avail = std::max(1, std::min(16, (int)std::thread::hardware_concurrency()));
    const int threads = rows < 4096 ? 1 : (int)std::min<int64_t>(avail, (int64_t)todo.size());
    std::atomic<size_t> at{0};
    run_chunks(threads, threads, [&](int, int64_t, int64_t) {
        for (size_t q; (q = at.fetch_add(1)) < todo.size();) {
            const int32_t i = todo[q];
            const int64_t r0 = inst_row0[i], n = size(i);
            const int32_t each = (int32_t)std::max<int64_t>(1, std::min<int64_t>(8, avail * n / rows));
            std::vector<int64_t> rp(n + 1, 0);
            std::vector<int32_t> cc;
            for (int64_t r = r0; r < r0 + n; ++r) {
                const int64_t s0 = h_slice_off[r / kSliceRows], w = (h_slice_off[r / kSliceRows + 1] - s0) / kSliceRows;
                for (int64_t e = 0; e < w; ++e) {
                    const int32_t g = h_col[s0 + e * kSliceRows + r % kSliceRows];
                    if (g != r) cc.push_back((int32_t)(g - r0));
                }
                rp[r - r0 + 1] = (int64_t)cc.size();
            }
            if (keep_local) {
                constexpr int64_t kRows = 256, kSamples = 16;
                std::vector<int64_t> tag(n, -1);
                int64_t own = 0, all = 0;
                for (int64_t k = 0, blocks = (n + kRows - 1) / kRows, m = std::min(blocks, kSamples); k < m; ++k) {
                    const int64_t a = k * blocks / m * kRows, b = std::min(n, a + kRows);
                    own += b - a;
                    all += b - a;
                    for (int64_t p = rp[a]; p < rp[b]; ++p) {
                        const int64_t c = cc[p];
                        if ((c < a || c >= b) && tag[c] != k) {
                            tag[c] = k;
                            ++all;
                        }
                    }
                }
                if (2 * all <= 5 * own) continue;
            }
            orders[i] = bisection_order(n, rp.data(), cc.data(), kChainMinTile, n < 4096 ? 1 : each);
        }
    });
    ch_orders = std::move(orders);
}

// the orders of one evaluation, in launches of nearly equal depth (at most D)
static void chain_split(int32_t n_orders, int32_t D, std::vector<int32_t> &depths) {
    const int32_t n_launch = (n_orders + D - 1) / D;
    depths.clear();
    for (int32_t l = 0, left = n_orders; l < n_launch; ++l) {
        depths.push_back(left / (n_launch - l));
        left -= depths.back();
    }
}

void Engine::ChainTab::release() {
    for (DevBuf *b : {&tiles, &tile0, &cnt, &toff, &loff, &rowmap, &lidx}) b->release();
    *this = ChainTab{};
}

Engine::ChainReach &Engine::chain_reach(int64_t T) {
    for (ChainReach &r : ch_reach)
        if (r.T == T) return r;
    ch_reach.push_back(ChainReach{T});
    return ch_reach.back();
}

// the tables of (T, cap), if the handle has them
bool Engine::chain_select(int64_t T, int32_t cap) {
    for (int32_t i = 0; i < kChainTabs; ++i)
        if (ch_tab[i].depth > 0 && ch_tab[i].T == T && ch_tab[i].cap == cap) {
            ch_tab[i].used = ++ch_clock;
            if (ch_sel != i) ++ch_stamp;
            ch_sel = i;
            return true;
        }
    return false;
}

// tile tables of T rows for D orders, on the device, in place of those not used for the longest time
tbpm_status Engine::chain_build(int64_t T, int32_t cap, int32_t D, int64_t rows, int64_t max_rows) {
    ChainTables t;
    chain_tables(h_slice_off, h_col, inst_row0, ch_orders, T, D, rows, max_rows, t, chain_width());
    if (t.depth < 1) return fail(TBPM_E_ARG, "no tile fits");
    const size_t nt = t.tiles.size();
    for (int32_t i = 0; i < kChainTabs; ++i)
        if (ch_tab[i].used < ch_tab[ch_sel].used) ch_sel = i;
    ChainTab &c = ch();
    ++ch_stamp;
    if (c.depth > 0) TRY_HIP(hipDeviceSynchronize(), "sync before tile rebuild");
    c.depth = 0;
    c.used = 0;
    hipError_t e = hipSuccess;
    auto up = [&](DevBuf &d, const void *src, size_t bytes) {
        if (e == hipSuccess) e = d.ensure(bytes);
        if (e == hipSuccess) e = hipMemcpy(d.ptr, src, bytes, hipMemcpyHostToDevice);
    };
    up(c.tiles, t.tiles.data(), sizeof(TileDesc) * nt);
    up(c.tile0, t.inst_tile0.data(), sizeof(int32_t) * t.inst_tile0.size());
    up(c.cnt, t.cnt.data(), sizeof(int32_t) * t.cnt.size());
    up(c.toff, t.toff.data(), sizeof(int32_t) * nt);
    up(c.loff, t.loff.data(), sizeof(int32_t) * nt);
    up(c.rowmap, t.rowmap.data(), sizeof(uint32_t) * t.rowmap.size());
    up(c.lidx, t.lidx.data(), sizeof(uint16_t) * t.lidx.size());
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();  // the caller goes on with another launch shape
        return fail(TBPM_E_OOM, "no memory for the chain tables");
    }
    TRY_HIP(e, "upload chain tables");
    c.T = T;
    c.cap = cap;
    c.n_tiles = (int32_t)nt;
    c.n_local = (int64_t)t.lidx.size() / std::max(chain_width(), 4);
    c.contiguous = t.contiguous;
    c.max_stage = t.max_stage;
    c.depth = t.depth;
    c.id = ++ch_builds;
    c.used = ++ch_clock;
    return TBPM_OK;
}

// Tile size and depth.  The more workgroups there are, the larger a tile may be
// (fewer rows evaluated and staged more than once); an operator too small to
// give every CU a workgroup takes small tiles and more orders per launch.
// Measured per time step of 17 orders (graphene L x L, S FP64 states): 64-row
// tiles of 17 orders 11.3 us against 20.5 us for 512-row tiles of 6 (L = 64,
// S = 1); 128 rows, 9 orders 14.3 us against 19.7 (L = 128); 512 rows, 6 orders
// 182 us against 195 for 256 rows, 9 orders and 319 for 128 rows, 9 orders
// (L = 512, S = 4).  One order per launch: 55, 63 and 531 us.
tbpm_status Engine::chain_prepare(int32_t s_user, bool fp32, int32_t n_orders, ChainShape &cs) {
    if (mat.max_width < 1 || mat.max_width > kChainWidth || n_orders < 2) return fail(TBPM_E_ARG, "rows too wide");
    cs.vs = fp32 && s_user > 1 ? 2 : 1;
    cs.n_blk = (s_user + cs.vs - 1) / cs.vs;
    const int64_t rows = chain_rows(mat.is_complex);
    const int64_t units = mat.n_rows * cs.n_blk;
    int64_t T = kChainMinTile;
    while (T < rows / 2 && T * 2 * 256 <= units) T *= 2;
    chain_orders();
    const int64_t max_rows = rows + rows / 4;
    for (; T >= kChainMinTile; T /= 2) {
        const int32_t cap = std::min<int32_t>(n_orders, T >= 512 ? 6 : (T >= 128 ? 9 : 17));
        if (!chain_select(T, cap)) {
            ChainReach &r = chain_reach(T);
            // a depth short of what was asked for is the rows' own, whatever is asked for
            if (r.tried < cap && r.reach == r.tried) {
                r.reach = chain_depth(h_slice_off, h_col, inst_row0, ch_orders, T, cap, rows, max_rows);
                r.tried = cap;
            }
            const int32_t D = std::min(cap, r.reach);
            if (D < std::min(n_orders, 3) || D >= r.refused) continue;
            tbpm_status st = chain_build(T, cap, D, rows, max_rows);
            if (st == TBPM_E_ARG) r.refused = D;
            if (st == TBPM_E_ARG) continue;
            if (st != TBPM_OK) return st;
        }
        // few tiles: their state blocks go to several workgroups each, up to what the
        // chip holds at once (two workgroups per CU, three of complex operators:
        // hofstadter 231 x 197, 3 states, 9.7 ms against 10.1 with two)
        const int64_t slots = mat.is_complex ? 768 : 512;
        cs.n_grp = (int32_t)std::min<int64_t>(cs.n_blk, std::max<int64_t>(1, (slots + ch().n_tiles - 1) / ch().n_tiles));
        chain_split(n_orders, ch().depth, cs.depths);
        return TBPM_OK;
    }
    return fail(TBPM_E_ARG, "no chain tile fits");
}

// One order of a wide operator per launch (wide.hip), for two blocks of states or
// more.  Tiles of up to 256 rows: a time step of bilayer 192^2 (17 orders) takes 328
// us with 16 FP32 states against 343 with 512-row tiles (two workgroups per CU
// instead of four) and 372 with 128 rows; the staged pass takes 433.  With one block
// there is nothing to share the matrix entries among (FP64, one state: 165 us
// against 155 staged).
tbpm_status Engine::wide_prepare(int32_t s_user, bool fp32, ChainShape &cs) {
    cs.vs = fp32 ? 2 : 1;
    cs.n_blk = (s_user + cs.vs - 1) / cs.vs;
    if (mat.max_width <= kChainWidth || mat.max_width > kWideWidth || mat.is_complex || cs.n_blk < 2 ||
        mat.n_rows * 16 >= ((int64_t)1 << 32))
        return fail(TBPM_E_ARG, "rows do not suit the wide pass");
    const int64_t units = mat.n_rows * cs.n_blk;
    int64_t T = kChainMinTile;
    while (T < kWideThreads && T * 2 * 256 <= units) T *= 2;
    chain_orders(true);
    for (; T >= kChainMinTile; T /= 2) {
        if (!chain_select(T, 1)) {
            ChainReach &r = chain_reach(T);
            if (r.refused <= 1) continue;
            tbpm_status st = chain_build(T, 1, 1, kWideThreads, kWideStage);
            if (st == TBPM_E_ARG) r.refused = 1;
            if (st == TBPM_E_ARG) continue;
            if (st != TBPM_OK) return st;
        }
        cs.n_grp = (int32_t)std::min<int64_t>(cs.n_blk, std::max<int64_t>(1, (512 + ch().n_tiles - 1) / ch().n_tiles));
        cs.depths.assign(1, 1);
        return TBPM_OK;
    }
    return fail(TBPM_E_ARG, "no tile fits");
}

// room for `need` more bytes and the tiles' matrix entries
bool Engine::chain_room(bool fp32, size_t need) {
    auto grow = [](const DevBuf &b, size_t n) { return n > b.bytes ? n : (size_t)0; };
    const size_t rb = fp32 ? 4 : 8;
    need += grow(ch_tval, rb * (mat.is_complex ? 2 : 1) * (size_t)ch().n_local * chain_width()) +
            grow(ch_tons, rb * (size_t)ch().n_local);
    if (need == 0) return true;
    size_t free_b = 0, total_b = 0;
    return hipMemGetInfo(&free_b, &total_b) == hipSuccess && need + ((size_t)256 << 20) <= free_b;
}

bool Engine::chain_fits(const ChainShape &cs, bool fp32, size_t vec) {
    auto grow = [](const DevBuf &b, size_t need) { return need > b.bytes ? need : (size_t)0; };
    size_t need = grow(v, vec) + grow(ba, vec) + grow(phi0, vec * (fp32 ? 2 : 1));
    if (cs.depths.size() > 1) need += grow(bb, vec) + grow(bc, vec);
    if (cs.depths.size() > 2) need += grow(bd, vec);
    return chain_room(fp32, need);
}

// The tiles' copies of the matrix entries, from the values the handle holds now
// (75 us for 2M rows; a propagation reads them once per launch).
tbpm_status Engine::chain_values(bool fp32, hipStream_t st) {
    const size_t rb = fp32 ? 4 : 8;
    const int32_t W = chain_width();
    ++ch_stamp;
    TRY_HIP(ch_tval.ensure(rb * (mat.is_complex ? 2 : 1) * (size_t)ch().n_local * W), "alloc chain values");
    TRY_HIP(ch_tons.ensure(rb * (size_t)ch().n_local), "alloc chain values");
    ChainTileTab t{(const int32_t *)ch().cnt.ptr, (const int32_t *)ch().toff.ptr, (const int32_t *)ch().loff.ptr,
                   (const uint32_t *)ch().rowmap.ptr, ch().depth, W};
    TRY_HIP(launch_chain_values(fp32, mat.is_complex, t, ch().n_tiles, mat, ch_tval.ptr, ch_tons.ptr, st),
            "launch chain values");
    return TBPM_OK;
}

ChainParams Engine::chain_params(const ChainShape &cs) const {
    ChainParams p{};
    p.tiles = (const TileDesc *)ch().tiles.ptr;
    p.n_tiles = ch().n_tiles;
    p.n_blk = cs.n_blk;
    p.n_grp = cs.n_grp;
    p.grp_blk = (cs.n_blk + cs.n_grp - 1) / cs.n_grp;
    p.table_depth = ch().depth;
    p.contiguous = ch().contiguous ? 1 : 0;
    p.n_inst = n_inst();
    p.n_rows = (uint32_t)mat.n_rows;
    p.cnt = (const int32_t *)ch().cnt.ptr;
    p.toff = (const int32_t *)ch().toff.ptr;
    p.loff = (const int32_t *)ch().loff.ptr;
    p.rowmap = (const uint32_t *)ch().rowmap.ptr;
    p.lidx = (const uint16_t *)ch().lidx.ptr;
    p.tval = ch_tval.ptr;
    p.tons = ch_tons.ptr;
    return p;
}

tbpm_status Engine::wide_launch(bool fp32, const ChainShape &cs, ChainParams &p, hipStream_t st) const {
    if (ch().depth != 1) return fail(TBPM_E_ARG, "the tile tables are not the wide pass's");
    p.lds_rows = ch().max_stage[1];
    hipError_t e = launch_pass_wide(fp32, chain_width(), cs.vs, ch().max_stage[0], p, st);
    if (e != hipSuccess) return hip_fail(e, "launch wide pass");
    return TBPM_OK;
}

tbpm_status Engine::chain_launch(bool fp32, const ChainShape &cs, const ChainParams &p, hipStream_t st) const {
    if (p.depth < 1 || p.depth > ch().depth) return fail(TBPM_E_ARG, "the tile tables serve fewer orders");
    hipError_t e = launch_chain(fp32, mat.is_complex, chain_width(), cs.vs, ch().max_stage[p.depth - 1],
                                ch().max_stage[p.depth], p, st);
    if (e != hipSuccess) return hip_fail(e, "launch chain");
    return TBPM_OK;
}

}  // namespace tbpm
