// Host side of the chain kernel (several Clenshaw orders per launch): when it
// is taken, the tile tables, and the launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <new>
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
// 5 to 8% of the rows, and takes 8 ms for 13456 of them).
void Engine::chain_orders(bool keep_local) {
    if (!ch_orders.empty()) return;
    const int32_t ni = n_inst();
    std::vector<std::vector<int32_t>> orders(ni);
    // the largest members first, up to 16 threads in all and 8 within a member
    // (13456 rows of 19 elements: 16 ms with one, 8 with eight; 12 graphene members of
    // 5000 to 20000 rows: 33 ms one member after another, 8 so)
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

Engine::ChainReach &Engine::chain_reach(int64_t T, int32_t cap) {
    for (ChainReach &r : ch_reach)
        if (r.T == T && r.cap == cap) return r;
    ch_reach.push_back(ChainReach{T, cap});
    return ch_reach.back();
}

const ChainSample &Engine::small_sample(ChainReach &r) {
    if (!r.has_small) chain_sample(r, 4, r.small);
    r.has_small = true;
    return r.small;
}

// (one hop of a wide operator's tiles differs less from tile to tile)
const ChainSample &Engine::full_sample(ChainReach &r) {
    if (!r.has_full) chain_sample(r, mat.max_width > kChainWidth ? 12 : 48, r.full);
    r.has_full = true;
    return r.full;
}

void Engine::chain_sample(const ChainReach &r, int32_t most, ChainSample &s) const {
    const bool wide = mat.max_width > kChainWidth;
    const int64_t rows = wide ? kWideThreads : chain_rows(mat.is_complex);
    (void)chain_depth(h_slice_off, h_col, inst_row0, ch_orders, r.T, r.cap, rows, wide ? kWideStage : rows + rows / 4, &s,
                      wide ? 1 : 0, most);
}

// Tiles cannot be more compact than balls of the row graph, whatever the row order:
// what these would cost rules operators out before an order is made for them.
ChainSample Engine::ball_sample(int64_t T, int32_t cap) {
    const bool wide = mat.max_width > kChainWidth;
    const double slack = 1.3;  // rows differ
    const double max_eval = slack * (wide ? kWideThreads : chain_rows(mat.is_complex));
    const double max_rows = wide ? slack * kWideStage : 1.25 * max_eval;
    if (ch_ball.empty()) ch_ball = ball_growth(h_slice_off, h_col, mat.n_rows, 1700);
    auto ball = [&](double r) {
        const size_t i = (size_t)r;
        return i + 1 >= ch_ball.size() ? ch_ball.back() : ch_ball[i] + (r - (double)i) * (ch_ball[i + 1] - ch_ball[i]);
    };
    ChainSample s;
    for (; T >= 1; T /= 2) {
        double r = 0.0;  // the ball of T rows
        while (r < (double)ch_ball.size() && ball(r + 1.0) <= (double)T) r += 1.0;
        const double step = ball(r + 1.0) - ball(r);
        if (step > 0.0) r += std::min(1.0, std::max(0.0, ((double)T - ball(r)) / step));
        const double own = std::max(1.0, ball(r));
        int32_t d = 0;
        while (d < cap && (double)T * ball(r + d) / own <= max_eval && (double)T * ball(r + d + 1) / own <= max_rows) ++d;
        if (d == 0 && wide && T > 1) continue;  // halved, as the tables would
        s.depth = d;
        s.tiles = (mat.n_rows + T - 1) / T;
        for (int32_t h = 0; h <= d; ++h) s.rows.push_back(ball(r + h) / own);
        s.sectors = s.rows;
        break;
    }
    return s;
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
        c.release();
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

// What one evaluation takes by the chain, and without it, in microseconds: the chain
// evaluates and reads rows of its shells more than once, and on operators whose
// shells grow fast that costs more than the launches and passes it saves.
//
// Two bounds per launch.  Memory: 5.4 TB/s for the 64-byte sectors of the staged rows
// (x), of the evaluated rows (psi and b_{j+2}), the own rows' outputs and the tables;
// shell rows far apart take a sector each.  Latency: every block of states of every
// workgroup takes some 3 us of loads and barriers and 0.35 us per order, in rounds of
// the workgroups that the chip holds.  Without the chain every pass streams its
// vectors, or costs a launch.  Estimate and measurement per time step of 17 orders, us:
//     states                          chain           one order per launch
//     graphene 320^2            1    33 (31)       106 (73)
//                              16   366 (242)      723 (667)
//     1% of its bonds rewired   4   238 (226)      227 (232)
//                              16   840 (823)      723 (690)
//     a matching on a ring, 200000 rows
//                               1   227 (169)      123 (129)
//                              16  3000 (1733)     706 (695)
//     diamond 2 x 30^3          1    47 (65)        60 (71)
//                               4   100 (127)       87 (82)
// Over 430 calls on lattices with 0 to 5% of their bonds rewired, ring matchings and
// three-dimensional lattices, by all methods, the choice is within 5% of one order (or
// two) per launch or faster; without it the chain was up to 3.2 times slower.
static double chain_rounds(int64_t groups, int32_t slots) {
    const double x = (double)groups / slots;
    return x <= 0.9 ? 1.0 : x + 0.5;  // the last round is partial, and the number of groups an estimate
}

double Engine::chain_us(const ChainSample &s, const ChainShape &cs, bool fp32, ChainUse use) const {
    const double n16 = 16.0 * (double)mat.n_rows, vec = n16 * cs.n_blk, rate = 5.4e6;  // bytes per us
    // bytes of matrix entries and local indices per evaluated row, in rows
    const double tab = (8.0 + 8.0 + (mat.is_complex ? 16.0 : 8.0) * chain_width()) / 16.0;
    const int32_t grp_blk = (cs.n_blk + cs.n_grp - 1) / cs.n_grp, groups = (cs.n_blk + grp_blk - 1) / grp_blk;
    const double rounds = chain_rounds(s.tiles * groups, chain_slots()) * grp_blk;
    // FP64 kernels for real rows of four elements spill a little (a tenth of their registers)
    const double spill = !fp32 && !mat.is_complex && chain_width() > 3 ? 1.35 : 1.0;
    auto order_us = [&](int32_t d) { return (3.0 + 0.35 * d) * spill; };
    // the adjoint's kernel keeps more in registers, and spills with four elements per row
    auto adjoint_us = [&](int32_t d) { return (4.0 + 0.5 * d) * (chain_width() <= 3 ? 1.0 : (mat.is_complex ? 1.4 : 2.0)); };
    auto launch = [&](int32_t d, double eval_streams, double own_rows, double block_us) {
        const double tables = n16 * groups * (tab * s.rows[d - 1] + 0.25 * s.rows[d]);
        const double bytes = vec * (s.sectors[d] + eval_streams * s.sectors[d - 1] + own_rows) + tables;
        return 2.5 + std::max(rounds * block_us, bytes / rate);
    };
    if (use == kUseHaydock) return 4.6 + launch(2, 1, 1, 2.0);  // u_{i-1} is read one hop out; and the sums
    double us = 0.0;
    for (const int32_t d : cs.depths) {
        if (use == kUseClenshaw) us += launch(d, 2, 2, order_us(d));
        // no psi; an order's vector, or J times it, is stored, and for one of the two recursions the last two
        if (use == kUseMoments) us += launch(d, 1, 1 + d, order_us(d));
        // the replay stores every order; the adjoint reads them back, and lambda
        if (use == kUseAdjoint) us += launch(d, 2, 2 + d, order_us(d)) + launch(d, 1, 4 + d, adjoint_us(d));
    }
    return us;
}

// pairs: two orders per launch where the fused shape is configured (none for Haydock).
// Such a launch reads the rows within two hops, whole sectors of them if a row's states
// are fewer bytes, and a sector for each matrix entry of a shell row: 26 us for two
// orders of the ring with one state (estimate 26), 41 (38) with four.
double Engine::plain_us(const ChainSample &s, int32_t s_user, bool fp32, int32_t n_orders, ChainUse use,
                        bool pairs) const {
    int32_t s_pad = 1;
    while (s_pad < s_user) s_pad <<= 1;
    const double row = (fp32 ? 8.0 : 16.0) * s_pad, vec = row * (double)mat.n_rows, rate = 5.4e6;
    const double w = mat.max_width, table = (8.0 + w * (mat.is_complex ? 20.0 : 12.0)) * (double)mat.n_rows;
    const double current = w * 20.0 * (double)mat.n_rows;  // a current operator's entries
    auto hop = [&](int32_t h) { return row >= 64.0 ? s.rows[h] : s.sectors[h]; };
    // one order per launch: no less than the launch, else a fixed part and the streams
    // (the general pass as it is configured for FP32 without a choice takes longer)
    const bool slow = fp32 && s_user > 1;
    const double gather = row >= 64.0 ? 0.0 : 0.5 * (s.sectors[1] - 1.0);
    const double order = std::max(slow ? 4.8 : 3.55, (slow ? 3.8 : 2.0) + ((4 + gather) * vec + table) / rate);
    double clenshaw = n_orders * order;
    if (pairs)
        clenshaw = 0.5 * n_orders *
                   std::max(slow ? 8.0 : 6.3, (slow ? 4.0 : 2.5) +
                                                  (vec * (hop(2) + 2 * hop(1) + 2) + table +
                                                   64.0 * w * (s.rows[1] - 1.0) * (double)mat.n_rows) / rate);
    switch (use) {
        case kUseMoments:  // half of the orders take a pass of the current operator as well
            return clenshaw + n_orders * std::max(1.75, 1.5 + 0.5 * current / rate);
        case kUseHaydock:  // two launches and two sums per iteration
            return std::max(16.5, 14.0 + (6 * vec + table) / 4.9e6);
        case kUseAdjoint: {  // replay, and an adjoint that updates the gradient
            const double all = n_orders * std::max(9.0, 5.0 + (13 * vec + 3.5 * table) / rate);
            return clenshaw + (pairs ? 0.75 : 1.0) * (all - n_orders * order);
        }
        default:
            return clenshaw;
    }
}

// Tile size and depth.  The more workgroups there are, the larger a tile may be
// (fewer rows evaluated and staged more than once); an operator too small to
// give every CU a workgroup takes small tiles and more orders per launch.
// Measured per time step of 17 orders (graphene L x L, S FP64 states): 64-row
// tiles of 17 orders 11.3 us against 20.5 us for 512-row tiles of 6 (L = 64,
// S = 1); 128 rows, 9 orders 14.3 us against 19.7 (L = 128); 512 rows, 6 orders
// 182 us against 195 for 256 rows, 9 orders and 319 for 128 rows, 9 orders
// (L = 512, S = 4).  One order per launch: 55, 63 and 531 us.
tbpm_status Engine::chain_prepare(int32_t s_user, bool fp32, int32_t n_orders, ChainShape &cs, ChainUse use,
                                  const ChainNeed &need) try {
    if (mat.max_width < 1 || mat.max_width > kChainWidth || n_orders < 2) return fail(TBPM_E_ARG, "rows too wide");
    cs.vs = fp32 && s_user > 1 ? 2 : 1;
    cs.n_blk = (s_user + cs.vs - 1) / cs.vs;
    const int64_t rows = chain_rows(mat.is_complex);
    const int64_t units = mat.n_rows * cs.n_blk;
    int64_t T = kChainMinTile;
    while (T < rows / 2 && T * 2 * 256 <= units) T *= 2;
    // few tiles: their state blocks go to several workgroups each, up to what the
    // chip holds at once
    const int64_t slots = chain_slots();
    const bool pairs = cfgs[fp32 ? 1 : 0].fused > 0 && n_orders >= 3;
    auto shape = [&](int64_t n_tiles, int32_t depth) {
        cs.n_grp = (int32_t)std::min<int64_t>(cs.n_blk, std::max<int64_t>(1, (slots + n_tiles - 1) / n_tiles));
        chain_split(n_orders, depth, cs.depths);
    };
    // times `margin` of what the same takes without the chain
    auto pays = [&](const ChainSample &s, double margin) {
        if (s.depth < std::min(n_orders, 3)) return false;
        shape(s.tiles, s.depth);
        return chain_us(s, cs, fp32, use) <= margin * plain_us(s, s_user, fp32, n_orders, use, pairs);
    };
    auto cap_of = [&](int64_t t) { return std::min<int32_t>(n_orders, t >= 512 ? 6 : (t >= 128 ? 9 : 17)); };
    // what the balls or a few tiles rule out is not looked at in full (0.1 ms for the
    // balls, 0.2 for four tiles, 1 to 3 for 48, and up to 20 for an order)
    bool any = false, sure = false;
    for (int64_t t = T; t >= kChainMinTile && !any; t /= 2) {
        const ChainSample ball = ball_sample(t, cap_of(t));
        any = pays(ball, 1.3);
        sure = pays(ball, 0.5);  // needs no small sample
    }
    if (!any) return fail(TBPM_E_ARG, "the chain does not pay");
    chain_orders();
    for (; T >= kChainMinTile; T /= 2) {
        const int32_t cap = cap_of(T);
        ChainReach &r = chain_reach(T, cap);
        if (r.refused || !(sure || pays(small_sample(r), 1.3)) || !pays(full_sample(r), 1.0)) continue;
        if (r.n_tiles > 0 && !pays(r.exact(), 1.0)) continue;
        const bool there = chain_select(T, cap);
        if (there) shape(ch().n_tiles, ch().depth);
        // looked at before the tables are built: near the limit every call would build them in vain
        if (need && !chain_room(fp32, there ? nullptr : &r.full, need(cs, there ? ch().n_tiles : r.full.tiles))) {
            chain_release();
            return fail(TBPM_E_OOM, "no memory for the chain");
        }
        if (!there) {
            tbpm_status st = chain_build(T, cap, r.full.depth, rows, rows + rows / 4);
            r.refused = st == TBPM_E_ARG;
            if (st == TBPM_E_ARG) continue;
            if (st != TBPM_OK) return st;
            r.n_tiles = ch().n_tiles;
            if (!pays(r.exact(), 1.0)) {
                ch().release();
                continue;
            }
            shape(ch().n_tiles, ch().depth);
        }
        return TBPM_OK;
    }
    return fail(TBPM_E_ARG, "no chain tile fits");
} catch (const std::bad_alloc &) {
    return fail(TBPM_E_OOM, "no host memory for the chain tables");  // the caller goes on with another launch shape
}

static int32_t wide_groups(int32_t n_blk, int64_t n_tiles) {
    return (int32_t)std::min<int64_t>(n_blk, std::max<int64_t>(1, (512 + n_tiles - 1) / n_tiles));
}

// One wide pass, and the same by the general or the staged pass, in microseconds.  A
// wide pass takes 3.6 us and, per block of states of a workgroup and round of 512
// workgroups, 0.8 us and 0.2 us for every shell row of a thread (a little more from
// the third on, which is not loaded ahead), or the sectors it reads at 12 TB/s from
// the caches; the others gather each element from the cache.  Estimate and
// measurement, us:
//     states                                  wide            general
//     bilayer 120^2, 19 elements       16    15 (15)       35 (33)
//     cubic 60^3, 6 elements           16    41 (44)       60 (54)
//     cubic 28^3                       16     8.2 (7.8)     7.9 (7.1)
//     6 random pairings, 50000 rows    16    33 (32)       16 (18)
//     20 random pairings, 20000 rows    4    18 (23)       11 (11)
double Engine::wide_us(const ChainSample &s, int32_t n_blk) const {
    const int32_t n_grp = wide_groups(n_blk, s.tiles), grp_blk = (n_blk + n_grp - 1) / n_grp;
    const int32_t groups = (n_blk + grp_blk - 1) / grp_blk;
    const double rounds = std::max(1.0, (double)(s.tiles * groups) / 512.0) * grp_blk;
    const double own = (double)mat.n_rows / (double)s.tiles, threads = 64.0 * std::ceil(own / 64.0);
    const double shell = own * (s.rows[1] - 1.0) / threads;
    const double n16 = 16.0 * (double)mat.n_rows, tab = (16.0 + 10.0 * chain_width()) / 16.0;
    const double bytes = n16 * (n_blk * (s.sectors[1] + 3.0) + groups * (tab + 0.25 * s.rows[1]));
    return 3.6 + std::max(bytes / 12.0e6, rounds * (0.8 + 0.2 * shell + 0.02 * mat.max_width) +
                                             grp_blk * 0.25 * std::max(0.0, shell - 2.0));
}

double Engine::wide_plain_us(int32_t s_user, bool fp32) const {
    int32_t s_pad = 1;
    while (s_pad < s_user) s_pad <<= 1;
    const double vec = (fp32 ? 8.0 : 16.0) * s_pad * (double)mat.n_rows, w = mat.max_width;
    return std::max(3.5 + 0.36 * w, 2.0 + vec * (3.0 + 0.45 * w) / 5.4e6);
}

// The order in which a wide pass's workgroups take the tiles, whatever the
// configuration's, which was chosen for another kernel: each XCD a contiguous range
// (1) while a vector leaves the caches room for the others, then runs of 64 tiles in
// turn (6), and runs of 32 (5) for the largest vectors.  Time of
// 70 samples (33 of the largest bilayer), ms, 16 states but for the 4 of one row:
//     order                                1       5       6
//     cubic 60^3, FP64       55 MB      52.2       -    56.2
//     bilayer 448^2, FP32   103 MB     109.9   108.7   108.6
//     bilayer 448^2, FP64   206 MB       231   223.5   224.8
//     cubic 110^3, FP64     341 MB       394   370.6   369.6
//     bilayer 1024^2, FP64, 4 states
//                           268 MB     202.2   199.8   197.9
//     bilayer 1024^2, FP32  537 MB     282.6   272.6   278.7
//                     FP64 1074 MB       563     529     544
int32_t Engine::wide_tile_order(const ChainShape &cs) const {
    const int64_t mb = 16 * mat.n_rows * cs.n_blk >> 20;
    return mb <= 96 ? 1 : (mb <= 384 ? 6 : 5);
}

// One order of a wide operator per launch (wide.hip), for two blocks of states or
// more.  Tiles of up to 256 rows: a time step of bilayer 192^2 (17 orders) takes 328
// us with 16 FP32 states against 343 with 512-row tiles (two workgroups per CU
// instead of four) and 372 with 128 rows; the staged pass takes 433.  With one block
// there is nothing to share the matrix entries among (FP64, one state: 165 us
// against 155 staged).
tbpm_status Engine::wide_prepare(int32_t s_user, bool fp32, ChainShape &cs, const ChainNeed &need) try {
    cs.vs = fp32 ? 2 : 1;
    cs.n_blk = (s_user + cs.vs - 1) / cs.vs;
    if (mat.max_width <= kChainWidth || mat.max_width > kWideWidth || mat.is_complex || cs.n_blk < 2 ||
        mat.n_rows * 16 >= ((int64_t)1 << 32))
        return fail(TBPM_E_ARG, "rows do not suit the wide pass");
    const int64_t units = mat.n_rows * cs.n_blk;
    int64_t T = kChainMinTile;
    while (T < kWideThreads && T * 2 * 256 <= units) T *= 2;
    auto pays = [&](const ChainSample &q, double margin) {
        return q.depth >= 1 && wide_us(q, cs.n_blk) <= margin * wide_plain_us(s_user, fp32);
    };
    bool any = false;
    for (int64_t t = T; t >= kChainMinTile && !any; t /= 2) any = pays(ball_sample(t, 1), 1.3);
    if (!any) return fail(TBPM_E_ARG, "the wide pass does not pay");
    chain_orders(true);
    for (; T >= kChainMinTile; T /= 2) {
        ChainReach &r = chain_reach(T, 1);
        if (r.refused || !pays(small_sample(r), 1.3) || !pays(full_sample(r), 1.0)) continue;
        if (r.n_tiles > 0 && !pays(r.exact(), 1.0)) continue;
        const bool there = chain_select(T, 1);
        if (need && !chain_room(fp32, there ? nullptr : &r.full, need(cs, there ? ch().n_tiles : r.full.tiles))) {
            chain_release();
            return fail(TBPM_E_OOM, "no memory for the wide pass");
        }
        if (!there) {
            tbpm_status st = chain_build(T, 1, 1, kWideThreads, kWideStage);
            r.refused = st == TBPM_E_ARG;
            if (st == TBPM_E_ARG) continue;
            if (st != TBPM_OK) return st;
            r.n_tiles = ch().n_tiles;
            if (!pays(r.exact(), 1.0)) {
                ch().release();
                continue;
            }
        }
        cs.n_grp = wide_groups(cs.n_blk, ch().n_tiles);
        cs.depths.assign(1, 1);
        return TBPM_OK;
    }
    return fail(TBPM_E_ARG, "no tile fits");
} catch (const std::bad_alloc &) {
    return fail(TBPM_E_OOM, "no host memory for the wide pass's tables");
}

// need bytes, and 256 MiB for everything else
bool Engine::free_memory(size_t need) {
    if (need == 0) return true;
    size_t free_b = 0, total_b = 0;
    return hipMemGetInfo(&free_b, &total_b) == hipSuccess && need + ((size_t)256 << 20) <= free_b;
}

void Engine::chain_release() {
    for (ChainTab &t : ch_tab) t.release();
    ch_tval.release();
    ch_tons.release();
    ch_sel = 0;
    ++ch_stamp;
}

// 512 MiB: a call on larger vectors (64 MiB each) takes hundreds of microseconds per
// time step, beside which allocating them again does not count.
void Engine::trim_states() {
    constexpr size_t kHistKeep = (size_t)512 << 20;
    if (ch_hist.bytes > kHistKeep) ch_hist.release();
}

bool Engine::chain_room(bool fp32, const ChainSample *sample, size_t need) {
    const double n = (double)mat.n_rows;
    const size_t rb = fp32 ? 4 : 8;
    const size_t n_local = sample ? (size_t)(n * sample->rows[sample->depth - 1]) : (size_t)ch().n_local;
    need += ch_tval.growth(rb * (mat.is_complex ? 2 : 1) * n_local * chain_width()) + ch_tons.growth(rb * n_local);
    if (sample)
        need += (size_t)(4 * n * sample->rows[sample->depth]) + 2 * n_local * std::max(chain_width(), 4) +
                (size_t)sample->tiles * (sizeof(TileDesc) + 4 * ((size_t)sample->depth + 3));
    if (free_memory(need)) return true;
    bool gave = ch_hist.bytes > 0;
    ch_hist.release();
    for (int32_t i = 0; i < kChainTabs; ++i)
        if (ch_tab[i].depth > 0 && (sample || i != ch_sel)) {
            ch_tab[i].release();
            gave = true;
        }
    if (sample) ++ch_stamp;
    return gave && free_memory(need);
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
