// Haydock recursion (paper, Sec. "Local density of states", the recursion
// method): one Lanczos chain per state of a block [rows][S] (S a power of
// two, S <= 64), all chains advanced together so that the matrix is read once
// per iteration for all of them.
//
// The normalised Lanczos vector l_i is never stored: the buffers hold
// u_i = b_i l_i (the unnormalised m_i of the recursion, or psi0 for i = 0),
// and a per-state scalar table hs[s] = {1/b_i, b_i/b_{i-1}, a_i/b_i, -}
// carries the normalisation (1/b_0 = 1/||psi0||).  One iteration is
//   k_hay_spmv : y = (H u_i)/b_i - (b_i/b_{i-1}) u_{i-1}   (= H l_i - b_i l_{i-1}),
//                partials of Re <u_i|y>/b_i                 (-> a_i)
//   k_hay_reduce(kA): a_i, hs[s].2 = a_i/b_i
//   k_hay_axpy : u_{i+1} = y - (a_i/b_i) u_i, over u_{i-1}, partials of ||u_{i+1}||^2
//   k_hay_reduce(kB): b_{i+1}, or 0 below the breakdown threshold (the chain
//                stays zero from then on: 1/b = 0 zeroes every later vector)
// so a_i = <l_i|H l_i - b_i l_{i-1}>, which equals <l_i|H|l_i> since l_i is
// orthogonal to l_{i-1} (the form that keeps better orthogonality in
// finite precision).  All reductions are FP64 per-tile partials summed in a
// fixed order, so results are reproducible for a given tiling.
//
// Streams per iteration: gather of u_i, u_{i-1}, y written (spmv); y, u_i
// read and u_{i+1} written (axpy): 6 state vectors plus the matrix.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_util.h"
#include "tbpm_internal.h"

namespace tbpm {
namespace {

enum HayReduce : int { kHayA = 0, kHayB = 1, kHayInit = 2 };
constexpr int kHayThreads = 1024;

// One thread per (row, state) element: on the headline lattice with 8 chains
// this runs ahead of units of 2 states (+3-7% per iteration) and of 4
// (+30%).  When every slice has the same width (uniform_w > 0) a row's slots
// come without the slice-offset loads.
template <bool CH>
__global__ __launch_bounds__(kWG) void k_hay_spmv(const TileDesc *__restrict__ tiles, int n_tiles, int xcd_remap,
                                                  int log2s, const int32_t *__restrict__ col,
                                                  const void *__restrict__ val, const uint32_t *__restrict__ soff,
                                                  int uniform_w, const double *__restrict__ onsite,
                                                  const d2 *__restrict__ u,
                                                  const d2 *__restrict__ uprev, d2 *__restrict__ y,
                                                  const double *__restrict__ hs, int32_t *counter,
                                                  double *__restrict__ partials) {
    using HV = typename std::conditional<CH, d2, double>::type;
    const HV *hvp = (const HV *)val;
    auto hv_ = [&](uint32_t slot) { return hvp[slot]; };
    const int tile = tile_of_block(blockIdx.x, n_tiles, xcd_remap);
    const TileDesc td = tiles[tile];
    if (counter && blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(counter, 1);
    const uint32_t smask = (1u << log2s) - 1u;
    const uint32_t s = threadIdx.x & smask;
    const double inv = hs[4 * s], cprev = hs[4 * s + 1];
    // 32-bit element indices: rows * S < 2^31 (checked by the entry point)
    const uint32_t n_u = (uint32_t)td.rows << log2s;
    const uint32_t row0 = (uint32_t)td.row0;
    constexpr int KG = 4;  // stored elements gathered per batch
    double dre = 0.0;
    for (uint32_t q = threadIdx.x; q < n_u; q += kWG) {
        const uint32_t r = row0 + (q >> log2s);
        const uint32_t sl = r / kSliceRows;
        uint32_t base;
        int w;
        if (uniform_w > 0) {
            w = uniform_w;
            base = sl * (uint32_t)(uniform_w * kSliceRows) + r % kSliceRows;
        } else {
            const uint32_t off = soff[sl];
            w = (int)((soff[sl + 1] - off) / kSliceRows);
            base = off + r % kSliceRows;
        }
        const uint32_t e = (r << log2s) + s;
        const d2 up = __builtin_nontemporal_load(uprev + e);  // read once
        const d2 ur = u[e];
        d2 acc;
        acc.x = onsite[r] * ur.x;
        acc.y = onsite[r] * ur.y;
        for (int k = 0; k < w; k += KG) {
            HV h[KG];
            uint32_t g[KG];
#pragma unroll
            for (int i = 0; i < KG; ++i) {
                const bool valid = k + i < w;
                const uint32_t slot = valid ? base + (uint32_t)(k + i) * kSliceRows : base;
                const HV hv = hv_(slot);
                g[i] = ((valid ? (uint32_t)col[slot] : r) << log2s) + s;
                h[i] = valid ? hv : HV{};
            }
#pragma unroll
            for (int i = 0; i < KG; ++i) acc = hmad(h[i], u[g[i]], acc);
        }
        d2 yv;
        yv.x = fma(inv, acc.x, -cprev * up.x);
        yv.y = fma(inv, acc.y, -cprev * up.y);
        __builtin_nontemporal_store(yv, y + e);
        dre = fma(ur.x * inv, yv.x, fma(ur.y * inv, yv.y, dre));
    }
    block_state_partials(dre, 0.0, 0.0, log2s, partials, tile, n_tiles);
}

// unext = y - (a_i/b_i) u  (unext may be the buffer of u_{i-1}), with the
// partials of ||unext||^2; with unext null it only measures ||y||^2.  The
// iteration walks it last tile to first (reverse), so it starts on the tiles
// whose y the product pass wrote last, and the next product pass starts on
// the tiles whose u_{i+1} it wrote last.
__global__ __launch_bounds__(kWG) void k_hay_axpy(const TileDesc *__restrict__ tiles, int n_tiles, int xcd_remap,
                                                  int reverse, int log2s, const d2 *y, const d2 *u, d2 *unext,
                                                  const double *__restrict__ hs, double *__restrict__ partials) {
    const int tile = tile_of_block(blockIdx.x, n_tiles, xcd_remap, reverse);
    const TileDesc td = tiles[tile];
    const uint32_t smask = (1u << log2s) - 1u;
    const uint32_t s = threadIdx.x & smask;
    const double c = unext ? hs[4 * s + 2] : 0.0;
    const uint32_t n_u = (uint32_t)td.rows << log2s;
    const uint32_t u0 = (uint32_t)td.row0 << log2s;
    double nrm = 0.0;
    for (uint32_t q = threadIdx.x; q < n_u; q += kWG) {
        const uint32_t e = u0 + q;
        d2 v = __builtin_nontemporal_load(y + e);  // read once
        if (unext) {
            const d2 ui = u[e];
            v.x = fma(-c, ui.x, v.x);
            v.y = fma(-c, ui.y, v.y);
            unext[e] = v;
        }
        nrm = fma(v.x, v.x, fma(v.y, v.y, nrm));
    }
    block_state_partials(0.0, 0.0, nrm, log2s, partials, tile, n_tiles);
}

// One workgroup per state: the fixed-order sum of the per-tile partials and
// the scalar update.  The iteration index is the device counter minus one
// (k_hay_spmv bumps it).
// First stage of a per-state sum over many per-tile partials: workgroup
// (g, s) adds values [g kFold, (g+1) kFold) of state s (row s of `in`, stride
// in_stride) in a fixed order and writes out[s n_fold + g].  One pass with
// all loads in flight, instead of one workgroup per state walking the whole
// row with dependent rounds of loads.
constexpr int kFold = 4 * kWG;

__global__ __launch_bounds__(kWG) void k_hay_fold(const double *__restrict__ in, int64_t in_stride, int n,
                                                  double *__restrict__ out, int n_fold) {
    __shared__ double red[kWG];
    const int g = blockIdx.x, s = blockIdx.y;
    const double *p = in + (int64_t)s * in_stride + (int64_t)g * kFold;
    const int m = min(kFold, n - g * kFold);
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int i = (int)threadIdx.x + q * kWG;
        v[q] = i < m ? p[i] : 0.0;
    }
    red[threadIdx.x] = (v[0] + v[1]) + (v[2] + v[3]);
    __syncthreads();
    for (int h = kWG / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[(int64_t)s * n_fold + g] = red[0];
}

// Final stage: workgroup s sums row s of `in` (n values, stride in_stride)
// and applies the Lanczos scalar update of `mode`.
__global__ __launch_bounds__(kWG) void k_hay_reduce(const double *__restrict__ in, int64_t in_stride, int n,
                                                    int s_user, int mode, double thr, double *__restrict__ hs,
                                                    int32_t *counter, int n_iter, double *__restrict__ a_out,
                                                    double *__restrict__ b_out) {
    __shared__ double red[kWG];
    const int s = blockIdx.x;
    const double *p = in + (int64_t)s * in_stride;
    // eight independent accumulators keep loads in flight; the order is fixed
    double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    int t = threadIdx.x;
    for (; t + 7 * kWG < n; t += 8 * kWG) {
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] += p[t + q * kWG];
    }
    for (; t < n; t += kWG) v[0] += p[t];
    red[threadIdx.x] = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    __syncthreads();
    for (int h = kWG / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    const double sum = red[0];
    double *h = hs + 4 * s;
    if (mode == kHayInit) {
        const double nrm = sqrt(sum);
        h[0] = nrm > 0.0 ? 1.0 / nrm : 0.0;
        h[1] = 0.0;
        h[2] = 0.0;
        h[3] = 0.0;
        if (s == 0) *counter = 0;
        return;
    }
    const int k = *(volatile const int32_t *)counter - 1;
    if (mode == kHayA) {
        h[2] = sum * h[0];
        if (k >= 0 && k < n_iter && s < s_user) a_out[(int64_t)k * s_user + s] = sum;
        return;
    }
    double b = sqrt(sum);
    double inv = 0.0;
    if (b > thr && h[0] != 0.0)
        inv = 1.0 / b;
    else
        b = 0.0;
    if (k >= 0 && k < n_iter && s < s_user) b_out[(int64_t)k * s_user + s] = b;
    h[1] = b * h[0];
    h[0] = inv;
}

// One iteration per launch, for operators of up to kChainWidth stored elements per
// row, on the chain kernel's tile tables (two hops of them), states in blocks of one:
//     u_{i+1} = (H u_i)/b_i - (a_i/b_i) u_i - (b_i/b_{i-1}) u_{i-1}
// on the tile's own rows and those one hop away (one per thread; u_i of the rows
// up to two hops away is in LDS), then H u_{i+1} on own rows, which is not
// stored: it gives <u_{i+1}|H u_{i+1}>, and with ||u_{i+1}||^2 and Re <u_{i+1}|u_i>
// the next a and b (k_hay_reduce3),
//     a_{i+1} = <u_{i+1}|H u_{i+1}>/b_{i+1}^2 - (b_{i+1}/b_i) Re <u_{i+1}|u_i>/b_{i+1},
// the same form of a as above.  first: the sums for u_0 = x alone.  u_i and
// u_{i-1} are read on other tiles' rows, so u_{i+1} goes to a third vector.
// Streams per iteration: u_i (and 35% of it again for the two hops), u_{i-1}
// (15%), u_{i+1}: 3.5 state vectors in one pass, and one sum, instead of 6 in two.
// Graphene 512^2, 8 states: 40 us and 4.6 us for the sums, 6 TB/s; the two-launch
// form 39 + 31 us and 18 us.
template <bool CH, int W>
__global__ __launch_bounds__(kHayThreads) void k_hay_step(const ChainParams p, const double *__restrict__ hs) {
    extern __shared__ __align__(16) unsigned char hay_mem[];
    using HV = typename std::conditional<CH, d2, double>::type;
    int grp = 0, tslot = (int)blockIdx.x;
    if (p.n_grp > 1) {
        const int r = (int)blockIdx.x >> 3;
        grp = r % p.n_grp;
        tslot = (r / p.n_grp) * 8 + ((int)blockIdx.x & 7);
        if (tslot >= p.n_tiles) return;  // the last group of 8 tiles is partial
    }
    const int blk0 = grp * p.grp_blk, blk1 = min(blk0 + p.grp_blk, p.n_blk);
    const int tile = tile_of_block(tslot, p.n_tiles, p.xcd_remap, p.reverse);
    if (p.bump && blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(p.counter, 1);
    if (blk0 >= blk1) return;
    const TileDesc td = p.tiles[tile];
    const int32_t *cnt = p.cnt + (int64_t)tile * (p.table_depth + 1);
    const int n_own = td.rows, n_eval = cnt[1], n_shell = cnt[2] - n_eval, n_tab = cnt[p.table_depth - 1];
    const uint32_t *rowmap = p.rowmap + p.toff[tile];
    const int64_t lo = p.loff[tile];
    const int tid = (int)threadIdx.x, nt = (int)blockDim.x, lane = tid & 63, wave = tid >> 6;
    const bool own = tid < n_own, eval = tid < n_eval, own_wave = (tid & ~63) < n_own;
    const int lr = min(tid, n_eval - 1);
    const uint32_t g = p.contiguous && lr < n_own ? (uint32_t)td.row0 + (uint32_t)lr : rowmap[lr];
    const uint32_t gs = tid < n_shell ? rowmap[n_eval + tid] : g;
    d2 *xs = (d2 *)hay_mem, *ys = xs + 2 * p.lds_rows;
    double *red = (double *)(ys + nt);  // [2][waves][3]

    HV h[W];
    uint32_t na[W];
    const double on = ((const double *)p.tons)[lo + lr];
    {
        const uint2 li = ((const uint2 *)p.lidx + lo)[lr];
#pragma unroll
        for (int k = 0; k < W; ++k) {
            h[k] = ((const HV *)p.tval + lo * W)[(int64_t)k * n_tab + lr];
            const uint32_t pair = k < 2 ? li.x : li.y;
            na[k] = (k & 1) ? pair >> 16 : pair & 0xffffu;
        }
    }
    auto row_of = [&](const void *base, int blk, uint32_t r) -> d2 & {
        return ((d2 *)base + (int64_t)blk * p.n_rows)[r];
    };
    // unconditional loads (lanes without a row repeat one)
    const void *b2p = p.b2 ? p.b2 : p.x;
    d2 px, psh, pb;
    auto load = [&](int blk) {
        px = row_of(p.x, blk, g);
        psh = row_of(p.x, blk, gs);
        pb = row_of(b2p, blk, g);
    };
    auto put = [&](int blk, d2 *buf) {
        if (eval) buf[tid] = px;
        if (tid < n_shell) buf[n_eval + tid] = psh;
        for (int l = tid + nt; l < n_shell; l += nt) buf[n_eval + l] = row_of(p.x, blk, rowmap[n_eval + l]);
    };
    // the partial sums of the block before (its waves' sums are behind a barrier)
    auto flush = [&](int blk, int par) {
        if (tid < 3) {
            double a = 0.0;
            for (int w = 0; w < (n_own + 63) / 64; ++w) a += red[(par * (nt / 64) + w) * 3 + tid];
            p.partials[((int64_t)blk * 3 + tid) * p.n_tiles + tile] = a;
        }
    };
    // inside: the neighbours of lanes without an own row may be out of buf's reach
    auto mul = [&](const d2 *buf, const d2 &self, bool inside) {
        d2 xc[W];
#pragma unroll
        for (int k = 0; k < W; ++k) xc[k] = buf[hay_place(own || !inside, na[k], (uint32_t)tid)];
        d2 acc;
        acc.x = on * self.x;
        acc.y = on * self.y;
#pragma unroll
        for (int k = 0; k < W; ++k) acc = hmad(h[k], xc[k], acc);
        return acc;
    };
    d2 *cur = xs, *oth = xs + p.lds_rows;
    load(blk0);
    put(blk0, cur);
    for (int blk = blk0; blk < blk1; ++blk) {
        const int par = (blk - blk0) & 1;
        const double s1 = hs[4 * blk], s3 = hs[4 * blk + 1], s2 = hs[4 * blk + 2];
        __syncthreads();
        const d2 u = px, um = pb;  // u_i, u_{i-1}
        if (blk + 1 < blk1) load(blk + 1);
        if (blk > blk0) flush(blk - 1, par ^ 1);
        d2 un = u;
        const d2 *src = cur;
        if (!p.first) {
            const d2 acc = mul(cur, u, false);
            un.x = fma(s1, acc.x, fma(-s3, um.x, -s2 * u.x));
            un.y = fma(s1, acc.y, fma(-s3, um.y, -s2 * u.y));
            if (eval) ys[tid] = un;
            if (own) row_of(p.out_last, blk, g) = un;
            src = ys;
            __syncthreads();
        }
        if (own_wave) {
            const d2 z = mul(src, un, true);
            double n2 = 0.0, hu = 0.0, cr = 0.0;
            if (own) {
                n2 = fma(un.x, un.x, un.y * un.y);
                hu = fma(un.x, z.x, un.y * z.y);
                cr = fma(un.x, u.x, un.y * u.y);
            }
            n2 = wave_sum(n2);
            hu = wave_sum(hu);
            cr = wave_sum(cr);
            if (lane == 63) {
                double *r = red + (par * (nt / 64) + wave) * 3;
                r[0] = n2;
                r[1] = hu;
                r[2] = cr;
            }
        }
        // the other half was read before the last barrier but one
        if (blk + 1 < blk1) put(blk + 1, oth);
        d2 *t = cur;
        cur = oth;
        oth = t;
    }
    __syncthreads();
    flush(blk1 - 1, (blk1 - 1 - blk0) & 1);
}

// The scalars after k_hay_step, from the sums over tiles in a fixed order: one
// workgroup per state.
__global__ __launch_bounds__(kWG) void k_hay_reduce3(const double *__restrict__ part, int n_tiles, int s_user, int first,
                                                     double thr, double *__restrict__ hs, int32_t *counter, int n_iter,
                                                     double *__restrict__ a_out, double *__restrict__ b_out) {
    __shared__ double red[3][kWG];
    const int s = blockIdx.x;
    const double *q = part + (int64_t)s * 3 * n_tiles;
    double v[3][4] = {};
    int t = threadIdx.x;
    for (; t + 3 * kWG < n_tiles; t += 4 * kWG) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int c = 0; c < 3; ++c) v[c][u] += q[(int64_t)c * n_tiles + t + u * kWG];
    }
    for (; t < n_tiles; t += kWG)
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c][0] += q[(int64_t)c * n_tiles + t];
#pragma unroll
    for (int c = 0; c < 3; ++c) red[c][threadIdx.x] = (v[c][0] + v[c][1]) + (v[c][2] + v[c][3]);
    __syncthreads();
    for (int w = kWG / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
#pragma unroll
            for (int c = 0; c < 3; ++c) red[c][threadIdx.x] += red[c][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    double *h = hs + 4 * s;
    const double old = first ? 0.0 : h[0];
    double b = sqrt(red[0][0]), inv = 0.0;
    if (first)
        inv = b > 0.0 ? 1.0 / b : 0.0;
    else if (b > thr && old != 0.0)
        inv = 1.0 / b;
    else
        b = 0.0;
    const double cprev = first ? 0.0 : b * old;
    const double a = inv * (inv * red[1][0]) - cprev * (inv * red[2][0]);
    const int k = first ? -1 : *(volatile const int32_t *)counter - 1;  // iteration
    if (k >= 0 && k < n_iter) b_out[(int64_t)k * s_user + s] = b;
    if (k + 1 < n_iter) a_out[(int64_t)(k + 1) * s_user + s] = a;
    h[0] = inv;
    h[1] = cprev;
    h[2] = a * inv;
    if (first && s == 0) *counter = 0;
}

// d(E_j) = -(1/pi) Im G_0(E_j + i eps), G_0 by the continued fraction from
// the deepest level up; one thread per (energy, state)
__global__ __launch_bounds__(kWG) void k_hay_ldos(const double *__restrict__ a, const double *__restrict__ b,
                                                  int n_iter, int n_states, const double *__restrict__ energies,
                                                  int64_t n_e, double eps, double *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x;
    if (i >= n_e * n_states) return;
    const int s = (int)(i % n_states);
    const int64_t j = i / n_states;
    const double zr = energies[j];
    double tr = zr - a[(int64_t)(n_iter - 1) * n_states + s], ti = eps;
    for (int q = n_iter - 2; q >= 0; --q) {
        const double bq = b[(int64_t)q * n_states + s];
        const double d = tr * tr + ti * ti;
        const double f = bq * bq / d;  // b^2 / t = f conj(t)
        tr = zr - a[(int64_t)q * n_states + s] - f * tr;
        ti = eps + f * ti;
    }
    out[i] = ti / (tr * tr + ti * ti) / M_PI;  // -Im(1/t)/pi
}

}  // namespace

hipError_t launch_hay_spmv(bool cplx, const TileDesc *tiles, int32_t n_tiles, int32_t xcd_remap, int32_t log2s,
                           const int32_t *col, const void *val, const uint32_t *slice_off, int32_t uniform_w,
                           const double *onsite, const double *u, const double *uprev, double *y, const double *hs,
                           int32_t *counter, double *partials, hipStream_t st) {
    if (cplx)
        hipLaunchKernelGGL(k_hay_spmv<true>, dim3((unsigned)n_tiles), dim3(kWG), 0, st, tiles, n_tiles, xcd_remap,
                           log2s, col, val, slice_off, uniform_w, onsite, (const d2 *)u, (const d2 *)uprev, (d2 *)y,
                           hs, counter, partials);
    else
        hipLaunchKernelGGL(k_hay_spmv<false>, dim3((unsigned)n_tiles), dim3(kWG), 0, st, tiles, n_tiles, xcd_remap,
                           log2s, col, val, slice_off, uniform_w, onsite, (const d2 *)u, (const d2 *)uprev, (d2 *)y,
                           hs, counter, partials);
    return hipGetLastError();
}

hipError_t launch_hay_axpy(const TileDesc *tiles, int32_t n_tiles, int32_t xcd_remap, int32_t reverse, int32_t log2s,
                           const double *y, const double *u, double *unext, const double *hs, double *partials,
                           hipStream_t st) {
    hipLaunchKernelGGL(k_hay_axpy, dim3((unsigned)n_tiles), dim3(kWG), 0, st, tiles, n_tiles, xcd_remap, reverse, log2s,
                       (const d2 *)y, (const d2 *)u, (d2 *)unext, hs, partials);
    return hipGetLastError();
}

int32_t hay_fold_count(int32_t n_tiles) { return n_tiles > kFold ? (n_tiles + kFold - 1) / kFold : 0; }

hipError_t launch_hay_reduce(const double *partials, int32_t n_tiles, int32_t s_pad, int32_t s_user, int32_t mode,
                             double thr, double *hs, int32_t *counter, int32_t n_iter, double *a_out, double *b_out,
                             double *fold, hipStream_t st) {
    const double *in = partials + (mode == kHayA ? 0 : 2 * (int64_t)n_tiles);
    int64_t stride = 3 * (int64_t)n_tiles;
    int n = n_tiles;
    const int32_t n_fold = hay_fold_count(n_tiles);
    if (n_fold > 0) {
        hipLaunchKernelGGL(k_hay_fold, dim3((unsigned)n_fold, (unsigned)s_pad), dim3(kWG), 0, st, in, stride, n_tiles,
                           fold, n_fold);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        in = fold;
        stride = n_fold;
        n = n_fold;
    }
    hipLaunchKernelGGL(k_hay_reduce, dim3((unsigned)s_pad), dim3(kWG), 0, st, in, stride, n, s_user, (int)mode, thr,
                       hs, counter, n_iter, a_out, b_out);
    return hipGetLastError();
}

hipError_t launch_hay_step(bool cplx, int width, int max_eval, int max_stage, ChainParams p, const double *hs,
                           hipStream_t st) {
    if (p.n_tiles <= 0) return hipSuccess;
    const unsigned nt = (unsigned)(max_eval + 63) / 64 * 64;
    const size_t lds = 16 * (2 * (size_t)max_stage + nt) + sizeof(double) * 6 * (nt / 64);
    if (max_eval < 1 || nt > kHayThreads || max_stage < max_eval || lds > 64 * 1024 || p.table_depth < 2 || width < 1 ||
        width > kChainWidth || p.n_blk < 1 || p.n_grp < 1 || p.grp_blk < 1)
        return hipErrorInvalidValue;
    p.lds_rows = max_stage;
    const dim3 grid(p.n_grp > 1 ? (unsigned)(((p.n_tiles + 7) / 8) * 8 * p.n_grp) : (unsigned)p.n_tiles), block(nt);
    if (cplx && width <= 3)
        hipLaunchKernelGGL((k_hay_step<true, 3>), grid, block, lds, st, p, hs);
    else if (cplx)
        hipLaunchKernelGGL((k_hay_step<true, 4>), grid, block, lds, st, p, hs);
    else if (width <= 3)
        hipLaunchKernelGGL((k_hay_step<false, 3>), grid, block, lds, st, p, hs);
    else
        hipLaunchKernelGGL((k_hay_step<false, 4>), grid, block, lds, st, p, hs);
    return hipGetLastError();
}

hipError_t launch_hay_reduce3(const double *partials, int32_t n_tiles, int32_t s_user, bool first, double thr, double *hs,
                              int32_t *counter, int32_t n_iter, double *a_out, double *b_out, hipStream_t st) {
    hipLaunchKernelGGL(k_hay_reduce3, dim3((unsigned)s_user), dim3(kWG), 0, st, partials, n_tiles, s_user, first ? 1 : 0,
                       thr, hs, counter, n_iter, a_out, b_out);
    return hipGetLastError();
}

hipError_t launch_hay_ldos(const double *a, const double *b, int32_t n_iter, int32_t n_states, const double *energies,
                           int64_t n_e, double eps, double *out, hipStream_t st) {
    const int64_t total = n_e * n_states;
    hipLaunchKernelGGL(k_hay_ldos, dim3((unsigned)((total + kWG - 1) / kWG)), dim3(kWG), 0, st, a, b, n_iter,
                       n_states, energies, n_e, eps, out);
    return hipGetLastError();
}

}  // namespace tbpm
