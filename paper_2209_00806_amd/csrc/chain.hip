// Several Clenshaw orders per launch (temporal blocking) for gfx950, for
// operators of at most kChainWidth stored elements per row.
//
// A launch evaluates `depth` consecutive orders of a time step,
//     b_j = alpha_j v + beta_j (H b_{j+1}) - b_{j+2}.
// The workgroup of a tile copies b_{j+1} of its own rows and of the rows up to
// depth hops away into LDS; order k is then evaluated on the rows up to depth -
// 1 - k hops away, from one LDS buffer into the other, with one barrier per
// order.  A tile's local rows are sorted by their distance (own rows, then
// shell after shell), so order k is a prefix of them, and one set of tables
// serves every depth up to the one it was built for.  A thread keeps the same
// NR local rows through all orders: psi, b_{j+1}, b_{j+2} and the rows' matrix
// entries stay in registers, and only the neighbours' values pass through LDS.
// Outputs go to memory only where a later launch (or the caller) reads them,
// and to buffers that no tile of the launch reads.
//
// States are stored in blocks of VS states, [block][row][VS] (16 bytes per row
// and block: one FP64 state or two FP32 states): a tile's own rows are
// contiguous at any state count, and a workgroup takes several blocks of its
// tile in turn with the matrix entries still in registers.
//
// What bounds it, on disordered graphene 1024 x 1024 with 8 FP64 states (three
// launches of 5-6 orders per time step, 512-row tiles): loads alone take 0.78 ms
// per time step and the orders alone 0.78 ms (LDS reads with 2.3-fold bank
// conflicts and the chain barrier -> LDS read -> FMAs -> LDS write), and two
// workgroups of 8 waves per CU overlap them to 1.17 ms.  Two orders per launch
// take 2.53 ms, bound by the streams of each launch.  Measured beside it: the
// next block prefetched into registers 1.81-1.97 ms (one workgroup per CU is
// left), prefetched into LDS by loads that write LDS directly 1.37 ms, one row
// per thread (1024 threads) 1.28 ms, two states per row and thread 1.87 ms, 256
// threads with 256-row tiles and 5 orders 1.29 ms.  Neighbour addresses without
// bank conflicts (wrong neighbours) would give 1.10 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "device_util.h"
#include "tbpm_internal.h"

namespace tbpm {
namespace {

__device__ __forceinline__ int read_lane(int x, int l) { return __builtin_amdgcn_readlane(x, l); }
__device__ __forceinline__ float read_lane(float x, int l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l));
}
__device__ __forceinline__ double read_lane(double x, int l) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, l);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Waves per SIMD: a real operator's thread fits 128 registers, which leaves room
// for two workgroups of 8 waves per CU; complex matrix entries take more, so
// their workgroups have 4 waves (three of them per CU).
constexpr int chain_waves(bool ch) { return ch ? 3 : 4; }

// The body of k_chain (Clenshaw orders) and k_chain_cheb (Chebyshev orders
//     T_{j+1} = 2 H~ T_j - T_{j-1},   T_1 = H~ T_0).
// kChainCurrent also applies a current operator to every T_j from the same
// neighbours in LDS.  In the adjoint (kChainAdjoint, T_j = alpha_j) lambda gains
// conj(c_{j+1}) alpha_{j+1}, and own row q adds to the gradient of its transposed
// elements (p, q) Re/Im of alpha_j[p] conj(w b_{j+1}[q]): alpha_j at p is read from
// LDS for the product anyway, b at the own row is the only stream of its own, and
// the sums over orders and state blocks stay in registers until the workgroup
// ends (one read-modify-write per tile and launch, no sum across lanes).
// Measured, DOS and its gradient on graphene 256^2, 4 FP64 states: 37.6 ms with the
// replay storing every order and the adjoint 5 or 6 orders per launch (27 us a
// launch, the replay's 25), 63.7 ms with two orders per launch of both, where the
// adjoint was bound by the read-modify-write of the gradient for every pair of
// orders and the sums over lanes.
template <typename R, bool CH, int W, int VS, int NT, int NR, int MODE>
__device__ __forceinline__ void chain_body(const ChainParams &p, const ChainCheb &ad) {
    extern __shared__ __align__(16) unsigned char chain_mem[];
    constexpr bool CHEB = MODE != kChainClenshaw, ADJ = MODE == kChainAdjoint, CUR = MODE == kChainCurrent;
    using V = VecT<R, VS>;
    using HV = typename HValT<R, CH>::T;
    // the groups of state blocks of a tile run on one XCD (workgroup g goes to XCD g & 7)
    int grp = 0, tslot = (int)blockIdx.x;
    if (p.n_grp > 1) {
        const int r = (int)blockIdx.x >> 3;
        grp = r % p.n_grp;
        tslot = (r / p.n_grp) * 8 + ((int)blockIdx.x & 7);
        if (tslot >= p.n_tiles) return;  // the last group of 8 tiles is partial
    }
    const int blk0 = grp * p.grp_blk, blk1 = min(blk0 + p.grp_blk, p.n_blk);
    const int tile = tile_of_block(tslot, p.n_tiles, p.xcd_remap, p.reverse);
    const TileDesc td = p.tiles[tile];
    const int32_t *cnt = p.cnt + (int64_t)tile * (p.table_depth + 1);
    const int depth = p.depth;
    const int n_own = td.rows;
    const int n_eval = cnt[depth - 1], n_stage = cnt[depth];
    const int n_tab = cnt[p.table_depth - 1];  // rows of the tile's matrix tables
    const uint32_t *rowmap = p.rowmap + p.toff[tile];
    const int64_t lo = p.loff[tile];
    const V *__restrict__ x = (const V *)p.x;
    const V *__restrict__ v = (const V *)p.v;
    const V *__restrict__ b2p = (const V *)p.b2;
    const uint2 *__restrict__ lidx = (const uint2 *)p.lidx + lo;
    const HV *__restrict__ tval = (const HV *)p.tval + lo * W;
    const R *__restrict__ tons = (const R *)p.tons + lo;
    const uint32_t row0 = (uint32_t)td.row0;
    const bool contig = p.contiguous != 0;
    auto grow_of = [&](int lr) -> uint32_t { return (contig && lr < n_own) ? row0 + (uint32_t)lr : rowmap[lr]; };

    // LDS: the outputs of even orders at 0 (NT * NR rows), b_{j+1} and the
    // outputs of odd orders behind them, so that both are constant offsets
    // from a row's address
    using LdsV = __attribute__((address_space(3))) V;
    constexpr uint32_t RB = sizeof(V), OFF = NT * NR * RB;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)chain_mem;
    auto at = [](uint32_t byte) -> LdsV & { return *(LdsV *)(uintptr_t)byte; };

    // lanes past the evaluated rows repeat the last one; what they write to LDS
    // no row reads
    HV h[NR][W];
    R on[NR];
    uint32_t na[NR][W];  // LDS byte addresses of the row's neighbours
    uint32_t g[NR];      // the rows
    const int tid = (int)threadIdx.x;
#pragma unroll
    for (int q = 0; q < NR; ++q) g[q] = grow_of(min(tid + q * NT, n_eval - 1));
    // the outermost shell's rows, one per thread and round
    const int n_shell = n_stage - n_eval;
    uint32_t gs = 0;
    if (tid < n_shell) gs = grow_of(n_eval + tid);
    V xo[NR], ps[NR], bq[NR], xs{};
    auto load_block = [&](int blk, V(&lx)[NR], V(&lv)[NR], V(&lb)[NR], V &ls) {
        const uint32_t eb = (uint32_t)blk * p.n_rows;
#pragma unroll
        for (int q = 0; q < NR; ++q) lx[q] = x[eb + g[q]];
        if (tid < n_shell) ls = x[eb + gs];
        if (p.b2) {
#pragma unroll
            for (int q = 0; q < NR; ++q) lb[q] = b2p[eb + g[q]];
        }
        if (p.v && p.v != p.x) {
#pragma unroll
            for (int q = 0; q < NR; ++q) lv[q] = v[eb + g[q]];
        }
    };
#pragma unroll
    for (int q = 0; q < NR; ++q) ps[q] = V{};
    {
        uint2 li[NR];
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            const int lr = min(tid + q * NT, n_eval - 1);
            li[q] = lidx[lr];
            on[q] = tons[lr];
#pragma unroll
            for (int k = 0; k < W; ++k) h[q][k] = tval[(int64_t)k * n_tab + lr];
        }
#pragma unroll
        for (int q = 0; q < NR; ++q)
#pragma unroll
            for (int k = 0; k < W; ++k) {
                const uint32_t pair = k < 2 ? li[q].x : li[q].y;
                na[q][k] = lds0 + ((k & 1) ? (pair >> 16) : (pair & 0xffffu)) * RB;
            }
    }
    const uint32_t own_at = lds0 + (uint32_t)tid * RB;
    const int wbase = __builtin_amdgcn_readfirstlane(tid);  // the wave's first row of slot 0

    // lane k holds order k's coefficient (the nonzero part of alpha) and its
    // number of rows: the loop reads them with readlane, where scalar loads
    // would make every order's LDS reads wait for them
    const PassCoef *cf = p.coef + (CHEB ? 0 : td.inst);
    R alpha_l = R(0), beta, beta_last;
    int lim_l;
    {
        const int k = min(tid & 63, depth - 1);
        lim_l = cnt[depth - 1 - k];
        if constexpr (CHEB) {
            beta = beta_last = (R)(2.0 * ad.inv_f);
        } else {
            const PassCoef c = cf[(int64_t)k * p.n_inst];
            alpha_l = (R)(c.ai != 0.0 ? c.ai : c.ar);
            if (p.turned && !(k & 1)) alpha_l = (R)c.ai;
            if (p.turned && (k & 1)) alpha_l = -(R)c.ar;
            beta = (R)cf[(int64_t)(p.first && depth > 1 ? 1 : 0) * p.n_inst].br;
            beta_last = (R)cf[(int64_t)(depth - 1) * p.n_inst].br;
        }
    }
    uint32_t eb = 0;
    // adjoint: the gradient sums of the own row (slot 0), its lambda and weighted b
    const bool own = tid < n_own;
    double ga[ADJ ? W : 1], gi[ADJ && CH ? W : 1], gd = 0.0;
    d2 lam, bw, bn, cc_l;
    // the current operator's elements of the own row
    d2 jv[CUR ? W : 1], jx;
    if constexpr (CUR) {
        const uint32_t sl = g[0] / kSliceRows, off = ad.slice_off[sl];
        const int w = (int)((ad.slice_off[sl + 1] - off) / kSliceRows);
#pragma unroll
        for (int i = 0; i < W; ++i) {
            jv[i].x = jv[i].y = 0.0;
            if (own && i < w) jv[i] = ((const d2 *)ad.jval)[off + i * kSliceRows + g[0] % kSliceRows];
        }
    }
    if constexpr (ADJ) {
#pragma unroll
        for (int i = 0; i < W; ++i) ga[i] = 0.0;
        if constexpr (CH) {
#pragma unroll
            for (int i = 0; i < W; ++i) gi[i] = 0.0;
        }
        cc_l = ((const d2 *)ad.cc)[min(tid & 63, depth - 1) + 1];
    }
    // b of order k at the own row
    auto load_b = [&](int k) {
        const char *src = ad.final_ && k + 1 == depth ? (const char *)ad.psi : (const char *)ad.bq + (int64_t)k * ad.bq_stride;
        d2 z;
        z.x = z.y = 0.0;
        return own ? ((const d2 *)src)[eb + g[0]] : z;
    };

    // B <- alpha psi + beta (H X) - B on the first N slots of this wave; IMAG:
    // alpha is imaginary (a its imaginary part)
    auto slots = [&](auto n_c, auto imag_c, V(&X)[NR], V(&B)[NR], R a, R bt, uint32_t rd) {
        constexpr int N = decltype(n_c)::value;
        constexpr bool IMAG = decltype(imag_c)::value;
        V xc[N][W];
#pragma unroll
        for (int q = 0; q < N; ++q)
#pragma unroll
            for (int i = 0; i < W; ++i) xc[q][i] = at(na[q][i] + rd);
        V acc[N];
        if constexpr (CUR) {
            jx.x = jx.y = 0.0;
#pragma unroll
            for (int i = 0; i < W; ++i) {
                jx.x = fma(jv[i].x, xc[0][i][0], fma(-jv[i].y, xc[0][i][1], jx.x));
                jx.y = fma(jv[i].x, xc[0][i][1], fma(jv[i].y, xc[0][i][0], jx.y));
            }
        }
        if constexpr (ADJ) {
            gd = fma(X[0][0], bw.x, fma(X[0][1], bw.y, gd));
#pragma unroll
            for (int i = 0; i < W; ++i) {
                ga[i] = fma(xc[0][i][0], bw.x, fma(xc[0][i][1], bw.y, ga[i]));
                if constexpr (CH) gi[i] = fma(xc[0][i][1], bw.x, fma(-xc[0][i][0], bw.y, gi[i]));
            }
        }
#pragma unroll
        for (int q = 0; q < N; ++q) {
            if constexpr (CHEB) {
                B[q] = -B[q];
            } else if constexpr (sizeof(R) == 8) {
#pragma unroll
                for (int i = 0; i < VS; ++i) {
                    if constexpr (IMAG) {
                        B[q][2 * i] = fma(-a, ps[q][2 * i + 1], -B[q][2 * i]);
                        B[q][2 * i + 1] = fma(a, ps[q][2 * i], -B[q][2 * i + 1]);
                    } else {
                        B[q][2 * i] = fma(a, ps[q][2 * i], -B[q][2 * i]);
                        B[q][2 * i + 1] = fma(a, ps[q][2 * i + 1], -B[q][2 * i + 1]);
                    }
                }
            }
            acc[q] = on[q] * X[q];
        }
#pragma unroll
        for (int i = 0; i < W; ++i)
#pragma unroll
            for (int q = 0; q < N; ++q) {
                if constexpr (CH)
                    unit_mad_cplx<R, VS>(h[q][i], xc[q][i], acc[q]);
                else
                    unit_mad_real<R, VS>(h[q][i], xc[q][i], acc[q]);
            }
#pragma unroll
        for (int q = 0; q < N; ++q) {
            if constexpr (sizeof(R) == 8) {
#pragma unroll
                for (int i = 0; i < 2 * VS; ++i) B[q][i] = fma(bt, acc[q][i], B[q][i]);
            } else {
                // FP32: the products and sums of the one-order kernels, each rounded
#pragma clang fp contract(off)
#pragma unroll
                for (int i = 0; i < VS; ++i) {
                    const R tr = IMAG ? -(a * ps[q][2 * i + 1]) : a * ps[q][2 * i];
                    const R ti = IMAG ? a * ps[q][2 * i] : a * ps[q][2 * i + 1];
                    B[q][2 * i] = (tr + bt * acc[q][2 * i]) - B[q][2 * i];
                    B[q][2 * i + 1] = (ti + bt * acc[q][2 * i + 1]) - B[q][2 * i + 1];
                }
            }
        }
    };
    // the first order of a time step: beta is complex, X = psi, no b_{j+2}
    auto first_order = [&]() {
        const PassCoef c = cf[0];
        const R ar = (R)c.ar, ai = (R)c.ai, br = (R)c.br, bi = (R)c.bi;
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            V acc = on[q] * xo[q];
#pragma unroll
            for (int i = 0; i < W; ++i) {
                const V xc = at(na[q][i] + OFF);
                if constexpr (CH)
                    unit_mad_cplx<R, VS>(h[q][i], xc, acc);
                else
                    unit_mad_real<R, VS>(h[q][i], xc, acc);
            }
#pragma unroll
            for (int i = 0; i < VS; ++i) {
                const R vr = xo[q][2 * i], vi = xo[q][2 * i + 1];
                const R hr = acc[2 * i], hi = acc[2 * i + 1];
                bq[q][2 * i] = ar * vr - ai * vi + (br * hr - bi * hi);
                bq[q][2 * i + 1] = ar * vi + ai * vr + (br * hi + bi * hr);
            }
        }
    };
    auto order = [&](auto imag_c, int k, V(&X)[NR], V(&B)[NR], uint32_t rd) {
        __syncthreads();
        const int act = read_lane(lim_l, k) - wbase;
        const R a = CHEB ? R(0) : read_lane(alpha_l, k);
        R bt = k + 1 == depth ? beta_last : beta;
        if constexpr (CHEB)
            if (ad.first && k == 0) bt = ad.inv_f;
        if constexpr (ADJ) {
            const bool j0 = ad.first && k == 0;
            // the weighted b of this order, and the load of the next one's
            const double w = j0 ? 1.0 : 2.0;
            bw = bn * w;
            if (ad.final_ && k + 1 == depth) {
                d2 bs;
                bs.x = ad.bs_re;
                bs.y = ad.bs_im;
                bw = cmul(bs, bn) * w;
            }
            if (k + 1 < depth) bn = load_b(k + 1);
        }
        if (NR >= 2 && act > NT)
            slots(std::integral_constant<int, NR>{}, imag_c, X, B, a, bt, rd);
        else if (act > 0)
            slots(std::integral_constant<int, 1>{}, imag_c, X, B, a, bt, rd);
        if constexpr (CUR)
            if (own) stv<true>((d2 *)((char *)ad.jout + (int64_t)k * ad.jout_stride) + (eb + g[0]), jx);
        if constexpr (ADJ) {
            d2 c, v0;
            c.x = read_lane(cc_l.x, k);
            c.y = read_lane(cc_l.y, k);
            v0.x = B[0][0];
            v0.y = B[0][1];
            lam += cmul(c, v0);
        }
    };
    auto keep = [&](int k, V(&B)[NR], uint32_t wr) {
        // inactive rows' values are written too: no row reads them
        if (k + 1 < depth) {
            const int act = read_lane(lim_l, k) - wbase;
#pragma unroll
            for (int q = 0; q < NR; ++q)
                if (act > q * NT) at(own_at + (uint32_t)(q * NT) * RB + wr) = B[q];
        }
        V *out = k + 1 == depth ? (V *)p.out_last : (k + 2 == depth ? (V *)p.out_prev : nullptr);
        if (p.out_all && k + 1 < depth) out = (V *)((char *)p.out_all + (int64_t)k * p.out_stride);
        if (out) {
#pragma unroll
            for (int q = 0; q < NR; ++q)
                if (tid + q * NT < n_own) stv<true>(out + (eb + g[q]), B[q]);
        }
    };
    for (int blk = blk0; blk < blk1; ++blk) {
        eb = (uint32_t)blk * p.n_rows;
#pragma unroll
        for (int q = 0; q < NR; ++q) bq[q] = V{};
        // the loads of one workgroup go ahead of the other's orders
        __builtin_amdgcn_s_setprio(1);
        load_block(blk, xo, ps, bq, xs);
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            if (tid + q * NT < n_eval) at(own_at + OFF + (uint32_t)(q * NT) * RB) = xo[q];
            if (!CHEB && p.v == p.x) ps[q] = xo[q];
            if (!CHEB && p.turned) {  // i psi: the first order's alpha is imaginary, the second's real
#pragma unroll
                for (int i = 0; i < VS; ++i) {
                    const R t = ps[q][2 * i];
                    ps[q][2 * i] = -ps[q][2 * i + 1];
                    ps[q][2 * i + 1] = t;
                }
            }
        }
        if (tid < n_shell) at(own_at + OFF + (uint32_t)n_eval * RB) = xs;
        for (int l = tid + NT; l < n_shell; l += NT)
            at(lds0 + OFF + (uint32_t)(n_eval + l) * RB) = x[eb + grow_of(n_eval + l)];
        if constexpr (ADJ) {
            bn = load_b(0);
            lam.x = lam.y = 0.0;
            if (ad.first) {
                d2 x0;
                x0.x = xo[0][0];
                x0.y = xo[0][1];
                lam = cmul(((const d2 *)ad.cc)[0], x0);
            } else if (own) {
                lam = ((const d2 *)ad.lam)[eb + g[0]];
            }
        }
        __builtin_amdgcn_s_setprio(0);
        for (int k = 0; k < depth; k += 2) {
            if (!CHEB && k == 0 && p.first) {
                __syncthreads();
                first_order();
#pragma unroll
                for (int q = 0; q < NR; ++q) xo[q] = V{};  // the second order has no b_{j+2}
            } else {
                order(std::integral_constant<bool, false>{}, k, xo, bq, OFF);
            }
            keep(k, bq, 0u);
            if (k + 1 < depth) {
                if (!CHEB && p.alt)
                    order(std::integral_constant<bool, true>{}, k + 1, bq, xo, 0u);
                else
                    order(std::integral_constant<bool, false>{}, k + 1, bq, xo, 0u);
                keep(k + 1, xo, OFF);
            }
        }
        if (depth & 1) {
#pragma unroll
            for (int q = 0; q < NR; ++q) xo[q] = bq[q];
        }
        if constexpr (ADJ) {
            if (own) {
                if (ad.final_ && blk < p.s_user)
                    lam += cmul(((const d2 *)ad.gcorr_l)[blk], ((const d2 *)p.phi0)[eb + g[0]]);
                ((d2 *)ad.lam)[eb + g[0]] = lam;
            }
        } else if (!CHEB && p.partials) {
            // <phi0|psi'> and ||psi'||^2 of the own rows, per state of the block
            double dre[VS], dim[VS], nrm[VS];
#pragma unroll
            for (int i = 0; i < VS; ++i) dre[i] = dim[i] = nrm[i] = 0.0;
            // the counter holds the step before those not summed yet
            const int64_t ckpt =
                p.ckpt_slot ? (int64_t)p.ckpt_slot[*(volatile const int32_t *)p.counter + 1 + p.local] : -1;
#pragma unroll
            for (int q = 0; q < NR; ++q) {
                if (tid + q * NT < n_own) {
#pragma unroll
                    for (int i = 0; i < VS; ++i) {
                        const d2 ph = ((const d2 *)p.phi0)[(int64_t)(eb + g[q]) * VS + i];
                        const double oxr = (double)xo[q][2 * i], oyi = (double)xo[q][2 * i + 1];
                        dre[i] = fma(ph.x, oxr, fma(ph.y, oyi, dre[i]));
                        dim[i] = fma(ph.x, oyi, fma(-ph.y, oxr, dim[i]));
                        nrm[i] = fma(oxr, oxr, fma(oyi, oyi, nrm[i]));
                        if (ckpt >= 0 && blk * VS + i < p.s_user) {
                            d2 oc;
                            oc.x = oxr;
                            oc.y = oyi;
                            const int64_t crow = p.perm ? (int64_t)p.perm[g[q]] : (int64_t)g[q];
                            ((d2 *)p.ckpt)[ckpt * p.ckpt_stride + crow * p.s_user + blk * VS + i] = oc;
                        }
                    }
                }
            }
            __syncthreads();  // the staged rows are dead: their LDS takes the partial sums
            double *red = reinterpret_cast<double *>(chain_mem);
            const int lane = tid & 63, wave = tid >> 6;
            const int own_waves = min(NT / 64, (n_own + 63) >> 6);
            if (wave < own_waves) {
#pragma unroll
                for (int i = 0; i < VS; ++i) {
                    const double a = wave_sum(dre[i]), b = wave_sum(dim[i]), c = wave_sum(nrm[i]);
                    if (lane == 63) {
                        red[(wave * VS + i) * 3] = a;
                        red[(wave * VS + i) * 3 + 1] = b;
                        red[(wave * VS + i) * 3 + 2] = c;
                    }
                }
            }
            __syncthreads();
            if (tid < 3 * VS) {
                double a = 0.0;
                for (int w = 0; w < own_waves; ++w) a += red[w * VS * 3 + tid];
                p.partials[((int64_t)blk * VS * 3 + tid) * p.n_tiles + tile] = a;
            }
        }
        if (blk + 1 < blk1) __syncthreads();  // the next block's rows overwrite the LDS
    }
    if constexpr (ADJ) {
        if (own) {
            const uint32_t row = g[0], sl = row / kSliceRows, off = ad.slice_off[sl];
            const int w = (int)((ad.slice_off[sl + 1] - off) / kSliceRows);
            HV *ga_out = (HV *)ad.gacc + (int64_t)grp * ad.ell_size + off + row % kSliceRows;
            ad.gdiag[(int64_t)grp * p.n_rows + row] += gd;
#pragma unroll
            for (int i = 0; i < W; ++i)
                if (i < w) {
                    if constexpr (CH) {
                        HV v = ga_out[i * kSliceRows];
                        v.x += ga[i];
                        v.y += gi[i];
                        ga_out[i * kSliceRows] = v;
                    } else {
                        ga_out[i * kSliceRows] += ga[i];
                    }
                }
        }
    }
}

template <typename R, bool CH, int W, int VS, int NT, int NR>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(chain_waves(CH)))) void k_chain(const ChainParams p) {
    chain_body<R, CH, W, VS, NT, NR, kChainClenshaw>(p, ChainCheb{});
}

template <bool CH, int W, int NT, int NR, int MODE>
__global__ __launch_bounds__(NT)
    __attribute__((amdgpu_waves_per_eu(chain_waves(CH)))) void k_chain_cheb(const ChainParams p, const ChainCheb ad) {
    chain_body<double, CH, W, 1, NT, NR, MODE>(p, ad);
}

// The tile tables' matrix entries: for every local row of a tile (up to
// table_depth - 1 hops away) its on-site energy and its stored elements, in the
// tile's local order.
template <typename HV, typename R>
__global__ __launch_bounds__(kWG) void k_chain_values(const ChainTileTab t, const HV *__restrict__ val,
                                                      const R *__restrict__ ons, const uint32_t *__restrict__ soff,
                                                      HV *__restrict__ tval, R *__restrict__ tons) {
    const int tile = blockIdx.x;
    const int n_tab = t.cnt[(int64_t)tile * (t.table_depth + 1) + t.table_depth - 1];
    const uint32_t *rowmap = t.rowmap + t.toff[tile];
    const int64_t lo = t.loff[tile];
    for (int lr = threadIdx.x; lr < n_tab; lr += kWG) {
        const uint32_t row = rowmap[lr];
        const uint32_t sl = row / kSliceRows;
        const uint32_t off = soff[sl];
        const int w = (int)((soff[sl + 1] - off) / kSliceRows);
        tons[lo + lr] = ons[row];
        for (int k = 0; k < t.width; ++k)
            tval[lo * t.width + (int64_t)k * n_tab + lr] =
                k < w ? val[off + (uint32_t)k * kSliceRows + row % kSliceRows] : HV{};
    }
}

// Second stage of the correlation for the steps of one replayed graph: one
// workgroup per (step, member, state) sums the per-tile partials of that
// member in a fixed order into sample counter + 1 + step; the last workgroup
// to finish advances the counter (every workgroup has read it by then).
__global__ __launch_bounds__(kWG) void k_chain_reduce(const ReduceParams p, int n_local, int64_t step_stride,
                                                      int32_t *counter, int advance) {
    __shared__ double red[3][kWG];
    const int k0 = *(volatile const int32_t *)counter;
    const int per = gridDim.x / n_local;
    const int step = blockIdx.x / per;
    const int rem = blockIdx.x % per;
    const int inst = rem / p.s_user;
    const int s = rem % p.s_user;
    const int t0 = p.inst_tile0[inst], t1 = p.inst_tile0[inst + 1];
    const int64_t nt = p.n_tiles;
    const double *q0 = p.partials + (int64_t)step * step_stride + (int64_t)s * 3 * nt;
    double a[2] = {0, 0}, b[2] = {0, 0}, c[2] = {0, 0};
    int t = t0 + threadIdx.x;
    for (; t + kWG < t1; t += 2 * kWG) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            a[u] += q0[t + u * kWG];
            b[u] += q0[nt + t + u * kWG];
            c[u] += q0[2 * nt + t + u * kWG];
        }
    }
    for (; t < t1; t += kWG) {
        a[0] += q0[t];
        b[0] += q0[nt + t];
        c[0] += q0[2 * nt + t];
    }
    red[0][threadIdx.x] = a[0] + a[1];
    red[1][threadIdx.x] = b[0] + b[1];
    red[2][threadIdx.x] = c[0] + c[1];
    __syncthreads();
    for (int h = kWG / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            red[0][threadIdx.x] += red[0][threadIdx.x + h];
            red[1][threadIdx.x] += red[1][threadIdx.x + h];
            red[2][threadIdx.x] += red[2][threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const int k = k0 + 1 + step;
        if (k >= 0 && k < p.n_steps) {
            const int64_t o = (int64_t)k * p.s_user + s;
            d2 cc;
            cc.x = red[0][0];
            cc.y = red[1][0];
            ((d2 *)p.corr[inst])[o] = cc;
            if (p.norm2[inst]) p.norm2[inst][o] = red[2][0];
            if (p.norm2_all) p.norm2_all[(int64_t)inst * p.n_steps * p.s_user + o] = red[2][0];
        }
        if (!advance) return;
        __threadfence();
        if (atomicAdd(counter + 1, 1) == (int)gridDim.x - 1) {
            atomicExch(counter + 1, 0);
            atomicExch(counter, k0 + n_local);
        }
    }
}

template <typename R, bool CH, int W, int VS>
hipError_t launch_chain_t(const ChainParams &p, size_t lds, hipStream_t st) {
    const dim3 grid(p.n_grp > 1 ? (unsigned)(((p.n_tiles + 7) / 8) * 8 * p.n_grp) : (unsigned)p.n_tiles);
    constexpr int NT = chain_threads(CH);
    hipLaunchKernelGGL((k_chain<R, CH, W, VS, NT, kChainRowsPerThread>), grid, dim3(NT), lds, st, p);
    return hipGetLastError();
}

template <typename R, int VS>
hipError_t launch_chain_r(bool cplx, int width, const ChainParams &p, size_t lds, hipStream_t st) {
    if (cplx) return width <= 3 ? launch_chain_t<R, true, 3, VS>(p, lds, st) : launch_chain_t<R, true, 4, VS>(p, lds, st);
    return width <= 3 ? launch_chain_t<R, false, 3, VS>(p, lds, st) : launch_chain_t<R, false, 4, VS>(p, lds, st);
}

}  // namespace

static bool chain_valid(bool cplx, int width, int max_eval, const ChainParams &p) {
    return p.depth >= 1 && p.depth <= p.table_depth && p.depth <= kChainMaxDepth && max_eval <= chain_rows(cplx) &&
           width >= 1 && width <= kChainWidth && p.n_blk >= 1 && p.n_grp >= 1 && p.grp_blk >= 1;
}

template <int MODE>
static void launch_cheb_t(bool cplx, int width, dim3 grid, size_t lds, const ChainParams &p, const ChainCheb &ad,
                          hipStream_t st) {
    constexpr int TR = chain_threads(false), TC = chain_threads(true), NR = kChainRowsPerThread;
    if (cplx && width <= 3)
        hipLaunchKernelGGL((k_chain_cheb<true, 3, TC, NR, MODE>), grid, dim3(TC), lds, st, p, ad);
    else if (cplx)
        hipLaunchKernelGGL((k_chain_cheb<true, 4, TC, NR, MODE>), grid, dim3(TC), lds, st, p, ad);
    else if (width <= 3)
        hipLaunchKernelGGL((k_chain_cheb<false, 3, TR, NR, MODE>), grid, dim3(TR), lds, st, p, ad);
    else
        hipLaunchKernelGGL((k_chain_cheb<false, 4, TR, NR, MODE>), grid, dim3(TR), lds, st, p, ad);
}

hipError_t launch_chain_cheb(int mode, bool cplx, int width, int max_own, int max_eval, int max_stage,
                             const ChainParams &p, const ChainCheb &ad, hipStream_t st) {
    if (p.n_tiles <= 0) return hipSuccess;
    // own rows are slot 0 of a thread
    if (!chain_valid(cplx, width, max_eval, p) || max_own > chain_threads(cplx)) return hipErrorInvalidValue;
    const int rows = chain_rows(cplx);
    const size_t lds = (size_t)16 * (rows + std::max(rows, max_stage));
    if (lds > 64 * 1024) return hipErrorInvalidValue;
    const dim3 grid(p.n_grp > 1 ? (unsigned)(((p.n_tiles + 7) / 8) * 8 * p.n_grp) : (unsigned)p.n_tiles);
    if (mode == kChainAdjoint)
        launch_cheb_t<kChainAdjoint>(cplx, width, grid, lds, p, ad, st);
    else if (mode == kChainCurrent)
        launch_cheb_t<kChainCurrent>(cplx, width, grid, lds, p, ad, st);
    else if (mode == kChainCheb)
        launch_cheb_t<kChainCheb>(cplx, width, grid, lds, p, ad, st);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_chain(bool fp32, bool cplx, int width, int vs, int max_eval, int max_stage, const ChainParams &p,
                        hipStream_t st) {
    if (p.n_tiles <= 0) return hipSuccess;
    const int rows = chain_rows(cplx);
    if (!chain_valid(cplx, width, max_eval, p)) return hipErrorInvalidValue;
    // both buffers, and at least the partial sums of the correlation
    const size_t lds = (size_t)(fp32 ? 8 : 16) * vs * (rows + std::max(rows, max_stage));
    if (lds > 64 * 1024) return hipErrorInvalidValue;
    if (fp32) {
        if (vs == 2) return launch_chain_r<float, 2>(cplx, width, p, lds, st);
        if (vs == 1) return launch_chain_r<float, 1>(cplx, width, p, lds, st);
        return hipErrorInvalidValue;
    }
    return vs == 1 ? launch_chain_r<double, 1>(cplx, width, p, lds, st) : hipErrorInvalidValue;
}

hipError_t launch_chain_values(bool fp32, bool cplx, const ChainTileTab &t, int32_t n_tiles, const DevMatrix &m,
                               void *tval, void *tons, hipStream_t st) {
    const dim3 grid((unsigned)n_tiles), block(kWG);
    if (fp32 && cplx)
        hipLaunchKernelGGL((k_chain_values<f2, float>), grid, block, 0, st, t, (const f2 *)m.val32, m.onsite32,
                           m.slice_off, (f2 *)tval, (float *)tons);
    else if (fp32)
        hipLaunchKernelGGL((k_chain_values<float, float>), grid, block, 0, st, t, (const float *)m.val32, m.onsite32,
                           m.slice_off, (float *)tval, (float *)tons);
    else if (cplx)
        hipLaunchKernelGGL((k_chain_values<d2, double>), grid, block, 0, st, t, (const d2 *)m.val64, m.onsite64,
                           m.slice_off, (d2 *)tval, (double *)tons);
    else
        hipLaunchKernelGGL((k_chain_values<double, double>), grid, block, 0, st, t, (const double *)m.val64,
                           m.onsite64, m.slice_off, (double *)tval, (double *)tons);
    return hipGetLastError();
}

hipError_t launch_chain_reduce(int n_inst, int n_local, int64_t step_stride, const ReduceParams &p, int32_t *counter,
                               bool advance, hipStream_t st) {
    hipLaunchKernelGGL(k_chain_reduce, dim3((unsigned)(n_local * n_inst * p.s_user)), dim3(kWG), 0, st, p, n_local,
                       step_stride, counter, advance ? 1 : 0);
    return hipGetLastError();
}

}  // namespace tbpm
