// One Clenshaw order per launch for real operators of up to kWideWidth stored
// elements per row:
//     b_j = alpha_j v + beta_j (H b_{j+1}) - b_{j+2}.
// A workgroup holds the matrix entries of its tile's rows (one row per thread)
// and the LDS places of their neighbours in registers, and takes several blocks
// of states in turn: per block and stored element a thread then has one
// 16-byte LDS read and the multiply-adds of the block's VS states, and no index
// or value load.  The rows of the next block (the tile's own and those one hop
// away) are loaded while a block is evaluated, and go into the other half of
// the LDS; one barrier per block.  States are stored in blocks, as for the chain
// kernel, so that own rows are contiguous at any state count.
//
// Measured, bilayer 192^2 (19 elements per row, 147456 rows), one pass: 16 FP32
// states 19.3 us (staged pass 25.5), 16 FP64 states 31.8 us (49.9), 4 FP64 states
// 14.7 us (17.1).  A block takes 1.5 us, its five streams at 8 TB/s; the rest, 7 us,
// is the launch, the chain of loads from the tile's descriptor to its rows, and the
// matrix entries.  Two orders per launch (one workgroup of 16 waves per CU, two
// more hops of rows) took 34.8 ms for what takes 21.0 ms here.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "device_util.h"
#include "tbpm_internal.h"

namespace tbpm {
namespace {

// on xo + H x of one row: its W neighbours are at byte offsets na (two in a
// register) from `base` in LDS.  The reads go in batches of KC, two batches in
// flight.
template <typename R, int W, int VS, int KC>
__device__ __forceinline__ VecT<R, VS> wide_row(const R (&h)[W], const uint32_t (&na)[W / 2], uint32_t base, R on,
                                                const VecT<R, VS> &xo) {
    using V = VecT<R, VS>;
    using LdsV = __attribute__((address_space(3))) V;
    V xb[2][KC];
    auto gather = [&](int i0) {
#pragma unroll
        for (int i = 0; i < KC; ++i)
            if (i0 + i < W) {
                // volatile: unpacked here, and not kept unpacked in twice the registers
                uint32_t at;
                if (i & 1)
                    asm volatile("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1"
                                 : "=v"(at) : "v"(base), "v"(na[(i0 + i) / 2]));
                else
                    asm volatile("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0"
                                 : "=v"(at) : "v"(base), "v"(na[(i0 + i) / 2]));
                xb[(i0 / KC) & 1][i] = *(LdsV *)(uintptr_t)at;
            }
    };
    gather(0);
    V acc = on * xo;
#pragma unroll
    for (int i0 = 0; i0 < W; i0 += KC) {
        // the sums so far pass through an empty statement that no read of a later
        // batch is moved over: all reads at once would spill
#pragma unroll
        for (int c = 0; c < 2 * VS; ++c) {
            R t = acc[c];
            asm volatile("" : "+v"(t)::"memory");
            acc[c] = t;
        }
        if (i0 + KC < W) gather(i0 + KC);
#pragma unroll
        for (int i = 0; i < KC; ++i)
            if (i0 + i < W) unit_mad_real<R, VS>(h[i0 + i], xb[(i0 / KC) & 1][i], acc);
    }
    return acc;
}

// alpha v + beta (H x)
template <typename R, int VS>
__device__ __forceinline__ VecT<R, VS> wide_order(const PassCoef &c, const VecT<R, VS> &v, const VecT<R, VS> &hx) {
    const R ar = (R)c.ar, ai = (R)c.ai, br = (R)c.br, bi = (R)c.bi;
    VecT<R, VS> o;
#pragma unroll
    for (int i = 0; i < VS; ++i) {
        const R vr = v[2 * i], vi = v[2 * i + 1];
        const R hr = hx[2 * i], hi = hx[2 * i + 1];
        o[2 * i] = ar * vr - ai * vi + (br * hr - bi * hi);
        o[2 * i + 1] = ar * vi + ai * vr + (br * hi + bi * hr);
    }
    return o;
}

// <phi0|psi'> and ||psi'||^2 of the tile's own rows, per state of block blk
// (o: psi' at own row g), through `red` (3 VS doubles per wave); with a slot, the
// states go to the checkpoint.  All threads of the workgroup take part.
template <typename R, int VS>
__device__ __forceinline__ void wide_partials(const ChainParams &p, int tile, int blk, bool own, uint32_t g, int64_t ckpt,
                                              const VecT<R, VS> &o, double *red) {
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int i = 0; i < VS; ++i) {
        double dre = 0.0, dim = 0.0, nrm = 0.0;
        if (own) {
            const d2 ph = ((const d2 *)p.phi0)[((int64_t)blk * p.n_rows + g) * VS + i];
            const double oxr = (double)o[2 * i], oyi = (double)o[2 * i + 1];
            dre = fma(ph.x, oxr, ph.y * oyi);
            dim = fma(ph.x, oyi, -(ph.y * oxr));
            nrm = fma(oxr, oxr, oyi * oyi);
            if (ckpt >= 0 && blk * VS + i < p.s_user) {
                d2 oc;
                oc.x = oxr;
                oc.y = oyi;
                const int64_t crow = p.perm ? (int64_t)p.perm[g] : (int64_t)g;
                ((d2 *)p.ckpt)[ckpt * p.ckpt_stride + crow * p.s_user + blk * VS + i] = oc;
            }
        }
        dre = wave_sum(dre);
        dim = wave_sum(dim);
        nrm = wave_sum(nrm);
        if (lane == 63) {
            red[(wave * VS + i) * 3] = dre;
            red[(wave * VS + i) * 3 + 1] = dim;
            red[(wave * VS + i) * 3 + 2] = nrm;
        }
    }
    __syncthreads();
    if (tid < 3 * VS) {
        double a = 0.0;
        for (int w = 0; w < (int)blockDim.x / 64; ++w) a += red[w * VS * 3 + tid];
        p.partials[((int64_t)blk * VS * 3 + tid) * p.n_tiles + tile] = a;
    }
}

template <typename R, int W, int VS>
__global__ __launch_bounds__(kWideThreads) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 8 ? 3 : 4))) void k_pass_wide(const ChainParams p) {
    extern __shared__ __align__(16) unsigned char wide_mem[];
    using V = VecT<R, VS>;
    constexpr int KC = 4;     // stored elements per batch of LDS reads
    constexpr int NSH = 2;    // shell rows per thread whose loads run ahead
    constexpr uint32_t RB = sizeof(V);
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
    if (p.bump && blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(p.counter, 1);
    if (blk0 >= blk1) return;
    const TileDesc td = p.tiles[tile];
    const PassCoef pc = p.coef[td.inst];
    const int n_own = td.rows, n_shell = p.cnt[2 * (int64_t)tile + 1] - n_own;
    const uint32_t *rowmap = p.rowmap + p.toff[tile];
    const int64_t lo = p.loff[tile];
    const int tid = (int)threadIdx.x, nt = (int)blockDim.x;
    const bool own = tid < n_own;
    const int lr = min(tid, n_own - 1);
    const uint32_t g = p.contiguous ? (uint32_t)td.row0 + (uint32_t)lr : rowmap[lr];
    uint32_t gs[NSH];
#pragma unroll
    for (int i = 0; i < NSH; ++i) gs[i] = tid + i * nt < n_shell ? rowmap[n_own + tid + i * nt] : g;

    using LdsV = __attribute__((address_space(3))) V;
    auto at = [](uint32_t byte) -> LdsV & { return *(LdsV *)(uintptr_t)byte; };
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)wide_mem;
    const uint32_t half = (uint32_t)p.lds_rows * RB;

    // matrix entries, and the neighbours' byte offsets in a half, two in a register
    R h[W];
    uint32_t na[W / 2];
    const R on = ((const R *)p.tons)[lo + lr];
    {
        // wave-uniform columns, 32-bit byte offsets within
        const R *tval = (const R *)p.tval + lo * W;
        const uint16_t *li = p.lidx + lo * W;
        auto col_at = [&](int k) { return (uint32_t)*(const uint16_t *)((const char *)(li + (int64_t)k * n_own) + (uint32_t)lr * 2u); };
#pragma unroll
        for (int k = 0; k < W; ++k)
            h[k] = *(const R *)((const char *)(tval + (int64_t)k * n_own) + (uint32_t)lr * (uint32_t)sizeof(R));
#pragma unroll
        for (int k = 0; k < W; k += 2) na[k / 2] = col_at(k) * RB | (col_at(k + 1) * RB) << 16;
    }

    // a block's vector: its place in memory is wave-uniform, rows are 32-bit byte offsets
    const int64_t bstride = (int64_t)p.n_rows * RB;
    auto row_of = [&](const void *base, int blk, uint32_t off) -> V & {
        return *(V *)((char *)base + blk * bstride + off);
    };
    // the loads of a block are unconditional (lanes without a row repeat one, absent
    // b_{j+2} is read from psi), so that a wait for them is no wait for later ones
    const void *b2p = p.b2 ? p.b2 : p.v;
    V px, psh[NSH], pv, pb;
    auto load = [&](int blk) {
        px = row_of(p.x, blk, g * RB);
#pragma unroll
        for (int i = 0; i < NSH; ++i) psh[i] = row_of(p.x, blk, gs[i] * RB);
        pv = row_of(p.v, blk, g * RB);
        pb = row_of(b2p, blk, g * RB);
    };
    auto put = [&](int blk, uint32_t base) {
        if (own) at(base + (uint32_t)tid * RB) = px;
#pragma unroll
        for (int i = 0; i < NSH; ++i)
            if (tid + i * nt < n_shell) at(base + (uint32_t)(n_own + tid + i * nt) * RB) = psh[i];
        for (int l = tid + NSH * nt; l < n_shell; l += nt)
            at(base + (uint32_t)(n_own + l) * RB) = row_of(p.x, blk, rowmap[n_own + l] * RB);
    };

    int64_t ckpt = -1;
    if (p.partials && p.ckpt_slot) ckpt = p.ckpt_slot[*(volatile const int32_t *)p.counter + 1 + p.local];
    uint32_t cur = lds0, oth = lds0 + half;
    auto step = [&](int blk, auto more_c) {
        constexpr bool MORE = decltype(more_c)::value;
        __syncthreads();
        const V vv = pv, bq = pb;
        if constexpr (MORE) load(blk + 1);
        const V xo = at(cur + (uint32_t)lr * RB);
        V o = wide_order<R, VS>(pc, vv, wide_row<R, W, VS, KC>(h, na, cur, on, xo));
        if (p.b2) o -= bq;
        if (own) row_of(p.out_last, blk, g * RB) = o;
        if (p.partials) wide_partials<R, VS>(p, tile, blk, own, g, ckpt, o, (double *)(wide_mem + 2 * half));
        if constexpr (MORE) {
            put(blk + 1, oth);  // that half was read before the barrier above
            const uint32_t t = cur;
            cur = oth;
            oth = t;
        }
    };
    load(blk0);
    put(blk0, lds0);
    int blk = blk0;
    for (; blk + 1 < blk1; ++blk) step(blk, std::integral_constant<bool, true>{});
    step(blk, std::integral_constant<bool, false>{});
}

template <typename R, int VS>
hipError_t launch_wide_t(int width, dim3 grid, dim3 block, size_t lds, const ChainParams &p, hipStream_t st) {
    switch (width) {
        case 6: hipLaunchKernelGGL((k_pass_wide<R, 6, VS>), grid, block, lds, st, p); break;
        case 8: hipLaunchKernelGGL((k_pass_wide<R, 8, VS>), grid, block, lds, st, p); break;
        case 10: hipLaunchKernelGGL((k_pass_wide<R, 10, VS>), grid, block, lds, st, p); break;
        case 12: hipLaunchKernelGGL((k_pass_wide<R, 12, VS>), grid, block, lds, st, p); break;
        case 14: hipLaunchKernelGGL((k_pass_wide<R, 14, VS>), grid, block, lds, st, p); break;
        case 16: hipLaunchKernelGGL((k_pass_wide<R, 16, VS>), grid, block, lds, st, p); break;
        case 18: hipLaunchKernelGGL((k_pass_wide<R, 18, VS>), grid, block, lds, st, p); break;
        case 20: hipLaunchKernelGGL((k_pass_wide<R, 20, VS>), grid, block, lds, st, p); break;
        case 22: hipLaunchKernelGGL((k_pass_wide<R, 22, VS>), grid, block, lds, st, p); break;
        case 24: hipLaunchKernelGGL((k_pass_wide<R, 24, VS>), grid, block, lds, st, p); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_pass_wide(bool fp32, int width, int vs, int max_own, const ChainParams &p, hipStream_t st) {
    if (p.n_tiles <= 0) return hipSuccess;
    if (max_own < 1 || max_own > kWideThreads || p.lds_rows < max_own || p.lds_rows > kWideStage || p.n_blk < 1 ||
        p.n_grp < 1 || p.grp_blk < 1 || p.table_depth != 1 || !p.v)
        return hipErrorInvalidValue;
    const unsigned nt = (unsigned)(max_own + 63) / 64 * 64;
    const size_t lds = 2 * (size_t)p.lds_rows * (fp32 ? 8 : 16) * vs + sizeof(double) * 3 * vs * (nt / 64);
    const dim3 grid(p.n_grp > 1 ? (unsigned)(((p.n_tiles + 7) / 8) * 8 * p.n_grp) : (unsigned)p.n_tiles), block(nt);
    if (fp32 && vs == 2) return launch_wide_t<float, 2>(width, grid, block, lds, p, st);
    if (!fp32 && vs == 1) return launch_wide_t<double, 1>(width, grid, block, lds, p, st);
    return hipErrorInvalidValue;
}

}  // namespace tbpm
