// Optical conductivity by propagation (paper, Sec. "Optical conductivity"):
// kernels around the Clenshaw passes.
//
//  * k_gather_values: the current operator J (values on H's CSR pattern) in
//    the sliced-ELL layout of H, through the slot -> CSR-position map.
//  * k_join: J psi0 and psi0 (internal row order, [rows][S padded]) side by
//    side in one block [rows][2S padded], so that one Chebyshev series of the
//    Fermi-Dirac operator serves both: f(H) [J psi0 | psi0].
//  * k_pack: from that block B and F = f(H) B, psi1 = (1 - f(H)) J psi0 =
//    B - F in columns 0..S-1 and psi2 = f(H) psi0 in S..2S-1 of one block
//    [n][2S] in the caller's row order, so that one propagation carries both.
//  * k_jcorr: per step, <psi2_s| J |psi1_s> for s < S from the propagated
//    block: J applied to the psi1 columns of each row (gathered over the
//    row's stored elements) and contracted with the row's psi2 columns; FP64
//    per-tile partials in the layout of the correlation, for k_reduce.
//  * k_ac_cond: the windowed sine transform of the Kubo formula, Eq. (AC).
//  * k_ac_kk: the imaginary part from the real part by the Kramers-Kronig
//    relation (the principal-value integral of the piecewise-linear,
//    even extension of Re sigma, as closed-form weights per grid point).
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "tbpm_internal.h"

namespace tbpm {
namespace {

__global__ __launch_bounds__(kWG) void k_gather_values(const int64_t *__restrict__ ell_csr, int64_t ell_size,
                                                       const d2 *__restrict__ csr_val, d2 *__restrict__ ell_val) {
    const int64_t stride = (int64_t)gridDim.x * kWG;
    for (int64_t q = (int64_t)blockIdx.x * kWG + threadIdx.x; q < ell_size; q += stride) {
        const int64_t pos = ell_csr[q];
        d2 v;
        v.x = 0.0;
        v.y = 0.0;
        if (pos >= 0) v = csr_val[pos];
        ell_val[q] = v;
    }
}

__global__ __launch_bounds__(kWG) void k_join(const d2 *__restrict__ jpsi, const d2 *__restrict__ psi,
                                              int64_t n_rows, int log2s, int log2s2, int log2sb, int S,
                                              d2 *__restrict__ out) {
    const int64_t total = n_rows << log2s2;
    const int64_t stride = (int64_t)gridDim.x * kWG;
    const int m2 = (1 << log2s2) - 1;
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < total; i += stride) {
        const int64_t r = i >> log2s2;
        const int c = (int)(i & m2);
        d2 v;
        v.x = 0.0;
        v.y = 0.0;
        if (c < S)
            v = jpsi[(r << log2s) + c];
        else if (c < 2 * S)
            v = psi[(r << log2s) + c - S];
        out[state_index(r, c, log2sb, n_rows)] = v;
    }
}

__global__ __launch_bounds__(kWG) void k_pack(const d2 *__restrict__ blk, const d2 *__restrict__ fblk,
                                              int64_t n_rows, int log2sb, int S, const int32_t *__restrict__ perm,
                                              d2 *__restrict__ out) {
    const int64_t total = n_rows * 2 * S;
    const int64_t stride = (int64_t)gridDim.x * kWG;
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < total; i += stride) {
        const int64_t r = i / (2 * S);
        const int c = (int)(i % (2 * S));
        const int64_t ro = perm ? (int64_t)perm[r] : r;
        const int64_t src = state_index(r, c, log2sb, n_rows);
        d2 v = fblk[src];
        if (c < S) {
            const d2 b = blk[src];
            v.x = b.x - v.x;
            v.y = b.y - v.y;
        }
        out[ro * 2 * S + c] = v;
    }
}

// state: the propagated block at precision R, states in blocks of 2^log2sb;
// thread t handles state t & (SP-1) of its rows (SP = 2^log2sp >= S); grid.y:
// the states of several time steps, state_stride elements apart (eight steps of
// graphene 256^2, whose 256 tiles alone leave three quarters of the chip idle:
// 13.6 us, one step 8.1)
template <typename R>
__global__ __launch_bounds__(kWG) void k_jcorr(const TileDesc *__restrict__ tiles, int n_tiles, int log2sp, int S,
                                               int log2sb, int64_t n_rows, const void *__restrict__ state,
                                               const uint32_t *__restrict__ soff, const int32_t *__restrict__ col,
                                               const d2 *__restrict__ jval, double *__restrict__ partials,
                                               int64_t state_stride, int64_t part_stride) {
    using C = typename CxT<R>::T;
    const C *psi = (const C *)state + blockIdx.y * state_stride;
    partials += blockIdx.y * part_stride;
    const TileDesc td = tiles[blockIdx.x];
    const uint32_t spm = (1u << log2sp) - 1u;
    const int64_t n_u = (int64_t)td.rows << log2sp;
    double dre = 0.0, dim = 0.0;
    for (int64_t u = threadIdx.x; u < n_u; u += kWG) {
        const int s = (int)(u & spm);
        if (s >= S) continue;
        const int64_t r = td.row0 + (u >> log2sp);
        const int64_t sl = r / kSliceRows;
        const uint32_t off = soff[sl];
        const int w = (int)((soff[sl + 1] - off) / kSliceRows);
        const int64_t base = off + r % kSliceRows;
        double ar = 0.0, ai = 0.0;
        for (int k = 0; k < w; ++k) {
            const int64_t slot = base + (int64_t)k * kSliceRows;
            const d2 j = jval[slot];
            const C x = psi[state_index(col[slot], s, log2sb, n_rows)];
            const double xr = (double)x.x, xi = (double)x.y;
            ar = fma(j.x, xr, fma(-j.y, xi, ar));
            ai = fma(j.x, xi, fma(j.y, xr, ai));
        }
        const C y = psi[state_index(r, S + s, log2sb, n_rows)];
        const double yr = (double)y.x, yi = (double)y.y;
        dre = fma(yr, ar, fma(yi, ai, dre));  // conj(y) * (ar + i ai)
        dim = fma(yr, ai, fma(-yi, ar, dim));
    }
    block_state_partials(dre, dim, 0.0, log2sp, partials, blockIdx.x, n_tiles);
}

// sigma(w_j) = (e^{-beta w_j} - 1) / (w_j A) dt sum_k w_k sin(w_j t_k) 2 Im Cbar_k,
// w_j = j pi / (N_t dt), sigma(0) = 0; the phase w_j t_k = pi (j k mod 2N)/N
// is reduced exactly in integers, the sum is compensated.
__global__ __launch_bounds__(kWG) void k_ac_cond(const d2 *__restrict__ corr, int n_steps, int n_states, double dt,
                                                 double beta, double area, int window, int log2l,
                                                 double *__restrict__ omegas, double *__restrict__ sigma) {
    __shared__ double c[kWG];
    const int lane = (int)threadIdx.x & ((1 << log2l) - 1);
    const int64_t j = ((int64_t)blockIdx.x * kWG + threadIdx.x) >> log2l;
    const int64_t two_n = 2 * (int64_t)n_steps;
    // m = j k mod 2N of the lane's terms k = 1 + lane, 1 + lane + L, ...
    int64_t m = (j * (1 + lane)) % two_n;
    const int64_t dm = (j << log2l) % two_n;
    double sum = 0.0, comp = 0.0;
    for (int k0 = 1; k0 < n_steps; k0 += kWG) {
        const int k = k0 + (int)threadIdx.x;
        double im = 0.0;
        if (k < n_steps) {
            for (int s = 0; s < n_states; ++s) im += corr[(int64_t)k * n_states + s].y;
            im /= n_states;
            im *= 2.0 * (window == TBPM_WIN_HANN ? 0.5 * (1.0 + cospi((double)k / n_steps)) : 1.0);
        }
        c[threadIdx.x] = im;
        __syncthreads();
        const int kn = min(kWG, n_steps - k0);
        if (j < n_steps) {
            for (int kk = lane; kk < kn; kk += 1 << log2l) {
                kadd(sum, comp, c[kk] * sinpi((double)m / n_steps));
                m += dm;
                if (m >= two_n) m -= two_n;
            }
        }
        __syncthreads();
    }
    sum = kadd_lanes(sum, comp, log2l);
    if (j >= n_steps || lane != 0) return;
    const double w_j = M_PI * j / (n_steps * dt);
    omegas[j] = w_j;
    sigma[j] = j == 0 ? 0.0 : (exp(-beta * w_j) - 1.0) / (w_j * area) * sum * dt;
}

// P int phi(u) / (u - m) du for the unit hat phi(u) = max(0, 1 - |u|):
//   g(m) = (1 - m) ln|1 - m| - (1 + m) ln|1 + m| + 2 m ln|m|   (0 ln 0 = 0),
// odd in m; for |m| >= 2 in the form -|m| log1p(-1/m^2) - log1p(2/(|m| - 1)),
// which has no cancellation between terms of size |m| ln|m|.
__device__ __forceinline__ double kk_hat(int64_t m) {
    const double a = (double)(m < 0 ? -m : m);
    double g;
    if (a < 2.0) {
        const double t1 = a == 1.0 ? 0.0 : (1.0 - a) * log(fabs(1.0 - a));
        const double t3 = a == 0.0 ? 0.0 : 2.0 * a * log(a);
        g = t1 - (1.0 + a) * log(1.0 + a) + t3;
    } else {
        g = -a * log1p(-1.0 / (a * a)) - log1p(2.0 / (a - 1.0));
    }
    return m < 0 ? -g : g;
}

// Im sigma_k = -(1/pi) P int Re sigma(|w|)/(w - w_k) dw on the grid w_j = j dw
// with Re sigma = sum_j y_j phi(w/dw - j) (linear between grid points, zero
// one spacing past the last) and its mirror image for w < 0: node 0 gives
// y_0 g(k), node j >= 1 gives y_j (g(k - j) + g(k + j)).  2^log2l
// lanes per k; the sum over j is compensated (Neumaier) and runs in a fixed order.
__global__ __launch_bounds__(kWG) void k_ac_kk(const double *__restrict__ re, int n, int log2l,
                                               double *__restrict__ im) {
    const int lane = (int)threadIdx.x & ((1 << log2l) - 1);
    const int64_t k = ((int64_t)blockIdx.x * kWG + threadIdx.x) >> log2l;
    double sum = 0.0, comp = 0.0;
    if (k < n)
        for (int j = lane; j < n; j += 1 << log2l)
            kadd(sum, comp, j == 0 ? re[0] * kk_hat(k) : re[j] * (kk_hat(k - j) + kk_hat(k + j)));
    sum = kadd_lanes(sum, comp, log2l);
    if (k < n && lane == 0) im[k] = -sum / M_PI;
}

int64_t grid_for_n(int64_t n) {
    int64_t b = (n + kWG - 1) / kWG;
    if (b > 65536) b = 65536;
    return b < 1 ? 1 : b;
}

// Chebyshev coefficients of the Fermi function from n samples g_q at cos(2 pi q/n)
// (n a power of two; g_{n-q} = g_q, so q <= n/2 suffices):
//     a_k = (4/n) [ (g_0 + (-1)^k g_{n/2})/2 + sum_{0<q<n/2} g_q cos(2 pi q k/n) ],
// half of it for k = 0.  2^log2l lanes per coefficient; the phase q k mod n is
// exact.  last: the largest k with |a_k| >= tol.
__global__ __launch_bounds__(kWG) void k_fermi_samples(double beta, double mu, double rescale, int n,
                                                       double *__restrict__ g) {
    const int q = blockIdx.x * kWG + threadIdx.x;
    if (q > n / 2) return;
    const double x = rescale * cospi(2.0 * (double)q / (double)n);
    const double v = 0.5 * (1.0 - tanh(0.5 * beta * (x - mu)));
    g[q] = q == 0 || q == n / 2 ? 0.5 * v : v;
}

__global__ __launch_bounds__(kWG) void k_fermi_cheb(const double *__restrict__ g, int n, int log2l, double tol,
                                                    double *__restrict__ a, int *__restrict__ last) {
    const int lane = (int)threadIdx.x & ((1 << log2l) - 1);
    const uint32_t k = (uint32_t)(((int64_t)blockIdx.x * kWG + threadIdx.x) >> log2l), mask = (uint32_t)n - 1u;
    const double step = 2.0 / (double)n;
    double sum = 0.0, comp = 0.0;
    if ((int)k < n / 2) {
        uint32_t m = ((uint32_t)lane * k) & mask;
        const uint32_t dm = (k << log2l) & mask;
        for (int q = lane; q <= n / 2; q += 1 << log2l) {
            kadd(sum, comp, g[q] * cospi((double)m * step));
            m = (m + dm) & mask;
        }
    }
    sum = kadd_lanes(sum, comp, log2l);
    if ((int)k >= n / 2 || lane != 0) return;
    const double v = (k == 0 ? 2.0 : 4.0) / (double)n * sum;
    a[k] = v;
    if (fabs(v) >= tol) atomicMax(last, (int)k);
}

__global__ void k_fermi_clear(int *last) { *last = 0; }

}  // namespace

hipError_t launch_fermi_cheb(double beta, double mu, double rescale, int32_t n, double tol, double *g, double *a,
                             int32_t *last, hipStream_t st) {
    if (n < 4 || (n & (n - 1)) || n > kFermiMaxSamples) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_fermi_clear, dim3(1), dim3(1), 0, st, last);
    hipLaunchKernelGGL(k_fermi_samples, dim3((unsigned)(n / 2 + kWG) / kWG), dim3(kWG), 0, st, beta, mu, rescale, n, g);
    const int l = transform_log2_lanes(n / 2);
    hipLaunchKernelGGL(k_fermi_cheb, dim3((unsigned)((((int64_t)n / 2) << l) + kWG - 1) / kWG), dim3(kWG), 0, st, g, n, l,
                       tol, a, last);
    return hipGetLastError();
}

hipError_t launch_gather_values(const int64_t *ell_csr, int64_t ell_size, const double *csr_val, double *ell_val,
                                hipStream_t st) {
    hipLaunchKernelGGL(k_gather_values, dim3((unsigned)grid_for_n(ell_size)), dim3(kWG), 0, st, ell_csr, ell_size,
                       (const d2 *)csr_val, (d2 *)ell_val);
    return hipGetLastError();
}

hipError_t launch_join(const double *jpsi, const double *psi, int64_t n_rows, int32_t log2s, int32_t log2s2,
                       int32_t log2sb, int32_t S, double *out, hipStream_t st) {
    hipLaunchKernelGGL(k_join, dim3((unsigned)grid_for_n(n_rows << log2s2)), dim3(kWG), 0, st, (const d2 *)jpsi,
                       (const d2 *)psi, n_rows, log2s, log2s2, log2sb, S, (d2 *)out);
    return hipGetLastError();
}

hipError_t launch_pack(const double *blk, const double *fblk, int64_t n_rows, int32_t log2sb, int32_t S,
                       const int32_t *perm, double *out, hipStream_t st) {
    hipLaunchKernelGGL(k_pack, dim3((unsigned)grid_for_n(n_rows * 2 * S)), dim3(kWG), 0, st, (const d2 *)blk,
                       (const d2 *)fblk, n_rows, log2sb, S, perm, (d2 *)out);
    return hipGetLastError();
}

hipError_t launch_jcorr(bool fp32, const TileDesc *tiles, int32_t n_tiles, int32_t log2sp, int32_t S, int32_t log2sb,
                        int64_t n_rows, const void *state, const uint32_t *slice_off, const int32_t *col, const double *jval,
                        double *partials, int32_t n_states, int64_t state_stride, int64_t part_stride, hipStream_t st) {
    const dim3 grid((unsigned)n_tiles, (unsigned)n_states);
    if (fp32)
        hipLaunchKernelGGL(k_jcorr<float>, grid, dim3(kWG), 0, st, tiles, n_tiles, log2sp, S, log2sb, n_rows, state,
                           slice_off, col, (const d2 *)jval, partials, state_stride, part_stride);
    else
        hipLaunchKernelGGL(k_jcorr<double>, grid, dim3(kWG), 0, st, tiles, n_tiles, log2sp, S, log2sb, n_rows, state,
                           slice_off, col, (const d2 *)jval, partials, state_stride, part_stride);
    return hipGetLastError();
}

hipError_t launch_ac_kk(const double *re, int32_t n, double *im, hipStream_t st) {
    const int l = transform_log2_lanes(n);
    hipLaunchKernelGGL(k_ac_kk, dim3((unsigned)((((int64_t)n << l) + kWG - 1) / kWG)), dim3(kWG), 0, st, re, n, l, im);
    return hipGetLastError();
}

hipError_t launch_ac_cond(const double *corr, int32_t n_steps, int32_t n_states, double dt, double beta, double area,
                          int window, double *omegas, double *sigma, hipStream_t st) {
    const int l = transform_log2_lanes(n_steps);
    hipLaunchKernelGGL(k_ac_cond, dim3((unsigned)((((int64_t)n_steps << l) + kWG - 1) / kWG)), dim3(kWG), 0, st,
                       (const d2 *)corr, n_steps, n_states, dt, beta, area, window, l, omegas, sigma);
    return hipGetLastError();
}

}  // namespace tbpm
