// Launch parameters and layout constants of the propagation kernels (the
// Clenshaw passes, the fused two-order pass, initialisation and the
// correlation reduction): everything these kernels see besides their own
// source and device_util.h.
#pragma once

#include <cstdint>

namespace tbpm {

// ---------------------------------------------------------------------------
// Device layout
// ---------------------------------------------------------------------------
// Off-diagonal part of H in sliced ELL: slices of kSliceRows consecutive
// rows; slice q holds width_q = (slice_off[q+1]-slice_off[q])/kSliceRows
// entries per row, stored column-major inside the slice, i.e. entry k of
// row r lives at slice_off[q] + k*kSliceRows + (r % kSliceRows).  Rows
// shorter than width_q are padded with (col = row, value = 0).
constexpr int kSliceRows = 32;
// Threads per workgroup of every streaming kernel (4 wave64s).
constexpr int kWG = 256;

// One workgroup's share of a Chebyshev pass: 'rows' consecutive rows of a
// single batch member 'inst', starting at global row 'row0'.
struct TileDesc {
    int64_t row0;
    int32_t rows;
    int32_t inst;
};

// Per-member coefficients of one pass: out = alpha*v + beta*(H x) - b2.
struct PassCoef {
    double ar, ai, br, bi;
};

// ---------------------------------------------------------------------------
// Kernel launch parameters
// ---------------------------------------------------------------------------
enum PassKind : int {
    kPassFirst = 0,   // x = v, no b2 buffer
    kPassNoB2 = 1,    // no b2 buffer
    kPassMid = 2,     // b2 buffer
    kPassLast = 3,    // b2 buffer, fused correlation
    kPassLastNoB2 = 4 // no b2 buffer, fused correlation
};

struct PassParams {
    const TileDesc *tiles;
    int32_t n_tiles;
    int32_t xcd_remap;
    int32_t log2s;  // log2 of the (padded) number of states
    int32_t bump_counter;
    const int32_t *col;
    const void *val;
    const uint32_t *slice_off;
    const void *onsite;
    const void *x;   // gathered vector (b_{j+1}, or v for the first pass)
    const void *v;   // psi_k
    const void *b2;  // b_{j+2}
    void *out;       // b_j or psi_{k+1}; may alias b2 or v element-wise
    const PassCoef *coef;  // [n_inst] of this pass
    int32_t *counter;      // device step counter
    // fused correlation (last pass)
    const double *phi0;    // complex128 [rows][S]
    int64_t phi0_ld;       // states per row of phi0 (>= S padded or the caller's S)
    double *partials;      // [S][3][n_tiles]
    // stored states (last pass): checkpoints or snapshots of psi(k dt)
    double *ckpt;              // complex128 [n_slots][rows][s_user], rows in the caller's order
    const int32_t *ckpt_slot;  // [n_steps]: slot of psi(k dt) in ckpt, or -1; null: none stored
    const int32_t *perm;       // internal row -> caller's row (single member), or null
    int64_t ckpt_stride;       // complex elements per slot (rows * s_user)
    int32_t s_user;
    // LDS staging (staged launch shape): tile t reads its own rows and the
    // external rows ucol[uoff[t] .. uoff[t+1]); lidx[slot] is the local row of
    // each ELL slot in that staged set
    const int32_t *uoff;
    const int32_t *ucol;
    const uint16_t *lidx;
    int32_t stage_units;   // LDS capacity in units (VS states)
    int32_t uniform_w;     // stored elements per row when every slice has that width, else 0
    int32_t reverse;  // walk the tiles last to first (see tile_of_block)
    // staged launch shape: log2 of the units of one state block of a row (at
    // most log2s - log2 VS); with several blocks, one workgroup per (tile,
    // block) stages and evaluates the tile's rows of that block, so the LDS
    // holds rows of one block
    int32_t log2ub;
};

// Two Clenshaw orders per launch (fused.hip).
enum PairKind : int {
    kPairFirst = 0,  // b_{M-2}, b_{M-3} from psi (x = psi, no b_{j+2})
    kPairMid = 1,    // b_j, b_{j-1} from b_{j+1} (x) and b_{j+2}
    kPairLast = 2,   // b_1 (kept in LDS only) and psi_{k+1} from b_2 (x) and b_3,
                     // with the fused correlation of psi_{k+1}
    kPairSecond = 3  // b_{M-3} (b_{M-1} folded into alpha1, no b_{j+2}) and
                     // b_{M-4} from b_{M-2} (x), after the first order ran alone
};

struct FusedParams {
    const TileDesc *tiles;
    int32_t n_tiles;
    int32_t xcd_remap;
    int32_t log2s;
    int32_t bump_counter;
    const int32_t *col;
    const void *val;
    const uint32_t *slice_off;
    const void *onsite;
    const void *x;     // b_{j+1} (or psi for kPairFirst), staged
    const void *v;     // psi
    const void *b2;    // b_{j+2} (kPairMid)
    void *out1;        // b_j on own rows (not written by kPairLast)
    void *out2;        // b_{j-1} on own rows; never a buffer the launch reads
    const PassCoef *coef1, *coef2;  // [n_inst] for orders j and j-1
    int32_t *counter;
    // 2-hop tiles: staged rows are own, then 1-hop (n1 of them), then 2-hop
    const int32_t *uoff;   // [n_tiles + 1] offsets into ucol
    const int32_t *n1;     // [n_tiles]
    const int32_t *ucol;   // 1-hop then 2-hop global rows of every tile
    const uint16_t *lidx;  // per ELL slot of an own row: local index (own or 1-hop)
    const int32_t *hoff;   // [n_tiles] offset of the tile's 1-hop index block in hidx
    const int32_t *hw;     // [n_tiles] entries per 1-hop row in that block
    const uint16_t *hidx;  // local indices of the stored elements of the 1-hop rows
    int32_t lds_units;     // LDS capacity in units: max over tiles of n_x + n_y
    int32_t uniform_w;     // stored elements per row when every slice has that width, else 0
    int32_t reverse;       // walk the tiles last to first (see tile_of_block)
    // fused correlation (kPairLast): as in PassParams
    const double *phi0;
    int64_t phi0_ld;
    double *partials;
};

// Time steps whose states one accumulation launch takes (k_qe_accum, k_jcorr).
constexpr int kHistSteps = 8;

// Several Clenshaw orders per launch (chain.hip).
constexpr int kChainMaxDepth = 24;  // orders per launch
constexpr int kChainWidth = 4;      // most stored elements per row
// Threads of a workgroup and local rows a thread evaluates: a tile's rows up to
// depth - 1 hops away are at most chain_rows.
constexpr int kChainRowsPerThread = 2;
constexpr int chain_threads(bool cplx) { return cplx ? 256 : 512; }
constexpr int chain_rows(bool cplx) { return chain_threads(cplx) * kChainRowsPerThread; }

// The wide pass (wide.hip): most stored elements per row, threads of a workgroup
// (one row each), and rows of a tile with those one hop away.
constexpr int kWideWidth = 24;
constexpr int kWideThreads = 256;
constexpr int kWideStage = 1280;

// Elements per row that the tile tables hold: up to 3, 4, or an even number (the wide
// pass keeps the places of two elements in a register).  Elements that are not there
// cost LDS reads and registers: bilayer 192^2, 21 elements, 16 FP32 states, 70 samples
// take 22.1 ms with 22 and 22.6 with 24, 16 FP64 states 36.4 and 37.3.
constexpr int chain_table_width(int max_width) {
    return max_width <= 3 ? 3 : (max_width + 1) / 2 * 2;
}

// The Haydock step's second product runs on whole waves, but the LDS it reads holds
// u_{i+1} of the evaluated rows only (one per thread), and the neighbours of a row
// that is not the tile's own may lie beyond them: such a lane reads its own place.
constexpr uint32_t hay_place(bool own, uint32_t neighbour, uint32_t tid) { return own ? neighbour : tid; }

struct ChainParams {
    const TileDesc *tiles;
    int32_t n_tiles;
    int32_t n_blk;         // state blocks of VS states
    int32_t n_grp, grp_blk;  // workgroups per tile and the state blocks each takes in turn
    int32_t xcd_remap;
    int32_t reverse;       // walk the tiles last to first (see tile_of_block)
    int32_t depth;         // orders of this launch
    int32_t table_depth;   // orders the tile tables serve
    int32_t contiguous;    // own rows are row0 .. row0 + rows - 1 (else through rowmap)
    int32_t n_inst;
    uint32_t n_rows;
    const int32_t *cnt;    // [n_tiles][table_depth + 1]: local rows up to h hops away
    const int32_t *toff;   // [n_tiles] offset of the tile's local rows in rowmap
    const int32_t *loff;   // [n_tiles] offset of the tile's rows in lidx, tval and tons
    const uint32_t *rowmap;
    const uint16_t *lidx;  // [row][4] local indices of the stored elements
    const void *tval;      // per tile [width][rows]
    const void *tons;
    const void *x;         // b_{j+1} (or psi), state blocks [n_blk][n_rows][VS]
    const void *v;         // psi; null: the alpha terms are absent
    const void *b2;        // b_{j+2}, or null
    void *out_last, *out_prev;  // the last order's and the last but one's outputs on own rows, or null
    void *out_all;         // or: every order but the last at out_all + k out_stride bytes
    int64_t out_stride;
    // alpha of the orders: with alt, real and imaginary in turn (real first, or
    // imaginary first with turned); without, all real.  beta is real except in
    // the first order of a time step (first), which may have any alpha and beta.
    int32_t alt, turned, first;
    const PassCoef *coef;  // [depth][n_inst]
    // fused correlation of the last order, or null
    const double *phi0;    // complex128, in state blocks
    double *partials;      // [S][3][n_tiles]
    // stored states of the fused correlation's launch, as in PassParams
    double *ckpt;
    const int32_t *ckpt_slot;
    int32_t local;  // steps since the counter was advanced
    int32_t *counter;
    const int32_t *perm;
    int64_t ckpt_stride;
    int32_t s_user;
    // the wide pass: rows of a half of the LDS; advance the step counter
    int32_t lds_rows, bump;
};

// Several orders of the Chebyshev recursion T_{j+1} = 2 H~ T_j - T_{j-1} per
// launch: x = T_j, b2 = T_{j-1} (null for j = 0), no v.
struct ChainCheb {
    double inv_f;
    const uint32_t *slice_off;
    int32_t first, final_;  // the launch holds j = 0 / the last order of a time step
    // kChainCurrent: jout + k jout_stride = J T_{j+k}, J without on-site entries
    // (complex, in the order of the sliced ELL's slots)
    const void *jval;
    void *jout;
    int64_t jout_stride;  // bytes
    // kChainAdjoint: T_j = alpha_j; per order the gradient of every stored element
    // and on-site energy from alpha_j at the neighbours and b_{j+1} at the own
    // row, and lambda
    const void *bq;        // b_{j+1} of the first order; the next orders' bq_stride bytes on
    int64_t bq_stride;
    const void *psi;       // last order of a time step (final): b_{M-1} = bs psi in bq's place
    double bs_re, bs_im;
    const double *cc;      // conj(c_j) from the first order's j on, complex
    const double *gcorr_l; // final: complex [s_user], lambda += gcorr_l phi0
    void *lam;             // lambda accumulator, state blocks
    void *gacc;            // [n_grp][ell_size] double (real H) or double2: own slot of (q, p), gradient of (p, q)
    double *gdiag;         // [n_grp][n_rows]
    int64_t ell_size;
};
enum { kChainClenshaw = 0, kChainAdjoint = 1, kChainCheb = 2, kChainCurrent = 3 };

struct ChainTileTab {
    const int32_t *cnt, *toff, *loff;
    const uint32_t *rowmap;
    int32_t table_depth, width;
};

struct InitParams {
    const TileDesc *tiles;
    int32_t n_tiles;
    int32_t log2s;
    int32_t s_user;
    const double *const *psi0;   // per member, [N_i][s_user] complex128
    const int64_t *inst_row0;    // per member, first global row
    void *v;                     // state buffer [rows][S] (R precision)
    double *phi0;                // padded FP64 copy [rows][S], or null
    double *partials;            // [S][3][n_tiles]
    int32_t *counter;
    const int32_t *perm;         // internal row -> caller's row in its member, or null
    // states in blocks of 2^log2sb, [block][n_rows][2^log2sb] (log2sb = log2s: one block)
    int32_t log2sb;
    int64_t n_rows;
};

struct ReduceParams {
    const double *partials;      // [S][3][n_tiles]
    int32_t n_tiles;
    const int32_t *inst_tile0;   // [n_inst + 1]
    int32_t log2s;
    int32_t s_user;
    int32_t n_steps;
    const int32_t *counter;
    double *const *corr;          // per member [n_steps][s_user] complex128
    double *const *norm2;         // per member, entries may be null
    double *norm2_all;            // [n_inst][n_steps][s_user], or null
};

}  // namespace tbpm
