// Device code of the small (w x w) factorisation behind the orthonormaliser, shared by the kernels
// that can run it: the stand-alone chol kernel and, as the last workgroup to arrive, the kernel that
// wrote the partial Gram matrices.
//
// Orthonormalisation (Section 2, "QR decomposition": Q-factor of the economic QR) is CholeskyQR2:
//   G = X^T X (fp64, exact products of the fp32 entries);  G_s = D G D with D = diag(G)^{-1/2};
//   G_s = R_s^T R_s (Cholesky, fp64);  X <- X (D R_s^{-1});  then the same once more on the result.
// The Q-factor it converges to is the one with a positive diagonal of R.  A pivot of the scaled
// Cholesky at step k equals (norm of column k's part orthogonal to the earlier columns / norm of
// column k)^2; if it is <= rank_tol^2 the column is declared dependent and its P~ column is zero.
#pragma once
#include <type_traits>

#include "psgd_dev.h"

namespace psgd {

// The first pass leaves an orthogonality error of about 1e-16/pivot (the smallest pivot of the scaled
// factorisation is about 1/cond^2 of the column-scaled matrix); below kSecondPassPivot the flag
// status[1] is set and the pass-2 code (which exits at once otherwise) does its work.
constexpr double kSecondPassPivot = 1e-6;
constexpr int kCholMaxGroups = 8;

// slot groups that sum the partial Gram matrices side by side (all kThreads threads busy for small w)
__host__ __device__ inline int chol_groups(int w) {
    const int ntri = (w * (w + 1)) / 2;
    int g = kThreads / ntri;
    return g < 1 ? 1 : (g > kCholMaxGroups ? kCholMaxGroups : g);
}
// Widths above the register path: 16 x 16 blocks of the upper triangle in LDS (chol_blocked) as long as these, one block row
// beside them and the vectors fit a workgroup's 160 KB, i.e. up to 11 blocks = 176; beyond that a packed triangle without
// blocking.
constexpr int kCholMaxBlocks = 11;
constexpr int kMaxWaveColumns = 3;     // columns of the widest block per lane of one wave
constexpr int kTjjStride = 17;         // row stride of the diagonal block's inverse (doubles)
__host__ __device__ inline bool chol_is_blocked(int w) { return w > kCholRegWidth && (w + 15) / 16 <= kCholMaxBlocks; }
// LDS bytes chol_body needs
__host__ __device__ inline size_t chol_lds_bytes(int w) {
    const int nbk = (w + 15) / 16;
    if (chol_is_blocked(w))
        return ((size_t)(nbk * (nbk + 1) / 2 + nbk) * 256 + 16 * kTjjStride + 16 * nbk) * sizeof(double) + (size_t)16 * nbk * sizeof(int);
    const int ntri = (w * (w + 1)) / 2;
    const int g = chol_groups(w);
    return ((size_t)(g > 1 ? g + 1 : 1) * ntri + 2 * w + 16 * nbk) * sizeof(double) + (size_t)(w + 2) * sizeof(int);
}
// the same for a launch that serves layers of any width up to w (the need is not monotone in w)
inline size_t chol_lds_bytes_upto(int w) {
    size_t b = 0;
    for (int v = 1; v <= w; ++v) b = chol_lds_bytes(v) > b ? chol_lds_bytes(v) : b;
    return b;
}

// squared column norms at or below this count as zero (far below anything fp32 data can produce, and
// keeps the reciprocal square root away from subnormal arguments)
constexpr double kTinyNorm2 = 1e-280;

// 1 / sqrt(x) for finite normal x > 0: hardware estimate refined by two Newton steps (full fp64 accuracy)
__device__ inline double rsqrt_nr(double x) {
    double y = __builtin_amdgcn_rsq(x);
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const double e = __builtin_fma(-(x * y), y, 1.0);
        y = __builtin_fma(0.5 * y, e, y);
    }
    return y;
}

// Power of two next to a column's scaling 1 / ||x||, kept within what fp32 can hold.  Z = X T columns multiplied by it
// give Y = M^T Z columns of norm about 1 where X = M Y' did with a Y' of such columns, so that a Y that is not
// orthonormalised (see Spread) does not drift out of range however small the gradients are.
__device__ inline double next_scale(double dsc) {
    if (!(dsc > 0.0)) return 1.0;
    const int e = __builtin_amdgcn_frexp_exp(dsc);
    return __builtin_ldexp(1.0, e > 110 ? 110 : (e < -110 ? -110 : e));
}

// Ordering point for LDS traffic inside one wavefront (its LDS accesses execute in program order; this
// keeps the compiler from moving them across).
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Value of v on lane I of each row of 16 lanes (a row broadcast on the data path: two moves, no scalar register in between.
// Lane reads into scalar registers cost these factorisations 30 to 60 cycles per updated row, most of their time).
template <int I> __device__ __forceinline__ double bcast_row(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x150 + I, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x150 + I, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
template <int I, int N, class F> __device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(static_cast<F&&>(f));
    }
}

template <int CTRL> __device__ __forceinline__ int dpp_or(int other, int v) {
    return __builtin_amdgcn_update_dpp(other, v, CTRL, 0xf, 0xf, false);
}

// What the factor R of X = Z R says about the Y = M^T Z that follows.  Left as it is, Y hands M M^T Z to the next
// factorisation in place of M (orthonormal Y), and every ratio of singular values that Z mixes counts twice:
//   - Columns out of order.  While a column of Z turns from a weak direction to one s times as strong, the pivot of the
//     weak one is s^-4 in place of s^-2.  From s = 300 on that is below rank_tol^2 = 1e-10, and the column counts as
//     dependent and is lost for the rest of the refresh.  A start block whose columns are sorted, or random, passes no
//     such point; one with the strong directions last does.
//   - Rounding along the leading vectors, 2^-17 or 2^-24 of sigma_1 (two or three operand planes), becomes
//     (sigma_1 / sigma_j)^2 of that in X's column j: above its own norm where sigma_j / sigma_1 < 2^-8 or 2^-12.
// So Y is orthonormalised in an iteration whose Z came with a column norm ||x_j|| more than 16 times an earlier R_ii (or
// nearly: powers of two), a pivot below 1e-2, or a smallest R_jj below 2^-11 (two planes 2^-7.5) of the largest column norm.
// Model on 400 x 300 matrices, blocks of 16 and 40, 3 to 16 iterations, geometric spectra and outliers over a flat rest
// with ratios of 1e2 to 3e4 in the block, sorted, random, permuted and ascending starts, against Y always orthonormal: no more
// columns lost, sin(theta) within 7 times (at 3e-7; two planes 1.1 times).  Never orthonormal: up to 4 columns with
// sin(theta) = 1 from a ratio of 5000 on; no limit on the pivots: 1e-4 in place of 4e-7.  R_jj in place of ||x_j|| misses
// columns that have just been passed on to an earlier one (5e-5 in place of 6e-7) unless the limit is 4, and then refreshes of
// an error-feedback run ask once each on average, where now one in eight does.
// In powers of two of squared norms; dependent columns do not count.
struct Spread {
    static constexpr int kNone = 1 << 20, kDisorder = 8;
    static constexpr double kPivot = 1e-2;
    int top = -kNone, low = kNone;      // largest column norm, smallest R_jj so far
    int disorder = 0;
    __device__ bool asks(int planes, double min_piv) const {
        return low < kNone && (disorder || min_piv < kPivot || top - low > (planes == 3 ? 22 : 15));
    }
    // one column (norm: ||x_j||^2, rjj: R_jj^2)
    __device__ void add(int norm, int rjj) {
        disorder |= norm - low > kDisorder;
        low = min(low, rjj);
        top = max(top, norm);
    }
    // the 16 columns of a block, one per lane of each row of 16 lanes (every lane of the wavefront ends up with the result)
    __device__ __forceinline__ void add_block(int norm, int rjj, bool counts) {
        const int e = counts ? rjj : kNone;
        int n = counts ? norm : -kNone;
        int before = dpp_or<0x111>(kNone, e);                                     // smallest of the lanes before
        before = min(before, dpp_or<0x111>(kNone, before));
        before = min(before, dpp_or<0x112>(kNone, before));
        before = min(before, dpp_or<0x114>(kNone, before));
        before = min(before, dpp_or<0x118>(kNone, before));
        disorder |= __ballot(n - min(before, low) > kDisorder) != 0;
        n = max(n, dpp_or<0x111>(-kNone, n));
        n = max(n, dpp_or<0x112>(-kNone, n));
        n = max(n, dpp_or<0x114>(-kNone, n));
        n = max(n, dpp_or<0x118>(-kNone, n));
        low = min(low, dpp_or<0x15f>(kNone, min(before, e)));                     // (lane 15 of the row)
        top = max(top, dpp_or<0x15f>(-kNone, n));
    }
};

// value of v on lane (row of lanes, I + row of lanes) of the caller's row of lanes
template <int I> __device__ __forceinline__ double bcast_by_row(double v) {
    int lo = 0, hi = 0;
    static_for<0, 4>([&](auto rc) {
        constexpr int r = decltype(rc)::value;
        lo = __builtin_amdgcn_update_dpp(lo, __double2loint(v), 0x150 + I + r, 1 << r, 0xf, false);
        hi = __builtin_amdgcn_update_dpp(hi, __double2hiint(v), 0x150 + I + r, 1 << r, 0xf, false);
    });
    return __hiloint2double(hi, lo);
}

// Right-looking factorisation A = R^T R of a scaled W x W matrix (W <= 16) by a wavefront in registers, without LDS traffic or
// barriers.  x and y are 16 x 16 matrices in the accumulator layout of v_mfma_f64_16x16x4_f64 (x[v]: row 4 v + (lane >> 4),
// column lane & 15), x the matrix (upper part, finite) and y an identity, which the row operations turn into R^{-T}: y[v] ends up as
// T[column][row], T = R^{-1}, and no separate inversion is needed.  Step k takes the multiples of row k, which one row of lanes
// holds, off the rows below with one MFMA each for x and y, the other rows of lanes supplying zeros.  The rows stay as they are
// (A = L D L^T): a step needs 1 / pivot, and the square roots, of all rows at once, come at the end.  What bounds the chain is that
// reciprocal and one MFMA (76 cycles): about 320 cycles a step (f64 operations wait while
// the other MFMA runs), and 425 with row k scaled by its square root and selected row by row in the step.
// A dependent column (flagged in badmask, or pivot not above tol2) makes row k of R the k-th row of the identity and skips
// the update.  rjj: R_jj of column j = lane & 15 (of the columns that are not dependent).  badmask, min_piv and rjj are the same in all
// rows of lanes.  Selects, not branches: at every merge point the compiler would copy the register array.
template <int W>
__device__ __forceinline__ void factor_in_registers(doublex4& x, doublex4& y, double tol2, int& badmask, double& min_piv, double& rjj) {
    const int j = threadIdx.x & 15, q = (threadIdx.x >> 4) & 3;
    const int bad = __builtin_amdgcn_readfirstlane(badmask);
    // (y's step is issued when the next pivot has been read: between the two MFMAs of a step the wave could issue nothing, and the
    // compiler's wait for x would count from the second)
    double m = 0.0;
    static_for<0, W>([&](auto kc) {
        constexpr int k = decltype(kc)::value, v = k >> 2, r = k & 3;
        double inv = 0.0;
        bool goes = false;
        if constexpr (k + 1 < W) {
            const double piv = bcast_row<k>(x[v]);                                // (means the pivot in row r of lanes only)
            goes = q == r && j > k && !((bad >> k) & 1) && piv > tol2;
            inv = __builtin_amdgcn_rcp(piv);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (k > 0) {
                y = __builtin_amdgcn_mfma_f64_16x16x4f64(m, y[(k - 1) >> 2], y, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int it = 0; it < 2; ++it) inv = __builtin_fma(__builtin_fma(-piv, inv, 1.0), inv, inv);
            m = x[v] * (goes ? -inv : 0.0);
            x = __builtin_amdgcn_mfma_f64_16x16x4f64(m, x[v], x, 0, 0, 0);
        } else if constexpr (k > 0) {
            y = __builtin_amdgcn_mfma_f64_16x16x4f64(m, y[(k - 1) >> 2], y, 0, 0, 0);
        }
    });
    // row k has not changed since step k: the pivots are x's diagonal
    double low = min_piv, diag = 1.0;
    badmask = bad;
    static_for<0, (W + 3) / 4>([&](auto vc) {
        constexpr int v = decltype(vc)::value;
        const double piv = bcast_by_row<4 * v>(x[v]);
        const bool good = piv > tol2 && !((bad >> (4 * v + q)) & 1);
        const double rinv = rsqrt_nr(good ? piv : 1.0);
        y[v] *= rinv;
        low = good && piv < low ? piv : low;
        diag = good && (j >> 2) == v ? piv * rinv : diag;                         // (column j's in row j & 3 of lanes)
        const unsigned long long deps = __ballot(!good);
        static_for<0, 4>([&](auto rc) {
            constexpr int r = decltype(rc)::value;
            badmask |= (int)((deps >> (16 * r)) & 1) << (4 * v + r);
        });
    });
    low = fmin(low, __shfl_xor(low, 16));
    min_piv = fmin(low, __shfl_xor(low, 32));
    rjj = __shfl(diag, 16 * (j & 3) + j);
}

// Adds a factorised block's columns to `spread`: lane j's R_jj is rjj / dsc (dsc = 1 / ||x_j||).
__device__ __forceinline__ void note_block(Spread& spread, double rjj, double dsc, bool counts) {
    const double norm = __builtin_amdgcn_rcp(counts ? dsc : 1.0);
    spread.add_block(__builtin_amdgcn_frexp_exp(norm * norm), __builtin_amdgcn_frexp_exp((rjj * norm) * (rjj * norm)), counts);
}

// What a factorisation inside the iteration notes (see IterationNote), where the wave that factorises keeps it in registers instead of
// the layer's eval and status words (scale: of column lane & 15).
struct IterationState {
    double scale = 1.0, shrunk = 0.0;
    int asks = 0, ends = 0;
};
constexpr double kLargest = 1e300;
// minimum over the 16 lanes of a row of lanes; over the wave
__device__ inline double min_lane16(double v) {
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) v = fmin(v, __shfl_xor(v, d));
    return v;
}
__device__ inline double min_wave(double v) {
    v = min_lane16(v);
    v = fmin(v, __shfl_xor(v, 16));
    return fmin(v, __shfl_xor(v, 32));
}
// What a factorisation tells the next iterations, by one wave.  low, low_r: smallest growth of all columns and of the first r
// (see log2_rho).  shrunk: log2 of what the error has come down by.
__device__ inline void note_iteration(const LayerDev& L, int note, int it, double low, double low_r, bool dependent, bool asks, IterationState* own) {
    constexpr int kFirst = kOrthYIterations + 1;          // the first iteration whose growth can be known
    double shrunk = it <= kFirst ? 0.0 : own ? own->shrunk : L.eval[L.wz];
    int ends = 0;
    if ((note & NOTE_GROWTH) && !dependent) {
        const float by = log2_rho(min(L.rows, L.cols), it, low, low_r);
        shrunk += it == kFirst ? (kFirst + 1) * by : by;
        if (!asks && shrunk + by <= (L.planes == 3 ? -37.8 : -29.9)) ends = it + 2;
    }
    if (own) {
        own->shrunk = shrunk;
        own->asks = asks ? 1 : 0;
        own->ends = ends;
    } else if ((threadIdx.x & 63) == 0) {
        L.eval[L.wz] = shrunk;
        if (ends > 0) L.status[11] = ends;
    }
}

// Start block of the subspace iteration beyond the columns of the warm start: uniform in (-1, 1) from a counter-based hash of
// (seed, layer, row, column).
__device__ inline uint32_t mix32(uint32_t x) {
    x ^= x >> 16; x *= 0x7feb352du; x ^= x >> 15; x *= 0x846ca68bu; x ^= x >> 16;
    return x;
}
__device__ inline float start_value(uint32_t seed, int layer, int i, int c) {
    uint32_t h = mix32(seed ^ mix32((uint32_t)layer * 0x9e3779b9u + 0x85ebca6bu));
    h = mix32(h ^ mix32((uint32_t)i + 0x632be5abu) ^ mix32((uint32_t)c * 0xc2b2ae35u + 0x27d4eb2fu));
    return (float)(h >> 8) * (2.0f / 16777216.0f) - 1.0f;
}

// Second-pass permission carried by a launch: -1 always, -2 never, else an iteration gate (kind 2).
__device__ inline bool allow2_of(const LayerDev& L, int a2gate) {
    if (a2gate == -1) return true;
    if (a2gate == -2) return false;
    return gate_open(L, a2gate);
}

// What the notes of a narrow factorisation are made from (column lane & 15).
struct NarrowFactor { double dsc, rjj, min_piv; int badmask; };
// The notes (see IterationNote), by the wave that has factorised; the next iteration needs them, not the application of the factor.
__device__ __forceinline__ void narrow_notes(const LayerDev& L, int w, int note, int it, const NarrowFactor& f, bool write_status, IterationState* own) {
    const int c = threadIdx.x & 15, jc = c < w ? c : 0;
    const bool good = c < w && !((f.badmask >> c) & 1);
    Spread spread;
    note_block(spread, f.rjj, f.dsc, good);
    const bool asks = spread.asks(L.planes, f.min_piv);
    if (write_status || own) {
        // (own: the caller keeps the state in registers, lane c column c's)
        const double csc = next_scale(f.dsc);
        const double norm = f.rjj * __builtin_amdgcn_rcp(good ? f.dsc : 1.0);
        const double prev = own ? own->scale : (note & NOTE_GROWTH) ? L.eval[jc] : 1.0;
        const double grew = good ? norm / prev : kLargest;
        note_iteration(L, note, it, min_lane16(grew), min_lane16(c < L.r ? grew : kLargest), (f.badmask & ((1 << w) - 1)) != 0, asks, own);
        if (own) own->scale = csc;
        else if ((threadIdx.x & 63) < w) L.eval[jc] = csc;
    }
    if (write_status && (threadIdx.x & 63) == 0) L.status[10] = asks ? 1 : 0;
}

// The factorisation for w <= 16 by one wavefront (see factor_in_registers).  g: the summed Gram matrix (packed upper triangle,
// LDS).  Same arithmetic and outputs as the general path of chol_body.  W: compiled width (w <= W); rows and columns
// w .. W-1 are those of an identity matrix.  later: the notes are left to the caller (narrow_notes).
template <int W>
__device__ __forceinline__ void chol_in_registers_w(const LayerDev& L, const double* g, int w, double tol2, int pass,
                                           bool allow2, double* tm, bool write_status, int* need2_out, int note,
                                           int it, NarrowFactor* later) {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));                           // (what depends on the lane is not kept in registers over the caller's loop)
    const int c = t & 15, q = (t >> 4) & 3;
    const int jc = c < w ? c : 0;
    const double djj = g[tri_idx(jc, jc, w)];
    const double dsc_own = djj > kTinyNorm2 ? rsqrt_nr(djj) : 0.0;
    int badmask = (int)(__ballot(c < w && !(dsc_own > 0.0)) & 0xffff);
    doublex4 x, y;
    static_for<0, 4>([&](auto vc) {
        constexpr int v = decltype(vc)::value;
        const int i = 4 * v + q;
        const double dsi = bcast_by_row<4 * v>(dsc_own);
        y[v] = i == c ? 1.0 : 0.0;
        const double xs = dsi > 0.0 && dsc_own > 0.0 ? g[tri_idx(i < w ? i : 0, jc, w)] * dsi * dsc_own : 0.0;
        x[v] = (i < w && c < w && i <= c) ? xs : y[v];
    });
    double min_piv = 1.0, rjj;
    factor_in_registers<W>(x, y, tol2, badmask, min_piv, rjj);
    const NarrowFactor f{dsc_own, rjj, min_piv, badmask};
    if (note & NOTE_SCALE) {                              // (uniform: every lane takes part in the broadcasts)
        const double csc = next_scale(dsc_own);
        static_for<0, 4>([&](auto vc) { constexpr int v = decltype(vc)::value; y[v] *= bcast_by_row<4 * v>(csc); });
    }
    if (later) *later = f;
    else if (note) narrow_notes(L, w, note, it, f, write_status, nullptr);
    // lane (q, c): entries 4 v + q of row c of tmat = D T with the dependent columns zeroed
    if (c < w) {
#pragma unroll
        for (int v = 0; v < W / 4; ++v) {
            const int i = 4 * v + q;
            if (i < w) tm[(int64_t)c * w + i] = ((badmask >> i) & 1) ? 0.0 : y[v] * dsc_own;
        }
    }
    if ((threadIdx.x & 63) == 0) {
        const int nbad = __popc(badmask & ((1 << w) - 1));
        const int need2 = (allow2 && min_piv < kSecondPassPivot) ? 1 : 0;
        if (need2_out) *need2_out = need2;
        if (write_status) {
            if (pass == 1) {
                L.status[0] = nbad;
                L.status[1] = need2;
            } else {
                L.status[0] = max(L.status[0], nbad);
            }
        }
    }
}

// note: see IterationNote (it: the iteration)
__device__ __forceinline__ void chol_in_registers(const LayerDev& L, const double* g, int w, double tol2, int pass,
                                         bool allow2, double* tm, bool write_status, int* need2_out, int note, int it = 0,
                                         NarrowFactor* later = nullptr) {
    if (w <= 4) chol_in_registers_w<4>(L, g, w, tol2, pass, allow2, tm, write_status, need2_out, note, it, later);
    else if (w <= 8) chol_in_registers_w<8>(L, g, w, tol2, pass, allow2, tm, write_status, need2_out, note, it, later);
    else if (w <= 12) chol_in_registers_w<12>(L, g, w, tol2, pass, allow2, tm, write_status, need2_out, note, it, later);
    else chol_in_registers_w<16>(L, g, w, tol2, pass, allow2, tm, write_status, need2_out, note, it, later);
}

// Diagonal 16 x 16 block of the blocked factorisation, by one wavefront in registers: factorises the block `blk` (row-major,
// upper part), leaves T_JJ = R_JJ^{-1} (all 16 x 16 of it) in `tjj` and updates the dependent-column flags and the smallest
// accepted pivot; with dsc (the block's 16 column scalings) also `spread` (columns from n_cols on are padding).  All 64 lanes
// of the wave call it.
__device__ __forceinline__ void chol_block16(const double* blk, double* tjj, double tol2, int* bad, double& min_piv,
                                             const double* dsc, int n_cols, Spread& spread) {
    const int c = threadIdx.x & 15, q = (threadIdx.x & 63) >> 4;
    doublex4 x, y;
    int badmask = (int)(__ballot(bad[c] != 0) & 0xffff);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int i = 4 * v + q;
        y[v] = i == c ? 1.0 : 0.0;
        x[v] = i <= c ? blk[16 * i + c] : 0.0;
    }
    double piv = 1.0, rjj;
    factor_in_registers<16>(x, y, tol2, badmask, piv, rjj);
    min_piv = piv < min_piv ? piv : min_piv;
    // lane (q, c) holds entries 4 v + q of row c of T_JJ
#pragma unroll
    for (int v = 0; v < 4; ++v) tjj[kTjjStride * c + 4 * v + q] = y[v];
    if (q == 0) bad[c] = (badmask >> c) & 1;
    if (dsc) note_block(spread, rjj, dsc[c], c < n_cols && !((badmask >> c) & 1));
}

// Cholesky factorisation and inverse of its factor in one sweep over 16 x 16 blocks: the row operations that turn A into R
// (A = R^T R) turn an identity into W = R^{-T}, and T = R^{-1} is its transpose.  In step J
//   panel      R_JK = T_JJ^T A_JK (K > J),  W_JK <- T_JJ^T W_JK (K <= J; this row of W is final and goes to tm)
//   trailing   A_IK -= R_JI^T R_JK (J < I <= K),  W_IK -= R_JI^T W_JK (K <= J < I)
// on the fp64 matrix cores, blocks dealt to the waves.  W_IK lives where A_KI was (row K of A is finished by then), row J
// of R in a buffer of its own, so one triangle of blocks holds everything; every operand is read row by row, 64 consecutive
// doubles per instruction.
// What bounds it is the chain of 16 steps inside each diagonal block (see factor_in_registers): one wave updates
// and factorises block J + 1 while the others run the rest of the trailing update of step J, and a step has two barriers.
// One workgroup, one slot, us at width 80, 128, 160: 24.3, 45.5, 63.9 with the blocks of the Gram matrix decoded one by one and scaled
// in a pass of their own, the square roots in the chain and T stored 8 bytes a row; 21.6, 38.1, 56.1 now (of the last 8 before the
// first block, 5 to 5.5 per block step, of which the chain 2.1 and the panel 1).
// g: the Gram matrix is the sum of n_slots packed triangles, sstr doubles apart.  smem: chol_lds_bytes(w).
// growth(inverse R_jj of the scaled matrix, column scaling, column dependent): called by wave 0 at the end, for column j = lane + 64 u.
template <class Growth>
__device__ __forceinline__ void chol_blocked(const double* gram_generic, int n_slots, int64_t sstr, int w, double tol2, bool scale,
                                    unsigned char* smem, double* __restrict__ tm, int& nbad, double& min_piv, Spread& spread, Growth&& growth) {
    const int nbk = (w + 15) / 16, wp = 16 * nbk, nblk = (nbk * (nbk + 1)) / 2;
    double* a = reinterpret_cast<double*>(smem);          // blocks (I, K), K >= I, row by row, each [16][16]
    double* rj = a + nblk * 256;                          // [nbk] blocks: row J of R
    double* tjj = rj + nbk * 256;                         // [16][17]
    double* dsc = tjj + 16 * kTjjStride;                  // [wp] scaling
    int* bad = reinterpret_cast<int*>(dsc + wp);          // [wp] dependent-column flags
    const PSGD_GLOBAL double* g = as_global(gram_generic);
    const int t = threadIdx.x, nt = blockDim.x;
    const int lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6), nw = nt >> 6, li = lane & 15, lk = lane >> 4;
    auto at = [&](int I, int K) { return a + (I * nbk - (I * (I - 1)) / 2 + (K - I)) * 256; };
    // ---- blocks of the Gram matrix, scaled, 256 threads per block; identity in the padding.  Which block is a scalar computation,
    // from the thread's block before.  The loads of a thread's first blocks go out before the scalings are known.
    const int ng = nt >> 8, grp = __builtin_amdgcn_readfirstlane(t >> 8), er = (t >> 4) & 15, ec = t & 15;
    int I = 0, K = grp;                                   // (K: counted from the diagonal until the row is known)
    while (I < nbk && K >= nbk - I) { K -= nbk - I; ++I; }
    const int lane_term = ec - er - (er * (er - 1)) / 2;
    auto load_blocks = [&](auto count) {
        constexpr int U = decltype(count)::value;
        bool first = true;
        for (int b0 = grp; first || b0 < nblk; b0 += U * ng) {
            double v[U];
            int off[U], pi[U], pj[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int bi = I < nbk ? I : 0, bj = I < nbk ? I + K : 0;
                // tri_idx(16 bi + er, 16 bj + ec, w), the terms of the lane apart; every lane loads: a conditional load is a branch, and
                // these would run one after the other
                const int o = 8 * bi * (2 * w - 16 * bi + 1) + 16 * (bj - bi) + (er * (w - 16 * bi) + lane_term);
                off[u] = (bi < bj || er <= ec) && 16 * bj + ec < w ? o : -1;
                v[u] = g[(unsigned)max(off[u], 0)];
                pi[u] = bi;
                pj[u] = bj;
                K += ng;
                while (I < nbk && K >= nbk - I) { K -= nbk - I; ++I; }
            }
            constexpr int D = U > 8 ? 2 : 4;
            for (int s0 = 1; s0 < n_slots; s0 += D) {
                double x[D][U];
#pragma unroll
                for (int d = 0; d < D; ++d)
#pragma unroll
                    for (int u = 0; u < U; ++u) x[d][u] = g[min(s0 + d, n_slots - 1) * sstr + max(off[u], 0)];
#pragma unroll
                for (int d = 0; d < D; ++d)
#pragma unroll
                    for (int u = 0; u < U; ++u) v[u] += s0 + d < n_slots ? x[d][u] : 0.0;
            }
            if (first) {
                first = false;
                for (int i = t; i < wp; i += nt) {
                    double d = 1.0;                       // (in the padding)
                    if (i < w) {
                        const int o = tri_idx(i, i, w);
                        d = g[o];
                        for (int s0 = 1; s0 < n_slots; s0 += 4) {
                            double p[4];
#pragma unroll
                            for (int q = 0; q < 4; ++q) p[q] = g[min(s0 + q, n_slots - 1) * sstr + o];
#pragma unroll
                            for (int q = 0; q < 4; ++q) d += s0 + q < n_slots ? p[q] : 0.0;
                        }
                    }
                    dsc[i] = d > kTinyNorm2 ? rsqrt_nr(d) : 0.0;
                    bad[i] = d > kTinyNorm2 ? 0 : 1;
                }
                __syncthreads();
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const double sc = dsc[16 * pi[u] + er] * dsc[16 * pj[u] + ec];
                // (a column that does not count may hold anything)
                if (b0 + u * ng < nblk)
                    a[(b0 + u * ng) * 256 + 16 * er + ec] = off[u] < 0 ? (pi[u] == pj[u] && er == ec ? 1.0 : 0.0) : sc > 0.0 ? v[u] * sc : 0.0;
            }
        }
    };
    if (nblk <= 4 * ng) load_blocks(std::integral_constant<int, 4>{});
    else load_blocks(std::integral_constant<int, 14>{});
    __syncthreads();
    min_piv = 1.0;
    // trailing update of step J for block (I, K), K >= I > J of A or K <= J < I of W
    auto update = [&](int J, int I, int K) {
        double* blk = K >= I ? at(I, K) : at(K, I);
        const double* __restrict__ ra = rj + I * 256;
        const double* __restrict__ rb = K > J ? rj + K * 256 : at(K, J);
        double av[4], bv[4];
        doublex4 d;
#pragma unroll
        for (int c = 0; c < 4; ++c) { av[c] = -ra[16 * (4 * c + lk) + li]; bv[c] = rb[16 * (4 * c + lk) + li]; }
#pragma unroll
        for (int v = 0; v < 4; ++v) d[v] = K == J ? 0.0 : blk[16 * (4 * v + lk) + li];      // (K = J: W_IJ starts at zero)
        __builtin_amdgcn_sched_barrier(0);                // (all loads first: they are made one by one between the MFMAs otherwise)
#pragma unroll
        for (int c = 0; c < 4; ++c) d = __builtin_amdgcn_mfma_f64_16x16x4f64(av[c], bv[c], d, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) blk[16 * (4 * v + lk) + li] = d[v];
    };
#pragma unroll 1
    for (int J = 0; J < nbk; ++J) {
        // ---- the rest of step J - 1: block (J, J) and its factorisation by wave 0, the other blocks by the other waves
        if (wv == 0) {
            if (J > 0) update(J - 1, J, J);
            wave_sync();
            chol_block16(at(J, J), tjj, tol2, bad + 16 * J, min_piv, scale ? dsc + 16 * J : nullptr, w - 16 * J, spread);
        } else if (J > 0) {
            // the blocks of rows I >= J one after the other, in each those of W (K < J), then those of A (K >= I)
            int I = J, k = wv - 1, row = J + (nbk - I);
#pragma unroll 1
            for (;;) {
                while (I < nbk && k >= row) { k -= row; ++I; --row; }
                if (I >= nbk) break;
                const int K = k < J ? k : I + (k - J);
                if (I != J || K != I) update(J - 1, I, K);
                k += nw - 1;
            }
        }
        __syncthreads();
        // ---- panel
#pragma unroll 1
        for (int K = wv; K < nbk; K += nw) {
            double* blk = K < J ? at(K, J) : at(J, K);
            double av[4], bv[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) { av[c] = tjj[kTjjStride * (4 * c + lk) + li]; bv[c] = blk[16 * (4 * c + lk) + li]; }
            // T[i][j], i in block K: the transpose of W_JK, zero below the diagonal and in the columns of dependent vectors.  The product
            // is formed transposed, lanes along j, so that a store covers runs of 128 bytes of T (8 bytes in each row of T otherwise,
            // most of the 1.4 us of a panel at width 160).
            const int j = 16 * J + li;
            doublex4 d = {0.0, 0.0, 0.0, 0.0};
            if (K > J) {
                bool dep[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) dep[v] = bad[16 * J + 4 * v + lk] != 0;
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int c = 0; c < 4; ++c) d = __builtin_amdgcn_mfma_f64_16x16x4f64(av[c], bv[c], d, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    rj[K * 256 + 16 * (4 * v + lk) + li] = dep[v] ? 0.0 : d[v];
                    const int i = 16 * K + 4 * v + lk;
                    if (i < w && j < w) tm[(int64_t)i * w + j] = 0.0;
                }
            } else {
                const double cj = bad[j] ? 0.0 : scale ? next_scale(dsc[j]) : 1.0;
                double ci[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) ci[v] = dsc[16 * K + 4 * v + lk];
                __builtin_amdgcn_sched_barrier(0);
                if (K < J) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) d = __builtin_amdgcn_mfma_f64_16x16x4f64(bv[c], av[c], d, 0, 0, 0);
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v) d[v] = tjj[kTjjStride * (4 * v + lk) + li];        // W_JJ = T_JJ^T
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 16 * K + 4 * v + lk;
                    blk[16 * li + 4 * v + lk] = d[v];
                    if (i < w && j < w) tm[(int64_t)i * w + j] = d[v] * ci[v] * cj;
                }
            }
        }
        __syncthreads();
    }
    nbad = 0;
    if (wv == 0) {
        for (int i0 = 0; i0 < w; i0 += 64) nbad += __popcll(__ballot(i0 + lane < w && bad[i0 + lane] != 0));
        growth([&](int j) { return at(j >> 4, j >> 4)[17 * (j & 15)]; }, dsc, bad);
    }
}

// Layers whose factorisation is cheap enough for every workgroup of the apply kernel to repeat it for
// itself (one kernel boundary less): register path, and few partial Gram matrices to add up.
// local_ok: launch-wide permission (all layers of the launch are narrow), the same in every kernel of the chain
__device__ inline bool local_chol(const LayerDev& L, int role, int local_ok) {
    const int len = side_len(L, side_of_role(L.transposed, role));
    return local_ok && L.thin[role].width <= kCholRegWidth &&
           len <= kLocalCholMaxRows;
}

// Sums the partial Gram matrices of thin[role] (packed upper triangles, slots of `slot_rows` rows, fixed
// order), scales to unit diagonal, Cholesky-factorises (upper, packed in LDS), inverts the factor in
// place and writes tmat = D R_s^{-1}.  pass 1 also decides whether the second CholeskyQR pass runs.
// Called by all threads of one workgroup per layer (256 or 1024: a multiple of 256 and a power of two); smem:
// chol_lds_bytes(w), 8-byte aligned.
// tm: where the w x w factor goes (the layer's tmat, or LDS of the caller); need2_out: optional LDS word
// that receives the second-pass decision; write_status: whether this caller owns the layer's status words; note, it: iteration_notes
// of the subspace iteration.
// gram_at: where the partial Gram matrices are (the layer's gram by default).
// NARROW: compiled for widths <= 16 only (the register path; nothing else is generated).
template <bool NARROW = false>
__device__ __forceinline__ void chol_body(const LayerDev& L, int role, double tol2, int pass, int slot_rows, bool allow2,
                                 unsigned char* smem, double* tm, bool write_status = true,
                                 int* need2_out = nullptr, int note = 0, const double* gram_at = nullptr, int it = 0) {
    const int side = side_of_role(L.transposed, role);
    const int n_slots = (side_len(L, side) + slot_rows - 1) / slot_rows;      // (kOneSlot: one, the sum of all)
    const int w = L.thin[role].width;
    const int ntri = (w * (w + 1)) / 2;
    const int64_t sstr = ntri;                            // distance between the matrices to add
    const int G = chol_groups(w);
    double* a = reinterpret_cast<double*>(smem);          // packed upper triangle
    double* ps = a + ntri;                                // [G][ntri] partial slot sums (G > 1)
    double* dsc = ps + (G > 1 ? G * ntri : 0);            // [w] scaling
    double* rdiag = dsc + w;                              // [w] diagonal of the inverse factor
    double* tcol = rdiag + w;                             // [w up to 16] copy of the column of R being replaced
    const int wp = (w + 15) & ~15;
    int* bad = reinterpret_cast<int*>(tcol + wp);         // [w] dependent-column flags
    const int t = threadIdx.x;
    const int nt = blockDim.x, nty = nt >> 4;             // threads, rows of the 16-wide thread grid
    const double* __restrict__ gram = gram_at ? gram_at : L.gram;
    const bool scale = (note & NOTE_SCALE) != 0;
    // (wave 0) the growth of its columns, and what follows from it; the scales of the iteration before are requested at the start
    double prev[kMaxWaveColumns];
    if constexpr (!NARROW) {
#pragma unroll
        for (int u = 0; u < kMaxWaveColumns; ++u) prev[u] = t < 64 && (note & NOTE_GROWTH) ? as_global(L.eval)[min(t + 64 * u, w - 1)] : 1.0;
    }
    double low = kLargest, low_r = kLargest;
    auto growth = [&](auto&& inverse_of, const double* dsc, const int* bad) {
        if (note == 0) return;
#pragma unroll
        for (int u = 0; u < kMaxWaveColumns; ++u) {
            const int j = t + 64 * u;
            if (j >= w) continue;
            if (!bad[j]) {
                const double grew = 1.0 / (inverse_of(j) * dsc[j]) / prev[u];
                low = fmin(low, grew);
                if (j < L.r) low_r = fmin(low_r, grew);
            }
            as_global(L.eval)[j] = next_scale(dsc[j]);
        }
        low = min_wave(low);
        low_r = min_wave(low_r);
    };
    auto outcome = [&](int nbad, double min_piv, const Spread& spread) {
        if (note && write_status) note_iteration(L, note, it, low, low_r, nbad > 0, spread.asks(L.planes, min_piv), nullptr);
        const int need2 = (allow2 && min_piv < kSecondPassPivot) ? 1 : 0;
        if (need2_out) *need2_out = need2;
        if (write_status) {
            if (pass == 1) {
                L.status[0] = nbad;
                L.status[1] = need2;
                if (scale) L.status[10] = spread.asks(L.planes, min_piv) ? 1 : 0;
            } else {
                L.status[0] = max(L.status[0], nbad);
            }
        }
    };
    if constexpr (!NARROW) {
        if (chol_is_blocked(w)) {
            int nbad = 0;
            double min_piv = 1.0;
            Spread spread;
            chol_blocked(gram, n_slots, sstr, w, tol2, scale, smem, tm, nbad, min_piv, spread, growth);
            if (t == 0) outcome(nbad, min_piv, spread);   // (wave 0 has factorised the diagonal blocks)
            return;
        }
    }
    if (G > 1 || NARROW) {
        // thread (e, g): entries e of slots g, g + G, ...; sixteen loads in flight, those past the end
        // re-read slot g and do not count
        const int g = t / ntri, e = t - g * ntri;
        if (g < G) {
            double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
            for (int sl = g; sl < n_slots; sl += 16 * G) {
                double x[16];
#pragma unroll
                for (int d = 0; d < 16; ++d) {
                    const int sd = sl + d * G;
                    x[d] = gram[(int64_t)(sd < n_slots ? sd : g) * sstr + e];
                }
#pragma unroll
                for (int d = 0; d < 16; ++d)
                    if (sl + d * G >= n_slots) x[d] = 0.0;
#pragma unroll
                for (int d = 0; d < 16; d += 4) { s0 += x[d]; s1 += x[d + 1]; s2 += x[d + 2]; s3 += x[d + 3]; }
            }
            (G > 1 ? ps + g * ntri : a)[e] = (s0 + s1) + (s2 + s3);
        }
        if (G > 1) {
            __syncthreads();
            if (t < ntri) {
                double s = 0.0;
                for (int g2 = 0; g2 < G; ++g2) s += ps[g2 * ntri + t];
                a[t] = s;
            }
        }
    } else {
        // one workgroup adds up everything: keep many loads in flight (four entries x 16 slots per thread, as
        // 16-byte loads where the slot stride keeps them aligned); the order of the sum is fixed
        typedef double doublex2 __attribute__((ext_vector_type(2)));
        const PSGD_GLOBAL double* gg = as_global(gram);
        if ((ntri & 1) == 0) {
            for (int e = 2 * t; e < ntri; e += 4 * nt) {
                const bool two = e + 2 * nt < ntri;
                const PSGD_GLOBAL double* g0 = gg + e;
                const PSGD_GLOBAL double* g1 = gg + (two ? e + 2 * nt : e);
                doublex2 p0 = {0.0, 0.0}, p1 = p0, p2 = p0, p3 = p0, q0 = p0, q1 = p0, q2 = p0, q3 = p0;
                int sl = 0;
                for (; sl + 16 <= n_slots; sl += 16) {
                    doublex2 x[16], y[16];
#pragma unroll
                    for (int d = 0; d < 16; ++d) {
                        x[d] = *reinterpret_cast<const PSGD_GLOBAL doublex2*>(g0 + (int64_t)(sl + d) * sstr);
                        y[d] = *reinterpret_cast<const PSGD_GLOBAL doublex2*>(g1 + (int64_t)(sl + d) * sstr);
                    }
#pragma unroll
                    for (int d = 0; d < 16; d += 4) {
                        p0 += x[d]; p1 += x[d + 1]; p2 += x[d + 2]; p3 += x[d + 3];
                        q0 += y[d]; q1 += y[d + 1]; q2 += y[d + 2]; q3 += y[d + 3];
                    }
                }
                for (; sl < n_slots; ++sl) {
                    p0 += *reinterpret_cast<const PSGD_GLOBAL doublex2*>(g0 + (int64_t)sl * sstr);
                    q0 += *reinterpret_cast<const PSGD_GLOBAL doublex2*>(g1 + (int64_t)sl * sstr);
                }
                const doublex2 ps2 = (p0 + p1) + (p2 + p3), qs2 = (q0 + q1) + (q2 + q3);
                a[e] = ps2.x; a[e + 1] = ps2.y;
                if (two) { a[e + 2 * nt] = qs2.x; a[e + 2 * nt + 1] = qs2.y; }
            }
        } else {
            for (int e = t; e < ntri; e += nt) {
                const PSGD_GLOBAL double* g0 = gg + e;
                double p0 = 0.0, p1 = 0.0, p2 = 0.0, p3 = 0.0;
                int sl = 0;
                for (; sl + 16 <= n_slots; sl += 16) {
                    double x[16];
#pragma unroll
                    for (int d = 0; d < 16; ++d) x[d] = g0[(int64_t)(sl + d) * sstr];
#pragma unroll
                    for (int d = 0; d < 16; d += 4) { p0 += x[d]; p1 += x[d + 1]; p2 += x[d + 2]; p3 += x[d + 3]; }
                }
                for (; sl < n_slots; ++sl) p0 += g0[(int64_t)sl * sstr];
                a[e] = (p0 + p1) + (p2 + p3);
            }
        }
    }
    __syncthreads();
    if (w <= kCholRegWidth) {
        if (t < 64) chol_in_registers(L, a, w, tol2, pass, allow2, tm, write_status, need2_out, note, it);
        return;
    }
    if constexpr (NARROW) return;
    for (int i = t; i < w; i += nt) {
        const double d = a[tri_idx(i, i, w)];
        dsc[i] = d > kTinyNorm2 ? rsqrt_nr(d) : 0.0;
        bad[i] = d > kTinyNorm2 ? 0 : 1;
    }
    __syncthreads();
    // threads as a 16 x 16 grid over (row, column): no integer division in the loops over the triangle
    const int tx = t & 15, ty = t >> 4;
    for (int i = ty; i < w; i += nty) {
        const int base = tri_idx(i, i, w) - i;
        for (int j = i + tx; j < w; j += 16) a[base + j] *= dsc[i] * dsc[j];
    }
    __syncthreads();
    // right-looking Cholesky, A = R^T R, R overwrites the strict upper triangle; 1 / R_kk goes to rdiag
    double min_piv = 1.0;
    Spread spread;
    for (int k = 0; k < w; ++k) {
        // every thread reads the pivot itself; the pivot entry is never overwritten, so two barriers
        // per step are enough
        const double piv = a[tri_idx(k, k, w)];
        const bool dep = bad[k] || !(piv > tol2);
        if (!dep && piv < min_piv) min_piv = piv;
        const int kbase = tri_idx(k, k, w) - k;             // a[tri_idx(k, j)] = a[kbase + j]
        if (dep) {
            if (t == 0) { bad[k] = 1; rdiag[k] = 1.0; }
            for (int j = k + 1 + t; j < w; j += nt) a[kbase + j] = 0.0;
        } else {
            const double rinv = rsqrt_nr(piv);
            if (t == 0) rdiag[k] = rinv;
            const double norm = __builtin_amdgcn_rcp(dsc[k]);
            spread.add(__builtin_amdgcn_frexp_exp(norm * norm), __builtin_amdgcn_frexp_exp(piv * (norm * norm)));
            for (int j = k + 1 + t; j < w; j += nt) a[kbase + j] *= rinv;
        }
        __syncthreads();
        if (!dep) {
            for (int i = k + 1 + ty; i < w; i += nty) {
                const double rki = a[kbase + i];
                const int base = tri_idx(i, i, w) - i;
                for (int j = i + tx; j < w; j += 16) a[base + j] -= rki * a[kbase + j];
            }
        }
        __syncthreads();
    }
    // inverse T of the upper-triangular factor, in place in the packed triangle (T_jj = 1 / R_jj is in rdiag):
    //   T_ij = -T_jj * sum_{l=i}^{j-1} T_il R_lj   (i < j; T_il already in place)
    // column by column, one thread per row i of the new column
    for (int j = 1; j < w; ++j) {
        for (int i = t; i < j; i += nt) tcol[i] = a[tri_idx(i, j, w)];
        __syncthreads();
        const double tjj = rdiag[j];
        for (int i = t; i < j; i += nt) {
            const int base = tri_idx(i, i, w) - i;
            double sacc = rdiag[i] * tcol[i];
            for (int l = i + 1; l < j; ++l) sacc += a[base + l] * tcol[l];
            a[base + j] = -tjj * sacc;
        }
        __syncthreads();
    }
    for (int i = ty; i < w; i += nty) {
        const int base = tri_idx(i, i, w) - i;
        for (int j = tx; j < w; j += 16) {
            double v = 0.0;
            if (!bad[j]) v = (i < j) ? a[base + j] : (i == j ? rdiag[i] : 0.0);
            tm[(int64_t)i * w + j] = v * dsc[i] * (scale ? next_scale(dsc[j]) : 1.0);
        }
    }
    if (t < 64) growth([&](int j) { return rdiag[j]; }, dsc, bad);
    if (t == 0) {
        int nbad = 0;
        for (int i = 0; i < w; ++i) nbad += bad[i];
        outcome(nbad, min_piv, spread);
    }
}

// True in exactly one workgroup of the `n_wg` that call it for a layer: the one that arrives last, after
// which everything the others wrote before their call is visible to it.  `counter` starts at zero and is
// zero again afterwards.  All threads of the workgroup must call it; flag points to an int in LDS.
__device__ inline bool last_to_arrive(int* counter, int n_wg, int* flag) {
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) {
        const int old = atomicAdd(counter, 1);
        *flag = (old == n_wg - 1) ? 1 : 0;
    }
    __syncthreads();
    const bool last = *flag != 0;
    if (last) {
        __threadfence();
        if (threadIdx.x == 0) *counter = 0;
    }
    return last;
}

}  // namespace psgd
