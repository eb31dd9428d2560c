// Whole compress steps of small layers in one launch (gfx950): one workgroup per layer holds M in LDS.
//
//   tiny_step     psgd_compress            M = mean G + E;  P~ = QR(M Q);  Q = M^T P~;  E = M - P~ Q^T     (Algorithm 1, SSP-Comp)
//   tiny_iterate  psgd_compress_refresh    M (left in E's buffer), the subspace iteration and the Gram matrix of its last Y;
//                                          Rayleigh-Ritz and the residual follow as in the general path
//
// What bounds such layers is latency: the general path runs six dependent launches of 3 to 11 us per step and as many per
// iteration, on less work than one compute unit does in the time.  Here everything between the first load and the last store
// stays in LDS.  M and the thin matrices are fp32 as in memory, the products run on v_mfma_f32_16x16x4_f32 (fp32 operands and
// sums: no operand planes), Gram matrices, factorisation and its application in fp64 as in the general path.  The product that E
// loses is the one that the updates apply (tiny_residual_planes; with three planes one that differs from it by roundings of fp32).
// A step of a 256 x 128 fp32 layer with four workers (with psgd_decompress) takes 39.1 us in the general path, 31.9 with the thin
// matrices row by row in LDS, read 4 bytes at a time, and E stored 4 bytes at a time, 25.0 now.  Of the 21.6 of its kernel 7.2 go to
// the gradients (one compute unit reads at 64 bytes per clock: 4.3 us for 640 KB), 2.3 to each product, 4 to E, 3.5 to Gram matrix,
// factorisation and its application.  A refresh at two to sixteen iterations 249 -> 222, an iteration 15 -> 13: products 2.9 and
// 3.4 (their MFMAs 1.7), Gram matrix 1.2, factorisation 3.6, application 1.1.
#include "thin_dev.h"

namespace psgd {

constexpr int kTinyThreads = 768;        // (the factorisation needs more registers than 1024 leave, and with 512 the products wait for LDS)
constexpr int kTinyWaves = kTinyThreads / 64;
constexpr int kTinyCols = 16;                          // columns of a thin matrix in LDS (zero from its width on)
constexpr int kTinyGramWaves = 4;                      // waves that share the rows of a Gram matrix
constexpr size_t kTinyScratch = kTinyGramWaves * 256 * sizeof(double);
constexpr size_t kTinyLds = 160 * 1024;
constexpr int64_t kTinyStepElements = 400000, kTinyRefreshElements = 2400000, kTinyRefreshAlways = 8192;

// Row stride of M in LDS, and of the thin matrices, which lie there column by column: whole 16-byte pieces, an odd number of them,
// so that the 16-byte pieces that 16 lanes read from 16 rows lie in different banks
__host__ __device__ inline int tiny_ldm(int cols) { return 4 * (((cols + 3) / 4) | 1); }
struct TinyLayout {
    size_t x, y, gram, flags, end;
    int ldx, ldy;                                          // of the thin matrices on the long and on the short side
};
__host__ __device__ inline TinyLayout tiny_layout_as(int rows, int cols, bool odd) {
    const int m = rows > cols ? rows : cols, n = rows > cols ? cols : rows;
    TinyLayout t;
    t.ldx = odd ? tiny_ldm(m) : (m + 3) & ~3;
    t.ldy = odd ? tiny_ldm(n) : (n + 3) & ~3;
    auto thin = [](int ld) {
        const size_t b = (size_t)kTinyCols * ld * sizeof(float);
        return b > kTinyScratch ? b : kTinyScratch;     // (each of the two also serves as the other's Gram scratch, and then for its factor)
    };
    t.x = (size_t)rows * tiny_ldm(cols) * sizeof(float);
    t.y = t.x + thin(t.ldx);
    t.gram = t.y + thin(t.ldy);
    t.flags = t.gram + 136 * sizeof(double);
    t.end = t.flags + 16;
    return t;
}
// (the thin matrices without the odd number of pieces where that is what makes the layer fit)
__host__ __device__ inline TinyLayout tiny_layout(int rows, int cols) {
    const TinyLayout t = tiny_layout_as(rows, cols, true);
    return t.end <= kTinyLds ? t : tiny_layout_as(rows, cols, false);
}
// Whether a layer's step, or refresh, fits (r: widest thin matrix of it).  n_arrays: gradients and E, which one compute unit reads at
// 0.06 to 0.1 ns per element: not longer than the general path's launches take.  us, one launch and the general path, psgd_compress
// alone: 256 x 128 fp32 r = 4, 8 workers 26 and 38, 11 (the last) 29 and 39; at 426000 elements, 12 workers, 41 and 41, at r = 16 46 and 44, 128 x
// 256 r = 16 48 and 43, 24 x 900 18 workers 56 and 42, though 128 x 128 25 workers 39 and 50 and bf16 31 to 42 and 36 to 54.
// A refresh has more launches to save, and a general launch over a matrix of kTinyRefreshAlways elements is one or two workgroups, which
// take as long per worker: 256 x 128 r = 4 where it runs four iterations, 64 workers 278 and 331, 96 (the last) 366 and 384, 128 455 and 408 (bf16 96
// 347 and 369, 128 428 and 414); 200 x 160 96 374 and 402; 128 x 128 256 workers 539 and 599; 64 x 64 279 and 600.  (With refresh_iters = 2 the
// general path is the faster one from 32 workers on, 165 and 162, 96 345 and 241: the rule does not look at the budget.)
// Not the number of layers, one workgroup each: 256 x 128, one worker, in a graph, step of 1, 256, 4096 layers 24, 36, 515 against
// 38, 100, 1199, refreshes at two iterations 92, 139, 1456 against 138, 280, 3002; 64 x 64 16, 19, 168 and 72, 93, 773 against 36, 64, 495 and 134, 204, 1451.
bool tiny_fits(int64_t rows, int64_t cols, int r, int n_arrays, bool refresh) {
    if (r > kCholRegWidth || rows * cols > (int64_t)(kTinyLds / sizeof(float))) return false;
    if (refresh ? n_arrays * (rows * cols - kTinyRefreshAlways) > kTinyRefreshElements : n_arrays * rows * cols > kTinyStepElements) return false;
    return tiny_layout((int)rows, (int)cols).end <= kTinyLds;
}

// M = (1 / N) sum of the gradients + E -> LDS (row stride ldm); store: also over E.  Sum in worker order, as everywhere.
template <bool BF, bool STORE>
__device__ __forceinline__ void tiny_form(const LayerDev& L, float* M, int ldm) {
    const int rows = L.rows, cols = L.cols, nw = L.n_workers, t = threadIdx.x;
    const int64_t ld = L.ld;
    PSGD_GLOBAL float* S = as_global(L.S);
    auto G = as_global(L.G);
    const float inv_n = 1.0f / (float)nw;
    const int cpr = (cols + 3) / 4, n_pieces = rows * cpr;       // 4-element pieces
    const float inv_cpr = 1.0f / (float)cpr;
    // D pieces of E and of up to NG gradients in flight per thread, 144 KB of the workgroup's
    constexpr int D = 4, NG = 2;
    for (int p0 = t; p0 < n_pieces; p0 += D * kTinyThreads) {
        unsigned row_c[D];                                       // row << 16 | first column (both below 2^16)
        floatx4 e[D], sum[D];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int p = min(p0 + d * kTinyThreads, n_pieces - 1);      // (past the end: the last piece again)
            int row = (int)(((float)p + 0.5f) * inv_cpr), c = p - row * cpr;
            if (c < 0) { --row; c += cpr; } else if (c >= cpr) { ++row; c -= cpr; }
            row_c[d] = (unsigned)row << 16 | (unsigned)(4 * c);
            e[d] = ld_stream<NT_E_IN>(reinterpret_cast<const PSGD_GLOBAL floatx4*>(S + (int64_t)row * ld + 4 * c));
        }
        auto elem = [&](int d) { return (int64_t)(row_c[d] >> 16) * ld + (row_c[d] & 0xffffu); };
        auto load = [&](int w, int d) -> floatx4 {
            if constexpr (BF) {
                const uintx2 v = ld_stream<NT_G>(reinterpret_cast<const PSGD_GLOBAL uintx2*>(reinterpret_cast<const PSGD_GLOBAL bf16_t*>(as_global(G[w])) + elem(d)));
                return floatx4{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u)};
            } else {
                return ld_stream<NT_G>(reinterpret_cast<const PSGD_GLOBAL floatx4*>(reinterpret_cast<const PSGD_GLOBAL float*>(as_global(G[w])) + elem(d)));
            }
        };
        for (int w0 = 0; w0 < nw; w0 += NG) {
            floatx4 g[NG][D];
#pragma unroll
            for (int q = 0; q < NG; ++q)
                if (w0 + q < nw) {
#pragma unroll
                    for (int d = 0; d < D; ++d) g[q][d] = load(w0 + q, d);
                }
#pragma unroll
            for (int q = 0; q < NG; ++q)
                if (w0 + q < nw) {
#pragma unroll
                    for (int d = 0; d < D; ++d) sum[d] = w0 + q == 0 ? g[q][d] : sum[d] + g[q][d];
                }
        }
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (p0 + d * kTinyThreads >= n_pieces) continue;
            const floatx4 x = sum[d] * inv_n + e[d];
            const int row = row_c[d] >> 16, c4 = row_c[d] & 0xffffu, left = cols - c4;
            *reinterpret_cast<floatx4*>(M + row * ldm + c4) = x;        // (past the last column: within the row, never used)
            if constexpr (STORE) {
                PSGD_GLOBAL float* sp = S + elem(d);
                if (left >= 4) *reinterpret_cast<PSGD_GLOBAL floatx4*>(sp) = x;
                else for (int q = 0; q < left; ++q) sp[q] = x[q];
            }
        }
    }
}

// One block of 16 reduction steps: a[q], b hold steps k0 + 4 lk + u (u = 0 .. 3) of Q tiles and of the thin operand, in two
// chains of sums each.  FIRST: the chains start here.  G = 0: 16 x 16 tiles, lane (li, lk) of b holds column li.  G = 1: the
// first 4 G columns only, in blocks of 4 x 4: four lanes of reduction steps keep sums of their own (8 clocks for 4 columns
// against 32 for 16); lane l of b[g] holds column 4 g + (l & 3) of the steps of lk = l >> 4.
template <int Q, int G, bool FIRST>
__device__ __forceinline__ void tiny_steps(const floatx4 (&a)[Q], const floatx4 (&b)[G ? G : 1], floatx4 (&c)[2][Q][G ? G : 1]) {
    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int g = 0; g < (G ? G : 1); ++g) {
                floatx4& d = c[u & 1][q][g];
                const floatx4 from = FIRST && u < 2 ? zero : d;
                if constexpr (G == 0) d = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q][u], b[g][u], from, 0, 0, 0);
                else d = __builtin_amdgcn_mfma_f32_4x4x1f32(a[q][u], b[g][u], from, 0, 0, 0);
            }
}

// X (m x w) = A Y.  ALONG: the reduction runs along the rows of M, A(i, k) = M[i][k] (m rows); else down its columns, A(i, k) =
// M[k][i].  Both operands of a wave's next 16 steps are requested before the products of these: one 16-byte read of the thin
// matrix for Q tiles of 16 rows, and 16 bytes of a row of M for each of them, or 4 Q bytes of four rows (tile q: columns Q i + q).  (4-byte reads,
// 8 for 4 MFMAs: 256 x 128 3.8 and 4.4 us, now 2.9 and 3.4, at r = 4 in blocks of 4 x 4 2.3 and 2.4.)
// fp32 sums run over 16 steps, their sums in pairs are fp64: with fp32 sums over a quarter of
// the reduction the result was 8 % further from 64 bits than that of the split operands' longer accumulators.
// fine: fp64 sums of single accumulators of 8 steps, for the last two products of a refresh.  One that ends when it has converged leaves
// its columns less settled, which the Rayleigh-Ritz step makes up for with another rounding of both factors (256 x 128 r = 4, error of E
// against 64 bits, mean of eight matrices: 6.38e-7 after 16 iterations without these sums, 6.36e-7 after 8 with them; in all products they take 3 % longer).
template <bool ALONG, int Q, int G>
__device__ __forceinline__ void tiny_mul_tiles(const float* M, int ldm, int m, int n, const float* Y, int ldy, float* X, int ldx, bool fine) {
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = lane & 15, lk = lane >> 4;
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    constexpr int NG = G ? G : 1;
    const int n32 = n & ~31;
    const float* bl = Y + (G ? li & 3 : li) * ldy + 4 * lk;
    for (int task = wv; 16 * Q * task < m; task += kTinyWaves) {
        const int i0 = 16 * Q * task;
        const float* ar[ALONG ? Q : 1];
        if constexpr (ALONG) {
#pragma unroll
            for (int q = 0; q < Q; ++q) ar[q] = M + min(i0 + 16 * q + li, m - 1) * ldm + 4 * lk;
        } else {
            ar[0] = M + 4 * lk * ldm + min(i0 + Q * li, ldm - Q);       // (columns past the last: their results are dropped)
        }
        struct Operands { floatx4 a[Q], b[NG]; };
        auto fetch = [&](Operands& o, int k0) {
#pragma unroll
            for (int g = 0; g < NG; ++g) o.b[g] = *reinterpret_cast<const floatx4*>(bl + 4 * g * ldy + k0);
            if constexpr (ALONG) {
#pragma unroll
                for (int q = 0; q < Q; ++q) o.a[q] = *reinterpret_cast<const floatx4*>(ar[q] + k0);
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float* p = ar[0] + (k0 + u) * ldm;
                    if constexpr (Q == 2) {
                        const floatx2 v = *reinterpret_cast<const floatx2*>(p);
                        o.a[0][u] = v.x;
                        o.a[1][u] = v.y;
                    } else {
                        o.a[0][u] = *p;
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);                 // (requested here, not where the registers of the last steps are free again)
        };
        double sum[Q][NG][4];
        floatx4 c[2][Q][NG];
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int g = 0; g < NG; ++g)
#pragma unroll
                for (int v = 0; v < 4; ++v) sum[q][g][v] = 0.0;
        auto add_up = [&](bool each) {
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int g = 0; g < NG; ++g)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        sum[q][g][v] += each ? (double)c[0][q][g][v] + (double)c[1][q][g][v] : (double)(c[0][q][g][v] + c[1][q][g][v]);
        };
        Operands now, next;
        if (n32 > 0) fetch(now, 0);
        for (int k0 = 0; k0 < n32; k0 += 32) {
            fetch(next, k0 + 16);
            tiny_steps<Q, G, true>(now.a, now.b, c);
            fetch(now, min(k0 + 32, n32 - 16));
            if (fine) {
                add_up(true);
                tiny_steps<Q, G, true>(next.a, next.b, c);
                add_up(true);
            } else {
                tiny_steps<Q, G, false>(next.a, next.b, c);
                add_up(false);
            }
        }
        for (int k0 = n32; k0 < n; k0 += 16) {                 // the last steps, those from n on as zeros
            const int kl = k0 + 4 * lk, at = kl < n ? k0 : -4 * lk;       // (reads stay within rows of whole 16-byte pieces)
#pragma unroll
            for (int g = 0; g < NG; ++g) now.b[g] = *reinterpret_cast<const floatx4*>(bl + 4 * g * ldy + at);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool in = kl + u < n;
#pragma unroll
                for (int g = 0; g < NG; ++g) now.b[g][u] = in ? now.b[g][u] : 0.f;
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const float x = ALONG ? ar[ALONG ? q : 0][at + u] : ar[0][(in ? k0 + u : -4 * lk) * ldm + q];
                    now.a[q][u] = in ? x : 0.f;
                }
            }
            tiny_steps<Q, G, true>(now.a, now.b, c);
            add_up(fine);
        }
        // row 4 lk + v of tile q, column li; G: row 4 (li >> 2) + v, column 4 g + (li & 3), after the sums over lk
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            int row = 4 * lk, col = li;
            bool mine = true;
            if constexpr (G > 0) {
                row = 4 * (li >> 2);
                col = 4 * g + (li & 3);
                mine = lk == g;
#pragma unroll
                for (int q = 0; q < Q; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        double s = sum[q][g][v];
                        s += __shfl_xor(s, 16);
                        sum[q][g][v] = s + __shfl_xor(s, 32);
                    }
            }
            if constexpr (ALONG || Q == 1) {
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const int i = i0 + 16 * q + row;
                    if (mine && i < m)
                        *reinterpret_cast<floatx4*>(X + col * ldx + i) = floatx4{(float)sum[q][g][0], (float)sum[q][g][1], (float)sum[q][g][2], (float)sum[q][g][3]};
                }
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int i = i0 + 2 * row + 4 * h;
                    if (mine && i < m)
                        *reinterpret_cast<floatx4*>(X + col * ldx + i) =
                            floatx4{(float)sum[0][g][2 * h], (float)sum[1][g][2 * h], (float)sum[0][g][2 * h + 1], (float)sum[1][g][2 * h + 1]};
                }
            }
        }
    }
}
// Two tiles per wave where that leaves two waves for each of the compute unit's four SIMDs (with one, its sums' additions and
// the end of the reduction are not hidden).  No barrier at the end.  (Columns of X that are not formed keep what they hold.)
template <int G>
__device__ __forceinline__ void tiny_mul_as(const float* M, int ldm, bool along, int m, int n, const float* Y, int ldy, float* X, int ldx, bool fine) {
    if (along) {
        if (m > 192) tiny_mul_tiles<true, 2, G>(M, ldm, m, n, Y, ldy, X, ldx, fine);
        else tiny_mul_tiles<true, 1, G>(M, ldm, m, n, Y, ldy, X, ldx, fine);
    } else {
        if (m > 192) tiny_mul_tiles<false, 2, G>(M, ldm, m, n, Y, ldy, X, ldx, fine);
        else tiny_mul_tiles<false, 1, G>(M, ldm, m, n, Y, ldy, X, ldx, fine);
    }
}
__device__ __forceinline__ void tiny_mul(const float* M, int ldm, bool along, int m, int n, int w, const float* Y, int ldy, float* X, int ldx) {
    if (w <= 4) tiny_mul_as<1>(M, ldm, along, m, n, Y, ldy, X, ldx, false);
    else tiny_mul_as<0>(M, ldm, along, m, n, Y, ldy, X, ldx, false);
}

// g = X^T X (packed upper triangle, fp64), X (len x w); red: kTinyScratch bytes
__device__ __forceinline__ void tiny_gram(const float* X, int ldx, int len, int w, double* red, double* g) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
    if (wv < kTinyGramWaves) {
        doublex4 acc = {0.0, 0.0, 0.0, 0.0};
        const float* xl = X + li * ldx + 4 * lk;
        for (int k0 = 16 * wv; k0 < len; k0 += 16 * kTinyGramWaves) {       // rows k0 + 4 lk + u
            const bool some = k0 + 4 * lk < len;
            const floatx4 x = *reinterpret_cast<const floatx4*>(some ? xl + k0 : X);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double d = k0 + 4 * lk + u < len ? (double)x[u] : 0.0;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(d, d, acc, 0, 0, 0);
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wv * 256 + 64 * v + lane] = acc[v];
    }
    __syncthreads();
    if (threadIdx.x < 256) {
        const int i = 4 * wv + lk;                         // (entry 64 v + lane of a block: row 4 v + lk, column li)
        double sum = 0.0;
#pragma unroll
        for (int q = 0; q < kTinyGramWaves; ++q) sum += red[q * 256 + threadIdx.x];
        if (i <= li && li < w) g[tri_idx(i, li, w)] = sum;
    }
    __syncthreads();
}

// X <- X T in place (len x w; T: w x w in LDS), fp64; a wave reads its 16 rows before it writes them
__device__ __forceinline__ void tiny_apply(float* X, int ldx, int len, int w, const double* tm) {
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = lane & 15, lk = lane >> 4;
    double t[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) t[u] = (4 * u + lk < w && li < w) ? tm[(4 * u + lk) * w + li] : 0.0;
    for (int tile = wv; 16 * tile < len; tile += kTinyWaves) {
        const int row = 16 * tile + li;
        float* xa = X + lk * ldx + min(row, len - 1);
        doublex4 acc = {0.0, 0.0, 0.0, 0.0};
        float a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = 4 * u + lk < w ? xa[4 * u * ldx] : 0.f;       // (the columns beyond may hold anything)
#pragma unroll
        for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(t[u], (double)a[u], acc, 0, 0, 0);
        // (column 4 v + lk of row li)
        if (row < len) {
#pragma unroll
            for (int v = 0; v < 4; ++v) xa[4 * v * ldx] = (float)acc[v];
        }
    }
    __syncthreads();
}

// thin result in LDS -> memory
__device__ __forceinline__ void tiny_store(const ThinRef& T, const float* X, int ldx, int len, int w) {
    PSGD_GLOBAL float* dst = as_global(T.ptr);
    const int ld = T.ld;
    for (int e = threadIdx.x; e < len * w; e += kTinyThreads) {
        const int row = e / w, c = e - row * w;
        dst[(int64_t)row * ld + c] = X[c * ldx + row];
    }
}

// outer-product operand copies (32 columns) of a thin matrix in LDS, zero beyond it
__device__ __forceinline__ void tiny_pack(const PackRef& K, int planes, const float* X, int ldx, int len, int lenP, int w) {
    PSGD_GLOBAL bf16_t* dn[kMaxPlanes];
#pragma unroll
    for (int k = 0; k < kMaxPlanes; ++k) dn[k] = as_global(K.n[k < planes ? k : 0]);
    for (int v = threadIdx.x; v < lenP * 4; v += kTinyThreads) {
        const int row = 32 * (v >> 7) + (v & 31), c0 = 16 * ((v >> 6) & 1) + 8 * ((v >> 5) & 1);
        bf16x8 o[kMaxPlanes];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool in = row < len && c0 + u < w;
            const float x = X[in ? (c0 + u) * ldx + row : 0];
            bf16_t q[kMaxPlanes];
            split_planes<kMaxPlanes>(in ? x : 0.f, q);
#pragma unroll
            for (int k = 0; k < kMaxPlanes; ++k) o[k][u] = q[k];
        }
#pragma unroll
        for (int k = 0; k < kMaxPlanes; ++k)
            if (k < planes) *reinterpret_cast<PSGD_GLOBAL bf16x8*>(dn[k] + 8 * v) = o[k];
    }
}

struct TinyLds {
    float *m, *x, *y;
    double *tmx, *tmy, *gram;                              // tmx, tmy: the factor of x, of y (where the other one was)
    int *need2, *asks_ends;                                // asks_ends: IterationState::asks + 2 ends
    int ldm, ldx, ldy;
    __device__ TinyLds(const LayerDev& L, unsigned char* smem) {
        const TinyLayout t = tiny_layout(L.rows, L.cols);
        m = reinterpret_cast<float*>(smem);
        x = reinterpret_cast<float*>(smem + t.x);
        y = reinterpret_cast<float*>(smem + t.y);
        tmx = reinterpret_cast<double*>(y);
        tmy = reinterpret_cast<double*>(x);
        gram = reinterpret_cast<double*>(smem + t.gram);
        need2 = reinterpret_cast<int*>(smem + t.flags);
        asks_ends = need2 + 1;
        ldm = tiny_ldm(L.cols);
        ldx = t.ldx;
        ldy = t.ldy;
    }
};

// Four consecutive elements of E, of row `row` from column c on
__device__ __forceinline__ void tiny_put(PSGD_GLOBAL float* out, int64_t ld, int rows, int cols, int row, int c, const floatx4& e) {
    if (row >= rows || c >= cols) return;
    PSGD_GLOBAL float* p = out + (int64_t)row * ld + c;
    if (c + 4 <= cols) *reinterpret_cast<PSGD_GLOBAL floatx4*>(p) = e;
    else for (int q = 0; q < cols - c; ++q) p[q] = e[q];
}

// E = M - X_L X_W^T from the two planes that tiny_pack has left in the operand copies (the same workgroup's stores, behind a
// barrier).  What the updates subtract is the product of these planes, 2^-17 from that of the factors themselves, and E has to hold
// what they leave: the same plane products in the same order as in the outer-product kernels, so that E plus the update is M to the
// rounding of E.
__device__ __forceinline__ void tiny_residual_planes(const LayerDev& L, const float* M, int ldm) {
    const int rows = L.rows, cols = L.cols;
    const int64_t ld = L.ld;
    PSGD_GLOBAL float* out = as_global(L.S);
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = lane & 31, lg = lane >> 5;
    const PSGD_GLOBAL bf16x8* l0 = reinterpret_cast<const PSGD_GLOBAL bf16x8*>(as_global(L.pack[SIDE_L].n[0]));
    const PSGD_GLOBAL bf16x8* l1 = reinterpret_cast<const PSGD_GLOBAL bf16x8*>(as_global(L.pack[SIDE_L].n[1]));
    const PSGD_GLOBAL bf16x8* w0 = reinterpret_cast<const PSGD_GLOBAL bf16x8*>(as_global(L.pack[SIDE_W].n[0]));
    const PSGD_GLOBAL bf16x8* w1 = reinterpret_cast<const PSGD_GLOBAL bf16x8*>(as_global(L.pack[SIDE_W].n[1]));
    const int nc = (cols + 31) / 32, n_tiles = ((rows + 31) / 32) * nc;
    for (int tile = wv; tile < n_tiles; tile += kTinyWaves) {
        const int I = tile / nc, J = tile - I * nc, row = 32 * I + li;
        // (fragment of a 32-row block: 128 pieces, of which the first 64 hold columns 0 .. 15)
        const bf16x8 a0 = w0[128 * J + lane], a1 = w1[128 * J + lane], b0 = l0[128 * I + lane], b1 = l1[128 * I + lane];
        floatx16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b0, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b1, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b0, acc, 0, 0, 0);
        const float* mr = M + min(row, rows - 1) * ldm;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int c = 32 * J + 8 * v + 4 * lg;
            const floatx4 x = *reinterpret_cast<const floatx4*>(mr + min(c, ldm - 4));
            tiny_put(out, ld, rows, cols, row, c, floatx4{x[0] - acc[4 * v], x[1] - acc[4 * v + 1], x[2] - acc[4 * v + 2], x[3] - acc[4 * v + 3]});
        }
    }
}

__global__ __launch_bounds__(kTinyThreads) void tiny_step_kernel(const LayerDev* __restrict__ layers, const int* __restrict__ ids, double tol2) {
    const LayerDev& L = layers[ids[blockIdx.x]];
    extern __shared__ __align__(16) unsigned char smem[];
    const TinyLds S(L, smem);
    const int tr = L.transposed, rows = L.rows, cols = L.cols, m = tr ? cols : rows, n = tr ? rows : cols, w = L.r, t = threadIdx.x;
    {
        const PSGD_GLOBAL float* q = as_global(L.thin[ROLE_Q].ptr);
        for (int e = t; e < n * w; e += kTinyThreads) { const int i = e / w; S.y[(e - i * w) * S.ldy + i] = q[e]; }
        for (int e = w * S.ldy + t; e < kTinyCols * S.ldy; e += kTinyThreads) S.y[e] = 0.f;
        for (int e = w * S.ldx + t; e < kTinyCols * S.ldx; e += kTinyThreads) S.x[e] = 0.f;
    }
    if (L.gdt == 0) tiny_form<false, false>(L, S.m, S.ldm); else tiny_form<true, false>(L, S.m, S.ldm);
    __syncthreads();
    tiny_mul(S.m, S.ldm, !tr, m, n, w, S.y, S.ldy, S.x, S.ldx);
    __syncthreads();
    for (int pass = 1; pass <= 2; ++pass) {
        tiny_gram(S.x, S.ldx, m, w, reinterpret_cast<double*>(S.y), S.gram);
        if (t < 64) chol_in_registers(L, S.gram, w, tol2, pass, pass == 1, S.tmx, true, S.need2, 0);
        __syncthreads();
        const bool again = *S.need2 != 0;
        tiny_apply(S.x, S.ldx, m, w, S.tmx);
        if (!again) break;                                 // (the second pass asks for no third)
    }
    const int side_x = tr ? SIDE_W : SIDE_L, side_y = tr ? SIDE_L : SIDE_W;
    tiny_mul(S.m, S.ldm, tr, n, m, w, S.x, S.ldx, S.y, S.ldy);
    // (P~ goes out while other waves are still at the product)
    tiny_store(L.thin[ROLE_P], S.x, S.ldx, m, w);
    tiny_pack(L.pack[side_x], L.planes, S.x, S.ldx, m, tr ? L.colsP : L.rowsP, w);
    __syncthreads();
    tiny_store(L.thin[ROLE_Q], S.y, S.ldy, n, w);
    tiny_pack(L.pack[side_y], L.planes, S.y, S.ldy, n, tr ? L.rowsP : L.colsP, w);
    if (L.planes == 2) {
        __syncthreads();
        tiny_residual_planes(L, S.m, S.ldm);
        return;
    }
    const float* xl = tr ? S.y : S.x;
    const float* xw = tr ? S.x : S.y;
    // E = M - P~ Q^T, 16 x 16 blocks, formed transposed (a lane then holds four consecutive elements of a row;
    // three planes hold the factors to fp32: the product of the planes and this one differ by roundings of fp32 sums)
    const int lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6), li = lane & 15, lk = lane >> 4;
    const int ldl = tr ? S.ldy : S.ldx, ldw = tr ? S.ldx : S.ldy, ldm = S.ldm;
    const int64_t ld = L.ld;
    PSGD_GLOBAL float* out = as_global(L.S);
    // a wave's share: a quarter of the blocks of a block row, kept in step with its operand of that row; all of one block, half of
    // two (as quarters, three of the twelve waves had all the blocks of up to 16 columns: step of 1036 x 9 fp32 41.0 -> 33.0 us, of 600 x 32 28.8 -> 26.4).
    // The larger quarters go round (rounded up, with the last waves idle: 400 x 70 r = 8, four workers 36.4 -> 34.8, 246 x 137 r = 2 27.7 -> 26.4)
    const int nr = (rows + 15) / 16, nc = (cols + 15) / 16, parts = min(nc - 1, 2);
    for (int share = wv; share < nr << parts; share += kTinyWaves) {
        const int I = share >> parts, part = (share + I) & ((1 << parts) - 1);
        const int row = 16 * I + li, rowc = min(row, rows - 1), j0 = (nc * part) >> parts, j1 = (nc * (part + 1)) >> parts;
        float a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = 4 * u < w ? xl[(4 * u + lk) * ldl + rowc] : 0.f;
        const float* mr = S.m + rowc * ldm + 4 * lk;
        const float* wb = xw + lk * ldw + li;
        for (int j = j0; j < j1; ++j) {
            const bool inside = 16 * j + 16 <= cols;           // (uniform)
            const floatx4 x = *reinterpret_cast<const floatx4*>(inside ? mr + 16 * j : S.m + rowc * ldm + min(16 * j + 4 * lk, ldm - 4));
            const float* b = inside ? wb + 16 * j : xw + lk * ldw + min(16 * j + li, cols - 1);
            floatx4 acc = {0.f, 0.f, 0.f, 0.f}, acc2 = acc, e;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                floatx4& c = u < 2 ? acc : acc2;
                if (4 * u < w) c = __builtin_amdgcn_mfma_f32_16x16x4f32(b[4 * u * ldw], a[u], c, 0, 0, 0);
            }
            if (w <= 8) {                                      // (one sum: the difference is rounded once either way)
                e = x - acc;
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v) e[v] = (float)((double)x[v] - ((double)acc[v] + (double)acc2[v]));
            }
            if (inside && row < rows) *reinterpret_cast<PSGD_GLOBAL floatx4*>(out + (int64_t)row * ld + 16 * j + 4 * lk) = e;
            else tiny_put(out, ld, rows, cols, row, 16 * j + 4 * lk, e);
        }
    }
}

// The subspace iteration of the refresh (see refresh_sequence for the steps; the second CholeskyQR pass on the last Z is made
// at once here).  iters: the budget.  Leaves Z and Y in their thin matrices and the Gram matrix of Y in the first slot.
__global__ __launch_bounds__(kTinyThreads) void tiny_iterate_kernel(const LayerDev* __restrict__ layers, const int* __restrict__ ids,
                                                                    double tol2, int iters, int warm, uint32_t seed) {
    const int lid = ids[blockIdx.x];
    const LayerDev& L = layers[lid];
    extern __shared__ __align__(16) unsigned char smem[];
    const TinyLds S(L, smem);
    const int tr = L.transposed, rows = L.rows, cols = L.cols, m = tr ? cols : rows, n = tr ? rows : cols, w = L.wz, t = threadIdx.x;
    int k_iters = refresh_iterations(L, iters);            // (read before anything is stored)
    {
        const ThinRef Q = L.thin[ROLE_Q];
        const PSGD_GLOBAL float* q = as_global(Q.ptr);
        const int n_copy = warm ? min(Q.width, w) : 0;
        for (int e = t; e < n * w; e += kTinyThreads) {
            const int i = e / w, c = e - i * w;
            S.y[c * S.ldy + i] = c < n_copy ? q[(int64_t)i * Q.ld + c] : start_value(seed, lid, i, c);
        }
        for (int e = w * S.ldy + t; e < kTinyCols * S.ldy; e += kTinyThreads) S.y[e] = 0.f;
    }
    if (L.gdt == 0) tiny_form<false, true>(L, S.m, S.ldm); else tiny_form<true, true>(L, S.m, S.ldm);
    __syncthreads();
    // (the last wave's, which makes the notes of a factorisation beside the product that follows: of the products of most sizes it has
    // no tile)
    IterationState state;
    bool asked = false;
#pragma unroll 1
    for (int it = 0; it < k_iters; ++it) {
        const bool last = it == k_iters - 1, grows = it > kOrthYIterations && !asked;
        int noted = 0;
        tiny_mul_as<0>(S.m, S.ldm, !tr, m, n, S.y, S.ldy, S.x, S.ldx, last);
        __syncthreads();
#pragma unroll 1
        for (int pass = 1; pass <= 2; ++pass) {
            tiny_gram(S.x, S.ldx, m, w, reinterpret_cast<double*>(S.y), S.gram);
            const int note = pass == 2 || last || it < kOrthYIterations ? 0 : grows ? NOTE_SCALE | NOTE_GROWTH : NOTE_SCALE;
            noted = note != 0 ? note : noted;
            if (t < 64) {
                NarrowFactor f;
                chol_in_registers(L, S.gram, w, tol2, pass, pass == 1 && last, S.tmx, true, S.need2, note, it, &f);
                if (note && t < 16) {
                    // (the Gram matrix has been read)
                    S.gram[t] = f.dsc;
                    S.gram[16 + t] = f.rjj;
                    if (t == 0) { S.gram[32] = f.min_piv; S.need2[2] = f.badmask; }
                }
            }
            __syncthreads();
            const bool again = *S.need2 != 0;
            tiny_apply(S.x, S.ldx, m, w, S.tmx);
            if (!again) break;
        }
        if (noted && t >= kTinyThreads - 64) {
            const NarrowFactor f{S.gram[t & 15], S.gram[16 + (t & 15)], S.gram[32], S.need2[2]};
            narrow_notes(L, w, noted, it, f, true, &state);
            if ((t & 63) == 0) *S.asks_ends = state.asks + 2 * state.ends;
        }
        tiny_mul_as<0>(S.m, S.ldm, tr, n, m, S.x, S.ldx, S.y, S.ldy, last);
        __syncthreads();
        if (it >= kOrthYIterations && !last) {
            asked = (*S.asks_ends & 1) != 0;
            const int ends = *S.asks_ends >> 1;
            if (ends > 0 && ends < k_iters) k_iters = ends;
        }
        if (!last && (it < kOrthYIterations || asked)) {
            tiny_gram(S.y, S.ldy, n, w, reinterpret_cast<double*>(S.x), S.gram);
            if (t < 64) chol_in_registers(L, S.gram, w, tol2, 1, false, S.tmy, true, S.need2, 0);
            __syncthreads();
            tiny_apply(S.y, S.ldy, n, w, S.tmy);
        }
    }
    tiny_store(L.thin[ROLE_ZP], S.x, S.ldx, m, w);
    tiny_store(L.thin[ROLE_ZQ], S.y, S.ldy, n, w);
    __syncthreads();
    tiny_gram(S.y, S.ldy, n, w, reinterpret_cast<double*>(S.x), S.gram);
    for (int e = t; e < (w * (w + 1)) / 2; e += kTinyThreads) as_global(L.gram)[e] = S.gram[e];
    if (t == 0) L.status[1] = 0;                           // (nothing is left to do for a second pass)
}

static hipError_t tiny_launch_size(const void* kfn, size_t lds) {
    return hipFuncSetAttribute(kfn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

// lds: the largest tiny_layout().end of the layers
hipError_t launch_tiny_step(const LayerDev* layers, const int* ids, int n_ids, size_t lds, double tol2, hipStream_t st) {
    hipError_t e = tiny_launch_size(reinterpret_cast<const void*>(tiny_step_kernel), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(tiny_step_kernel, dim3(n_ids), dim3(kTinyThreads), lds, st, layers, ids, tol2);
    return hipGetLastError();
}

hipError_t launch_tiny_iterate(const LayerDev* layers, const int* ids, int n_ids, size_t lds, double tol2, int iters, int warm,
                               uint32_t seed, hipStream_t st) {
    hipError_t e = tiny_launch_size(reinterpret_cast<const void*>(tiny_iterate_kernel), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(tiny_iterate_kernel, dim3(n_ids), dim3(kTinyThreads), lds, st, layers, ids, tol2, iters, warm, seed);
    return hipGetLastError();
}

size_t tiny_lds_bytes(int64_t rows, int64_t cols) { return tiny_layout((int)rows, (int)cols).end; }

}  // namespace psgd
