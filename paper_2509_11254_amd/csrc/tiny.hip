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
// A step of a 256 x 128 fp32 layer with four workers (with psgd_decompress) 39.1 -> 32 us, of a 64 x 64 one 38.2 -> 16, sixteen
// of 104 x 104 43.5 -> 23; a refresh 559 -> 288, 425 -> 156, 601 -> 240.  Of the 28 us of the first, 8 go to the gradients (one
// compute unit reads at 64 bytes per clock: 4.3 us for 640 KB), the rest to LDS round trips of the products.
#include "thin_dev.h"

namespace psgd {

constexpr int kTinyThreads = 768;        // (the factorisation needs more registers than 1024 leave, and with 512 the products wait for LDS)
constexpr int kTinyWaves = kTinyThreads / 64;
constexpr int kTinyStride = 16;                        // floats per row of a thin matrix in LDS
constexpr int kTinyGramWaves = 4;                      // waves that share the rows of a Gram matrix
constexpr size_t kTinyScratch = kTinyGramWaves * 256 * sizeof(double);
constexpr size_t kTinyLds = 160 * 1024;
constexpr int64_t kTinyStepElements = 400000, kTinyRefreshElements = 2400000, kTinyRefreshAlways = 8192;

// Row stride of M in LDS: whole 16-byte pieces, an odd number of them, so that 16 rows times 4 columns (the A operand of M Y) lie
// in 64 different banks
__host__ __device__ inline int tiny_ldm(int cols) { return 4 * (((cols + 3) / 4) | 1); }
struct TinyLayout { size_t x, y, tm, gram, flags, end; };
__host__ __device__ inline TinyLayout tiny_layout(int rows, int cols) {
    const int m = rows > cols ? rows : cols, n = rows > cols ? cols : rows;
    auto thin = [](int len) {
        const size_t b = ((size_t)len * kTinyStride * sizeof(float) + 15) & ~(size_t)15;
        return b > kTinyScratch ? b : kTinyScratch;     // (each of the two also serves as the other's Gram scratch)
    };
    TinyLayout t;
    t.x = (size_t)rows * tiny_ldm(cols) * sizeof(float);
    t.y = t.x + thin(m);
    t.tm = t.y + thin(n);
    t.gram = t.tm + 256 * sizeof(double);
    t.flags = t.gram + 136 * sizeof(double);
    t.end = t.flags + 16;
    return t;
}
// Whether a layer's step, or refresh, fits (r: widest thin matrix of it).  n_arrays: gradients and E, which one compute unit reads at
// 0.08 to 0.1 ns per element: not longer than the general path's launches take.  256 x 128 fp32, us: step, 8 workers 33 against 41, 11
// workers 42.4 and 42.8.  A refresh has more launches to save, and a general launch over a matrix of kTinyRefreshAlways elements is
// one or two workgroups, which take as long per worker: 256 x 128 at two iterations, 64 workers 309 against 350, 96 398 and 398, 128
// 481 and 440 (bf16 96 379 and 390, 128 456 and 386); 200 x 160 96 403 and 429, 128 491 and 472; 128 x 128 256 workers 566 and 616;
// 64 x 64 301 and 578.  Not the number of layers, one workgroup each: 256 x 128, one worker, step of 1, 256, 4096 layers 26,
// 37, 599 against 37, 102, 1250, refreshes at two iterations 170, 259, 2600 against 365, 812, 8250; 64 x 64 10, 13, 178 against 36, 65, 522.
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

// X (m x w) = A Y, A(i, k) = M[i si + k sk] (m x n), Y (n x w): a wave per 16 rows, the operands of the next 16 steps of the reduction
// requested before the products of these.  fp32 sums run over 16 steps, their sums in pairs are fp64: with fp32 sums over a quarter of
// the reduction the result was 8 % further from 64 bits than that of the split operands' longer accumulators.
// fine: fp64 sums of single accumulators of 8 steps, for the last two products of a refresh.  One that ends when it has converged leaves
// its columns less settled, which the Rayleigh-Ritz step makes up for with another rounding of both factors (256 x 128 r = 4, error of E
// against 64 bits, mean of eight matrices: 6.38e-7 after 16 iterations without these sums, 6.36e-7 after 8 with them; in all products they take 3 % longer).
__device__ __forceinline__ void tiny_mul(const float* M, int si, int sk, int m, int n, const float* Y, int w, float* X, bool fine = false) {
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = lane & 15, lk = lane >> 4;
    int oa[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) oa[u] = (4 * u + lk) * sk;
    const float* bl = Y + lk * kTinyStride + li;
    const int n16 = n & ~15;
    for (int tile = wv; 16 * tile < m; tile += kTinyWaves) {
        const float* ar = M + min(16 * tile + li, m - 1) * si;
        double sum[4] = {0.0, 0.0, 0.0, 0.0};
        float a[4], b[4];
        const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
        auto fetch = [&](int k0) {
#pragma unroll
            for (int u = 0; u < 4; ++u) { a[u] = ar[k0 * sk + oa[u]]; b[u] = bl[(k0 + 4 * u) * kTinyStride]; }
        };
        if (n16 > 0) fetch(0);
        floatx4 c0 = zero, c1 = zero;
        for (int k0 = 0; k0 < n16; k0 += 16) {
            float ac[4], bc[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) { ac[u] = a[u]; bc[u] = li < w ? b[u] : 0.f; }
            fetch(min(k0 + 16, n16 - 16));
            c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(ac[0], bc[0], c0, 0, 0, 0);
            c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(ac[2], bc[2], c1, 0, 0, 0);
            c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(ac[1], bc[1], c0, 0, 0, 0);
            c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(ac[3], bc[3], c1, 0, 0, 0);
            if (fine) {
#pragma unroll
                for (int v = 0; v < 4; ++v) sum[v] += (double)c0[v] + (double)c1[v];
                c0 = zero;
                c1 = zero;
            } else if ((k0 & 16) || k0 + 16 >= n16) {
                const floatx4 c = c0 + c1;
#pragma unroll
                for (int v = 0; v < 4; ++v) sum[v] += (double)c[v];
                c0 = zero;
                c1 = zero;
            }
        }
        for (int k0 = n16; k0 < n; k0 += 4) {
            const int k = k0 + lk, kc = min(k, n - 1);
            const float av = ar[kc * sk], bv = Y[kc * kTinyStride + li];
            const floatx4 c = __builtin_amdgcn_mfma_f32_16x16x4f32(k < n ? av : 0.f, k < n && li < w ? bv : 0.f, zero, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) sum[v] += (double)c[v];
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 16 * tile + 4 * lk + v;
            if (row < m) X[row * kTinyStride + li] = (float)sum[v];       // (columns from w on: zero)
        }
    }
    __syncthreads();
}

// g = X^T X (packed upper triangle, fp64), X (len x w); red: kTinyScratch bytes
__device__ __forceinline__ void tiny_gram(const float* X, int len, int w, double* red, double* g) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
    if (wv < kTinyGramWaves) {
        doublex4 acc = {0.0, 0.0, 0.0, 0.0};
        const float* xl = X + lk * kTinyStride + li;
        constexpr int step = 4 * kTinyGramWaves;
        int k0 = 4 * wv;
        for (; k0 + 3 * step + 4 <= len; k0 += 4 * step) {       // (four whole steps)
            float x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = xl[(k0 + u * step) * kTinyStride];
#pragma unroll
            for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x[u], (double)x[u], acc, 0, 0, 0);
        }
        for (; k0 < len; k0 += step) {
            const float x0 = X[min(k0 + lk, len - 1) * kTinyStride + li];
            const double x = k0 + lk < len ? (double)x0 : 0.0;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x, x, acc, 0, 0, 0);
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
__device__ __forceinline__ void tiny_apply(float* X, int len, int w, const double* tm) {
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = lane & 15, lk = lane >> 4;
    double b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) b[u] = (4 * u + lk < w && li < w) ? tm[(4 * u + lk) * w + li] : 0.0;
    for (int tile = wv; 16 * tile < len; tile += kTinyWaves) {
        const float* xa = X + min(16 * tile + li, len - 1) * kTinyStride + lk;
        doublex4 acc = {0.0, 0.0, 0.0, 0.0};
        float a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = xa[4 * u];
#pragma unroll
        for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[u], b[u], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 16 * tile + 4 * v + lk;
            if (row < len) X[row * kTinyStride + li] = (float)acc[v];
        }
    }
    __syncthreads();
}

// thin result in LDS -> memory
__device__ __forceinline__ void tiny_store(const ThinRef& T, const float* X, int len, int w) {
    PSGD_GLOBAL float* dst = as_global(T.ptr);
    const int ld = T.ld;
    for (int e = threadIdx.x; e < len * w; e += kTinyThreads) {
        const int row = e / w, c = e - row * w;
        dst[(int64_t)row * ld + c] = X[row * kTinyStride + c];
    }
}

// outer-product operand copies (32 columns) of a thin matrix in LDS, zero beyond it.  KEEP: the first two planes also replace the
// matrix in LDS, eight columns of a row (32 bytes) by those of plane 0 and those of plane 1.
template <bool KEEP>
__device__ __forceinline__ void tiny_pack(const PackRef& K, int planes, float* X, int len, int lenP, int w) {
    PSGD_GLOBAL bf16_t* dn[kMaxPlanes];
#pragma unroll
    for (int k = 0; k < kMaxPlanes; ++k) dn[k] = as_global(K.n[k < planes ? k : 0]);
    for (int v = threadIdx.x; v < lenP * 4; v += kTinyThreads) {
        const int row = 32 * (v >> 7) + (v & 31), c0 = 16 * ((v >> 6) & 1) + 8 * ((v >> 5) & 1);
        bf16x8 o[kMaxPlanes];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool in = row < len && c0 + u < w;
            const float x = X[in ? row * kTinyStride + c0 + u : 0];
            bf16_t q[kMaxPlanes];
            split_planes<kMaxPlanes>(in ? x : 0.f, q);
#pragma unroll
            for (int k = 0; k < kMaxPlanes; ++k) o[k][u] = q[k];
        }
#pragma unroll
        for (int k = 0; k < kMaxPlanes; ++k)
            if (k < planes) *reinterpret_cast<PSGD_GLOBAL bf16x8*>(dn[k] + 8 * v) = o[k];
        if (KEEP && row < len && c0 < 16) {                    // (what this thread alone has read)
            bf16x8* own = reinterpret_cast<bf16x8*>(X + row * kTinyStride + c0);
            own[0] = o[0];
            own[1] = o[1];
        }
    }
}

struct TinyLds {
    float *m, *x, *y;
    double *tm, *gram;
    int *need2, *asks_ends;                                // asks_ends: IterationState::asks + 2 ends
    int ldm;
    __device__ TinyLds(const LayerDev& L, unsigned char* smem) {
        const TinyLayout t = tiny_layout(L.rows, L.cols);
        m = reinterpret_cast<float*>(smem);
        x = reinterpret_cast<float*>(smem + t.x);
        y = reinterpret_cast<float*>(smem + t.y);
        tm = reinterpret_cast<double*>(smem + t.tm);
        gram = reinterpret_cast<double*>(smem + t.gram);
        need2 = reinterpret_cast<int*>(smem + t.flags);
        asks_ends = need2 + 1;
        ldm = tiny_ldm(L.cols);
    }
};

// E = M - X_L X_W^T from the two planes that tiny_pack has left in place of the factors.  What the updates subtract is the
// product of these planes, 2^-17 from that of the factors themselves, and E has to hold what they leave: the same plane products
// in the same order as in the outer-product kernels, so that E plus the update is M to the rounding of E.  (bf16 gradients, four
// workers, compress alone: 256 x 128 28.8 us with the fp32 product of the factors, 26.0 with this; 64 x 64 11.4 and 11.6.  Splitting the
// factors here again, 31.0 and 12.1.)
__device__ __forceinline__ void tiny_residual_planes(const LayerDev& L, const float* M, int ldm, const float* xl, const float* xw) {
    const int rows = L.rows, cols = L.cols;
    const int64_t ld = L.ld;
    PSGD_GLOBAL float* out = as_global(L.S);
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = lane & 31, lg = lane >> 5;
    const int nc = (cols + 31) / 32, n_tiles = ((rows + 31) / 32) * nc;
    for (int tile = wv; tile < n_tiles; tile += kTinyWaves) {
        const int I = tile / nc, J = tile - I * nc, row0 = 32 * I + 4 * lg, col = 32 * J + li;
        const bf16x8* a = reinterpret_cast<const bf16x8*>(xl + min(32 * I + li, rows - 1) * kTinyStride + 8 * lg);
        const bf16x8* b = reinterpret_cast<const bf16x8*>(xw + min(col, cols - 1) * kTinyStride + 8 * lg);
        floatx16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[1], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[0], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[0], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = row0 + 8 * (v >> 2) + (v & 3);
            if (row < rows && col < cols) out[(int64_t)row * ld + col] = M[row * ldm + col] - acc[v];
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
        for (int e = t; e < n * w; e += kTinyThreads) { const int i = e / w; S.y[i * kTinyStride + e - i * w] = q[e]; }
    }
    if (L.gdt == 0) tiny_form<false, false>(L, S.m, S.ldm); else tiny_form<true, false>(L, S.m, S.ldm);
    __syncthreads();
    // M_log(i, k): row i, column k of the matrix with the long side first
    const int sl = tr ? 1 : S.ldm, ss = tr ? S.ldm : 1;
    tiny_mul(S.m, sl, ss, m, n, S.y, w, S.x);
    for (int pass = 1; pass <= 2; ++pass) {
        tiny_gram(S.x, m, w, reinterpret_cast<double*>(S.y), S.gram);
        if (t < 64) chol_in_registers(L, S.gram, w, tol2, pass, pass == 1, S.tm, true, S.need2, 0);
        __syncthreads();
        const bool again = *S.need2 != 0;
        tiny_apply(S.x, m, w, S.tm);
        if (!again) break;                                 // (the second pass asks for no third)
    }
    tiny_mul(S.m, ss, sl, n, m, S.x, w, S.y);
    tiny_store(L.thin[ROLE_P], S.x, m, w);
    tiny_store(L.thin[ROLE_Q], S.y, n, w);
    float* xl = tr ? S.y : S.x;
    float* xw = tr ? S.x : S.y;
    if (L.planes == 2) {
        __syncthreads();                                   // (what tiny_store reads is replaced)
        tiny_pack<true>(L.pack[SIDE_L], 2, xl, rows, L.rowsP, w);
        tiny_pack<true>(L.pack[SIDE_W], 2, xw, cols, L.colsP, w);
        __syncthreads();
        tiny_residual_planes(L, S.m, S.ldm, xl, xw);
        return;
    }
    tiny_pack<false>(L.pack[SIDE_L], L.planes, xl, rows, L.rowsP, w);
    tiny_pack<false>(L.pack[SIDE_W], L.planes, xw, cols, L.colsP, w);
    // E = M - P~ Q^T, 16 x 16 blocks, four of them at a time (three planes hold the factors to fp32: the product of the planes and
    // this one differ by roundings of fp32 sums)
    const int lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6), li = lane & 15, lk = lane >> 4;
    const int nc = (cols + 15) / 16, n_tiles = ((rows + 15) / 16) * nc;
    const int64_t ld = L.ld;
    PSGD_GLOBAL float* out = as_global(L.S);
    constexpr int B = 4;
    for (int tile0 = wv; tile0 < n_tiles; tile0 += B * kTinyWaves) {
        floatx4 acc[B], acc2[B];
        int row0[B], col[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int tile = min(tile0 + b * kTinyWaves, n_tiles - 1), I = tile / nc, J = tile - I * nc;      // (scalar; the last again)
            row0[b] = 16 * I;
            col[b] = 16 * J + li;
            const float* la = xl + min(16 * I + li, rows - 1) * kTinyStride + lk;
            const float* wb = xw + min(col[b], cols - 1) * kTinyStride + lk;
            acc[b] = acc2[b] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                floatx4& c = u < 2 ? acc[b] : acc2[b];
                if (4 * u < w) c = __builtin_amdgcn_mfma_f32_16x16x4f32(la[4 * u], wb[4 * u], c, 0, 0, 0);
            }
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            if (tile0 + b * kTinyWaves >= n_tiles) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = row0[b] + 4 * lk + v;
                if (row < rows && col[b] < cols) out[(int64_t)row * ld + col[b]] = (float)((double)S.m[row * S.ldm + col[b]] - ((double)acc[b][v] + (double)acc2[b][v]));
            }
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
            S.y[i * kTinyStride + c] = c < n_copy ? q[(int64_t)i * Q.ld + c] : start_value(seed, lid, i, c);
        }
    }
    if (L.gdt == 0) tiny_form<false, true>(L, S.m, S.ldm); else tiny_form<true, true>(L, S.m, S.ldm);
    __syncthreads();
    const int sl = tr ? 1 : S.ldm, ss = tr ? S.ldm : 1;
    IterationState state;                                  // (wave 0's)
    bool asked = false;
#pragma unroll 1
    for (int it = 0; it < k_iters; ++it) {
        const bool last = it == k_iters - 1, grows = it > kOrthYIterations && !asked;
        tiny_mul(S.m, sl, ss, m, n, S.y, w, S.x, last);
#pragma unroll 1
        for (int pass = 1; pass <= 2; ++pass) {
            tiny_gram(S.x, m, w, reinterpret_cast<double*>(S.y), S.gram);
            if (t < 64) {
                const int note = pass == 2 || last || it < kOrthYIterations ? 0 : grows ? NOTE_SCALE | NOTE_GROWTH : NOTE_SCALE;
                chol_in_registers(L, S.gram, w, tol2, pass, pass == 1 && last, S.tm, true, S.need2, note, it, &state);
                if (note && t == 0) *S.asks_ends = state.asks + 2 * state.ends;
            }
            __syncthreads();
            const bool again = *S.need2 != 0;
            tiny_apply(S.x, m, w, S.tm);
            if (!again) break;
        }
        if (it >= kOrthYIterations && !last) {
            asked = (*S.asks_ends & 1) != 0;
            const int ends = *S.asks_ends >> 1;
            if (ends > 0 && ends < k_iters) k_iters = ends;
        }
        tiny_mul(S.m, ss, sl, n, m, S.x, w, S.y, last);
        if (!last && (it < kOrthYIterations || asked)) {
            tiny_gram(S.y, n, w, reinterpret_cast<double*>(S.x), S.gram);
            if (t < 64) chol_in_registers(L, S.gram, w, tol2, 1, false, S.tm, true, S.need2, 0);
            __syncthreads();
            tiny_apply(S.y, n, w, S.tm);
        }
    }
    tiny_store(L.thin[ROLE_ZP], S.x, m, w);
    tiny_store(L.thin[ROLE_ZQ], S.y, n, w);
    __syncthreads();
    tiny_gram(S.y, n, w, reinterpret_cast<double*>(S.x), S.gram);
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
