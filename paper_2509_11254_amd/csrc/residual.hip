// Rank-w outer product on MFMA fused with the error-feedback residual (gfx950).
//
//   residual    S <- S - X_L X_W^T     E_{t+1} = M - P~ Q_t^T        (Algorithm 2, error update)
//               (FORM: S holds E_t, not M; M = mean G + E is formed again on the way, Eq. (7a))
//   decompress  out <- X_L X_W^T       Delta_hat = P~ Q_t^T          (Algorithm 1, return value)
//   msgd        m <- mu m + X_L X_W^T;  X <- X - eta m               (Eq. (7c): momentum SGD on Delta_hat)
//   adam        Adam / AdamW moments and weights from X_L X_W^T      (the base optimizer of Section 5's runs)
//
// Both thin operands arrive pre-split into two or three bf16 planes in fragment order; the
// product keeps the 3 (two planes) or 6 (three planes) largest plane products, accumulated in fp32 by
// v_mfma_f32_32x32x16_bf16.  A workgroup owns a
// 128 x 128 tile; wave v owns rows 32v..32v+31 and all 128 columns as four 32 x 32 MFMA blocks.  With wide operands it owns 128
// columns of 8 to 32 such row blocks (rpw), which its 8 or 16 waves take in turn: the column operand is staged in LDS once,
// after that no wave waits for another.
// MFMA block q, column lane i is bound to matrix column 4*i + q, so that after the four blocks each
// lane holds 4 consecutive columns of 16 rows: S is then read and written with 16-byte accesses
// straight from/to the accumulator layout and never goes through LDS.
#include <type_traits>

#include "psgd_dev.h"

namespace psgd {

constexpr int RT = 128;   // tile rows and columns

template <int PL> __device__ inline bool keep_term(int ka, int kb) { return PL == 2 ? (ka + kb <= 1) : (ka + kb <= 2); }

// The thin operands of one tile: planes of the column side (wk) and of the row side (lk), in fragment order (frag_piece).
template <int PL>
struct OuterOperands { const PSGD_GLOBAL bf16_t *wk[PL], *lk[PL]; };
// kept: the copies that a compress step with a deferred residual leaves of its P~ and Q (in the layers that defer: the launch
// addresses only those) instead of the working ones
template <int PL>
__device__ inline OuterOperands<PL> outer_operands(const LayerDev& L, int kept) {
    OuterOperands<PL> O;
#pragma unroll
    for (int k = 0; k < PL; ++k) {
        O.wk[k] = as_global(kept ? L.lzf[SIDE_W][k] : L.pack[SIDE_W].n[k]);
        O.lk[k] = as_global(kept ? L.lzf[SIDE_L][k] : L.pack[SIDE_L].n[k]);
    }
#pragma unroll
    for (int k = 0; k < PL; ++k) asm volatile("" ::"s"(O.wk[k]), "s"(O.lk[k]));      // (all pointers in one round trip)
    return O;
}

// LDS layout of the column operand of a tile: matrix column j = cb*128 + jj belongs to MFMA block q = jj & 3 as its lane jj >> 2;
// 16-byte piece (k-step ks, half lg) of it is piece q (64 KS + 2) + 64 ks + 32 lg + (jj >> 2) of the plane, so that a wavefront reads
// its fragment (q, ks) as 1 KB of consecutive memory, and, by the two pieces between the blocks, eight lanes that write
// neighbouring columns of a fragment reach all banks.
template <int NB> constexpr int kOuterBlock = (64 * 2 * NB + 2) * 8;        // elements of one MFMA block
template <int NB> constexpr int kOuterPlane = 4 * kOuterBlock<NB>;

struct NothingMore { __device__ void operator()() const {} };
// Column operand of a tile -> LDS (its 128 rows are one run of whole fragments, thread t takes pieces t, t + NT, ..).  SB pieces
// per thread are requested together.  Ends with a barrier.
template <int NB, int PL, int W, int SB, class F = NothingMore>
__device__ inline void outer_stage(const OuterOperands<PL>& O, int cb, bf16_t* b_pl, F&& requested = F{}) {
    constexpr int KS = 2 * NB, NT = 64 * W;
    constexpr int NP = (RT / 32) * KS * 64, NI = (NP + NT - 1) / NT;         // 16-byte pieces per plane, and per thread
    const int t = threadIdx.x;
    const int64_t col_frag = (int64_t)cb * (RT / 32) * KS * 512;
#pragma unroll
    for (int i0 = 0; i0 < NI; i0 += SB) {
        uintx4 tmp[SB][PL];
#pragma unroll
        for (int i = 0; i < SB; ++i) {
            const int v = t + (i0 + i) * NT;
#pragma unroll
            for (int k = 0; k < PL; ++k)
                if (i0 + i < NI && (NP % NT == 0 || v < NP)) tmp[i][k] = *reinterpret_cast<const PSGD_GLOBAL uintx4*>(O.wk[k] + col_frag + 8 * v);
        }
        if (i0 == 0) {
            __builtin_amdgcn_sched_barrier(0);
            requested();
        }
#pragma unroll
        for (int i = 0; i < SB; ++i) {
            const int v = t + (i0 + i) * NT;
            const int frag = v >> 6, blk = frag / KS;
            const int jj = 32 * blk + (v & 31);
            const int off = (jj & 3) * kOuterBlock<NB> + (64 * (frag - blk * KS) + (v & 32) + (jj >> 2)) * 8;
#pragma unroll
            for (int k = 0; k < PL; ++k)
                if (i0 + i < NI && (NP % NT == 0 || v < NP)) *reinterpret_cast<uintx4*>(b_pl + k * kOuterPlane<NB> + off) = tmp[i][k];
        }
    }
    __syncthreads();
}

// Product of the 32-row block r32 of the row side with the 128 columns of block cb, by one wavefront.
// KGH = half the k-steps whose row operand is held in registers at a time with two planes (a quarter with three):
// small for the kernels that also hold a tile of M or of the optimizer state, or that want more workgroups per CU
// STAGE: the column operand goes to LDS on the way (else outer_stage has been called)
// requested: called when the first requests are out, for the scalar loads of what the caller needs after the product
template <int NB, int PL, int KGH, bool STAGE, class F = NothingMore>   // cp = 32*NB columns of the thin operands (reduction length), PL bf16 planes
__device__ inline void outer_tile(const OuterOperands<PL>& O, int r32, int cb, bf16_t* b_pl, floatx16 (&acc)[4], F&& requested = F{}) {
    constexpr int KS = 2 * NB;         // k-steps of 16
    constexpr int KG = (PL == 2 ? 2 * KGH : KGH) > 0 ? (PL == 2 ? 2 * KGH : KGH) : 1;
    constexpr int NG = (KS + KG - 1) / KG;
    const int lane = threadIdx.x & 63;
    // Every global round trip on the way to the first MFMA is a stretch in which this workgroup moves no
    // matrix bytes, so the requests go out together: the first batch of the column operand, then the first group of this wave's
    // row operand.
    const int64_t row_frag = (int64_t)r32 * KS * 512;
    bf16x8 av[2][KG][PL];
    auto load_rows = [&](int g, bf16x8 (&dst)[KG][PL]) {
#pragma unroll
        for (int j = 0; j < KG; ++j)
            if (g * KG + j < KS) {
#pragma unroll
                for (int k = 0; k < PL; ++k)
                    dst[j][k] = *reinterpret_cast<const PSGD_GLOBAL bf16x8*>(O.lk[k] + row_frag + (g * KG + j) * 512 + 8 * lane);
            }
    };
    auto rows_and_more = [&]() {
        load_rows(0, av[0]);
        __builtin_amdgcn_sched_barrier(0);
        requested();
    };
    if constexpr (STAGE) outer_stage<NB, PL, 4, (KGH < 2 ? 2 : 4)>(O, cb, b_pl, rows_and_more); else rows_and_more();
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[q][v] = 0.f;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        if (g + 1 < NG) load_rows(g + 1, av[(g + 1) & 1]);      // next group in flight during this one's MFMAs
#pragma unroll
        for (int j = 0; j < KG; ++j) {
            const int ks = g * KG + j;
            if (ks >= KS) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int boff = q * kOuterBlock<NB> + (64 * ks + lane) * 8;
                bf16x8 bv[PL];
#pragma unroll
                for (int k = 0; k < PL; ++k) bv[k] = *reinterpret_cast<const bf16x8*>(b_pl + k * kOuterPlane<NB> + boff);
#pragma unroll
                for (int sum = 2 * (PL - 1); sum >= 0; --sum)
#pragma unroll
                    for (int ka = 0; ka < PL; ++ka) {
                        const int kb = sum - ka;
                        if (kb >= 0 && kb < PL && keep_term<PL>(ka, kb))
                            acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[g & 1][j][ka], bv[kb], acc[q], 0, 0, 0);
                    }
            }
        }
    }
}

// 16 bytes of worker w's gradient at element offset off, widened to fp32
__device__ inline floatx4 load_grad4(const LayerDev& L, int w, int64_t off) {
    const PSGD_GLOBAL void* gw = as_global(as_global(L.G)[w]);
    if (L.gdt == 0) return ld_stream<NT_G>(reinterpret_cast<const PSGD_GLOBAL floatx4*>(reinterpret_cast<const PSGD_GLOBAL float*>(gw) + off));
    const uintx2 v = ld_stream<NT_G>(reinterpret_cast<const PSGD_GLOBAL uintx2*>(reinterpret_cast<const PSGD_GLOBAL bf16_t*>(gw) + off));
    return floatx4{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
                   __uint_as_float(v.y & 0xffff0000u)};
}

template <int NB, int PL, bool FORM, int W>
__global__ __launch_bounds__(64 * W, W == 4 ? 2 : 1) void residual_kernel(const LayerDev* __restrict__ layers,
                                                                       const int* __restrict__ ids, int rpw, int kept) {
    const LayerDev& L = layers[ids[blockIdx.y]];
    const int n_r32 = (L.rows + 31) / 32, n_cb = (L.cols + RT - 1) / RT;
    const int n_rg = (n_r32 + rpw - 1) / rpw;      // groups of rpw 32-row blocks, one workgroup each
    const int tile = blockIdx.x;
    if (tile >= n_rg * n_cb) return;
    const int cb = tile % n_cb, r32_0 = (tile / n_cb) * rpw, r32_1 = min(n_r32, r32_0 + rpw);
    extern __shared__ __align__(16) unsigned char smem[];
    bf16_t* b_pl = reinterpret_cast<bf16_t*>(smem);

    constexpr bool MULTI = W > 4;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 31, lg = lane >> 5;
    // (the layer's numbers are read once, here: the compiler cannot move a scalar load across a store that might alias
    // it, and read in place every store of the epilogue waited for a round trip to the scalar cache of its own)
    const int rows = L.rows, cols = L.cols;
    const int64_t ld = L.ld;
    const int col = cb * RT + 4 * li;
    const bool col_ok = col < cols;
    const OuterOperands<PL> ops = outer_operands<PL>(L, kept);
    float* const S = L.S;
    if constexpr (MULTI) outer_stage<NB, PL, W, 4>(ops, cb, b_pl);
    auto one_block = [&](int r32) {
        const bool interior = 32 * r32 + 32 <= rows && cb * RT + RT <= cols;     // (uniform) nothing to decide per lane
        // issue the 16 loads of M first; the operand staging and the MFMAs hide their latency
        // addresses = uniform base of tile row 8*(v>>2) + (v&3) (scalar registers) + one per-lane offset
        PSGD_GLOBAL float* tile0 = as_global(S) + (int64_t)(32 * r32) * ld + cb * RT;
        const unsigned lane_byte = ((unsigned)(4 * lg) * (unsigned)ld + 4 * li) * 4u;   // < 2^32
        const int row_lane = 32 * r32 + 4 * lg;
        auto at = [&](int k) {
            return reinterpret_cast<PSGD_GLOBAL float*>(reinterpret_cast<PSGD_GLOBAL char*>(tile0 + (int64_t)k * ld) + lane_byte);
        };
        floatx4 m[16];
        auto load_m = [&](auto whole) {
            const int nw = FORM ? L.n_workers : 1;
            const float inv_n = 1.0f / (float)nw;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int k = 8 * (v >> 2) + (v & 3);
                m[v] = floatx4{0.f, 0.f, 0.f, 0.f};
                if (decltype(whole)::value || (col_ok && row_lane + k < rows)) {
                    m[v] = ld_stream<NT_M_RES>(reinterpret_cast<const PSGD_GLOBAL floatx4*>(at(k)));
                    if (FORM) {
                        // same arithmetic and order as the product kernel's FORM path: (sum of workers) / N + E
                        const int64_t off = (int64_t)(32 * r32 + k) * ld + cb * RT + (lane_byte >> 2);
                        floatx4 g = load_grad4(L, 0, off);
                        for (int w = 1; w < nw; ++w) g += load_grad4(L, w, off);
                        m[v] = g * inv_n + m[v];
                    }
                }
            }
        };
        if (interior) load_m(std::true_type{}); else load_m(std::false_type{});
        floatx16 acc[4];
        outer_tile<NB, PL, 1, !MULTI>(ops, r32, cb, b_pl, acc);
        if (interior) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const floatx4 e = {m[v].x - acc[0][v], m[v].y - acc[1][v], m[v].z - acc[2][v], m[v].w - acc[3][v]};
                st_stream<NT_E_OUT>(reinterpret_cast<PSGD_GLOBAL floatx4*>(at(8 * (v >> 2) + (v & 3))), e);
            }
            return;
        }
        if (!col_ok) return;
        const bool full = col + 3 < cols;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int k = 8 * (v >> 2) + (v & 3);
            if (row_lane + k >= rows) continue;
            floatx4 e;
            e.x = m[v].x - acc[0][v]; e.y = m[v].y - acc[1][v]; e.z = m[v].z - acc[2][v]; e.w = m[v].w - acc[3][v];
            PSGD_GLOBAL float* p = at(k);
            if (full) {
                st_stream<NT_E_OUT>(reinterpret_cast<PSGD_GLOBAL floatx4*>(p), e);
            } else {
                p[0] = e.x;
                if (col + 1 < cols) p[1] = e.y;
                if (col + 2 < cols) p[2] = e.z;
            }
        }
    };
    if constexpr (MULTI) {
        for (int r32 = r32_0 + wv; r32 < r32_1; r32 += W) {
            asm volatile("" ::: "memory");      // (or the reads of the staged operand are hoisted, and spill)
            one_block(r32);
        }
    } else {
        one_block(r32_0 + wv);
    }
}

// Write-only: nothing but other workgroups' stores hides this one's operand round trip and MFMA phase, so as many
// workgroups per compute unit as the operand tile in LDS allows (four at NB * PL <= 6).
template <int NB, int PL, int W>
__global__ __launch_bounds__(64 * W, W == 4 ? (NB * PL <= 6 ? 4 : 2) : 1) void decompress_kernel(const LayerDev* __restrict__ layers,
                                                              const int* __restrict__ ids, int rpw, int kept,
                                                              void* const* __restrict__ outs, int out_bf16) {
    const int lid = ids[blockIdx.y];
    const LayerDev& L = layers[lid];
    const int n_r32 = (L.rows + 31) / 32, n_cb = (L.cols + RT - 1) / RT;
    const int n_rg = (n_r32 + rpw - 1) / rpw;      // groups of rpw 32-row blocks, one workgroup each
    const int tile = blockIdx.x;
    if (tile >= n_rg * n_cb) return;
    const int cb = tile % n_cb, r32_0 = (tile / n_cb) * rpw, r32_1 = min(n_r32, r32_0 + rpw);
    extern __shared__ __align__(16) unsigned char smem[];
    bf16_t* b_pl = reinterpret_cast<bf16_t*>(smem);
    constexpr bool MULTI = W > 4;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 31, lg = lane >> 5;
    const int col = cb * RT + 4 * li;
    // (what the stores need is read before them: the compiler cannot move a scalar load across a store that might
    // alias it, and left in place every one of the 16 stores waited for its own round trip to the scalar cache.  But not
    // before the operands are requested, which the first MFMA waits for: scalar loads are waited for all together)
    const int rows = L.rows, cols = L.cols;
    int64_t ld = 0;
    void* outp = nullptr;
    if constexpr (MULTI) { ld = L.ld; outp = outs[lid]; }
    const OuterOperands<PL> ops = outer_operands<PL>(L, kept);
    if constexpr (MULTI) outer_stage<NB, PL, W, 4>(ops, cb, b_pl);
    auto one_block = [&](int r32) {
        const int row_base = 32 * r32 + 4 * lg;
        floatx16 acc[4];
        outer_tile<NB, PL, 2, !MULTI>(ops, r32, cb, b_pl, acc, [&]() { if constexpr (!MULTI) { ld = L.ld; outp = outs[lid]; } });
        const int64_t off0 = (int64_t)row_base * ld + col;
        if (32 * r32 + 32 <= rows && cb * RT + RT <= cols) {
            // interior tile: sixteen stores, nothing to decide
            if (out_bf16) {
                PSGD_GLOBAL bf16_t* p = as_global(reinterpret_cast<bf16_t*>(outp)) + off0;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    bf16x4 o;
                    o[0] = (bf16_t)acc[0][v]; o[1] = (bf16_t)acc[1][v]; o[2] = (bf16_t)acc[2][v]; o[3] = (bf16_t)acc[3][v];
                    st_stream<NT_DEC>(reinterpret_cast<PSGD_GLOBAL bf16x4*>(p + (int64_t)(8 * (v >> 2) + (v & 3)) * ld), o);
                }
            } else {
                PSGD_GLOBAL float* p = as_global(reinterpret_cast<float*>(outp)) + off0;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const floatx4 o = {acc[0][v], acc[1][v], acc[2][v], acc[3][v]};
                    st_stream<NT_DEC>(reinterpret_cast<PSGD_GLOBAL floatx4*>(p + (int64_t)(8 * (v >> 2) + (v & 3)) * ld), o);
                }
            }
            return;
        }
        if (col >= cols) return;
        const bool full = col + 3 < cols;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = row_base + 8 * (v >> 2) + (v & 3);
            if (row >= rows) continue;
            const float d[4] = {acc[0][v], acc[1][v], acc[2][v], acc[3][v]};
            const int64_t off = (int64_t)row * ld + col;
            if (out_bf16) {
                PSGD_GLOBAL bf16_t* p = as_global(reinterpret_cast<bf16_t*>(outp)) + off;
                if (full) {
                    bf16x4 o;
                    o[0] = (bf16_t)d[0]; o[1] = (bf16_t)d[1]; o[2] = (bf16_t)d[2]; o[3] = (bf16_t)d[3];
                    st_stream<NT_DEC>(reinterpret_cast<PSGD_GLOBAL bf16x4*>(p), o);
                } else {
                    for (int q = 0; q < 4; ++q) if (col + q < cols) p[q] = (bf16_t)d[q];
                }
            } else {
                PSGD_GLOBAL float* p = as_global(reinterpret_cast<float*>(outp)) + off;
                if (full) {
                    floatx4 o = {d[0], d[1], d[2], d[3]};
                    st_stream<NT_DEC>(reinterpret_cast<PSGD_GLOBAL floatx4*>(p), o);
                } else {
                    for (int q = 0; q < 4; ++q) if (col + q < cols) p[q] = d[q];
                }
            }
        }
    };
    if constexpr (MULTI) {
        for (int r32 = r32_0 + wv; r32 < r32_1; r32 += W) {
            asm volatile("" ::: "memory");      // (or the reads of the staged operand are hoisted, and spill)
            one_block(r32);
        }
    } else {
        one_block(r32_0 + wv);
    }
}

// Decompress fused with the momentum-SGD update of Eq. (7c): Delta_hat never goes to memory.
//   m_t = mu m_{t-1} + P~ Q^T,   X_{t+1} = X_t - eta m_t      (both rows x cols fp32 with the layer's ld, in place)
template <int NB, int PL, int W>
__global__ __launch_bounds__(64 * W, W == 4 ? 2 : 1) void msgd_kernel(const LayerDev* __restrict__ layers,
                                                           const int* __restrict__ ids, int rpw, int kept,
                                                           float* const* __restrict__ moms,
                                                           float* const* __restrict__ xs, float mu, float eta) {
    const int lid = ids[blockIdx.y];
    const LayerDev& L = layers[lid];
    const int n_r32 = (L.rows + 31) / 32, n_cb = (L.cols + RT - 1) / RT;
    const int n_rg = (n_r32 + rpw - 1) / rpw;      // groups of rpw 32-row blocks, one workgroup each
    const int tile = blockIdx.x;
    if (tile >= n_rg * n_cb) return;
    const int cb = tile % n_cb, r32_0 = (tile / n_cb) * rpw, r32_1 = min(n_r32, r32_0 + rpw);
    extern __shared__ __align__(16) unsigned char smem[];
    bf16_t* b_pl = reinterpret_cast<bf16_t*>(smem);
    constexpr bool MULTI = W > 4;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 31, lg = lane >> 5;
    const int rows = L.rows, cols = L.cols;          // (read once, before any store: see residual_kernel)
    const int64_t ld = L.ld;
    const int col = cb * RT + 4 * li;
    const bool col_ok = col < cols;
    const OuterOperands<PL> ops = outer_operands<PL>(L, kept);
    float *const mom = moms[lid], *const xp = xs[lid];
    if constexpr (MULTI) outer_stage<NB, PL, W, 4>(ops, cb, b_pl);
    auto one_block = [&](int r32) {
        const bool interior = 32 * r32 + 32 <= rows && cb * RT + RT <= cols;
        const int64_t tile_off = (int64_t)(32 * r32) * ld + cb * RT;
        PSGD_GLOBAL float* m0 = as_global(mom) + tile_off;
        PSGD_GLOBAL float* x0 = as_global(xp) + tile_off;
        const unsigned lane_byte = ((unsigned)(4 * lg) * (unsigned)ld + 4 * li) * 4u;   // < 2^32
        const int row_lane = 32 * r32 + 4 * lg;
        auto at = [&](PSGD_GLOBAL float* base, int k) {
            return reinterpret_cast<PSGD_GLOBAL float*>(reinterpret_cast<PSGD_GLOBAL char*>(base + (int64_t)k * ld) + lane_byte);
        };
        // momentum and weights of the tile are requested first; the operand staging and the MFMAs hide the latency
        floatx4 mo[16], xo[16];
        auto load_state = [&](auto whole) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int k = 8 * (v >> 2) + (v & 3);
                mo[v] = floatx4{0.f, 0.f, 0.f, 0.f};
                xo[v] = floatx4{0.f, 0.f, 0.f, 0.f};
                if (decltype(whole)::value || (col_ok && row_lane + k < rows)) {
                    mo[v] = ld_stream<NT_OPT_IN>(reinterpret_cast<const PSGD_GLOBAL floatx4*>(at(m0, k)));
                    xo[v] = ld_stream<NT_OPT_IN>(reinterpret_cast<const PSGD_GLOBAL floatx4*>(at(x0, k)));
                }
            }
        };
        if (interior) load_state(std::true_type{}); else load_state(std::false_type{});
        floatx16 acc[4];
        outer_tile<NB, PL, 1, !MULTI>(ops, r32, cb, b_pl, acc);
        if (interior) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int k = 8 * (v >> 2) + (v & 3);
                const floatx4 d = {acc[0][v], acc[1][v], acc[2][v], acc[3][v]};
                const floatx4 mn = mo[v] * mu + d;
                const floatx4 xn = xo[v] - mn * eta;
                st_stream<NT_OPT_OUT>(reinterpret_cast<PSGD_GLOBAL floatx4*>(at(m0, k)), mn);
                st_stream<NT_OPT_OUT>(reinterpret_cast<PSGD_GLOBAL floatx4*>(at(x0, k)), xn);
            }
            return;
        }
        if (!col_ok) return;
        const bool full = col + 3 < cols;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int k = 8 * (v >> 2) + (v & 3);
            if (row_lane + k >= rows) continue;
            const floatx4 d = {acc[0][v], acc[1][v], acc[2][v], acc[3][v]};
            const floatx4 mn = mo[v] * mu + d;
            const floatx4 xn = xo[v] - mn * eta;
            PSGD_GLOBAL float* pm = at(m0, k);
            PSGD_GLOBAL float* px = at(x0, k);
            if (full) {
                st_stream<NT_OPT_OUT>(reinterpret_cast<PSGD_GLOBAL floatx4*>(pm), mn);
                st_stream<NT_OPT_OUT>(reinterpret_cast<PSGD_GLOBAL floatx4*>(px), xn);
            } else {
                for (int q = 0; q < 4; ++q)
                    if (col + q < cols) { pm[q] = mn[q]; px[q] = xn[q]; }
            }
        }
    };
    if constexpr (MULTI) {
        for (int r32 = r32_0 + wv; r32 < r32_1; r32 += W) {
            asm volatile("" ::: "memory");      // (or the reads of the staged operand are hoisted, and spill)
            one_block(r32);
        }
    } else {
        one_block(r32_0 + wv);
    }
}

// Decompress fused with Adam on Delta_hat (the base optimizer of the paper's pre-training and fine-tuning runs,
// Section 5 and Appendix C; the update itself is the published one, with decoupled weight decay):
//   m <- b1 m + (1 - b1) D,  v <- b2 v + (1 - b2) D^2,  X <- X - step m / (sqrt(v) rs2 + eps) - decay X
// with step = eta / (1 - b1^t), rs2 = 1 / sqrt(1 - b2^t), decay = eta lambda folded by the host.
struct AdamArgs { float b1, b2, c1, c2, step, rs2, eps, decay; };

template <int NB, int PL, int W>
__global__ __launch_bounds__(64 * W, W == 4 ? 2 : 1) void adam_kernel(const LayerDev* __restrict__ layers,
                                                           const int* __restrict__ ids, int rpw, int kept,
                                                           float* const* __restrict__ m1s,
                                                           float* const* __restrict__ m2s,
                                                           float* const* __restrict__ xs, AdamArgs a) {
    const int lid = ids[blockIdx.y];
    const LayerDev& L = layers[lid];
    const int n_r32 = (L.rows + 31) / 32, n_cb = (L.cols + RT - 1) / RT;
    const int n_rg = (n_r32 + rpw - 1) / rpw;      // groups of rpw 32-row blocks, one workgroup each
    const int tile = blockIdx.x;
    if (tile >= n_rg * n_cb) return;
    const int cb = tile % n_cb, r32_0 = (tile / n_cb) * rpw, r32_1 = min(n_r32, r32_0 + rpw);
    extern __shared__ __align__(16) unsigned char smem[];
    bf16_t* b_pl = reinterpret_cast<bf16_t*>(smem);
    constexpr bool MULTI = W > 4;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 31, lg = lane >> 5;
    const int rows = L.rows, cols = L.cols;          // (read once, before any store: see residual_kernel)
    const int64_t ld = L.ld;
    const int col = cb * RT + 4 * li;
    const bool col_ok = col < cols;
    const OuterOperands<PL> ops = outer_operands<PL>(L, kept);
    float *const mp = m1s[lid], *const vp = m2s[lid], *const xp = xs[lid];
    if constexpr (MULTI) outer_stage<NB, PL, W, 4>(ops, cb, b_pl);
    auto one_block = [&](int r32) {
        const bool interior = 32 * r32 + 32 <= rows && cb * RT + RT <= cols;
        const int64_t tile_off = (int64_t)(32 * r32) * ld + cb * RT;
        PSGD_GLOBAL float* m0 = as_global(mp) + tile_off;
        PSGD_GLOBAL float* v0 = as_global(vp) + tile_off;
        PSGD_GLOBAL float* x0 = as_global(xp) + tile_off;
        const unsigned lane_byte = ((unsigned)(4 * lg) * (unsigned)ld + 4 * li) * 4u;   // < 2^32
        const int row_lane = 32 * r32 + 4 * lg;
        auto at = [&](PSGD_GLOBAL float* base, int k) {
            return reinterpret_cast<PSGD_GLOBAL float*>(reinterpret_cast<PSGD_GLOBAL char*>(base + (int64_t)k * ld) + lane_byte);
        };
        // the two moments of the tile are requested before the product (its staging and MFMAs hide their latency);
        // the weights, needed last, are read in the epilogue
        floatx4 mo[16], vo[16];
        auto load_state = [&](auto whole) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int k = 8 * (v >> 2) + (v & 3);
                mo[v] = floatx4{0.f, 0.f, 0.f, 0.f};
                vo[v] = floatx4{0.f, 0.f, 0.f, 0.f};
                if (decltype(whole)::value || (col_ok && row_lane + k < rows)) {
                    mo[v] = ld_stream<NT_OPT_IN>(reinterpret_cast<const PSGD_GLOBAL floatx4*>(at(m0, k)));
                    vo[v] = ld_stream<NT_OPT_IN>(reinterpret_cast<const PSGD_GLOBAL floatx4*>(at(v0, k)));
                }
            }
        };
        if (interior) load_state(std::true_type{}); else load_state(std::false_type{});
        floatx16 acc[4];
        outer_tile<NB, PL, 1, !MULTI>(ops, r32, cb, b_pl, acc);
        auto update = [&](int v, const floatx4& xo, floatx4& mn, floatx4& vn, floatx4& xn) {
            const floatx4 d = {acc[0][v], acc[1][v], acc[2][v], acc[3][v]};
            mn = mo[v] * a.b1 + d * a.c1;
            vn = vo[v] * a.b2 + (d * d) * a.c2;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                xn[q] = xo[q] - a.step * (mn[q] / (sqrtf(vn[q]) * a.rs2 + a.eps)) - a.decay * xo[q];
        };
        if (interior) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                floatx4 xo[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) xo[u] = ld_stream<NT_OPT_IN>(reinterpret_cast<const PSGD_GLOBAL floatx4*>(at(x0, 8 * g + u)));
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int v = 4 * g + u, k = 8 * g + u;
                    floatx4 mn, vn, xn;
                    update(v, xo[u], mn, vn, xn);
                    st_stream<NT_OPT_OUT>(reinterpret_cast<PSGD_GLOBAL floatx4*>(at(m0, k)), mn);
                    st_stream<NT_OPT_OUT>(reinterpret_cast<PSGD_GLOBAL floatx4*>(at(v0, k)), vn);
                    st_stream<NT_OPT_OUT>(reinterpret_cast<PSGD_GLOBAL floatx4*>(at(x0, k)), xn);
                }
            }
            return;
        }
        if (!col_ok) return;
        const bool full = col + 3 < cols;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            floatx4 xo[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = 8 * g + u;
                xo[u] = floatx4{0.f, 0.f, 0.f, 0.f};
                if (row_lane + k < rows) {
                    if (full) xo[u] = ld_stream<NT_OPT_IN>(reinterpret_cast<const PSGD_GLOBAL floatx4*>(at(x0, k)));
                    else for (int q = 0; q < 4; ++q) if (col + q < cols) xo[u][q] = at(x0, k)[q];
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int v = 4 * g + u, k = 8 * g + u;
                if (row_lane + k >= rows) continue;
                floatx4 mn, vn, xn;
                update(v, xo[u], mn, vn, xn);
                PSGD_GLOBAL float* pm = at(m0, k);
                PSGD_GLOBAL float* pv = at(v0, k);
                PSGD_GLOBAL float* px = at(x0, k);
                if (full) {
                    st_stream<NT_OPT_OUT>(reinterpret_cast<PSGD_GLOBAL floatx4*>(pm), mn);
                    st_stream<NT_OPT_OUT>(reinterpret_cast<PSGD_GLOBAL floatx4*>(pv), vn);
                    st_stream<NT_OPT_OUT>(reinterpret_cast<PSGD_GLOBAL floatx4*>(px), xn);
                } else {
                    for (int q = 0; q < 4; ++q)
                        if (col + q < cols) { pm[q] = mn[q]; pv[q] = vn[q]; px[q] = xn[q]; }
                }
            }
        }
    };
    if constexpr (MULTI) {
        for (int r32 = r32_0 + wv; r32 < r32_1; r32 += W) {
            asm volatile("" ::: "memory");      // (or the reads of the staged operand are hoisted, and spill)
            one_block(r32);
        }
    } else {
        one_block(r32_0 + wv);
    }
}

// waves of a workgroup that walks over more than one tile
template <int NB, int PL> constexpr int kOuterWaves = NB * PL >= kOuterManyWaves ? 8 : 4;

static size_t outer_lds_bytes(int nb, int planes) { return (size_t)planes * 4 * (128 * nb + 2) * 16; }

template <int NB, int PL>
static hipError_t launch_outer_nb(bool decomp, bool form, bool kept, const LayerDev* layers, const int* ids, int n_ids,
                                  int max_tiles, int rpw, void* const* outs, int out_bf16, hipStream_t st) {
    constexpr int W = kOuterWaves<NB, PL>;
    dim3 grid(max_tiles, n_ids), block(rpw > 4 ? 64 * W : kThreads);
    const size_t lds = outer_lds_bytes(NB, PL);
    // (kept copies exist up to width 128)
    if (kept && NB > 4) return hipErrorInvalidValue;
    if (decomp) {
        constexpr int WD = W == 4 ? 4 : 16;        // (nothing but the operands in registers)
        if (rpw > 8) block = dim3(64 * WD);
        auto kfn = rpw > 8 ? decompress_kernel<NB, PL, WD> : rpw > 4 ? decompress_kernel<NB, PL, W> : decompress_kernel<NB, PL, 4>;
        if (lds > 48 * 1024) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kfn, grid, block, lds, st, layers, ids, rpw, kept ? 1 : 0, outs, out_bf16);
    } else if (form) {
        if (kept) return hipErrorInvalidValue;      // (the deferred residual lives in the stored M)
        auto kfn = rpw > 4 ? residual_kernel<NB, PL, true, W> : residual_kernel<NB, PL, true, 4>;
        if (lds > 48 * 1024) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kfn, grid, block, lds, st, layers, ids, rpw, kept ? 1 : 0);
    } else {
        auto kfn = rpw > 4 ? residual_kernel<NB, PL, false, W> : residual_kernel<NB, PL, false, 4>;
        if (lds > 48 * 1024) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kfn, grid, block, lds, st, layers, ids, rpw, kept ? 1 : 0);
    }
    return hipGetLastError();
}

template <int NB, int PL>
static hipError_t launch_msgd_nb(const LayerDev* layers, const int* ids, int n_ids, int max_tiles, int rpw, float* const* moms,
                                 float* const* xs, float mu, float eta, bool kept, hipStream_t st) {
    constexpr int W = kOuterWaves<NB, PL>;
    dim3 grid(max_tiles, n_ids), block(rpw > 4 ? 64 * W : kThreads);
    const size_t lds = outer_lds_bytes(NB, PL);
    if (kept && NB > 4) return hipErrorInvalidValue;
    auto kfn = rpw > 4 ? msgd_kernel<NB, PL, W> : msgd_kernel<NB, PL, 4>;
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kfn, grid, block, lds, st, layers, ids, rpw, kept ? 1 : 0, moms, xs, mu, eta);
    return hipGetLastError();
}

// moms, xs: device arrays of per-layer device pointers; kept: as for launch_outer
hipError_t launch_msgd(int nb, int planes, const LayerDev* layers, const int* ids, int n_ids, int max_tiles, int rpw,
                       float* const* moms, float* const* xs, float mu, float eta, bool kept, hipStream_t st) {
    if (n_ids <= 0 || max_tiles <= 0) return hipSuccess;
#define PSGD_CASE(N)                                                                                       \
    case N:                                                                                                \
        return planes == 2 ? launch_msgd_nb<N, 2>(layers, ids, n_ids, max_tiles, rpw, moms, xs, mu, eta, kept, st)   \
                           : launch_msgd_nb<N, 3>(layers, ids, n_ids, max_tiles, rpw, moms, xs, mu, eta, kept, st);
    switch (nb) {
        PSGD_CASE(1) PSGD_CASE(2) PSGD_CASE(3) PSGD_CASE(4) PSGD_CASE(5) PSGD_CASE(6)
        default: return hipErrorInvalidValue;
    }
#undef PSGD_CASE
}

template <int NB, int PL>
static hipError_t launch_adam_nb(const LayerDev* layers, const int* ids, int n_ids, int max_tiles, int rpw, float* const* m1s,
                                 float* const* m2s, float* const* xs, const AdamArgs& a, bool kept, hipStream_t st) {
    constexpr int W = kOuterWaves<NB, PL>;
    dim3 grid(max_tiles, n_ids), block(rpw > 4 ? 64 * W : kThreads);
    const size_t lds = outer_lds_bytes(NB, PL);
    if (kept && NB > 4) return hipErrorInvalidValue;
    auto kfn = rpw > 4 ? adam_kernel<NB, PL, W> : adam_kernel<NB, PL, 4>;
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kfn, grid, block, lds, st, layers, ids, rpw, kept ? 1 : 0, m1s, m2s, xs, a);
    return hipGetLastError();
}

// m1s, m2s, xs: device arrays of per-layer device pointers; coef = {b1, b2, 1 - b1, 1 - b2, eta / (1 - b1^t),
// 1 / sqrt(1 - b2^t), eps, eta * weight decay}
hipError_t launch_adam(int nb, int planes, const LayerDev* layers, const int* ids, int n_ids, int max_tiles, int rpw,
                       float* const* m1s, float* const* m2s, float* const* xs, const float* coef, bool kept,
                       hipStream_t st) {
    if (n_ids <= 0 || max_tiles <= 0) return hipSuccess;
    const AdamArgs a = {coef[0], coef[1], coef[2], coef[3], coef[4], coef[5], coef[6], coef[7]};
#define PSGD_CASE(N)                                                                                       \
    case N:                                                                                                \
        return planes == 2 ? launch_adam_nb<N, 2>(layers, ids, n_ids, max_tiles, rpw, m1s, m2s, xs, a, kept, st)     \
                           : launch_adam_nb<N, 3>(layers, ids, n_ids, max_tiles, rpw, m1s, m2s, xs, a, kept, st);
    switch (nb) {
        PSGD_CASE(1) PSGD_CASE(2) PSGD_CASE(3) PSGD_CASE(4) PSGD_CASE(5) PSGD_CASE(6)
        default: return hipErrorInvalidValue;
    }
#undef PSGD_CASE
}

// kept: the factors are the fragment-order copies that the last compress step left in the addressed layers (all of
// them defer their residual)
hipError_t launch_outer(int nb, int planes, bool decomp, bool form, bool kept, const LayerDev* layers, const int* ids,
                        int n_ids, int max_tiles, int rpw, void* const* outs, int out_bf16, hipStream_t st) {
    if (n_ids <= 0 || max_tiles <= 0) return hipSuccess;
#define PSGD_CASE(N)                                                                                              \
    case N:                                                                                                       \
        return planes == 2 ? launch_outer_nb<N, 2>(decomp, form, kept, layers, ids, n_ids, max_tiles, rpw, outs, out_bf16, st) \
                           : launch_outer_nb<N, 3>(decomp, form, kept, layers, ids, n_ids, max_tiles, rpw, outs, out_bf16, st);
    switch (nb) {
        PSGD_CASE(1) PSGD_CASE(2) PSGD_CASE(3) PSGD_CASE(4) PSGD_CASE(5) PSGD_CASE(6)
        default: return hipErrorInvalidValue;
    }
#undef PSGD_CASE
}

}  // namespace psgd
