// Kernels on the thin (len x w) matrices of the compressor: operand packing, reduction of the
// split products, the orthonormaliser, the Rayleigh-Ritz step of the refresh, random start blocks.
//
// The small factorisation of the orthonormaliser (CholeskyQR2) is in thin_dev.h.
#include <string.h>

#include "thin_dev.h"

namespace psgd {

// --------------------------------------------------------------------------------------------
// pack: thin fp32 (len x width, ld) -> split-bf16 operand copies (PackRef).
// --------------------------------------------------------------------------------------------
// grid.z walks the roles to pack (role_a, then role_b when two are asked for); which: 1 = outer-product copies (what
// the outer-product kernels read), 2 = transposed copies (what the products read), 3 = both
__global__ __launch_bounds__(kThreads) void pack_kernel(const LayerDev* __restrict__ layers,
                                                        const int* __restrict__ ids, int role_a, int role_b,
                                                        int cp, int which) {
    const LayerDev& L = layers[ids[blockIdx.y]];
    const int role = blockIdx.z == 0 ? role_a : role_b;
    const int side = side_of_role(L.transposed, role);
    const int len = side_len(L, side), lenP = side_lenP(L, side);
    const int i0 = blockIdx.x * 64;
    if (i0 >= lenP) return;
    const ThinRef T = L.thin[role];
    extern __shared__ __align__(16) unsigned char smem[];
    float* tile = reinterpret_cast<float*>(smem);      // [64][cp + 1]
    const int tw = cp + 1;
    // eight loads per thread are issued before their LDS stores
    const PSGD_GLOBAL float* src = as_global(T.ptr);
    for (int e0 = 0; e0 < 64 * cp; e0 += 8 * kThreads) {
        float v[8];
#pragma unroll
        for (int d = 0; d < 8; ++d) {
            const int e = e0 + d * kThreads + threadIdx.x;
            const int i = e / cp, c = e % cp;
            v[d] = (e < 64 * cp && i0 + i < len && c < T.width) ? src[(int64_t)(i0 + i) * T.ld + c] : 0.f;
        }
#pragma unroll
        for (int d = 0; d < 8; ++d) {
            const int e = e0 + d * kThreads + threadIdx.x;
            if (e < 64 * cp) tile[(e / cp) * tw + e % cp] = v[d];
        }
    }
    __syncthreads();
    write_packs(L.pack[side], L.planes, tile, tw, cp, i0, 64, lenP, which);
}

// role_b < 0: one role
hipError_t launch_pack(const LayerDev* layers, const int* ids, int n_ids, int max_lenP, int role_a, int role_b,
                       int cp, int which, hipStream_t st) {
    if (n_ids <= 0) return hipSuccess;
    dim3 grid(max_lenP / 64, n_ids, role_b >= 0 ? 2 : 1), block(kThreads);
    const size_t lds = (size_t)64 * (cp + 1) * sizeof(float);
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(pack_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(pack_kernel, grid, block, lds, st, layers, ids, role_a, role_b, cp, which);
    return hipGetLastError();
}

// --------------------------------------------------------------------------------------------
// iterations the next refresh of these layers will run: the largest per-layer count.  The host fetches it asynchronously and
// stops launching iterations past it (they would find every gate closed).
// --------------------------------------------------------------------------------------------
__global__ __launch_bounds__(64) void max_iterations_kernel(const LayerDev* __restrict__ layers, const int* __restrict__ ids,
                                                            int n_ids, int mx, int* __restrict__ out) {
    int k = 1;
    for (int i = threadIdx.x; i < n_ids; i += 64) k = max(k, refresh_iterations(layers[ids[i]], mx));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) k = max(k, __shfl_xor(k, off));
    if (threadIdx.x == 0) out[0] = k;
}

hipError_t launch_max_iterations(const LayerDev* layers, const int* ids, int n_ids, int mx, int* out, hipStream_t st) {
    if (n_ids <= 0) return hipSuccess;
    hipLaunchKernelGGL(max_iterations_kernel, dim3(1), dim3(64), 0, st, layers, ids, n_ids, mx, out);
    return hipGetLastError();
}

// --------------------------------------------------------------------------------------------
// chol: one workgroup per layer runs the factorisation on the partial Gram matrices that the producing
// kernel has left (used when that kernel cannot hand over to it itself).
// --------------------------------------------------------------------------------------------
template <int NT>
__global__ __launch_bounds__(NT) void chol_kernel(const LayerDev* __restrict__ layers,
                                                  const int* __restrict__ ids, int role, double tol2,
                                                  int pass, int slot_rows_n, int slot_rows_t, int gate, int a2gate,
                                                  int local_ok) {
    const LayerDev& L = layers[ids[blockIdx.y]];
    if (!gate_open(L, gate)) return;
    if (pass == 2 && L.status[1] == 0) return;
    if (pass == 1 && local_chol(L, role, local_ok)) return;       // the apply kernel factorises for itself
    extern __shared__ __align__(16) unsigned char smem[];
    chol_body(L, role, tol2, pass, L.transposed ? slot_rows_t : slot_rows_n, allow2_of(L, a2gate), smem, L.tmat, true, nullptr,
              pass == 1 ? iteration_notes(L, role, gate) : 0, nullptr, gate & 0xff);
}

// --------------------------------------------------------------------------------------------
// gram sum: the partial Gram matrices of thin[role] (one per slot_rows_n rows in the layers stored with rows >= cols, per
// slot_rows_t in the others) added up, fixed order, the sum left in the first
// slot.  A workgroup owns 64 entries and its four waves every fourth slot each, 16 loads in flight per thread: the sum of
// 64 slots of width 160 (6.6 MB) is a microsecond-scale pass over the chip instead of the factorisation's one workgroup
// reading all of it.
// --------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void gram_sum_kernel(const LayerDev* __restrict__ layers, const int* __restrict__ ids,
                                                            int role, int slot_rows_n, int slot_rows_t, int gate, int flagged) {
    __shared__ double part[4][64];
    const LayerDev& L = layers[ids[blockIdx.y]];
    if (!gate_open(L, gate)) return;       // (the slots of a layer whose iteration is over hold what its Ritz step needs)
    if (flagged && L.status[1] == 0) return;
    const int slot_rows = L.transposed ? slot_rows_t : slot_rows_n;
    const int n_slots = (side_len(L, side_of_role(L.transposed, role)) + slot_rows - 1) / slot_rows;
    const int w = L.thin[role].width;
    const int ntri = (w * (w + 1)) / 2;
    if ((int)blockIdx.x * 64 >= ntri || n_slots <= 1) return;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + lane;
    PSGD_GLOBAL double* g = as_global(L.gram) + (e < ntri ? e : 0);
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    for (int sl = wv; sl < n_slots; sl += 64) {
        double x[16];
#pragma unroll
        for (int d = 0; d < 16; ++d) x[d] = g[(int64_t)(sl + 4 * d < n_slots ? sl + 4 * d : wv) * ntri];
#pragma unroll
        for (int d = 0; d < 16; ++d) if (sl + 4 * d >= n_slots) x[d] = 0.0;
#pragma unroll
        for (int d = 0; d < 16; d += 4) { s0 += x[d]; s1 += x[d + 1]; s2 += x[d + 2]; s3 += x[d + 3]; }
    }
    part[wv][lane] = (s0 + s1) + (s2 + s3);
    __syncthreads();
    if (wv == 0 && e < ntri) g[0] = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
}

// w: the widest of the layers' blocks; gate: iteration gate of the refresh (-1: none); flagged: only the layers whose
// second-pass flag is set
hipError_t launch_gram_sum(const LayerDev* layers, const int* ids, int n_ids, int w, int role, int slot_rows_n, int slot_rows_t,
                           int gate, int flagged, hipStream_t st) {
    if (n_ids <= 0) return hipSuccess;
    const int ntri = (w * (w + 1)) / 2;
    hipLaunchKernelGGL(gram_sum_kernel, dim3((ntri + 63) / 64, n_ids), dim3(kThreads), 0, st, layers, ids, role, slot_rows_n, slot_rows_t, gate, flagged);
    return hipGetLastError();
}

// Widths above 32 get 512 threads: the panels and trailing updates of the blocked factorisation are dealt to the waves
// (1024 threads halve the registers a thread may hold, and measured slower).
hipError_t launch_chol(const LayerDev* layers, const int* ids, int n_ids, int w, int role, double tol2, int pass,
                       int slot_rows_n, int slot_rows_t, int gate, int a2gate, int local_ok, hipStream_t st) {
    if (n_ids <= 0) return hipSuccess;
    const bool wide = w > 32;
    dim3 grid(1, n_ids), block(wide ? 512 : kThreads);
    const size_t lds = chol_lds_bytes_upto(w);
    auto kfn = wide ? chol_kernel<512> : chol_kernel<kThreads>;
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kfn, grid, block, lds, st, layers, ids, role, tol2, pass, slot_rows_n, slot_rows_t, gate, a2gate,
                       local_ok);
    return hipGetLastError();
}

// --------------------------------------------------------------------------------------------
// apply: thin[dst] (len x w_out) <- thin[src] (len x w_in) * tmat[:, :w_out]   (fp64 accumulate);
// w_in and w_out are the widths of the two thin matrices, tmat is w_in x w_in row-major.  One kernel for launches whose
// layers are all narrow (width <= 16, in place), one for widths up to 96, one beyond.
// In place (dst == src) is allowed: a workgroup reads its 64 rows completely before writing them.
// Fused follow-ups, chosen by `mode` and the layer's second-pass flag:
//   APPLY_PASS1  (upper-triangular tmat): flag set   -> also the partial Gram matrix of the result (the narrow kernel's last
//                                                       workgroup to finish factorises their sum)
//                                         flag clear -> result is final: operand copies if cp > 0
//   APPLY_PASS1_ONLY (the same)         : final + operand copies whatever the flag says: the second pass, if the flag asks
//                                       for one, is run later on the result
//   APPLY_PASS2  (upper-triangular tmat): flag clear -> nothing to do; else final + operand copies
//   APPLY_RITZ   (full tmat)            : final + operand copies if cp > 0 (not in the narrow kernel)
// --------------------------------------------------------------------------------------------
enum ApplyMode { APPLY_PASS1 = 1, APPLY_PASS2 = 2, APPLY_RITZ = 3, APPLY_PASS1_ONLY = 4 };

// LDS bytes of the narrow kernel's x tile and result tile, 16-byte rounded
__host__ __device__ inline size_t apply_main_lds(int w, int cp) {
    const int ow = (cp > 16 ? cp : 16) + 1;
    const size_t b = (size_t)kGramRows2 * (ow + w + 1) * sizeof(float);
    return (b + 15) & ~(size_t)15;
}

// Narrow layers (width <= 16).  It carries the per-workgroup factorisation of the first pass and the hand-over to that of the
// second.  ITER: inside the subspace iteration, where a factorisation also notes what its successor needs (see Spread); the
// step's launches are 0.4 us shorter without that code.
template <bool ITER>
__global__ __launch_bounds__(kThreads) void apply_kernel(const LayerDev* __restrict__ layers,
                                                         const int* __restrict__ ids, int role, int mode, int cp,
                                                         int gate, int a2gate, double tol2, int which, int slot_rows) {
    __shared__ int s_last;
    __shared__ int s_need2;
    const LayerDev& L = layers[ids[blockIdx.y]];
    if (ITER && !gate_open(L, gate)) return;
    const int side = side_of_role(L.transposed, role);
    const int len = side_len(L, side), lenP = side_lenP(L, side);
    const int i0 = blockIdx.x * kGramRows2;
    if (i0 >= lenP) return;
    const ThinRef X = L.thin[role];
    const int w = X.width;
    extern __shared__ __align__(16) unsigned char smem[];
    const size_t main_lds = apply_main_lds(w, cp);
    const double* __restrict__ tm = L.tmat;
    int need2;
    const int t = threadIdx.x;
    // x tile (64 x w): one contiguous block of the thin matrix when ld == width (always the case for the
    // library's own buffers and for P, Q), fetched with one 16-byte load per thread over the flat range
    const bool flat_x = X.ld == w && (w & 3) == 0;
    const int n_valid = (min(len, i0 + kGramRows2) - i0) * w;               // elements that exist
    floatx4 xpre = {0.f, 0.f, 0.f, 0.f};
    // partial Gram matrices of the second pass: behind those of the first where other workgroups may still have to read these
    double* gram2 = L.gram;
    const int ntri = (w * (w + 1)) / 2;
    const bool local = (mode == APPLY_PASS1 || mode == APPLY_PASS1_ONLY) && local_chol(L, role, 1);
    if (local) {
        // small factorisation repeated by every workgroup; the first one records the outcome.  The
        // workgroup's own rows are requested first so that their latency overlaps the factorisation.
        if (flat_x && 4 * t < n_valid) xpre = *reinterpret_cast<const PSGD_GLOBAL floatx4*>(as_global(X.ptr) + (int64_t)i0 * X.ld + 4 * t);
        double* tml = reinterpret_cast<double*>(smem + main_lds);
        const int rows1 = L.transposed ? kGramRows1 : slot_rows;
        gram2 += (int64_t)((len + rows1 - 1) / rows1) * ntri;
        chol_body<true>(L, role, tol2, 1, rows1, allow2_of(L, a2gate), smem + main_lds + w * w * sizeof(double),
                        tml, blockIdx.x == 0, &s_need2, ITER ? iteration_notes(L, role, gate) : 0, nullptr, gate & 0xff);
        __syncthreads();
        need2 = s_need2;
        tm = tml;
    } else {
        need2 = L.status[1];
    }
    if (mode == APPLY_PASS2 && !need2) return;
    const bool do_gram = (mode == APPLY_PASS1) && need2;
    const bool do_pack = !do_gram && cp > 0;
    if (i0 >= (do_pack ? lenP : len)) return;
    const int ow = (cp > 16 ? cp : 16) + 1;           // stride of the result tile (zero padded to cp)
    const int xs = w + 1;                             // row stride of the x tile
    float* sx = reinterpret_cast<float*>(smem);       // [64][xs]  x tile
    float* so = sx + (size_t)kGramRows2 * xs;         // [64][ow]  result tile
    const int tx = t & 63, ty = t >> 6;
    const float inv_w = 1.0f / (float)w;
    if (flat_x) {
        if (!local && 4 * t < n_valid) xpre = *reinterpret_cast<const PSGD_GLOBAL floatx4*>(as_global(X.ptr) + (int64_t)i0 * X.ld + 4 * t);
        const int f = 4 * t;
        if (f < kGramRows2 * w) {
            int row = (int)(((float)f + 0.5f) * inv_w);
            int c = f - row * w;
            if (c < 0) { --row; c += w; } else if (c >= w) { ++row; c -= w; }
            float* dd = sx + row * xs + c;
            dd[0] = xpre.x; dd[1] = xpre.y; dd[2] = xpre.z; dd[3] = xpre.w;
        }
    } else {
        for (int i = ty; i < kGramRows2; i += 4) {
            const bool in = i0 + i < len;
            const float* __restrict__ xr = X.ptr + (int64_t)(in ? i0 + i : 0) * X.ld;
            if (tx < w) sx[i * xs + tx] = in ? xr[tx] : 0.f;
        }
    }
    for (int e = t; e < kGramRows2 * ow; e += kThreads) so[e] = 0.f;
    // The product runs on the fp64 matrix cores (v_mfma_f64_16x16x4_f64): wave v owns rows 16v..16v+15 of the tile.
    // A operand = x (fp32 in LDS, widened per use), B operand = tmat; lane: row / column index li, k index lk.
    const int li = tx & 15, lk = tx >> 4;
    double b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) b[u] = (4 * u + lk < w && li < w) ? tm[(4 * u + lk) * w + li] : 0.0;
    __syncthreads();
    const float* __restrict__ xa = sx + (16 * ty + li) * xs + lk;
    doublex4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (4 * u < w) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(4 * u + lk < w ? (double)xa[4 * u] : 0.0, b[u], acc, 0, 0, 0);
    if (li < w) {
#pragma unroll
        for (int v = 0; v < 4; ++v) so[(16 * ty + 4 * v + lk) * ow + li] = (float)acc[v];
    }
    __syncthreads();
    if (flat_x) {
        // contiguous result block: one 16-byte store per thread (rows past the end are cut off)
        const int f = 4 * t;
        if (f < n_valid) {
            int row = (int)(((float)f + 0.5f) * inv_w);
            int c = f - row * w;
            if (c < 0) { --row; c += w; } else if (c >= w) { ++row; c -= w; }
            const float* __restrict__ sr = so + row * ow + c;
            *reinterpret_cast<PSGD_GLOBAL floatx4*>(as_global(X.ptr) + (int64_t)i0 * X.ld + f) = floatx4{sr[0], sr[1], sr[2], sr[3]};
        }
    } else {
        for (int i = ty; i < kGramRows2 && i0 + i < len; i += 4)
            if (tx < w) X.ptr[(int64_t)(i0 + i) * X.ld + tx] = so[i * ow + tx];
    }
    if (do_gram) {
        gram_tile_f64(so, ow, kGramRows2, w, gram2 + (int64_t)blockIdx.x * ntri);
        const int n_wg = (len + kGramRows2 - 1) / kGramRows2;
        if (last_to_arrive(&L.status[7], n_wg, &s_last))
            chol_body<true>(L, role, tol2, 2, kGramRows2, false, smem, L.tmat, true, nullptr, 0, gram2);
    } else if (do_pack) {
        write_packs(L.pack[side], L.planes, so, ow, cp, i0, kGramRows2, lenP, which & 3, (which & 4) ? L.lzf[side] : nullptr);
    }
}

// --------------------------------------------------------------------------------------------
// The same product for blocks up to 96 wide, as a streaming pass: with a block of tmat staged per 32 output columns from L2
// behind barriers and 66 KB of LDS per workgroup it spent its time on latency, not bytes (224 matrices, 1.58 M rows of width
// 64: 0.70 ms for 1.6 GB of traffic).  Here a workgroup keeps the part of tmat it needs in LDS for its whole life -- per
// 16-column tile of the result only the rows above the diagonal block when tmat is triangular -- and walks over
// many 64-row tiles of its layer; the rows of the next tile are requested before the MFMA phase of the current one.
// --------------------------------------------------------------------------------------------
constexpr int kApplyStreamMaxWidth = 96;
constexpr int kTmStride = 17;        // doubles per row of a 16-column tile of tmat in LDS

__host__ __device__ inline int apply_tm_rows(int ct, int kpad, bool upper) {
    const int k = 16 * (ct + 1);
    return (upper && k < kpad) ? k : kpad;
}
// kp16 > 0: the variant with tmat in registers (reduction length padded to 16 kp16, no tmat in LDS)
__host__ __device__ inline size_t apply_stream_lds(int w_in, int w_out, int cp, bool upper, int kp16) {
    const int kpad = kp16 > 0 ? 16 * kp16 : ((w_in + 3) & ~3), n_ct = (w_out + 15) / 16;
    size_t rows = 0;
    for (int ct = 0; ct < n_ct && kp16 == 0; ++ct) rows += (size_t)apply_tm_rows(ct, kpad, upper);
    const int ow = (cp > 16 * n_ct ? cp : 16 * n_ct) + 1;
    return rows * kTmStride * sizeof(double) + (size_t)kGramRows2 * (kpad + 1 + ow) * sizeof(float);
}

// KP16 > 0: for a triangular tmat of width <= 16 KP16 the wave's fragments of it (tile ct: 4 (ct + 1) steps of the
// reduction) stay in registers for the workgroup's whole life and the MFMA phase reads nothing but them and the rows:
// with the fragments in LDS every MFMA waits on two LDS reads, and the phase ran at a third of the matrix cores' rate.
// KP16 = 0: fragments from LDS (a full tmat, the Ritz step, or widths whose fragments do not fit the registers).
template <int KP16>
__global__ __launch_bounds__(kThreads) void apply_stream_kernel(const LayerDev* __restrict__ layers,
                                                                const int* __restrict__ ids, int src_role, int dst_role,
                                                                int mode, int cp, int gate, int w_out_max, int which) {
    const LayerDev& L = layers[ids[blockIdx.y]];
    if (!gate_open(L, gate)) return;
    if (blockIdx.z != 0) {
        src_role = ROLE_ZQ;
        dst_role = ROLE_Q;
    }
    const int need2 = L.status[1];
    if (mode == APPLY_PASS2 && !need2) return;
    const bool do_gram = (mode == APPLY_PASS1) && need2;
    const bool do_pack = !do_gram && cp > 0;
    const int side = side_of_role(L.transposed, src_role);
    const int len = side_len(L, side), lenP = side_lenP(L, side);
    const int n_tiles = ((do_pack ? lenP : len) + kGramRows2 - 1) / kGramRows2;
    if ((int)blockIdx.x >= n_tiles) return;
    const ThinRef X = L.thin[src_role];
    const ThinRef Y = L.thin[dst_role];
    const int w_in = X.width, w_out = Y.width;
    const bool upper = mode != APPLY_RITZ;
    const int kpad = KP16 > 0 ? 16 * KP16 : ((w_in + 3) & ~3);
    const int n_ct = (w_out + 15) / 16;
    const int n_ct_max = (w_out_max + 15) / 16;
    const int ow = (cp > 16 * n_ct_max ? cp : 16 * n_ct_max) + 1;    // stride of the result tile (zero padded to cp)
    const int xs = kpad + 1;
    extern __shared__ __align__(16) unsigned char smem[];
    double* tl = reinterpret_cast<double*>(smem);                    // tiles of tmat, tile ct: apply_tm_rows x 17
    int tm_rows_all = 0;
    int tm_rows[kApplyStreamMaxWidth / 16], tm_off[kApplyStreamMaxWidth / 16];     // (uniform)
#pragma unroll
    for (int ct = 0; ct < kApplyStreamMaxWidth / 16; ++ct) {
        tm_rows[ct] = (KP16 == 0 && ct < n_ct) ? apply_tm_rows(ct, kpad, upper) : 0;
        tm_off[ct] = tm_rows_all;
        tm_rows_all += tm_rows[ct];
    }
    float* sx = reinterpret_cast<float*>(tl + (size_t)tm_rows_all * kTmStride);   // [64][xs]  x tile
    float* so = sx + (size_t)kGramRows2 * xs;                                     // [64][ow]  result tile
    const int t = threadIdx.x;
    const int lane = t & 63, wv = t >> 6;
    const int li = lane & 15, lk = lane >> 4;
    // ---- tmat -> LDS (eight loads per thread in flight), zero where the matrix ends
    {
        const double* __restrict__ tm = L.tmat;
        const int tcols = min(w_out, w_in);
        int off = 0;
        for (int ct = 0; ct < n_ct && KP16 == 0; ++ct) {
            const int rows = apply_tm_rows(ct, kpad, upper);
            for (int e0 = 0; e0 < rows * 16; e0 += 8 * kThreads) {
                double tv[8];
#pragma unroll
                for (int d = 0; d < 8; ++d) {
                    const int e = e0 + d * kThreads + t;
                    const int k = e >> 4, c = 16 * ct + (e & 15);
                    tv[d] = (e < rows * 16 && k < w_in && c < tcols) ? tm[(int64_t)k * w_in + c] : 0.0;
                }
#pragma unroll
                for (int d = 0; d < 8; ++d) {
                    const int e = e0 + d * kThreads + t;
                    if (e < rows * 16) tl[(off + (e >> 4)) * kTmStride + (e & 15)] = tv[d];
                }
            }
            off += rows;
        }
        for (int e = t; e < kGramRows2 * ow; e += kThreads) so[e] = 0.f;
    }
    constexpr int NTB = KP16 > 0 ? 2 * KP16 * (KP16 + 1) : 1;
    double tb[NTB];                                              // tile ct, step ks at 2 ct (ct + 1) + ks
    if (KP16 > 0) {
        const double* __restrict__ tm = L.tmat;
        const int tcols = min(w_out, w_in);
#pragma unroll
        for (int ct = 0; ct < KP16; ++ct)
#pragma unroll
            for (int ks = 0; ks < 4 * (ct + 1); ++ks) {
                const int k = 4 * ks + lk, c = 16 * ct + li;
                tb[2 * ct * (ct + 1) + ks] = (k < w_in && c < tcols) ? tm[(int64_t)k * w_in + c] : 0.0;
            }
    }
    // ---- the rows of a tile: one contiguous block of the thin matrix when ld == width, fetched with 16-byte loads
    const bool flat_x = X.ld == w_in && (w_in & 3) == 0;
    const bool flat_y = Y.ld == w_out && (w_out & 3) == 0;
    const float inv_wi = 1.0f / (float)w_in, inv_wo = 1.0f / (float)w_out;
    constexpr int XP = kApplyStreamMaxWidth / 16;          // 16-byte pieces per thread at the widest
    floatx4 xr[XP];
    auto load_x = [&](int tile) {
        const int i0 = tile * kGramRows2;
        const int n_valid = (min(len, i0 + kGramRows2) - i0) * w_in;
        const PSGD_GLOBAL float* xp = as_global(X.ptr) + (int64_t)i0 * X.ld;
#pragma unroll
        for (int d = 0; d < XP; ++d) {
            const int f = 4 * (d * kThreads + t);
            xr[d] = floatx4{0.f, 0.f, 0.f, 0.f};
            if (f < n_valid) xr[d] = *reinterpret_cast<const PSGD_GLOBAL floatx4*>(xp + f);
        }
    };
    int tile = blockIdx.x;
    if (flat_x) load_x(tile);
    for (; tile < n_tiles; tile += gridDim.x) {
        const int i0 = tile * kGramRows2;
        // ---- x tile -> LDS (zero beyond the matrix and in the columns up to the padded reduction length)
        if (flat_x) {
#pragma unroll
            for (int d = 0; d < XP; ++d) {
                const int f = 4 * (d * kThreads + t);
                if (f >= kGramRows2 * w_in) continue;
                int row = (int)(((float)f + 0.5f) * inv_wi);
                int c = f - row * w_in;
                if (c < 0) { --row; c += w_in; } else if (c >= w_in) { ++row; c -= w_in; }
                float* dd = sx + row * xs + c;
                dd[0] = xr[d].x; dd[1] = xr[d].y; dd[2] = xr[d].z; dd[3] = xr[d].w;
            }
            if (kpad > w_in)
                for (int e = t; e < kGramRows2 * (kpad - w_in); e += kThreads)
                    sx[(e / (kpad - w_in)) * xs + w_in + e % (kpad - w_in)] = 0.f;        // (uniform widths: rarely)
        } else {
            for (int i = wv; i < kGramRows2; i += 4) {
                const bool in = i0 + i < len;
                const float* __restrict__ xrow = X.ptr + (int64_t)(in ? i0 + i : 0) * X.ld;
                for (int c = lane; c < kpad; c += 64) sx[i * xs + c] = (in && c < w_in) ? xrow[c] : 0.f;
            }
        }
        __syncthreads();
        if (flat_x && tile + (int)gridDim.x < n_tiles) load_x(tile + gridDim.x);
        // ---- wave v: rows 16 v .. 16 v + 15 of the tile (fp64 matrix cores).  All column tiles advance together along
        // the reduction index: one read of the row operand serves them all, and their accumulators are independent
        // chains (a tile by itself is a chain of dependent MFMAs, each behind two LDS reads).
        if constexpr (KP16 > 0) {
            const float* __restrict__ xa = sx + (16 * wv + li) * xs + lk;
            double a[4 * KP16];
#pragma unroll
            for (int ks = 0; ks < 4 * KP16; ++ks) a[ks] = (double)xa[4 * ks];
            doublex4 acc[KP16];
#pragma unroll
            for (int ct = 0; ct < KP16; ++ct) acc[ct] = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int ks = 0; ks < 4 * KP16; ++ks)
#pragma unroll
                for (int ct = ks / 4; ct < KP16; ++ct)
                    acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ks], tb[2 * ct * (ct + 1) + ks], acc[ct], 0, 0, 0);
#pragma unroll
            for (int ct = 0; ct < KP16; ++ct)
                if (ct < n_ct) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) so[(16 * wv + 4 * v + lk) * ow + 16 * ct + li] = (float)acc[ct][v];
                }
        } else {
            const float* __restrict__ xa = sx + (16 * wv + li) * xs + lk;
            const double* __restrict__ sb = tl + lk * kTmStride + li;
            doublex4 acc[kApplyStreamMaxWidth / 16];
#pragma unroll
            for (int ct = 0; ct < kApplyStreamMaxWidth / 16; ++ct) acc[ct] = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
            for (int k = 0; k < kpad; k += 4) {
                const double a = (double)xa[k];
#pragma unroll
                for (int ct = 0; ct < kApplyStreamMaxWidth / 16; ++ct)
                    if (ct < n_ct && k < tm_rows[ct])
                        acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, sb[(tm_off[ct] + k) * kTmStride], acc[ct], 0, 0, 0);
            }
#pragma unroll
            for (int ct = 0; ct < kApplyStreamMaxWidth / 16; ++ct)
                if (ct < n_ct) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) so[(16 * wv + 4 * v + lk) * ow + 16 * ct + li] = (float)acc[ct][v];
                }
        }
        __syncthreads();
        // ---- rows of the result
        const int rows_valid = min(len, i0 + kGramRows2) - i0;
        if (flat_y) {
            const int n_valid = rows_valid * w_out;
            PSGD_GLOBAL float* yp = as_global(Y.ptr) + (int64_t)i0 * Y.ld;
            for (int f = 4 * t; f < n_valid; f += 4 * kThreads) {
                int row = (int)(((float)f + 0.5f) * inv_wo);
                int c = f - row * w_out;
                if (c < 0) { --row; c += w_out; } else if (c >= w_out) { ++row; c -= w_out; }
                const float* __restrict__ sr = so + row * ow + c;
                *reinterpret_cast<PSGD_GLOBAL floatx4*>(yp + f) = floatx4{sr[0], sr[1], sr[2], sr[3]};
            }
        } else {
            for (int i = wv; i < rows_valid; i += 4) {
                float* __restrict__ yr = Y.ptr + (int64_t)(i0 + i) * Y.ld;
                for (int c = lane; c < w_out; c += 64) yr[c] = so[i * ow + c];
            }
        }
        if (do_gram) gram_tile_f64(so, ow, kGramRows2, w_out, L.gram + (int64_t)tile * ((w_out * (w_out + 1)) / 2));
        else if (do_pack) write_packs(L.pack[side], L.planes, so, ow, cp, i0, kGramRows2, lenP, which & 3, (which & 4) ? L.lzf[side] : nullptr);
        __syncthreads();
    }
}

// --------------------------------------------------------------------------------------------
// The same product for blocks wider than the streaming kernel's.  Their tmat (205 KB at width 160) fits neither registers nor
// LDS; staged 32 columns at a time behind barriers on four waves per 64 rows, with 128 tiles of 64 rows (8192 x 128), that
// chain of round trips was all of 45 us.  Here sixteen waves share a tile: wave (row group, column
// group) walks every fourth 16-column tile of the result along the reduction index with the fragments of tmat loaded
// straight from L2, four steps ahead.
// --------------------------------------------------------------------------------------------
// PARTS: a workgroup that leaves a partial Gram matrix takes PARTS tiles of ROWS rows for it, kGramRows2 in all.  The second
// factorisation is one workgroup, which adds these matrices up: 256 of 32 rows took it 522 us at 8192 x 128, 128 of 64 rows 285.
constexpr int kApplyWideThreads = 1024;
template <int ROWS, int PARTS>
__global__ __launch_bounds__(kApplyWideThreads) void apply_wide_kernel(const LayerDev* __restrict__ layers,
                                                                       const int* __restrict__ ids, int src_role,
                                                                       int dst_role, int mode, int cp, int gate, int w_in_max,
                                                                       int w_out_max, int which) {
    const LayerDev& L = layers[ids[blockIdx.y]];
    if (!gate_open(L, gate)) return;
    if (blockIdx.z != 0) {
        src_role = ROLE_ZQ;
        dst_role = ROLE_Q;
    }
    const int need2 = L.status[1];
    if (mode == APPLY_PASS2 && !need2) return;
    const bool do_gram = (mode == APPLY_PASS1) && need2;
    const bool do_pack = !do_gram && cp > 0;
    const int side = side_of_role(L.transposed, src_role);
    const int len = side_len(L, side), lenP = side_lenP(L, side);
    const int i0 = blockIdx.x * ROWS;
    if (i0 >= (do_pack ? lenP : len)) return;
    if (PARTS > 1 && do_gram && blockIdx.x % PARTS != 0) return;       // (the workgroup of the first of these rows takes them all)
    const int parts = PARTS > 1 && do_gram ? PARTS : 1;
    const ThinRef X = L.thin[src_role];
    const ThinRef Y = L.thin[dst_role];
    const int w_in = X.width, w_out = Y.width;
    const bool upper = mode != APPLY_RITZ;
    const int kpad = (w_in + 15) & ~15, n_ct = (w_out + 15) / 16;
    const int xs = ((w_in_max + 15) & ~15) + 1;
    const int wo16 = (w_out_max + 15) & ~15, ow = (cp > wo16 ? cp : wo16) + 1;
    extern __shared__ __align__(16) unsigned char smem[];
    float* sx = reinterpret_cast<float*>(smem);            // [ROWS][xs]  x tile, zero beyond the matrix
    float* so = sx + (size_t)ROWS * xs;                    // [PARTS ROWS][ow]  result tile, zero beyond w_out
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, li = lane & 15, lk = lane >> 4;
    constexpr int RG = ROWS / 16, CG = kApplyWideThreads / 64 / RG;
    const int rg = wv % RG, cg = wv / RG;
    const float* __restrict__ xa = sx + (16 * rg + li) * xs + lk;
    const PSGD_GLOBAL double* __restrict__ tm = as_global(L.tmat);
    for (int part = 0; part < parts; ++part) {
        const int p0 = i0 + part * ROWS;
        float* po = so + (size_t)(part * ROWS) * ow;
        if (part > 0) __syncthreads();                     // (the x tile has been read)
        for (int i = wv; i < ROWS; i += kApplyWideThreads / 64) {
            const bool in = p0 + i < len;
            const PSGD_GLOBAL float* xr = as_global(X.ptr) + (int64_t)(in ? p0 + i : 0) * X.ld;
            for (int c = lane; c < kpad; c += 64) sx[i * xs + c] = (in && c < w_in) ? xr[c] : 0.f;
            for (int c = lane; c < ow; c += 64) po[i * ow + c] = 0.f;
        }
        __syncthreads();
        for (int ct = cg; ct < n_ct; ct += CG) {
            const int col = 16 * ct + li;
            const int kend = upper ? min(kpad, 16 * (ct + 1)) : kpad;
            const bool col_ok = col < w_in;
            auto frag = [&](int k) {                           // (k + lk may pass the end: that row counts as zero)
                const bool ok = col_ok && k + lk < w_in;
                const double v = tm[ok ? (int64_t)(k + lk) * w_in + col : 0];
                return ok ? v : 0.0;
            };
            doublex4 acc = {0.0, 0.0, 0.0, 0.0};
            double b[4], bn[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) b[u] = frag(4 * u);
            for (int k = 0; k < kend; k += 16) {
#pragma unroll
                for (int u = 0; u < 4; ++u) bn[u] = frag(k + 16 + 4 * u);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)xa[k + 4 * u], b[u], acc, 0, 0, 0);
#pragma unroll
                for (int u = 0; u < 4; ++u) b[u] = bn[u];
            }
            if (col < w_out) {
#pragma unroll
                for (int v = 0; v < 4; ++v) po[(16 * rg + 4 * v + lk) * ow + col] = (float)acc[v];
            }
        }
    }
    __syncthreads();
    const int rows_valid = min(len, i0 + parts * ROWS) - i0;
    for (int i = wv; i < rows_valid; i += kApplyWideThreads / 64) {
        PSGD_GLOBAL float* yr = as_global(Y.ptr) + (int64_t)(i0 + i) * Y.ld;
        for (int c = lane; c < w_out; c += 64) yr[c] = so[i * ow + c];
    }
    if (do_gram) gram_tile_f64(so, ow, PARTS * ROWS, w_out, L.gram + (int64_t)(blockIdx.x / PARTS) * ((w_out * (w_out + 1)) / 2));
    else if (do_pack) write_packs<0, kApplyWideThreads>(L.pack[side], L.planes, so, ow, cp, i0, ROWS, lenP, which & 3, (which & 4) ? L.lzf[side] : nullptr);
}

// Rows per workgroup of apply_wide_kernel: 32 where 64 leave compute units idle, up to one workgroup of 64 per unit (kernel, 8192 x 160
// 24 -> 16 us, 8192 x 128 20 -> 14; step of 4096 x 4096 bf16 r = 128 218 -> 212 us).  With more tiles its reads of tmat are what grows,
// and what is left is within 1 % either way: 20000 x 2048 r = 100 534 and, on 32 rows, 531 us, refreshes of three 8192 x 4096
// r = 128 2739 and 2707, of fourteen 2048 x 2048 r = 110 2458 and 2469.  Where the launch may leave Gram matrices, up to half of
// that: beyond, the workgroups that leave them are more than half the units and twice as long (16384 x 2048 r = 100, 256 tiles: step
// 346 either way, 663 and 688 where its second pass is asked for).
static int apply_rows(int max_lenP, int n_ids, int mode) {
    return (max_lenP / kGramRows2) * n_ids <= (mode == APPLY_PASS1 ? 128 : 256) ? 32 : kGramRows2;
}

// w_in / w_out: upper bounds of the operand widths over the addressed layers (LDS sizing only)
// small: every layer of the launch is narrow (w_in <= 16) and the chain runs the per-workgroup factorisation
// mode APPLY_RITZ: ROLE_ZP -> ROLE_P, and in the same launch (z = 1) ROLE_ZQ -> ROLE_Q, which shares nothing with it but tmat
// (as two launches: 9 us more per refresh of 256 x 128 r = 4, 12 of 4096 x 4096 r = 8)
// stream_wgs: workgroups per layer of apply_stream_kernel above width 64 (see one_round; 0: as below)
// slot_rows: rows per partial Gram matrix that the first pass's per-workgroup factorisation adds up in the row-major layers
// (the others: 128)
// which: operand copies to leave when cp > 0 (1 = outer-product, 2 = transposed, 3 = both; + 4: the outer-product ones are
// the layer's kept copies where it has them -- the P~ of a compress step with a deferred residual)
hipError_t launch_apply(const LayerDev* layers, const int* ids, int n_ids, int max_lenP, int w_in, int w_out,
                        int src_role, int dst_role, int mode, int cp, int gate, int a2gate, double tol2,
                        bool small, int which, int slot_rows, int stream_wgs, hipStream_t st) {
    if (n_ids <= 0) return hipSuccess;
    if (w_out > w_in || (small && (w_in > kCholRegWidth || w_out != w_in || src_role != dst_role || mode == APPLY_RITZ))) return hipErrorInvalidValue;
    const int n_sides = mode == APPLY_RITZ ? 2 : 1;
    dim3 grid(max_lenP / kGramRows2, n_ids), block(kThreads);
    if (!small && w_in <= kApplyStreamMaxWidth) {
        // (triangular tmat up to width 80: its fragments fit the registers)
        const int kp16 = (mode != APPLY_RITZ && w_in <= 80) ? (w_in + 15) / 16 : 0;
        // a few rounds of workgroups over the whole launch, each walking several tiles of its layer
        // (config 4, width 64: 0.54 ms with one round of 512 workgroups, 0.43 with four, 0.42 with eight, 0.45 with 16)
        // Above width 64 one round where the caller has counted it out (see one_round; at width 40 in bf16 5018 us and 5053)
        int per_layer = w_in > 64 && stream_wgs > 0 ? stream_wgs : (8 * 512 + n_ids - 1) / n_ids;
        if (per_layer > (int)grid.x) per_layer = grid.x;
        if (per_layer < 1) per_layer = 1;
        const size_t lds = apply_stream_lds(w_in, w_out, cp, mode != APPLY_RITZ, kp16);
        // (widths up to 16 are the `small` chain's: kp16 >= 2 here)
        auto kfn = kp16 == 2 ? apply_stream_kernel<2> : kp16 == 3 ? apply_stream_kernel<3>
                 : kp16 == 4 ? apply_stream_kernel<4> : kp16 == 5 ? apply_stream_kernel<5> : apply_stream_kernel<0>;
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kfn, dim3(per_layer, n_ids, n_sides), block, lds, st, layers, ids, src_role, dst_role,
                           mode, cp, gate, w_out, which);
        return hipGetLastError();
    }
    if (!small) {
        const int wi16 = (w_in + 15) & ~15, wo16 = (w_out + 15) & ~15;
        const int rows = apply_rows(max_lenP, n_ids, mode), rows_out = mode == APPLY_PASS1 ? kGramRows2 : rows;
        const size_t lds = ((size_t)rows * (wi16 + 1) + (size_t)rows_out * ((cp > wo16 ? cp : wo16) + 1)) * sizeof(float);
        auto kfn = rows == kGramRows2 ? apply_wide_kernel<kGramRows2, 1>
                 : mode == APPLY_PASS1 ? apply_wide_kernel<32, kGramRows2 / 32> : apply_wide_kernel<32, 1>;
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kfn, dim3(max_lenP / rows, n_ids, n_sides), dim3(kApplyWideThreads), lds, st, layers, ids, src_role, dst_role, mode, cp,
                           gate, w_in, w_out, which);
        return hipGetLastError();
    }
    // (w_in: upper bound over the layers, every size here grows with it)
    size_t lds = apply_main_lds(w_in, cp);
    if (mode == APPLY_PASS1 || mode == APPLY_PASS1_ONLY) {
        if (chol_lds_bytes_upto(w_in) > lds) lds = chol_lds_bytes_upto(w_in);           // second-pass factorisation
        lds += (size_t)w_in * w_in * sizeof(double) + chol_lds_bytes_upto(w_in);        // per-workgroup factorisation
    }
    auto kfn = gate >= 0 ? apply_kernel<true> : apply_kernel<false>;
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kfn, grid, block, lds, st, layers, ids, src_role, mode, cp, gate, a2gate, tol2, which, slot_rows);
    return hipGetLastError();
}

// --------------------------------------------------------------------------------------------
// start block of the subspace iteration: columns [0, n_copy) from thin[src_role] (warm start), the others from start_value.
// --------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void init_block_kernel(const LayerDev* __restrict__ layers,
                                                              const int* __restrict__ ids, int dst_role,
                                                              int src_role, int warm, uint32_t seed) {
    const int lid = ids[blockIdx.y];
    const LayerDev& L = layers[lid];
    const int side = side_of_role(L.transposed, dst_role);
    const int len = side_len(L, side);
    const ThinRef Y = L.thin[dst_role];
    const ThinRef X = L.thin[src_role];
    const int n_copy = warm ? min(X.width, Y.width) : 0;
    const int64_t total = (int64_t)len * Y.width;
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < total; e += (int64_t)gridDim.x * kThreads) {
        const int i = (int)(e / Y.width), c = (int)(e % Y.width);
        float v;
        if (c < n_copy) {
            v = X.ptr[(int64_t)i * X.ld + c];
        } else {
            v = start_value(seed, lid, i, c);
        }
        Y.ptr[(int64_t)i * Y.ld + c] = v;
    }
}

hipError_t launch_init_block(const LayerDev* layers, const int* ids, int n_ids, int max_len, int w, int dst_role,
                             int src_role, int warm, uint32_t seed, hipStream_t st) {
    if (n_ids <= 0) return hipSuccess;
    const int64_t total = (int64_t)max_len * w;
    int gx = (int)((total + kThreads * 4 - 1) / (kThreads * 4));
    if (gx < 1) gx = 1;
    dim3 grid(gx, n_ids), block(kThreads);
    hipLaunchKernelGGL(init_block_kernel, grid, block, 0, st, layers, ids, dst_role, src_role, warm, seed);
    return hipGetLastError();
}

// --------------------------------------------------------------------------------------------
// Rayleigh-Ritz: eigen-decomposition of the w x w Gram matrix H = Y^T Y (Y = M^T Z, Z orthonormal)
// by cyclic two-sided Jacobi in fp64: jacobi_block_kernel up to width 160, jacobi_kernel above, with H and a slice of the accumulated
// rotations V in LDS.
// On exit tmat[:, k] is the eigenvector of the k-th largest eigenvalue, so that P~ = Z tmat[:, :r] are
// the leading left singular vectors (Definition 3) and Q = Y tmat[:, :r] = M^T P~.  status gets
// sigma_1 and sigma_r = sqrt(eigenvalue), and the iteration count the next refresh needs.
// --------------------------------------------------------------------------------------------
constexpr int kJacobiMaxSweeps = 30;

// Storage of the symmetric matrix H of even order n in LDS: n rows of S doubles, S the odd one of n / 2 + 1 and
// n / 2 + 2; entry (i, j) lives in row i at column d = (j - i) mod n if d <= n / 2 (for d = n / 2 in the row of the
// smaller index), otherwise it is entry (j, i) of row j.  About as many doubles as a packed triangle.  The lanes
// of a rotation step hold neighbouring rotation pairs at a fixed distance, so the entries they touch together
// move along a diagonal: by +-1 in both indices (address stride S) or by +1 and -1 (stride S - 2).  Both are
// odd, so 32 lanes reading doubles fall on 32 different even banks; the packed triangle's strides vary with the
// row and collide.
__host__ __device__ inline int sym_stride(int n) { return (n / 2 + 1) | 1; }
__device__ inline int sym_idx(int i, int j, int n) {
    int d = j - i;
    d += d < 0 ? n : 0;
    const bool own = 2 * d < n || (2 * d == n && i < j);
    return own ? __mul24(i, sym_stride(n)) + d : __mul24(j, sym_stride(n)) + (n - d);      // (24-bit multiply: full rate)
}

// The round-robin tournament on n players (n even): n / 2 slots, slot k pairs the players at positions 2k ("top")
// and 2k + 1 ("bottom").  Position 0 keeps its player; after every round the others move one place round the ring
// top[1] -> bottom[0] -> bottom[1] -> ... -> bottom[n/2 - 1] -> top[n/2 - 1] -> ... -> top[2] -> top[1].
// In round rd the players (matrix indices) in slot k are
//   top: n - 1 for k = 0, else (rd + k) mod (n - 1);   bottom: (rd - k) mod (n - 1),
// and after n - 1 rounds everybody is back where round 0 had them.
__device__ inline int jacobi_next_pos(int x, int n) {
    const int half = n / 2, k = x >> 1;
    if (x == 0 || n <= 2) return x;
    if ((x & 1) == 0) return k == 1 ? 1 : x - 2;            // top[k] -> top[k - 1], top[1] -> bottom[0]
    return k == half - 1 ? n - 2 : x + 2;                   // bottom[k] -> bottom[k + 1], the last one -> top[half - 1]
}
__device__ inline int jacobi_top(int k, int rd, int n) {
    if (k == 0) return n - 1;
    const int p = rd + k;
    return p >= n - 1 ? p - (n - 1) : p;
}
__device__ inline int jacobi_bottom(int k, int rd, int n) {
    const int q = rd - k;
    return q < 0 ? q + (n - 1) : q;
}
// position in round 0 of matrix index j (inverse of jacobi_top / jacobi_bottom at rd = 0)
__device__ inline int jacobi_pos0(int j, int n) {
    const int half = n / 2;
    if (j == n - 1) return 0;
    if (j == 0) return 1;
    return j < half ? 2 * j : 2 * (n - 1 - j) + 1;
}

// Rotation that annihilates apq of a 2 x 2 diagonal block: the half of the angle whose cosine and sine are |d| / h and b / h, d =
// aqq - app, b = 2 apq, h^2 = d^2 + b^2, so (c, s) is (1 + |d| / h, +-b / h) normalised.
__device__ inline void jacobi_angle(double app, double apq, double aqq, double& c, double& sn) {
    const bool turns = fabs(apq) > 1e-150 && apq * apq > 1e-36 * fabs(app * aqq);
    const double d = aqq - app, b = 2.0 * apq;
    const double ih = rsqrt_nr(turns ? __builtin_fma(d, d, b * b) : 1.0);     // (of a normal number, by the test above)
    const double x = turns ? __builtin_fma(fabs(d), ih, 1.0) : 1.0;
    const double y = turns ? (d >= 0.0 ? b : -b) * ih : 0.0;
    const double in = rsqrt_nr(__builtin_fma(x, x, y * y));
    c = x * in;
    sn = y * in;
}
// J^T A J for the off-diagonal block (slot k1) x (slot k2) ...
__device__ inline void jacobi_rotate(double c1, double s1, double c2, double s2, double app, double apq, double aqp, double aqq, double (&o)[4]) {
    // rows: (top, bottom) <- (c1 top - s1 bottom, s1 top + c1 bottom)
    const double rpp = c1 * app - s1 * aqp, rpq = c1 * apq - s1 * aqq;
    const double rqp = s1 * app + c1 * aqp, rqq = s1 * apq + c1 * aqq;
    // columns: likewise with slot k2's rotation
    o[0] = c2 * rpp - s2 * rpq;
    o[1] = s2 * rpp + c2 * rpq;
    o[2] = c2 * rqp - s2 * rqq;
    o[3] = s2 * rqp + c2 * rqq;
}
// ... and for a diagonal one (upper part)
__device__ inline void jacobi_rotate_diag(double c, double s, double app, double apq, double aqq, double& opp, double& opq, double& oqq) {
    opp = c * c * app - 2.0 * c * s * apq + s * s * aqq;
    opq = (c * c - s * s) * apq + c * s * (app - aqq);
    oqq = s * s * app + 2.0 * c * s * apq + c * c * aqq;
}
__device__ inline void jacobi_note(double c, double sn, int n, int rd, int k, double* cs, int* pq) {
    const int half = n / 2;
    cs[k] = c; cs[half + k] = sn;
    pq[k] = jacobi_top(k, rd, n); pq[half + k] = jacobi_bottom(k, rd, n);      // the columns of V the slot holds in round rd
}
// Slot k's rotation of round rd from the H of that round (stored by position)
__device__ inline void jacobi_rotation(const double* a, int n, int rd, int k, double* cs, int* pq) {
    double c, sn;
    jacobi_angle(a[sym_idx(2 * k, 2 * k, n)], a[sym_idx(2 * k, 2 * k + 1, n)], a[sym_idx(2 * k + 1, 2 * k + 1, n)], c, sn);
    jacobi_note(c, sn, n, rd, k, cs, pq);
}
// rank of eigenvalue j = number of eigenvalues that come before it (ties by index); eval (or null): the eigenvalues in that order
__device__ inline void ritz_ranks(const double* lam, int* rank_of, int w, double* eval) {
    for (int j = threadIdx.x; j < w; j += blockDim.x) {
        const double lj = lam[j];
        int rank = 0;
        for (int k = 0; k < w; ++k) {
            const double lk = lam[k];
            rank += (lk > lj || (lk == lj && k < j)) ? 1 : 0;
        }
        rank_of[j] = rank;
        if (eval) eval[rank] = lj;
    }
}
// What a refresh leaves in the layer's status words, from the Ritz values in L.eval; by the threads of one workgroup.
constexpr int kJacobiMaxWidth = 200;       // of jacobi_kernel: five 2 x 2 blocks per thread
__device__ inline void ritz_notes(const LayerDev& L, int w, int sweeps, float* sigma_out) {
    const int t = threadIdx.x, r = L.r;
    // Iterations for a cut without a gap (see refresh_iterations).  Where the count that the subspace needs is out of
    // reach, what is asked of the step is its error (Lemma 2 / Eq. (6): ||M - P~ P~^T M||^2 = sum_{i > r} sigma_i^2
    // at the optimum).  Direction i <= r of the block, still off by sin(theta_i) <= (theta_b / theta_i)^k after k
    // iterations from any start (theta: Ritz values = squared singular value estimates), costs at most
    // sin^2(theta_i) (theta_i - theta_b) on top of the optimum: the directions well above the cut cost nothing after
    // two iterations, the ones in the cluster at the cut have little to lose.  The count is the smallest k for which
    // the sum of these is below 1e-5 of ||M||^2 >= sum of the Ritz values: a tenth of the 1e-4 the step is held to,
    // because the Ritz values are those of the layer's previous refresh and error feedback has flattened the spectrum
    // further since (with 5e-5 the counts came out at 3 to 10 and left 1e-4 to 3e-4).
    // Measured on 7B-shaped bf16 layers (sigma_{b+1} / sigma_r = 0.98): after 3 steps of error feedback 2 iterations
    // leave 3e-6 ||M||^2; after 60 steps, with ||E|| = 0.3 ||M||, 4 leave 1.8e-4, 8 leave 5.8e-5, 16 leave 1.5e-5.
    // (one wave, in a fixed order; the powers by a product per count, as pow() takes a microsecond of the chain for each)
    int ke = 255;
    if (t < 64) {
        constexpr int kEach = (kJacobiMaxWidth + 63) / 64;
        const double lb = w > r ? L.eval[w - 1] : 0.0;
        double tr = 0.0, term[kEach], rho2[kEach];
#pragma unroll
        for (int u = 0; u < kEach; ++u) {
            const int i = t + 64 * u;
            const double li = i < w ? L.eval[i] : 0.0;
            tr += fmax(li, 0.0);
            const bool counts = i < r && lb > 0.0 && li > lb;
            const double rho = counts ? lb / li : 0.0;
            rho2[u] = rho * rho;
            term[u] = counts ? rho2[u] * rho2[u] * (li - lb) : 0.0;
        }
        for (int o = 32; o > 0; o >>= 1) tr += __shfl_xor(tr, o);
        for (int k = 2; k <= 64; ++k) {
            double part = 0.0;
#pragma unroll
            for (int u = 0; u < kEach; ++u) part += term[u];
            for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o);
            if (part <= 1e-5 * tr) {
                ke = k;
                break;
            }
#pragma unroll
            for (int u = 0; u < kEach; ++u) term[u] *= rho2[u];
        }
    }
    for (int k = t; k < r; k += blockDim.x) {
        const float sg = (float)sqrt(fmax(L.eval[k], 0.0));
        if (sigma_out) sigma_out[k] = sg;
        if (k == 0) L.status[2] = __float_as_int(sg);
        if (k == r - 1) L.status[3] = __float_as_int(sg);
    }
    if (t == 0) {
        // The iteration contracts the error of the leading r-dimensional subspace by about
        // rho = theta_b / theta_r per step (theta = Ritz values, the smallest one of the block standing
        // in for sigma_{b+1}^2); the next refresh of this layer needs as many steps as 1e-5 takes (a tenth of
        // the 1e-4 bar on the subspace), plus one.  (Error feedback drives M towards rho = 1: what is not
        // sent accumulates in E until it is as large as what is.  The launches cap the count, see gate_open.)
        int k_next = 255;
        const double lr = L.eval[r - 1], lb = L.eval[w - 1];
        if (w > r && lr > 0.0 && lb >= 0.0) {
            const double rho = lb / lr;
            if (rho < 0.999) k_next = (rho <= 1e-12) ? 2 : (int)ceil(log(1e-5) / log(rho)) + 1;
        }
        L.status[4] = max(2, min(255, k_next));
        L.status[9] = ke;
        L.status[11] = 0;
        L.status[5] = sweeps;
        L.status[8] = min(L.status[8] + 1, 1 << 20);
    }
}

// Widths above kJacobiBlockWidth, round-robin ordering with w/2 disjoint rotations per round.
// grid = (slices, layers): every workgroup of a layer repeats the (deterministic) iteration on H and
// accumulates the rotations into its own slice of v_rows rows of V, which is independent of the other rows.
//
// H is stored by POSITION in the tournament, not by matrix index: the 2 x 2 block (slot k1) x (slot k2) sits at
// the same LDS addresses in every round, is rotated by the two slots' rotations, and its four entries are written
// to where the tournament moves their row and column players.  Source and destination addresses of a thread's
// blocks are therefore computed once.  A round:
//   read and rotate | barrier | write | barrier | the next round's rotations from the new diagonal blocks, while the other
//   waves run V <- V J | barrier
// V stays indexed by matrix index.
// NBLK: 2 x 2 blocks of H per thread, at least (w/2)(w/2 + 1)/2 over the workgroup.
template <int NBLK>
__global__ __launch_bounds__(1024) void jacobi_kernel(const LayerDev* __restrict__ layers,
                                                      const int* __restrict__ ids, int role, int v_rows,
                                                      int slot_rows, float* __restrict__ sigma_out) {
    const LayerDev& L = layers[ids[blockIdx.y]];
    const int w = L.thin[role].width;
    const int n_slots = (side_len(L, side_of_role(L.transposed, role)) + slot_rows - 1) / slot_rows;
    const int n = (w + 1) & ~1;      // even size for the round-robin schedule (a zero row/column is added)
    const int half = n / 2;
    const int row0 = blockIdx.x * v_rows;
    const int nv = min(v_rows, n - row0);              // rows of V kept by this workgroup
    extern __shared__ __align__(16) unsigned char smem[];
    double* csb = reinterpret_cast<double*>(smem);     // two buffers of [half] cos, [half] sin
    double* red = csb + 2 * n;                         // [2][16] per-wave partial sums of the convergence test
    double* a = red + 32;                              // H, n rows of sym_stride(n) (see sym_idx)
    double* v = a + n * sym_stride(n);                 // v_rows x n slice of the accumulated rotations
    int* pqb = reinterpret_cast<int*>(v + v_rows * n); // two buffers of [half] top, [half] bottom matrix indices
    const int t = threadIdx.x;
    const int nt = blockDim.x;
    const int txw = nt >= 512 ? 32 : 16, tyw = nt / txw;   // threads as a tyw x txw grid: no integer division
    const int tx = t & (txw - 1), ty = t / txw;
    // H = sum of the partial Gram matrices (upper triangle) left by the last product's epilogue, entry
    // (position x, position y) = H of the matrix indices that round 0 puts there
    const int ntri = (w * (w + 1)) / 2;
    for (int x = ty; x < n; x += tyw) {
        const int k = x >> 1, i = (x & 1) ? jacobi_bottom(k, 0, n) : jacobi_top(k, 0, n);
        for (int y = x + tx; y < n; y += txw) {
            const int ky = y >> 1, j = (y & 1) ? jacobi_bottom(ky, 0, n) : jacobi_top(ky, 0, n);
            double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
            if (i < w && j < w) {
                const double* g = L.gram + tri_idx(min(i, j), max(i, j), w);
                int sp = 0;
                for (; sp + 4 <= n_slots; sp += 4) {
                    s0 += g[(int64_t)sp * ntri]; s1 += g[(int64_t)(sp + 1) * ntri];
                    s2 += g[(int64_t)(sp + 2) * ntri]; s3 += g[(int64_t)(sp + 3) * ntri];
                }
                for (; sp < n_slots; ++sp) s0 += g[(int64_t)sp * ntri];
            }
            a[sym_idx(x, y, n)] = (s0 + s1) + (s2 + s3);
        }
    }
    for (int i = ty; i < nv; i += tyw)
        for (int j = tx; j < n; j += txw) v[i * n + j] = (row0 + i == j) ? 1.0 : 0.0;
    // The unordered pairs {k1, k2} of slots (k1 = k2 included), i.e. the 2 x 2 blocks of H that hold one stored
    // copy each, dealt evenly to the threads once: block e is k1 = e mod half, k2 = k1 + e / half (mod half); the
    // distances e / half = 0 .. half / 2 reach every pair once (the last distance, for even half, only from the
    // lower k1).  Per entry: source address | destination address << 16 (both below 2^16 doubles).
    int bk[NBLK], n_blk = 0;                                   // k1 | k2 << 8
    unsigned adr[NBLK][4];
    {
        const int total = (half * (half + 1)) / 2;
#pragma unroll
        for (int b = 0; b < NBLK; ++b) {
            const int e = t + b * nt;
            bk[b] = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) adr[b][q] = 0;
            if (e < total) {
                const int dk = e / half, k1 = e - dk * half;
                int k2 = k1 + dk;
                k2 -= k2 >= half ? half : 0;
                bk[b] = k1 | (k2 << 8);
                n_blk = b + 1;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    // entry q of the block: row 2 k1 + (q >> 1), column 2 k2 + (q & 1); a diagonal block's entry 2
                    // (bottom, top) is the stored entry 1 again and is left out when the block is written
                    const int x = 2 * k1 + (q >> 1), y = 2 * k2 + (q & 1);
                    adr[b][q] = (unsigned)sym_idx(x, y, n) |
                                ((unsigned)sym_idx(jacobi_next_pos(x, n), jacobi_next_pos(y, n), n) << 16);
                }
            }
        }
    }
    __syncthreads();
    int cur = 0, sweeps = 0;
    for (int sweep = 0; sweep < kJacobiMaxSweeps; ++sweep) {
        // convergence: off-diagonal mass relative to the diagonal.  The per-wave partial sums are added in wave order
        // by every thread for itself: the same bits in every thread and in every workgroup of the layer, whose
        // slices of V only fit together if all of them run the same number of sweeps.
        double off = 0.0, dia = 0.0;
        for (int i = ty; i < n; i += tyw)
            for (int j = i + tx; j < n; j += txw) {
                const double x = a[sym_idx(i, j, n)];
                if (i == j) dia += x * x; else off += 2.0 * x * x;
            }
        for (int o = 32; o > 0; o >>= 1) { off += __shfl_down(off, o); dia += __shfl_down(dia, o); }
        if ((t & 63) == 0) { red[t >> 6] = off; red[16 + (t >> 6)] = dia; }
        __syncthreads();
        double off_all = 0.0, dia_all = 0.0;
        for (int wq = 0; wq < (nt >> 6); ++wq) { off_all += red[wq]; dia_all += red[16 + wq]; }
        const bool done = off_all <= 1e-20 * dia_all;
        if (done) break;
        sweeps = sweep + 1;
        if (t < half) jacobi_rotation(a, n, 0, t, csb + cur * n, pqb + cur * n);
        __syncthreads();
        for (int rd = 0; rd < n - 1; ++rd) {
            const double* cs = csb + cur * n;
            const int* pq = pqb + cur * n;
            // H <- J^T H J on this thread's blocks: rows by slot k1's rotation, columns by slot k2's
            double o[NBLK][4];
#pragma unroll
            for (int b = 0; b < NBLK; ++b) {
                if (b >= n_blk) break;
                const int k1 = bk[b] & 0xff, k2 = bk[b] >> 8;
                const double c1 = cs[k1], s1 = cs[half + k1];
                const double app = a[adr[b][0] & 0xffffu], apq = a[adr[b][1] & 0xffffu];
                const double aqp = a[adr[b][2] & 0xffffu], aqq = a[adr[b][3] & 0xffffu];
                if (k1 == k2) {
                    // (aqp is apq here)
                    jacobi_rotate_diag(c1, s1, app, apq, aqq, o[b][0], o[b][1], o[b][3]);
                    o[b][2] = 0.0;
                } else {
                    jacobi_rotate(c1, s1, cs[k2], cs[half + k2], app, apq, aqp, aqq, o[b]);
                }
            }
            __syncthreads();
#pragma unroll
            for (int b = 0; b < NBLK; ++b) {
                if (b >= n_blk) break;
                const bool diag = (bk[b] & 0xff) == (bk[b] >> 8);
                a[adr[b][0] >> 16] = o[b][0];
                a[adr[b][1] >> 16] = o[b][1];
                if (!diag) a[adr[b][2] >> 16] = o[b][2];
                a[adr[b][3] >> 16] = o[b][3];
            }
            __syncthreads();
            if (rd + 1 < n - 1 && t < half) jacobi_rotation(a, n, rd + 1, t, csb + (cur ^ 1) * n, pqb + (cur ^ 1) * n);
            for (int i = ty; i < nv; i += tyw)
                for (int k = tx; k < half; k += txw) {
                    const int p = pq[k], q = pq[half + k];
                    const double c = cs[k], sn = cs[half + k];
                    const double vx = v[i * n + p], vy = v[i * n + q];
                    v[i * n + p] = c * vx - sn * vy;
                    v[i * n + q] = sn * vx + c * vy;
                }
            __syncthreads();
            cur ^= 1;
        }
    }
    __syncthreads();
    // eigenvalue of matrix index j (= column j of V): the diagonal entry at the position round 0 gives j, where
    // every sweep ends
    double* lam = csb;                                 // [n], the rotation buffers are free now
    for (int j = t; j < n; j += nt) { const int x = jacobi_pos0(j, n); lam[j] = a[sym_idx(x, x, n)]; }
    __syncthreads();
    int* rank_of = pqb;                                // (2 n entries available)
    double* __restrict__ tm = L.tmat;
    ritz_ranks(lam, rank_of, w, blockIdx.x == 0 ? L.eval : nullptr);
    __syncthreads();
    for (int i = ty; i < nv; i += tyw)
        if (row0 + i < w)
            for (int j = tx; j < w; j += txw) tm[(int64_t)(row0 + i) * w + rank_of[j]] = v[i * n + j];
    if (blockIdx.x == 0) ritz_notes(L, w, sweeps, sigma_out);
}

// v of lane (lane ^ 2^B), B < 3, and of lane (lane ^ 8 * 2^B): moves on the data path, no LDS
template <int CTRL> __device__ __forceinline__ double dpp_move(double v) {
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true),
                            __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true));
}
template <int B> __device__ __forceinline__ double from_column(double v) {
    if constexpr (B == 0) return dpp_move<0xb1>(v);                   // quad_perm 1 0 3 2
    else if constexpr (B == 1) return dpp_move<0x4e>(v);              // quad_perm 2 3 0 1
    else return dpp_move<0x1b>(dpp_move<0x141>(v));                   // half rows mirrored (^ 7), quad_perm 3 2 1 0 (^ 3)
}
template <int B> __device__ __forceinline__ int swapped_rows(int v) {
    // (the first result has each upper row replaced by the lower one, the second each lower row by the upper one)
    if constexpr (B == 1) {
        const auto x = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return threadIdx.x & 16 ? x[0] : x[1];
    } else {
        const auto x = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return threadIdx.x & 32 ? x[0] : x[1];
    }
}
template <int B> __device__ __forceinline__ double from_row(double v) {
    if constexpr (B == 0) return dpp_move<0x128>(v);                  // row_ror 8
    else return __hiloint2double(swapped_rows<B>(__double2hiint(v)), swapped_rows<B>(__double2loint(v)));
}
__device__ __forceinline__ double from_lane(int byte_address, double v) {
    return __hiloint2double(__builtin_amdgcn_ds_bpermute(byte_address, __double2hiint(v)),
                            __builtin_amdgcn_ds_bpermute(byte_address, __double2loint(v)));
}

// ---- Jacobi on 8 x 8 blocks, widths up to kJacobiBlockWidth.
// One wave works on the 16 indices of a pair of blocks (a 16 x 16 part of H) in registers: lane (k1, k2) holds the 2 x 2 block
// (slot k1) x (slot k2), and rows k1 and k1 + 8 of slot k2's columns of the part's accumulated rotations.  A phase pairs the indices that
// differ in bit `split` and below: slot k holds the index with that bit 0 and the k-th other bits, and the one with that bit 1 and
// the k ^ g-th; the 2^split rounds run g through a Gray code, so that between rounds one bit of k changes.  Split 3: the pairs
// across the two blocks, 2, 1 and 0: those inside both.
constexpr int kJacobiBlockWidth = 160;
__device__ inline int block_at(int I, int K) { return ((K * (K + 1)) / 2 + I) * 64; }     // I <= K
// entry of a block; the columns of a row are permuted so that neither rows nor columns meet on a bank
__device__ inline int in_block(int i, int k) { return 8 * i + (k ^ i); }
// entry (e, f) of the pair's 16 x 16 part, p < q
__device__ inline int in_pair(int e, int f, int pp, int pq, int qq) {
    const int i = e & 7, k = f & 7;
    return (e ^ f) & 8 ? pq + (e & 8 ? in_block(k, i) : in_block(i, k)) : (e & 8 ? qq : pp) + in_block(i, k);
}
// h: blocks of H, jac: 16 x 16 rotations of this pair, row by row
template <int SPLIT>
__device__ __forceinline__ void jacobi_phase(double* h, double* jac, int pp, int pq, int qq, bool first) {
    constexpr int low = (1 << SPLIT) - 1;
    const int lane = threadIdx.x & 63, k1 = lane >> 3, k2 = lane & 7;
    const int e0 = (k1 & low) | ((k1 & ~low) << 1), e1 = e0 | (1 << SPLIT);
    const int f0 = (k2 & low) | ((k2 & ~low) << 1), f1 = f0 | (1 << SPLIT);
    const int from1 = 4 * 9 * k1, from2 = 4 * 9 * k2;
    double x[4] = {h[in_pair(e0, f0, pp, pq, qq)], h[in_pair(e0, f1, pp, pq, qq)], h[in_pair(e1, f0, pp, pq, qq)], h[in_pair(e1, f1, pp, pq, qq)]};
    double u0, u1, v0, v1;
    if (first) {
        u0 = k1 == f0 ? 1.0 : 0.0; u1 = k1 == f1 ? 1.0 : 0.0;
        v0 = k1 + 8 == f0 ? 1.0 : 0.0; v1 = k1 + 8 == f1 ? 1.0 : 0.0;
    } else {
        u0 = jac[16 * k1 + f0]; u1 = jac[16 * k1 + f1];
        v0 = jac[16 * k1 + 128 + f0]; v1 = jac[16 * k1 + 128 + f1];
    }
    static_for<0, low + 1>([&](auto round) {
        constexpr int rd = decltype(round)::value;
        double c, s, o[4];
        jacobi_angle(x[0], x[1], x[3], c, s);                         // (of use on lanes k1 = k2)
        const double c1 = from_lane(from1, c), s1 = from_lane(from1, s), c2 = from_lane(from2, c), s2 = from_lane(from2, s);
        jacobi_rotate(c1, s1, c2, s2, x[0], x[1], x[2], x[3], o);
        const double t0 = c2 * u0 - s2 * u1, t1 = c2 * v0 - s2 * v1;
        u1 = s2 * u0 + c2 * u1;
        v1 = s2 * v0 + c2 * v1;
        u0 = t0;
        v0 = t1;
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = o[q];
        if constexpr (SPLIT > 0) {
            constexpr int bit = rd < low ? __builtin_ctz(rd + 1) : SPLIT - 1;      // (the last one back to g = 0)
            x[1] = from_column<bit>(x[1]);
            x[2] = from_row<bit>(x[2]);
            x[3] = from_row<bit>(from_column<bit>(x[3]));
            u1 = from_column<bit>(u1);
            v1 = from_column<bit>(v1);
        }
    });
    auto put = [&](int e, int f, double val) {
        if (e > f) return;
        h[in_pair(e, f, pp, pq, qq)] = val;
        if (!((e ^ f) & 8)) h[in_pair(f, e, pp, pq, qq)] = val;
    };
    put(e0, f0, x[0]);
    put(e0, f1, x[1]);
    put(e1, f0, x[2]);
    put(e1, f1, x[3]);
    jac[16 * k1 + f0] = u0;
    jac[16 * k1 + f1] = u1;
    jac[16 * k1 + 128 + f0] = v0;
    jac[16 * k1 + 128 + f1] = v1;
}

// The same outcome as jacobi_kernel.  A sweep is a tournament of the nb blocks of 8 indices: in each round nb / 2 waves rotate
// their pair's 16 x 16 part and accumulate the rotations J (the pairs across the two blocks; in a sweep's first round those inside
// them too), then all waves apply them, H_ab <- J_a^T H_ab J_b and V <- V J_b in 16 x 16 parts on the fp64 matrix cores.
// H: upper triangle of blocks in LDS (width 160: 149 of 160 KB with 16 rows of V; 168 does not fit); V^T: nb * 8 columns of v_rows (a
// multiple of 16) each.
// What bounds it: the instructions of the rotating waves, 8 rounds of about 600 cycles (of 1000 where three of ten such waves share
// a SIMD), then the matrix cores and addresses of the update, 4000 cycles at width 80 and 11000 at 160.  A rotation at a time over the
// whole of H moves all of H through LDS for each of 8 nb - 1 rounds per sweep (0.7 us per round at width 16, 1.1 at 80, 2.2 at 160).
// us per decomposition that way and this: one layer of width 12 54 -> 26, 16 53 -> 24, 40 187 -> 97, 120 815 -> 493, 144 1552 ->
// 863, 160 1772 -> 750; 7 layers of width 80 488 to 578 -> 240 to 253, 64 601 -> 302; 128 of width 104 1088 -> 571, 256 of 24 131 -> 79.
template <int NT>
__global__ __launch_bounds__(NT) void jacobi_block_kernel(const LayerDev* __restrict__ layers, const int* __restrict__ ids, int role,
                                                          int v_rows, int slot_rows, float* __restrict__ sigma_out) {
    const LayerDev& L = layers[ids[blockIdx.y]];
    const int w = L.thin[role].width;
    const int n_slots = (side_len(L, side_of_role(L.transposed, role)) + slot_rows - 1) / slot_rows;
    const int np = (w + 15) / 16, nb = 2 * np, n = 8 * nb, n_blk = (nb * (nb + 1)) / 2;
    const int row0 = blockIdx.x * v_rows;
    if (row0 >= w) return;                                 // (a narrower layer than the launch's widest)
    extern __shared__ __align__(16) unsigned char smem[];
    double* h = reinterpret_cast<double*>(smem);
    double* jac = h + n_blk * 64;                          // [np][16][16]
    double* vt = jac + np * 256;                           // [n][v_rows]
    double* red = vt + n * v_rows;                         // [2][16] per-wave partial sums of the convergence test
    const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6), li = lane & 15, lk = lane >> 4;
    constexpr int nw = NT / 64;
    // wave wv's blocks (I, K), I <= K: wv, wv + nw, ... column by column
    auto each_block = [&](auto&& f) {
        int K = 0, I = wv;
        for (int b = wv; b < n_blk; b += nw, I += nw) {
            while (I > K) I -= ++K;
            f(b, I, K);
        }
    };
    const int bi = lane >> 3, bk = lane & 7;
    const int ntri = (w * (w + 1)) / 2;
    each_block([&](int b, int I, int K) {
        const int i = 8 * I + bi, j = 8 * K + bk;
        double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
        if (i < w && j < w) {
            const PSGD_GLOBAL double* g = as_global(L.gram) + tri_idx(min(i, j), max(i, j), w);
            int sp = 0;
            for (; sp + 4 <= n_slots; sp += 4) {
                s0 += g[(int64_t)sp * ntri]; s1 += g[(int64_t)(sp + 1) * ntri];
                s2 += g[(int64_t)(sp + 2) * ntri]; s3 += g[(int64_t)(sp + 3) * ntri];
            }
            for (; sp < n_slots; ++sp) s0 += g[(int64_t)sp * ntri];
        }
        h[b * 64 + in_block(bi, bk)] = (s0 + s1) + (s2 + s3);
    });
    for (int j = wv; j < n; j += nw)
        for (int i = lane; i < v_rows; i += 64) vt[j * v_rows + i] = row0 + i == j ? 1.0 : 0.0;
    __syncthreads();
    const int n_tiles = (np * (np - 1)) / 2, n_items = n_tiles + np * (v_rows / 16);
    auto blocks_of = [&](int pair, int rd, int& p, int& q) {
        const int x = jacobi_top(pair, rd, nb), y = jacobi_bottom(pair, rd, nb);
        p = min(x, y);
        q = max(x, y);
    };
    // entries (li & 7, 4 c + lk) of a block and the other way round
    const int at_row[2] = {in_block(li & 7, lk), in_block(li & 7, 4 + lk)}, at_col[2] = {in_block(lk, li & 7), in_block(4 + lk, li & 7)};
    int sweeps = 0;
    for (int sweep = 0; sweep < kJacobiMaxSweeps; ++sweep) {
        // convergence: off-diagonal mass relative to the diagonal, added up in a fixed order: the same bits in every workgroup of
        // the layer, whose slices of V only fit together if all of them run the same number of sweeps
        double off = 0.0, dia = 0.0;
        each_block([&](int b, int I, int K) {
            const double x = h[b * 64 + in_block(bi, bk)];
            if (I != K) off += 2.0 * x * x;
            else if (bi == bk) dia += x * x;
            else off += x * x;
        });
        for (int o = 32; o > 0; o >>= 1) { off += __shfl_down(off, o); dia += __shfl_down(dia, o); }
        if (lane == 0) { red[wv] = off; red[16 + wv] = dia; }
        __syncthreads();
        double off_all = 0.0, dia_all = 0.0;
        for (int q = 0; q < nw; ++q) { off_all += red[q]; dia_all += red[16 + q]; }
        if (off_all <= 1e-20 * dia_all) break;
        sweeps = sweep + 1;
#pragma unroll 1
        for (int rd = 0; rd < nb - 1; ++rd) {
#pragma unroll 1
            for (int b = wv; b < np; b += nw) {
                int p, q;
                blocks_of(b, rd, p, q);
                const int pp = block_at(p, p), pq = block_at(p, q), qq = block_at(q, q);
                if (rd == 0) {
                    jacobi_phase<2>(h, jac + 256 * b, pp, pq, qq, true);
                    wave_sync();
                    jacobi_phase<1>(h, jac + 256 * b, pp, pq, qq, false);
                    wave_sync();
                    jacobi_phase<0>(h, jac + 256 * b, pp, pq, qq, false);
                    wave_sync();
                }
                jacobi_phase<3>(h, jac + 256 * b, pp, pq, qq, rd != 0);
            }
            __syncthreads();
            int a = 0, k = wv;                             // tile (a, a + 1 + k) of the upper triangle of pairs
#pragma unroll 1
            for (int item = wv; item < n_items; item += nw, k += nw) {
                if (item < n_tiles) {
                    while (k >= np - 1 - a) { k -= np - 1 - a; ++a; }
                    const int b = a + 1 + k;
                    int pa, qa, pb, qb;
                    blocks_of(a, rd, pa, qa);
                    blocks_of(b, rd, pb, qb);
                    // T = H_ab: as the A operand lane (li, lk) reads row li; the product's row 4 v + lk, column li.  [half of a][half of b]
                    const int rows[2] = {pa, qa}, cols[2] = {pb, qb};
                    int base[2][2];
                    bool turned[2][2];
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            turned[i][j] = rows[i] > cols[j];
                            base[i][j] = block_at(min(rows[i], cols[j]), max(rows[i], cols[j]));
                        }
                    double tv[4], ja[4], jb[4];
                    int out[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const int z = c >> 1;
                        const int by_row0 = base[0][z] + (turned[0][z] ? at_col[c & 1] : at_row[c & 1]);
                        const int by_row1 = base[1][z] + (turned[1][z] ? at_col[c & 1] : at_row[c & 1]);
                        tv[c] = h[li & 8 ? by_row1 : by_row0];
                        const int by_col0 = base[z][0] + (turned[z][0] ? at_row[c & 1] : at_col[c & 1]);
                        const int by_col1 = base[z][1] + (turned[z][1] ? at_row[c & 1] : at_col[c & 1]);
                        out[c] = li & 8 ? by_col1 : by_col0;
                        jb[c] = jac[256 * b + 64 * c + lane];
                        ja[c] = jac[256 * a + 64 * c + lane];
                    }
                    // (without the fence the loads are made one by one between the MFMAs)
                    __builtin_amdgcn_sched_barrier(0);
                    doublex4 x = {0.0, 0.0, 0.0, 0.0}, y = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int c = 0; c < 4; ++c) x = __builtin_amdgcn_mfma_f64_16x16x4f64(tv[c], jb[c], x, 0, 0, 0);
                    // (row 4 v + lk of T J_b is what the B operand of step v takes)
#pragma unroll
                    for (int c = 0; c < 4; ++c) y = __builtin_amdgcn_mfma_f64_16x16x4f64(ja[c], x[c], y, 0, 0, 0);
#pragma unroll
                    for (int v = 0; v < 4; ++v) h[out[v]] = y[v];
                } else {
                    const int e = item - n_tiles, b = e % np, r0 = 16 * (e / np);
                    int p, q;
                    blocks_of(b, rd, p, q);
                    double* v0 = vt + 8 * p * v_rows + r0 + li;
                    double* v1 = vt + 8 * q * v_rows + r0 + li;
                    double jb[4], xv[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        jb[c] = jac[256 * b + 64 * c + lane];
                        xv[c] = (c & 2 ? v1 : v0)[(4 * (c & 1) + lk) * v_rows];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    doublex4 y = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int c = 0; c < 4; ++c) y = __builtin_amdgcn_mfma_f64_16x16x4f64(jb[c], xv[c], y, 0, 0, 0);
#pragma unroll
                    for (int v = 0; v < 4; ++v) (v & 2 ? v1 : v0)[(4 * (v & 1) + lk) * v_rows] = y[v];
                }
            }
            __syncthreads();
        }
    }
    __syncthreads();
    double* lam = jac;                                     // [n], and the ranks: the rotations are done
    int* rank_of = reinterpret_cast<int*>(lam + n);
    for (int j = t; j < n; j += NT) lam[j] = h[block_at(j >> 3, j >> 3) + in_block(j & 7, j & 7)];
    __syncthreads();
    ritz_ranks(lam, rank_of, w, blockIdx.x == 0 ? L.eval : nullptr);
    __syncthreads();
    double* __restrict__ tm = L.tmat;
    for (int i = wv; i < min(v_rows, w - row0); i += nw)
        for (int j = lane; j < w; j += 64) tm[(int64_t)(row0 + i) * w + rank_of[j]] = vt[j * v_rows + i];
    if (blockIdx.x == 0) ritz_notes(L, w, sweeps, sigma_out);
}

size_t jacobi_lds_bytes(int w, int v_rows) {
    const int n = (w + 1) & ~1;
    return (size_t)(2 * n + 32 + n * sym_stride(n) + v_rows * n) * sizeof(double) + (size_t)2 * n * sizeof(int);
}

size_t jacobi_block_lds_bytes(int w, int v_rows) {
    const int np = (w + 15) / 16, nb = 2 * np;
    return (size_t)(nb * (nb + 1) / 2 * 64 + np * 256 + 8 * nb * v_rows + 32) * sizeof(double);
}

// slot_rows: rows per partial Gram matrix of thin[role] (kOneSlot: gram_sum_kernel has added them up)
hipError_t launch_jacobi(const LayerDev* layers, const int* ids, int n_ids, int w, int role, int slot_rows, float* sigma_out,
                         hipStream_t st) {
    if (n_ids <= 0) return hipSuccess;
    constexpr size_t kLdsCap = 159 * 1024;     // of the 160 KB a workgroup can have
    // rows of V per workgroup: as few as its kernel takes while the chip has idle compute units, and no more than fit in LDS
    const int slices = 256 / n_ids < 1 ? 1 : 256 / n_ids;
    size_t lds;
    int v_rows;
    if (w <= kJacobiBlockWidth) {
        v_rows = ((w + slices - 1) / slices + 15) / 16 * 16;
        while (v_rows > 16 && jacobi_block_lds_bytes(w, v_rows) > kLdsCap) v_rows -= 16;
        lds = jacobi_block_lds_bytes(w, v_rows);
        const int threads = w <= 48 ? 256 : w <= 96 ? 512 : 1024;
        auto kfn = threads == 256 ? jacobi_block_kernel<256> : threads == 512 ? jacobi_block_kernel<512> : jacobi_block_kernel<1024>;
        if (lds > kLdsCap) return hipErrorInvalidValue;
        if (lds > 48 * 1024) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kfn, dim3((w + v_rows - 1) / v_rows, n_ids), dim3(threads), lds, st, layers, ids, role, v_rows, slot_rows, sigma_out);
        return hipGetLastError();
    }
    const int n = (w + 1) & ~1;
    v_rows = (n + slices - 1) / slices;
    v_rows = v_rows < 8 ? 8 : v_rows;
    while (v_rows > 1 && jacobi_lds_bytes(w, v_rows) > kLdsCap) --v_rows;
    v_rows = v_rows > n ? n : v_rows;
    lds = jacobi_lds_bytes(w, v_rows);
    if (lds > kLdsCap || w > kJacobiMaxWidth) return hipErrorInvalidValue;
    // (with four or five blocks per thread the kernel spills a few registers; 512 threads with twice the registers measured slower)
    constexpr int kThreadsWide = 1024;
    auto kfn = ((n / 2) * (n / 2 + 1)) / 2 <= 4 * kThreadsWide ? jacobi_kernel<4> : jacobi_kernel<5>;
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kfn, dim3((n + v_rows - 1) / v_rows, n_ids), dim3(kThreadsWide), lds, st, layers, ids, role, v_rows, slot_rows, sigma_out);
    return hipGetLastError();
}

// --------------------------------------------------------------------------------------------
// Host tables (layer descriptors, pointer tables, id lists) reach the workspace as kernel arguments: the runtime
// copies a launch's arguments before the launch call returns, so the host arrays may be rewritten or go out of
// scope at once, nothing depends on how the runtime stages copies from pageable memory, and no copy node ever
// re-reads a host array.  One launch carries kPutBytes bytes.
// --------------------------------------------------------------------------------------------
constexpr int kPutBytes = 2048;
struct PutChunk { uint4 w[kPutBytes / 16]; };

__global__ __launch_bounds__(kPutBytes / 16) void put_kernel(uint4* __restrict__ dst, PutChunk c, int n16) {
    if ((int)threadIdx.x < n16) dst[threadIdx.x] = c.w[threadIdx.x];
}

// dst: device, 16-byte aligned, with room for `bytes` rounded up to 16 (the tail is written as zeros)
hipError_t launch_put(void* dst, const void* src_host, size_t bytes, hipStream_t st) {
    const unsigned char* src = static_cast<const unsigned char*>(src_host);
    unsigned char* d = static_cast<unsigned char*>(dst);
    for (size_t o = 0; o < bytes; o += kPutBytes) {
        const size_t n = bytes - o < (size_t)kPutBytes ? bytes - o : (size_t)kPutBytes;
        PutChunk c;
        memset(&c, 0, sizeof(c));
        memcpy(&c, src + o, n);
        hipLaunchKernelGGL(put_kernel, dim3(1), dim3(kPutBytes / 16), 0, st, reinterpret_cast<uint4*>(d + o), c,
                           (int)((n + 15) / 16));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// status words of the addressed layers <- 0 (a workspace seen for the first time: "iterations the next refresh
// needs" = unknown, arrival counters at rest)
__global__ __launch_bounds__(64) void clear_status_kernel(const LayerDev* __restrict__ layers, const int* __restrict__ ids) {
    const LayerDev& L = layers[ids[blockIdx.x]];
    if (threadIdx.x < kStatusWords) as_global(L.status)[threadIdx.x] = 0;
}

hipError_t launch_clear_status(const LayerDev* layers, const int* ids, int n_ids, hipStream_t st) {
    if (n_ids <= 0) return hipSuccess;
    hipLaunchKernelGGL(clear_status_kernel, dim3(n_ids), dim3(64), 0, st, layers, ids);
    return hipGetLastError();
}

// plain copy, 16 bytes per thread per iteration (profiler calibration / attainable copy bandwidth)
__global__ __launch_bounds__(kThreads) void copy_kernel(uint4* __restrict__ dst, const uint4* __restrict__ src,
                                                        size_t n_vec) {
    for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < n_vec; i += (size_t)gridDim.x * kThreads)
        dst[i] = src[i];
}

hipError_t launch_copy(void* dst, const void* src, size_t n_bytes, hipStream_t st) {
    const size_t n_vec = n_bytes / 16;
    if (n_vec == 0) return hipSuccess;
    size_t gx = (n_vec + kThreads - 1) / kThreads;
    if (gx > 256 * 64) gx = 256 * 64;
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)gx), dim3(kThreads), 0, st, reinterpret_cast<uint4*>(dst),
                       reinterpret_cast<const uint4*>(src), n_vec);
    return hipGetLastError();
}

}  // namespace psgd
