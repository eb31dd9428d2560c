// Host side of the C ABI declared in include/psgd.h: argument checks, launch planning, workspace
// layout, pointer-table upload, and the sequences of batched launches that make up one SSP-Comp
// step, one SVD-Comp step (Algorithm 1) and the reconstruction.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "../../include/psgd.h"
#include "psgd_dev.h"

namespace psgd {
hipError_t launch_prod(int nb, int planes, bool colmode, bool form, bool lazy, bool onew, const LayerDev* layers,
                       const int* ids, int n_ids, int max_tiles, int out_role, int epi, int gate, int nt_s, hipStream_t st);
hipError_t launch_form_row(int nb, int planes, bool gbf, bool onew, int lazy, const LayerDev* layers, const int* ids,
                           int n_ids, int max_tiles, int out_role, int epi, int nt_m, const int* xtab, int xstride,
                           int xtiles, hipStream_t st);
bool form_row_supported(int nb, int planes, bool gbf, bool onew, bool lazy);
hipError_t launch_col_prod(int nb, int planes, const LayerDev* layers, const int* ids, int n_ids, int max_tiles,
                           int out_role, int epi, int gate, int nt_s, const int* xtab, int xstride, int xtiles,
                           hipStream_t st);
bool col_prod_supported(int nb);
hipError_t launch_row_prod(int nb, int planes, const LayerDev* layers, const int* ids, int n_ids, int max_tiles,
                           int out_role, int epi, int gate, int nt_s, const int* xtab, int xstride, int xtiles,
                           hipStream_t st);
bool row_prod_supported(int nb);
hipError_t launch_outer(int nb, int planes, bool decomp, bool form, bool kept, const LayerDev* layers, const int* ids,
                        int n_ids, int max_tiles, int rpw, void* const* outs, int out_bf16, hipStream_t st);
hipError_t launch_max_iterations(const LayerDev* layers, const int* ids, int n_ids, int mx, int* out, hipStream_t st);
hipError_t launch_msgd(int nb, int planes, const LayerDev* layers, const int* ids, int n_ids, int max_tiles, int rpw,
                       float* const* moms, float* const* xs, float mu, float eta, bool kept, hipStream_t st);
hipError_t launch_adam(int nb, int planes, const LayerDev* layers, const int* ids, int n_ids, int max_tiles, int rpw,
                       float* const* m1s, float* const* m2s, float* const* xs, const float* coef, bool kept,
                       hipStream_t st);
hipError_t launch_finish(bool p_like, int kind_n, int kind_t, const LayerDev* layers, const int* ids, int n_ids, int max_blocks,
                         int cp, int out_role, int epi, int gate, int chol_gate, int a2gate, double tol2, int w,
                         int local_ok, hipStream_t st);
hipError_t launch_thin_gram(const LayerDev* layers, const int* ids, int n_ids, int max_blocks, int role, int cp,
                            int gate, int flagged, hipStream_t st);
hipError_t launch_pack(const LayerDev* layers, const int* ids, int n_ids, int max_lenP, int role_a, int role_b,
                       int cp, int which, hipStream_t st);
hipError_t launch_chol(const LayerDev* layers, const int* ids, int n_ids, int w, int role, double tol2, int pass,
                       int slot_rows_n, int slot_rows_t, int gate, int a2gate, int local_ok, hipStream_t st);
hipError_t launch_gram_sum(const LayerDev* layers, const int* ids, int n_ids, int w, int role, int slot_rows_n, int slot_rows_t,
                           int gate, int flagged, hipStream_t st);
int finish_rows(int w, int max_blocks, int n_ids);
hipError_t launch_apply(const LayerDev* layers, const int* ids, int n_ids, int max_lenP, int w_in, int w_out,
                        int src_role, int dst_role, int mode, int cp, int gate, int a2gate, double tol2,
                        bool small, int which, int slot_rows, int stream_wgs, hipStream_t st);
hipError_t launch_init_block(const LayerDev* layers, const int* ids, int n_ids, int max_len, int w, int dst_role,
                             int src_role, int warm, uint32_t seed, hipStream_t st);
hipError_t launch_jacobi(const LayerDev* layers, const int* ids, int n_ids, int w, int role, int slot_rows, float* sigma_out,
                         hipStream_t st);
bool tiny_fits(int64_t rows, int64_t cols, int r, int n_arrays, bool refresh);
size_t tiny_lds_bytes(int64_t rows, int64_t cols);
hipError_t launch_tiny_step(const LayerDev* layers, const int* ids, int n_ids, size_t lds, double tol2, hipStream_t st);
hipError_t launch_tiny_iterate(const LayerDev* layers, const int* ids, int n_ids, size_t lds, double tol2, int iters, int warm,
                               uint32_t seed, hipStream_t st);
hipError_t launch_copy(void* dst, const void* src, size_t n_bytes, hipStream_t st);
hipError_t launch_put(void* dst, const void* src_host, size_t bytes, hipStream_t st);
hipError_t launch_clear_status(const LayerDev* layers, const int* ids, int n_ids, hipStream_t st);
enum ApplyModeHost { APPLY_PASS1 = 1, APPLY_PASS2 = 2, APPLY_RITZ = 3, APPLY_PASS1_ONLY = 4 };
}  // namespace psgd

using namespace psgd;

namespace {

constexpr int kMaxWidth = 192;      // widest thin block (packed Cholesky factor and product operands must fit in LDS)
constexpr int kTargetTiles = 1024;  // workgroups per forming-pass launch we try to reach by splitting the reduction
constexpr int kTargetTilesPlain = 512;   // ... per launch of a product that only reads M: half as many, twice as long-lived
                                         // (config 2: pass 2a 20.4 -> 18.6 us, its refresh step 1.00 -> 0.96 ms)
constexpr int kTargetTilesWide = 256;    // ... at thin widths of 64 and more (see choose_split)
constexpr int kMaxSplit = 32;
constexpr int64_t kMaxLd = (int64_t)1 << 23;   // largest leading dimension (elements)

inline int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

struct Plan {            // host copy of what a layer needs
    psgd_layer_desc d;
    int transposed;
    int rowsP, colsP;
    int m, n;
    int wz = 0;                             // this layer's block width in the subspace iteration: at least r, at most n
    int split[SPLIT_KINDS][2] = {{1, 1}, {1, 1}, {1, 1}, {1, 1}};   // reduction splits of its products, as in LayerDev (see plan_splits)
    int split_alone[2] = {1, 1};            // SPLIT_ITER of the layer by itself (psgd_refresh)
};

struct Lists {
    std::vector<int> norm, tr;   // layer ids stored row-major as logical / as the transpose
};

}  // namespace

struct psgd_ctx {
    uint64_t serial = 0;     // unique per context (the built-in workspace remembers whose contents it holds)
    int n_layers = 0;
    int n_workers = 0;
    psgd_options opt{};
    std::vector<Plan> plan;
    Lists lists;
    int rmax = 0;
    int cpc = 0;     // packed width of the compress step: 32 * ceil(rmax / 32)
    int wz = 0;      // widest block of the subspace iteration (r + oversampling, multiple of 8), see Plan::wz
    int cpz = 0;     // its packed width: wz rounded up to a multiple of 32
    int cpmax = 0;   // max(cpc, cpz)
    int planes = 2;  // bf16 planes per fp32 operand of the MFMA products (2: 3 products, 3: 6 products)
    bool reform_m = false;   // SSP step forms M = mean G + E in every pass instead of storing it over E
    bool lazy = false;       // deferred residual: E_{t+1} = M - P~ Q^T is applied by the next forming pass
    bool lazy_tr = false;    // ... also for the layers stored with rows < cols (column-mode forming pass: width 32 only)
    bool pending = false;    // the E buffers of the row-major layers hold M_t, their residual is still owed
    double kernel_bytes[3] = {0.0, 0.0, 0.0};   // algorithmic bytes of the three streaming kernels of one SSP step
    int grad_kind = 0;                          // 1: every layer has fp32 gradients, 2: every layer bf16, 0: mixed
    bool nt_m = false;                          // the row-major layers' M is too large to be found in a cache again
    bool nt_read = false;                       // ... the M of all layers
    // XCD table of the forming pass on 32 x 256 tiles (see form_row_kernel): 16 rows of xstride ints; built when the
    // row-major layers are many enough to be dealt evenly to the 8 XCDs
    std::vector<int> hXtab, hXtabC;             // (forming pass; column-mode product: other tile counts)
    int xstride = 0, xtiles = 0, xtiles_c = 0;
    size_t off_xtab = 0, off_xtab_c = 0;
    // workspace layout (byte offsets)
    // The gradient pointer table and the layer descriptors (which point into it) exist kGSlots times: a caller
    // that rotates between a few sets of gradient buffers finds its table already on the device.
    static constexpr int kGSlots = 4;
    size_t off_layers_s[kGSlots] = {}, off_gtab_s[kGSlots] = {};
    size_t off_iters = 0;            // one int: most iterations any layer's next refresh will run
    size_t off_ids = 0, off_outs = 0, off_moms = 0, off_m2s = 0, off_xs = 0;
    size_t off_alone[2] = {0, 0};    // partial sums of psgd_refresh, which splits for one layer (a context of one: the layer's own)
    std::vector<size_t> off_layer;   // start of each layer's private region
    size_t ws_bytes = 0;
    // cached tables
    void* bound_ws = nullptr;
    void* outs_ws = nullptr;     // workspace that holds the current table of decompress outputs
    void* msgd_ws = nullptr;     // ... and of the momentum and weight buffers of psgd_decompress_msgd / _adam
    void* m2_ws = nullptr;       // ... and of the second-moment buffers of psgd_decompress_adam
    int stream_wgs[2][2] = {};                  // of steps, of refreshes (see one_round)
    // every layer's step (plain, one power iteration) or refresh runs in one workgroup that holds M in LDS (tiny.hip)
    bool tiny_step = false, tiny_refresh = false;
    size_t tiny_lds = 0;
    void* factors_ws = nullptr;  // workspace whose outer-product operand copies are the P~, Q of the last compress call
    bool factors_kept = false;   // ... a call with a deferred residual: in the layers that defer they are the kept copies
    bool tables_valid = false;
    std::vector<const void*> hG;                       // the caller's current table
    std::vector<const void*> hGs[kGSlots];             // what each device slot holds (empty: nothing yet)
    int cur_slot = 0, next_victim = 0;
    std::vector<float*> hE, hQ, hP;
    std::vector<void*> hOut;
    std::vector<float*> hMom, hM2, hX;
    std::vector<int> hIds;
    std::vector<LayerDev> hLayers;   // n_layers + 1 (last = scratch descriptor of single-layer calls)
    int last_hip = 0;
    double algo_bytes = 0.0;
    // The per-layer iteration counts of the next refresh are decided on the device.  Their maximum is copied to
    // pinned host memory after every batched refresh (asynchronously, with an event behind it); a later refresh
    // that finds the event complete launches only that many iterations instead of the whole budget.
    // A copy describes the counts as the refresh it was enqueued behind left them: it is used by the very next
    // batched refresh on the same workspace and by no other (refresh_seq), and not at all if something else has
    // changed the counts in between (iters_gen: a single-layer psgd_refresh, another workspace, a reset).  The
    // copies go through a small ring of pinned words, so that a loop that runs ahead of the GPU (tau = 1) still
    // has a free word for every refresh; when none is free the next refresh launches the whole budget.  Whatever
    // the host launches, the device never runs an iteration that was not launched (see gate_open).
    static constexpr int kIterSlots = 4;
    struct IterFetch { int* h = nullptr; hipEvent_t ev = nullptr; bool pending = false; int gen = 0; uint64_t seq = 0; };
    IterFetch fetch[kIterSlots];
    bool fetch_ready = false;        // pinned words and events exist
    bool fetch_failed = false;       // ... could not be created: every refresh launches the whole budget
    int fetch_last = -1;             // slot of the copy enqueued behind the last batched refresh (-1: none)
    uint64_t refresh_seq = 0;        // batched refreshes run so far
    int iters_gen = 0;
    // optional timing of the three streaming kernels with event pairs on the caller's stream
    bool prof_on = false;
    int prof_mask = (1 << PSGD_PROF_TAGS) - 1;   // which of the tagged launches are timed
    std::vector<hipEvent_t> prof_ev;      // pairs (start, stop)
    std::vector<int> prof_tag;            // tag of each pair
    size_t prof_used = 0;                 // pairs recorded so far
};

namespace {

int fail_hip(psgd_ctx* c, hipError_t e) {
    c->last_hip = (int)e;
    return PSGD_E_HIP;
}

#define PSGD_TRY(expr)                                   \
    do {                                                 \
        hipError_t e__ = (expr);                         \
        if (e__ != hipSuccess) return fail_hip(ctx, e__); \
    } while (0)

// PSGD_FORM_ROW=0 (environment, measurement knob): forming passes use the 128 x 64 kernel everywhere
bool form_row_env() {
    static int v = -1;
    if (v < 0) {
        const char* e = std::getenv("PSGD_FORM_ROW");
        v = (e && e[0] == '0') ? 0 : 1;
    }
    return v == 1;
}

// Whether a product of the row-major layers runs on 32 x 256 tiles (form_row_kernel, row_prod_kernel, col_prod_kernel) at
// operand width 32 nb.  lazy: a forming pass that also applies the owed residual.
bool on_wide_tiles(const psgd_ctx* c, bool p_like, bool form, int nb, bool lazy) {
    if (!form_row_env()) return false;
    if (!form) return p_like ? row_prod_supported(nb) : col_prod_supported(nb);
    return p_like && c->grad_kind != 0 && form_row_supported(nb, c->planes, c->grad_kind == 2, c->n_workers == 1, lazy);
}

// Floats of partial sums per row of one side's result (0: rows, 1: columns) that the products of layer p can need: pieces
// times width, the most over the launches of the compress-type calls (alone: those of psgd_refresh).
int64_t part_width(const psgd_ctx* c, const Plan& p, int side, bool alone) {
    int64_t most = 0;
    auto launch = [&](bool p_like, bool form, bool iter, bool lazy) {
        const int mode = p_like == (p.transposed == 0) ? 0 : 1;
        if (mode != side) return;
        const int nb = (iter ? c->cpz : c->cpc) / 32;
        const int kind = !p.transposed && on_wide_tiles(c, p_like, form, nb, lazy) ? SPLIT_V2 : split_kind(form, iter ? 0 : -1);
        const int split = alone && kind == SPLIT_ITER ? p.split_alone[mode] : p.split[kind][mode];
        if (split > 1) most = std::max<int64_t>(most, (int64_t)split * (iter ? p.wz : p.d.r));
    };
    if (alone) {
        launch(true, false, true, false);
        launch(false, false, true, false);
        return most;
    }
    for (bool iter : {false, true}) {
        launch(true, true, iter, false);                              // M formed
        if (c->lazy) launch(true, true, iter, true);
        launch(true, false, iter, false);                             // M read (the step: further power iterations)
        launch(false, false, iter, false);
        if (c->reform_m && !iter) launch(false, true, iter, false);
    }
    return most;
}

struct LayerRegion {
    size_t part[2], pack[2][6], lzf[2][3], z[2], gram, tmat, eval, status, end;
};

// byte layout of one layer's private workspace region, relative to its start
LayerRegion layer_region(const psgd_ctx* c, const Plan& p) {
    LayerRegion R{};
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = (size_t)round_up((int64_t)(o + bytes), 256); return at; };
    const int lenP[2] = {p.rowsP, p.colsP};
    for (int s = 0; s < 2; ++s) {
        int64_t width = part_width(c, p, s, false);
        if (c->n_layers == 1) width = std::max(width, part_width(c, p, s, true));      // (see off_alone)
        R.part[s] = take((size_t)width * lenP[s] * sizeof(float));
    }
    for (int s = 0; s < 2; ++s)
        for (int k = 0; k < 2 * c->planes; ++k) R.pack[s][k] = take((size_t)lenP[s] * c->cpmax * sizeof(bf16_t));
    if (c->lazy && (!p.transposed || c->lazy_tr))
        for (int s = 0; s < 2; ++s)
            for (int k = 0; k < c->planes; ++k) R.lzf[s][k] = take((size_t)lenP[s] * c->cpc * sizeof(bf16_t));
    const int len[2] = {(int)p.d.rows, (int)p.d.cols};
    for (int s = 0; s < 2; ++s) R.z[s] = take((size_t)len[s] * p.wz * sizeof(float));
    const size_t w2 = (size_t)(p.wz + 2) * (p.wz + 2);
    const int max_lenP = lenP[0] > lenP[1] ? lenP[0] : lenP[1];
    // one partial Gram matrix per 64 rows of the widest block as a full square (as packed triangles: one per 32 rows), or triangles per
    // 32 and per 64 rows of a narrow P (the first pass of its factorisation and, while that is being read, the second)
    const size_t tri = (size_t)p.d.r * (p.d.r + 1) / 2, pass12 = p.d.r <= 16 ? (size_t)(kGramRows2 / 32 + 1) * tri : 0;
    R.gram = take((size_t)(max_lenP / kGramRows2) * std::max(w2, pass12) * sizeof(double));
    R.tmat = take(w2 * sizeof(double));
    R.eval = take((size_t)(p.wz + 2) * sizeof(double));
    R.status = take(kStatusWords * sizeof(int));
    R.end = o;
    return R;
}

// PSGD_TARGET_TILES (environment, tuning knob): workgroups a product launch should reach; 0 = not set
int target_tiles_env() {
    static int v = -1;
    if (v < 0) {
        const char* e = std::getenv("PSGD_TARGET_TILES");
        v = e ? std::atoi(e) : 0;
        if (v < 1) v = 0;
    }
    return v;
}

// Reduction split of a launch with `base_tiles` output blocks.  cp: packed width of the thin operand.  At widths
// of 64 and more one workgroup per compute unit is the target with three planes: the partial products that finish_kernel has
// to add up grow with the width, and the wide product kernels do not gain from more workgroups (4096 x 4096: the step at
// r = 64 takes 0.325 ms with 1024 workgroups, 0.302 with 256; at r = 128 0.514 and 0.473; at r = 16 and 32 it is
// the other way round).
// Two per compute unit with two planes up to width 128: where a compute unit has room for two (the forming pass, and the products
// that only read M up to width 96), and at width 128 also for the latter, of which one fits, for their shorter walks.  8192 x 8192 bf16
// r = 128, us per step with 512 and 256 of them: 413 and 399, 4096 x 4096 216 and 203, 8192 x 2048 r = 110 208 and 194, but four
// 4096 x 4096 438 and 464, three 11008 x 4096 r = 100 873 and 884, the 14 matrices of two 1B-shaped blocks 751 and 765, and with 256
// the error of Q is up to a tenth larger (3.99e-7 and 4.03e-7, 4.46e-7 and 4.92e-7).  With three planes one fits, and 4096 x 4096
// fp32 r = 128 took 307 us with 512 workgroups against 288.  run: the width the products run at, wider than the step's cp in a
// refresh's iteration (8192 x 8192 bf16 r = 128 at width 160: 6.38 ms with 512 workgroups, 6.18 with 256; 2048 x 8192 r = 104 4.52 and 4.36).
int split_target(bool form, int cp, int run, int planes) {
    int target = target_tiles_env();
    if (target == 0) target = cp >= 64 ? (planes == 2 && run <= 128 ? 2 : 1) * kTargetTilesWide : (form ? kTargetTiles : kTargetTilesPlain);
    else if (!form && target > kTargetTilesPlain) target = target / 2;
    return target;
}
// A launch that does not reach the target by itself is split, although from three quarters of it on the split costs more
// than it fills (25000 x 2048 fp32 r = 100, 196 workgroups of 256: 661 us per step in halves, 621 whole): the longer walks'
// fp32 sums leave 1.4 to 1.7 times the error (E 6.2e-6 and 9.4e-6).  Left whole are launches of one orientation from three
// quarters on where base_all, the batch's blocks of both orientations, reaches the target (the forming pass of the 22 matrices of
// a 1B-shaped model stored as the transpose, 968 workgroups, is 0.1 ms faster than in halves with their finish_kernel).
int choose_split(int64_t base_tiles, int min_chunks, bool form, int cp, int run, int planes, int64_t base_all) {
    const int target = split_target(form, cp, run, planes);
    if (base_tiles >= target || (4 * base_tiles >= 3 * target && base_all >= target)) return 1;
    int64_t s = (target + base_tiles - 1) / base_tiles;
    if (s > kMaxSplit) s = kMaxSplit;
    if (s > min_chunks) s = min_chunks;
    if (s < 1) s = 1;
    return (int)s;
}

// Splits of one kind of product over the layers of one launch (a launch serves the layers of one orientation, and the
// launches follow each other, so each has to fill the GPU by itself).  A layer has tiles(p) output blocks, each a walk over
// chunks(p) steps; with fewer blocks than the target the walks are cut into pieces of about the same number of steps, and
// none into fewer pieces than an equal split of all would make (the longer the walk, the larger the error of its fp32 sum).
// Either no layer of a launch is split or all are (their sums then all come from finish_kernel).
// Measured against one split per batch, bounded by its shortest walk: eight small matrices of 64 x 24 to 1000 x 264, fp32,
// r = 8: products 115 -> 38 us, step with momentum SGD 163 -> 94 us; two 1B-shaped fp32 blocks at r = 16 939 -> 866 us (two
// matrices of them are stored as the transpose, 32 workgroups of their row product).
template <class Tiles, class Chunks>
void plan_splits(std::vector<Plan>& plan, const std::vector<int>& ids, bool form, int cp, int run, int planes, Tiles tiles, Chunks chunks,
                 bool both, SplitKind kind, int mode) {
    int64_t base = 0, steps = 0, base_all = 0;
    int most = 1, least = 1 << 30;
    for (int l : ids) {
        base += tiles(plan[l]);
        steps += (int64_t)tiles(plan[l]) * chunks(plan[l]);
        most = std::max(most, (int)chunks(plan[l]));
        least = std::min(least, (int)chunks(plan[l]));
    }
    if (base == 0) return;
    if (both) for (const Plan& p : plan) base_all += tiles(p);
    const int s = choose_split(base, most, form, cp, run, planes, base_all);
    if (s <= 1) return;
    // Steps per workgroup: with walks of one length as many pieces as choose_split says, with several lengths the fewest
    // steps that keep the launch within its target (before the equal split's number, whose pieces of the short walks end early
    // and make room: the column product of the two blocks above 866 -> 870 us per step, error of Q 1.6e-7 -> 1.1e-7).
    int64_t per = 1;
    if (steps != base * most) {
        auto total = [&](int64_t q) {
            int64_t n = 0;
            for (int l : ids) n += (int64_t)tiles(plan[l]) * std::max<int64_t>(2, std::min<int64_t>((chunks(plan[l]) + q - 1) / q, kMaxSplit));
            return n;
        };
        const int64_t target = split_target(form, cp, run, planes);
        per = std::max<int64_t>(1, steps / target);
        while (per < most && total(per) > target) ++per;
    }
    const int equal = choose_split(base, least, form, cp, run, planes, base_all);
    for (int l : ids) {
        const int64_t mine = steps == base * most ? s : std::max<int64_t>(equal, (chunks(plan[l]) + per - 1) / per);
        plan[l].split[kind][mode] = (int)std::max<int64_t>(2, std::min<int64_t>(mine, kMaxSplit));
    }
}

// The splits of all launches.  one_split: one number per kind of product for the whole context, bounded by its shortest walk
// and planned for the fewer workgroups.
void plan_all(psgd_ctx* c, bool one_split) {
    auto row_tiles = [](const Plan& p) { return (int)((p.d.rows + 127) / 128); };
    auto col_tiles = [](const Plan& p) { return (int)((p.d.cols + 127) / 128); };
    auto row_chunks = [](const Plan& p) { return (int)((p.d.cols + 63) / 64); };
    auto col_chunks = [](const Plan& p) { return (int)((p.d.rows + 63) / 64); };
    auto row_tiles_v2 = [](const Plan& p) { return p.rowsP / 32; };
    auto col_tiles_v2 = [](const Plan& p) { return (p.colsP + 255) / 256; };
    auto row_chunks_v2 = [](const Plan& p) { return (int)((p.d.cols + 255) / 256); };
    auto col_chunks_v2 = [](const Plan& p) { return (int)((p.d.rows + 31) / 32); };
    std::vector<int> all(c->n_layers);
    for (int l = 0; l < c->n_layers; ++l) all[l] = l;
    auto plan = [&](const std::vector<int>& ids, SplitKind kind, int mode, bool form, int cp, int run, auto tiles, auto chunks) {
        if (!one_split) {
            plan_splits(c->plan, ids, form, cp, run, c->planes, tiles, chunks, kind != SPLIT_V2, kind, mode);
            return;
        }
        int64_t base = 0;
        int least = 1 << 30;
        for (int l : ids) { base += tiles(c->plan[l]); least = std::min(least, chunks(c->plan[l])); }
        const int s = base > 0 ? choose_split(base, least, form, cp, kMaxWidth, c->planes, 0) : 1;
        for (int l : ids) c->plan[l].split[kind][mode] = s;
    };
    for (Plan& p : c->plan)
        for (auto& k : p.split) k[0] = k[1] = 1;
    for (const std::vector<int>* ids : {&c->lists.norm, &c->lists.tr}) {
        const std::vector<int>& of = one_split ? all : *ids;
        plan(of, SPLIT_M, 0, false, c->cpc, c->cpc, row_tiles, row_chunks);
        plan(of, SPLIT_M, 1, false, c->cpc, c->cpc, col_tiles, col_chunks);
        plan(of, SPLIT_ITER, 0, false, c->cpc, c->cpz, row_tiles, row_chunks);
        plan(of, SPLIT_ITER, 1, false, c->cpc, c->cpz, col_tiles, col_chunks);
        plan(of, SPLIT_FORM, 0, true, c->cpc, c->cpc, row_tiles, row_chunks);
        plan(of, SPLIT_FORM, 1, true, c->cpc, c->cpc, col_tiles, col_chunks);
    }
    // on 32 x 256 tiles: the forming pass of the row-major layers (and the row products that share its split) and their
    // column products
    plan(c->lists.norm, SPLIT_V2, 0, true, 32, 32, row_tiles_v2, row_chunks_v2);
    plan(c->lists.norm, SPLIT_V2, 1, false, 32, 32, col_tiles_v2, col_chunks_v2);
    for (Plan& p : c->plan) {
        p.split_alone[0] = choose_split(row_tiles(p), row_chunks(p), false, c->cpz, one_split ? kMaxWidth : c->cpz, c->planes, 0);
        p.split_alone[1] = choose_split(col_tiles(p), col_chunks(p), false, c->cpz, one_split ? kMaxWidth : c->cpz, c->planes, 0);
    }
}

// Workspace layout for the planned splits: offsets and total.
void lay_out(psgd_ctx* c) {
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = (size_t)round_up((int64_t)(o + bytes), 256); return at; };
    for (int k = 0; k < psgd_ctx::kGSlots; ++k) c->off_layers_s[k] = take((size_t)(c->n_layers + 1) * sizeof(LayerDev));
    c->off_ids = take((3 * (size_t)c->n_layers + 1) * sizeof(int));
    c->off_iters = take(psgd_ctx::kIterSlots * sizeof(int));
    c->off_xtab = take((size_t)16 * c->xstride * sizeof(int) + 16);
    c->off_xtab_c = take((size_t)16 * c->xstride * sizeof(int) + 16);
    for (int k = 0; k < psgd_ctx::kGSlots; ++k) c->off_gtab_s[k] = take((size_t)c->n_layers * c->n_workers * sizeof(void*));
    c->off_outs = take((size_t)c->n_layers * sizeof(void*));
    c->off_moms = take((size_t)c->n_layers * sizeof(void*));
    c->off_xs = take((size_t)c->n_layers * sizeof(void*));
    c->off_m2s = take((size_t)c->n_layers * sizeof(void*));
    for (int s = 0; s < 2 && c->n_layers > 1; ++s) {
        size_t most = 0;
        for (const Plan& p : c->plan) most = std::max(most, (size_t)part_width(c, p, s, true) * (s == 0 ? p.rowsP : p.colsP) * sizeof(float));
        c->off_alone[s] = take(most);
    }
    c->off_layer.resize(c->n_layers);
    for (int l = 0; l < c->n_layers; ++l) {
        c->off_layer[l] = o;
        o += layer_region(c, c->plan[l]).end;
    }
    c->ws_bytes = o;
}

void build_layer_dev(psgd_ctx* c, char* ws, int l, int slot, LayerDev* out) {
    const Plan& p = c->plan[l];
    const LayerRegion R = layer_region(c, p);
    char* base = ws + c->off_layer[l];
    LayerDev L{};
    L.rows = (int)p.d.rows; L.cols = (int)p.d.cols; L.ld = p.d.ld; L.r = p.d.r; L.wz = p.wz;
    L.gdt = p.d.grad_dtype; L.n_workers = c->n_workers; L.transposed = p.transposed; L.planes = c->planes;
    L.rowsP = p.rowsP; L.colsP = p.colsP;
    std::memcpy(L.split, p.split, sizeof(L.split));
    L.G = reinterpret_cast<const void* const*>(ws + c->off_gtab_s[slot]) + (size_t)l * c->n_workers;
    L.S = c->hE.empty() ? nullptr : c->hE[l];
    const int side_p = side_of_role(p.transposed, ROLE_P), side_q = side_of_role(p.transposed, ROLE_Q);
    L.thin[ROLE_P] = ThinRef{c->hP.empty() ? nullptr : c->hP[l], p.d.r, p.d.r};
    L.thin[ROLE_Q] = ThinRef{c->hQ.empty() ? nullptr : c->hQ[l], p.d.r, p.d.r};
    L.thin[ROLE_ZP] = ThinRef{reinterpret_cast<float*>(base + R.z[side_p]), p.wz, p.wz};
    L.thin[ROLE_ZQ] = ThinRef{reinterpret_cast<float*>(base + R.z[side_q]), p.wz, p.wz};
    for (int s = 0; s < 2; ++s) {
        L.part[s] = reinterpret_cast<float*>(base + R.part[s]);
        for (int k = 0; k < c->planes; ++k) {
            L.pack[s].n[k] = reinterpret_cast<bf16_t*>(base + R.pack[s][2 * k]);
            L.pack[s].t[k] = reinterpret_cast<bf16_t*>(base + R.pack[s][2 * k + 1]);
            L.lzf[s][k] = (c->lazy && (!p.transposed || c->lazy_tr)) ? reinterpret_cast<bf16_t*>(base + R.lzf[s][k]) : nullptr;
        }
    }
    L.gram = reinterpret_cast<double*>(base + R.gram);
    L.tmat = reinterpret_cast<double*>(base + R.tmat);
    L.eval = reinterpret_cast<double*>(base + R.eval);
    L.status = reinterpret_cast<int*>(base + R.status);
    *out = L;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Refresh the cached host tables from the caller's; returns true when the device copy is stale.
template <typename T, typename U>
bool sync_table(std::vector<T>& cache, U const* user, size_t n) {
    if (!user) return false;
    bool changed = cache.size() != n;
    if (changed) cache.assign(n, nullptr);
    for (size_t i = 0; i < n; ++i)
        if (cache[i] != (T)user[i]) { cache[i] = (T)user[i]; changed = true; }
    return changed;
}

int check_table(const void* const* tab, size_t n) {
    if (!tab) return PSGD_E_INVALID_ARG;
    for (size_t i = 0; i < n; ++i) {
        if (!tab[i]) return PSGD_E_INVALID_ARG;
        if (!aligned16(tab[i])) return PSGD_E_ALIGN;
    }
    return PSGD_OK;
}

// Whether work put on `st` is being recorded into a graph instead of executed.
static bool is_capturing(hipStream_t st) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    const bool yes = hipStreamIsCapturing(st, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return yes;
}

// Upload what has changed: the layer descriptors and id lists (new workspace, or new E/Q/P
// pointers) and/or the table of gradient pointers.  Stream-ordered, so launches already queued keep
// seeing the old tables.
int upload_tables(psgd_ctx* ctx, void* workspace, hipStream_t st, bool desc_changed, bool g_changed) {
    char* ws = reinterpret_cast<char*>(workspace);
    const bool fresh = !ctx->tables_valid || ctx->bound_ws != workspace;
    const int nl = ctx->n_layers;
    if (fresh || desc_changed || g_changed) {
        // Under stream capture nothing may be uploaded: a copy node would read this context's host arrays again at
        // every replay, and the clearing of a new workspace's status words would become a memset node.  The one
        // thing that is allowed to differ from the last eager call is which of the gradient tables already on the
        // device is used.
        bool slot_known = false;
        for (int k = 0; k < psgd_ctx::kGSlots; ++k) slot_known |= !ctx->hG.empty() && ctx->hGs[k] == ctx->hG;
        const bool upload = fresh || desc_changed || (g_changed && !ctx->hG.empty() && !slot_known);
        if (upload && is_capturing(st)) {
            ctx->tables_valid = false;      // the host copies are ahead of the device now: upload all next time
            return PSGD_E_CAPTURE;
        }
    }
    // (tables go to the device as kernel arguments, launch_put: the host arrays are free again when it returns)
    if (fresh) ctx->iters_gen++;   // the iteration counts live in the workspace: a bound fetched from another one is void
    if (fresh || desc_changed) {
        ctx->hLayers.resize(nl + 1);
        for (int slot = 0; slot < psgd_ctx::kGSlots; ++slot) {
            for (int l = 0; l < nl; ++l) build_layer_dev(ctx, ws, l, slot, &ctx->hLayers[l]);
            ctx->hLayers[nl] = ctx->hLayers[0];
            PSGD_TRY(launch_put(ws + ctx->off_layers_s[slot], ctx->hLayers.data(), (size_t)(nl + 1) * sizeof(LayerDev), st));
        }
    }
    if (fresh) {
        std::vector<int>& ids = ctx->hIds;
        ids.assign(3 * (size_t)nl + 1, 0);
        for (int l = 0; l < nl; ++l) ids[l] = l;
        for (size_t i = 0; i < ctx->lists.norm.size(); ++i) ids[nl + i] = ctx->lists.norm[i];
        for (size_t i = 0; i < ctx->lists.tr.size(); ++i) ids[2 * (size_t)nl + i] = ctx->lists.tr[i];
        ids[3 * (size_t)nl] = nl;   // id of the scratch descriptor
        PSGD_TRY(launch_put(ws + ctx->off_ids, ids.data(), ids.size() * sizeof(int), st));
        if (!ctx->hXtab.empty()) PSGD_TRY(launch_put(ws + ctx->off_xtab, ctx->hXtab.data(), ctx->hXtab.size() * sizeof(int), st));
        if (!ctx->hXtabC.empty()) PSGD_TRY(launch_put(ws + ctx->off_xtab_c, ctx->hXtabC.data(), ctx->hXtabC.size() * sizeof(int), st));
    }
    if (fresh)
        for (auto& v : ctx->hGs) v.clear();
    if ((fresh || g_changed) && !ctx->hG.empty()) {
        // a slot that already holds this table, else the next one in turn
        int slot = -1;
        for (int k = 0; k < psgd_ctx::kGSlots; ++k)
            if (ctx->hGs[k] == ctx->hG) slot = k;
        if (slot < 0) {
            slot = ctx->next_victim;
            ctx->next_victim = (ctx->next_victim + 1) % psgd_ctx::kGSlots;
            ctx->hGs[slot] = ctx->hG;
            PSGD_TRY(launch_put(ws + ctx->off_gtab_s[slot], ctx->hG.data(), ctx->hG.size() * sizeof(void*), st));
        }
        ctx->cur_slot = slot;
    }
    if (fresh) {
        // status words of a new workspace start at zero ("iterations the next refresh needs" = unknown); a fill
        // kernel, not a memset, so that nothing on this path would ever become a memset node of a graph
        PSGD_TRY(launch_clear_status(reinterpret_cast<const LayerDev*>(ws + ctx->off_layers_s[0]),
                                     reinterpret_cast<const int*>(ws + ctx->off_ids), nl, st));
    }
    ctx->bound_ws = workspace;
    ctx->tables_valid = true;
    return PSGD_OK;
}

struct Launcher {
    psgd_ctx* ctx;
    char* ws;
    hipStream_t st;
    const LayerDev* layers;
    const int *ids_all, *ids_norm, *ids_tr;
    int n_all, n_norm, n_tr;
    // geometry maxima over the layers addressed by this launcher
    int max_rows = 0, max_cols = 0, max_rowsP = 0, max_colsP = 0;
    // 128 x 128 tiles of an outer product: of all layers, and workgroups of the layer with the most of them at 4, 8, 16 and 32
    // blocks of 32 rows each
    int64_t tiles_all = 0;
    static constexpr int kOuterGroups = 4;
    int tiles_rg[kOuterGroups] = {};
    struct Geometry {       // of the layers of one orientation
        int blocks[2] = {0, 0};                     // 128-row blocks of a row-mode / column-mode result
        int tiles[SPLIT_KINDS][2] = {};             // workgroups per layer of a product
        bool split[SPLIT_KINDS][2] = {};            // (all layers of a launch are split or none is)
        int longest = 0, shortest_max = 0;          // largest long side (P) and largest short side (Q)
    } norm, tr;
    int gram_rows_n = kGramRows1, gram_rows_t = kGramRows1;   // rows per Gram slot of the last product, per orientation
    hipError_t err = hipSuccess;
    bool prof_mute = false;   // the refresh's products are not part of the per-kernel timing
    bool capturing = false;   // the stream records into a graph: no event records
    int gate = -1;            // iteration gate of the launches inside the subspace iteration (-1: none)
    bool keep_e = false;      // FORM products leave E in place (M is formed again by the later passes)
    bool lazy_form = false;   // the forming pass of the row-major layers also applies their pending residual
    bool lazy_share = false;  // ... and the transposed operand copies of Q_{t-1} are what the step before left: they hold
                              // the kept Q, which the pass then need not read
    bool kept_packs = false;  // compress step with a deferred residual: the outer-product operand copies of its P~ and Q
                              // are the kept ones in the layers that have them
    int stream_wgs[2] = {0, 0};   // launch_apply on a P-like, a Q-like result
    bool use_xtab = true;     // PSGD_XTAB=0 (environment, measurement knob): plain layer-by-layer launch order
    bool use_xtab_c = true;   // PSGD_XTAB_C=0 (likewise): the same for the column-mode product alone

    // Whether the partial Gram matrices of a rows x w result are added up by a launch of their own, and the factorisation is
    // another one (see kWideWidth, kSumSlots).
    static bool sums_first(int w, int rows) {
        return w > kWideWidth || (w > kCholRegWidth && rows > kSumSlots * kGramRows1);
    }
    void note(hipError_t e) { if (err == hipSuccess && e != hipSuccess) err = e; }
    // event pair around one tagged launch group (only when profiling is on and pairs are left)
    int prof_begin(int tag) {
        if (prof_mute || capturing || !ctx->prof_on || !((ctx->prof_mask >> tag) & 1) || ctx->prof_used >= ctx->prof_ev.size() / 2) return -1;
        const int k = (int)ctx->prof_used++;
        ctx->prof_tag[k] = tag;
        note(hipEventRecord(ctx->prof_ev[2 * k], st));
        return k;
    }
    void prof_end(int k) { if (k >= 0) note(hipEventRecord(ctx->prof_ev[2 * k + 1], st)); }
    int max_len() const { return max_rows > max_cols ? max_rows : max_cols; }
    int max_lenP() const { return max_rowsP > max_colsP ? max_rowsP : max_colsP; }

    // operand copies of caller-supplied thin matrices: the transposed ones for a product, the others for an
    // outer-product kernel
    enum { PACK_OUTER = 1, PACK_TRANSPOSED = 2 };
    void pack(int role, int cp, int which, int role_b = -1) {
        note(launch_pack(layers, ids_all, n_all, max_lenP(), role, role_b, cp, which, st));
    }
    // product whose result is P-like (lives on the long side) or Q-like, stored in thin[out_role];
    // chol_gate >= -1: the first CholeskyQR pass on the result follows at once (see prod_orth)
    void prod(bool p_like, bool form, int nb, int out_role, int epi, int chol_gate = -2, int a2gate = -2,
              double tol2 = 0.0, int w = 0, bool small = false) {
        // normal storage: P-like result is L-side -> row mode; transposed storage: column mode
        const int k = prof_begin(p_like ? PSGD_PROF_SWEEP1 : PSGD_PROF_SWEEP2);
        const int ef = epi | (keep_e ? EPI_KEEP_E : 0) | (kept_packs && epi == EPI_PACK ? EPI_KEPT : 0);
        const bool onew = ctx->n_workers == 1;
        const SplitKind kind = (SplitKind)split_kind(form, gate);      // (where prod_kernel runs)
        const int mode_n = p_like ? 0 : 1, mode_t = 1 - mode_n;
        // forming pass on row-major layers at compress-step widths: the kernel built on 32 x 256 tiles
        // (never inside the gated part of the subspace iteration: its first product carries gate iteration 0,
        // which is open for every layer)
        const bool on_wide = n_norm > 0 && on_wide_tiles(ctx, p_like, form, nb, lazy_form);
        const bool v2 = on_wide && form;
        // (the XCD table pays where the thin operands are a large part of what a workgroup reads: width 64)
        const int* xtab = (ctx->xstride > 0 && use_xtab && nb >= 2 && ids_norm == ids_all + ctx->n_layers)
                              ? reinterpret_cast<const int*>(ws + ctx->off_xtab) : nullptr;
        // the same product on a matrix that is already formed (the refresh's iteration, further power steps)
        const bool r2 = on_wide && !form && p_like;
        const bool gram32 = (v2 || r2) && !norm.split[SPLIT_V2][0] && epi == EPI_GRAM && chol_gate >= -1 && (!small || norm.longest <= kLocalGram32);
        // the second product on row-major layers at those widths likewise
        const bool c2 = on_wide && !form && !p_like;
        const int* xtab_c = (ctx->xstride > 0 && use_xtab && use_xtab_c && nb >= 2 && ids_norm == ids_all + ctx->n_layers)
                                ? reinterpret_cast<const int*>(ws + ctx->off_xtab_c) : nullptr;
        if (c2) note(launch_col_prod(nb, ctx->planes, layers, ids_norm, n_norm, norm.tiles[SPLIT_V2][1], out_role, ef, gate, ctx->nt_m ? 1 : 0, xtab_c, ctx->xstride, ctx->xtiles_c, st));
        else if (r2) note(launch_row_prod(nb, ctx->planes, layers, ids_norm, n_norm, norm.tiles[SPLIT_V2][0], out_role, gram32 ? ef : (ef & ~EPI_KIND_MASK), gate, ctx->nt_m ? 1 : 0, xtab, ctx->xstride, ctx->xtiles, st));
        else if (v2) note(launch_form_row(nb, ctx->planes, ctx->grad_kind == 2, onew, lazy_form ? (lazy_share ? 2 : 1) : 0, layers, ids_norm, n_norm, norm.tiles[SPLIT_V2][0], out_role, gram32 ? ef : (ef & ~EPI_KIND_MASK), ctx->nt_m ? 1 : 0, xtab, ctx->xstride, ctx->xtiles, st));
        else note(launch_prod(nb, ctx->planes, !p_like, form, form && p_like && lazy_form, onew, layers, ids_norm, n_norm, norm.tiles[kind][mode_n], out_role, ef, gate, ctx->nt_read ? 1 : 0, st));
        // (the row product of the layers stored with rows < cols stays on 128 x 64 tiles: 990 x 3741 fp32 r = 6 72.8 us per step
        // against 76.2 on 32 x 256 tiles, eight 2048 x 5632 r = 16 530 against 556, 22 of them in bf16 r = 32 1327 against 1358,
        // four 4096 x 11008 r = 64 1015 against 1089; single long ones are up to 5 % faster there, 1024 x 100000 712 and 695)
        note(launch_prod(nb, ctx->planes, p_like, form, form && p_like && lazy_form && ctx->lazy_tr, onew, layers, ids_tr, n_tr, tr.tiles[kind][mode_t], out_role, ef, gate, ctx->nt_read ? 1 : 0, st));
        prof_end(k);
        // split reductions are completed (and the epilogue run) by a second, small launch, whose last
        // workgroup per layer also factorises the Gram matrix; unsplit products need a launch for that
        const bool rv2 = v2 || r2;
        const SplitKind kind_n = rv2 || c2 ? SPLIT_V2 : kind;
        const bool split_n = n_norm > 0 && norm.split[kind_n][mode_n], split_t = n_tr > 0 && tr.split[kind][mode_t];
        // Wide blocks, and long ones: the partial Gram matrices are added up by a launch that spreads over the chip, and one
        // launch of the factorisation serves both orientations.
        const int ww = w > 0 ? w : 32 * nb;
        const bool wide = sums_first(ww, p_like ? std::max(norm.longest, tr.longest) : std::max(norm.shortest_max, tr.shortest_max));
        const int fin_gate = wide ? -2 : chol_gate;
        int fin_rows = kGramRows1;
        if (split_n || split_t) {
            // (one launch for both orientations where both are split)
            const int* ids = split_n && split_t ? ids_all : split_n ? ids_norm : ids_tr;
            const int n_ids = split_n && split_t ? n_all : split_n ? n_norm : n_tr;
            const int most = std::max(split_n ? norm.blocks[mode_n] : 0, split_t ? tr.blocks[mode_t] : 0);
            fin_rows = finish_rows(ww, most, n_ids);
            note(launch_finish(p_like, kind_n, kind, layers, ids, n_ids, most, 32 * nb, out_role, epi | (ef & EPI_KEPT), gate, fin_gate, a2gate, tol2, ww, small ? 1 : 0, st));
        }
        // (an unsplit launch of that kernel writes one partial Gram matrix per 32-row block itself; only where the apply kernel
        // factorises for itself and would have more than 64 of them to add up, a small pass over the result leaves one
        // per 128 rows)
        if (rv2 && !split_n && epi == EPI_GRAM && !gram32) note(launch_thin_gram(layers, ids_norm, n_norm, norm.blocks[0], out_role, 32 * nb, gate, 0, st));
        gram_rows_n = gram32 ? 32 : split_n ? fin_rows : kGramRows1;
        gram_rows_t = split_t ? fin_rows : kGramRows1;
        if (chol_gate >= -1) {
            // (the many 32-row slots are added up before at any width; the launches for an orthonormal Y that only a few
            // layers ask for are kept few: there the factorisation adds the slots up itself)
            // (up to 2048 rows: 70 matrices of 400 x 400 to 1072 x 400 bf16 r = 37 3.45 -> 3.35 ms, 4096 x 4096 r = 112 4.47 -> 4.66)
            const bool few = wide && chol_gate >= 0 && (chol_gate & kGateIfAsked) && std::max(norm.shortest_max, tr.shortest_max) <= 2048;
            if (wide && !few) note(launch_gram_sum(layers, ids_all, n_all, ww, out_role, gram_rows_n, gram_rows_t, chol_gate, 0, st));
            else if (gram32 && !small) note(launch_gram_sum(layers, ids_norm, n_norm, ww, out_role, gram_rows_n, gram_rows_t, chol_gate, 0, st));
            if (wide) {
                note(launch_chol(layers, ids_all, n_all, w, out_role, tol2, 1, few ? gram_rows_n : kOneSlot, few ? gram_rows_t : kOneSlot, chol_gate, a2gate, 0, st));
            } else {
                // (not where the apply kernel factorises every layer for itself)
                const bool local_n = small && (p_like ? norm.longest : norm.shortest_max) <= kLocalCholMaxRows;
                const bool local_t = small && (p_like ? tr.longest : tr.shortest_max) <= kLocalCholMaxRows;
                if (!split_n && !local_n) note(launch_chol(layers, ids_norm, n_norm, w, out_role, tol2, 1, gram32 ? kOneSlot : kGramRows1, 0, chol_gate, a2gate, small ? 1 : 0, st));
                if (!split_t && !local_t) note(launch_chol(layers, ids_tr, n_tr, w, out_role, tol2, 1, 0, kGramRows1, chol_gate, a2gate, small ? 1 : 0, st));
            }
        }
    }
    // thin[out_role] = product as in prod(), then CholeskyQR2 on it: the first pass always, the second
    // when the first one's pivots ask for it (decided on the device) and `pass2` allows it.  Inside the
    // subspace iteration the second pass is only wanted where exact orthonormality matters: on Z in a
    // layer's last iteration; that iteration only notes the need, see second_pass_deferred.  cp > 0: also leave the
    // split-bf16 operand copies of the result.
    enum Pass2 { PASS2_NEVER = 0, PASS2_ALWAYS = 1, PASS2_DEFERRED = 2 };
    // if_asked (Y of the subspace iteration): only for the layers whose Z asked for it; the others' product leaves the operand
    // copies, and the launches behind it find nothing to do.
    void prod_orth(bool p_like, bool form, int nb, int out_role, int w, double tol2, int cp, int kind, Pass2 pass2, bool if_asked = false) {
        const int g = gate < 0 ? -1 : gate_with_kind(gate, kind) | (if_asked ? kGateIfAsked : 0);
        const int a2 = pass2 == PASS2_ALWAYS ? -1 : (pass2 == PASS2_NEVER || gate < 0) ? -2 : gate_with_kind(gate, 2);
        // narrow blocks everywhere: the apply kernel factorises per workgroup and hands over to the second
        // factorisation itself; otherwise the second factorisation is a launch of its own
        const bool small = w <= 16;
        // (inside the iteration only products read the result: no outer-product copies)
        const int wh = gate >= 0 ? PACK_TRANSPOSED : (PACK_OUTER | PACK_TRANSPOSED | (kept_packs ? 4 : 0));
        prod(p_like, form, nb, out_role, if_asked ? EPI_ITERATE : EPI_GRAM, g, a2, tol2, w, small);
        note(launch_apply(layers, ids_all, n_all, max_lenP(), w, w, out_role, out_role, pass2 == PASS2_ALWAYS ? APPLY_PASS1 : APPLY_PASS1_ONLY, cp, g, a2, tol2, small, wh, gram_rows_n, stream_wgs[p_like ? 0 : 1], st));
        if (pass2 == PASS2_ALWAYS) {
            if (!small) note(launch_chol(layers, ids_all, n_all, w, out_role, tol2, 2, kGramRows2, kGramRows2, g, -2, 0, st));
            note(launch_apply(layers, ids_all, n_all, max_lenP(), w, w, out_role, out_role, APPLY_PASS2, cp, g, a2, tol2, small, wh, 0, stream_wgs[p_like ? 0 : 1], st));
        }
    }
    // The second CholeskyQR pass on Z after the subspace iteration, for the layers whose last factorisation of Z asked for
    // it (nearly none): Z <- Z T2, and as Y = M^T Z is linear in Z, Y <- Y T2; then the Gram matrix of Y anew.  One set of
    // launches that find nothing to do, where the second pass inside the iteration was one per iteration (the host does
    // not know which is a layer's last): 0.1 ms of a refresh with 16 iterations at widths above 16.
    void second_pass_deferred(int w, int cp, double tol2) {
        const bool wide = sums_first(w, max_len());
        const int blocks = (max_lenP() + 127) / 128;
        note(launch_thin_gram(layers, ids_all, n_all, blocks, ROLE_ZP, cp, -1, 1, st));
        if (wide) note(launch_gram_sum(layers, ids_all, n_all, w, ROLE_ZP, kGramRows1, kGramRows1, -1, 1, st));
        note(launch_chol(layers, ids_all, n_all, w, ROLE_ZP, tol2, 2, wide ? kOneSlot : kGramRows1, wide ? kOneSlot : kGramRows1, -1, -2, 0, st));
        for (int role : {ROLE_ZP, ROLE_ZQ})
            note(launch_apply(layers, ids_all, n_all, max_lenP(), w, w, role, role, APPLY_PASS2, 0, -1, -2, tol2, w <= 16, 0, 0, stream_wgs[role == ROLE_ZP ? 0 : 1], st));
        note(launch_thin_gram(layers, ids_all, n_all, blocks, ROLE_ZQ, cp, -1, 1, st));
        if (w > kWideWidth) note(launch_gram_sum(layers, ids_all, n_all, w, ROLE_ZQ, kGramRows1, kGramRows1, -1, 1, st));     // (as Jacobi expects them)
    }
    // the same CholeskyQR2 on a thin[out_role] that the caller supplied: its Gram slots come from a pass of their own
    void orth_given(int out_role, int w, double tol2, int cp) {
        const bool small = w <= 16;
        const int blocks = (max_lenP() + 127) / 128;
        note(launch_thin_gram(layers, ids_all, n_all, blocks, out_role, cp, -1, 0, st));
        const bool wide = sums_first(w, max_len());
        if (wide) note(launch_gram_sum(layers, ids_all, n_all, w, out_role, kGramRows1, kGramRows1, -1, 0, st));
        if (!small || max_len() > kLocalCholMaxRows) note(launch_chol(layers, ids_all, n_all, w, out_role, tol2, 1, wide ? kOneSlot : kGramRows1, wide ? kOneSlot : kGramRows1, -1, -1, small ? 1 : 0, st));
        note(launch_apply(layers, ids_all, n_all, max_lenP(), w, w, out_role, out_role, APPLY_PASS1, cp, -1, -1, tol2, small, 3, kGramRows1, stream_wgs[0], st));
        if (!small) note(launch_chol(layers, ids_all, n_all, w, out_role, tol2, 2, kGramRows2, kGramRows2, -1, -2, 0, st));
        note(launch_apply(layers, ids_all, n_all, max_lenP(), w, w, out_role, out_role, APPLY_PASS2, cp, -1, -1, tol2, small, 3, 0, stream_wgs[0], st));
    }
    // 32-row blocks per workgroup of the outer-product kernels and the grid that goes with them.  Four blocks, one per wave, and the
    // column operand staged for one tile, up to nb * planes = 6.  Wider operands leave a compute unit room for two such
    // workgroups (nb * planes = 8) or one, which stages, multiplies and stores one after the other: there 8 or 16 waves
    // share one staged operand and walk down 8 to 32 blocks, as many as still give every compute unit a workgroup
    // (8192 x 8192 r = 128, four blocks and 32: three planes residual 194 -> 133 us, decompress 153 -> 99, momentum SGD 266 -> 223;
    // two planes 128 -> 120, 72 -> 56 into bf16; 4096 x 4096 three planes 49 -> 38.  2048 x 2048, 64 tiles too few: 12.4 and 15.1.
    // nb * planes = 6, 7B-shaped block: residual 311 against 343, Adam 910 and 935)
    int outer_log_groups(int nb) const {
        if (nb * ctx->planes < kOuterManyWaves) return 0;
        int i = kOuterGroups - 1;
        while (i > 0 && (tiles_all >> i) < 256) --i;
        return i;
    }
    int outer_rows(int nb) const { return 4 << outer_log_groups(nb); }
    int outer_tiles(int nb) const { return tiles_rg[outer_log_groups(nb)]; }
    void residual(int nb, bool form = false) {
        const int k = prof_begin(PSGD_PROF_RESIDUAL);
        note(launch_outer(nb, ctx->planes, false, form, false, layers, ids_all, n_all, outer_tiles(nb), outer_rows(nb), nullptr, 0, st));
        prof_end(k);
    }
    // deferred residual: the layers that defer keep their operands; the others (stored with rows < cols, at
    // widths above 32) take their residual at once
    // (the layers that defer need no launch: the step's apply and product kernels have written their kept copies)
    void residual_deferred(int nb) {
        if (ctx->lazy_tr) return;
        const int k = prof_begin(PSGD_PROF_RESIDUAL);
        note(launch_outer(nb, ctx->planes, false, false, false, layers, ids_tr, n_tr, outer_tiles(nb), outer_rows(nb), nullptr, 0, st));
        prof_end(k);
    }
    // E <- M - (kept P~)(kept Q)^T for the layers that defer: what the deferred residual still owes
    void residual_owed(int nb) {
        const int k = prof_begin(PSGD_PROF_RESIDUAL);
        if (ctx->lazy_tr) note(launch_outer(nb, ctx->planes, false, false, true, layers, ids_all, n_all, outer_tiles(nb), outer_rows(nb), nullptr, 0, st));
        else note(launch_outer(nb, ctx->planes, false, false, true, layers, ids_norm, n_norm, outer_tiles(nb), outer_rows(nb), nullptr, 0, st));
        prof_end(k);
    }
};

void geometry(const Plan& p, Launcher& L) {
    auto mx = [](int& a, int b) { if (b > a) a = b; };
    mx(L.max_rows, (int)p.d.rows); mx(L.max_cols, (int)p.d.cols);
    mx(L.max_rowsP, p.rowsP); mx(L.max_colsP, p.colsP);
    const int rb = (int)((p.d.rows + 127) / 128), cb = (int)((p.d.cols + 127) / 128);
    L.tiles_all += (int64_t)rb * cb;
    for (int i = 0; i < Launcher::kOuterGroups; ++i) mx(L.tiles_rg[i], ((rb + (1 << i) - 1) >> i) * cb);
    Launcher::Geometry& g = p.transposed ? L.tr : L.norm;
    mx(g.longest, p.m); mx(g.shortest_max, p.n);
    mx(g.blocks[0], rb); mx(g.blocks[1], cb);
    for (int k = 0; k < SPLIT_KINDS; ++k) {
        mx(g.tiles[k][0], (k == SPLIT_V2 ? p.rowsP / 32 : rb) * p.split[k][0]);
        mx(g.tiles[k][1], (k == SPLIT_V2 ? (p.colsP + 255) / 256 : cb) * p.split[k][1]);
        for (int m = 0; m < 2; ++m) g.split[k][m] |= p.split[k][m] > 1;
    }
}

// Workgroups per layer of a launch of apply_stream_kernel above width 64 on all of `plan` (side: 0 P-like results, 1 Q-like) that make
// one round of two per compute unit: a workgroup loads 30 KB of the factor's fragments once for several tiles, and no second
// round runs half empty.  The most that leave the layers together, each of which uses no more than it has tiles, at 512, and the launch at
// 4096, the others of which find nothing to do.  0, as many as launch_apply takes at any width: up to one and a half rounds of tiles,
// and above eight, and where a long layer beside short ones would walk more tiles per workgroup than there are rounds (refresh: a thirty-second
// part more is still the faster side).  us per refresh, several rounds and one: 772 tiles (7B-shaped block r = 64) 7860 and 7800, 782 (50000 x 1024 r = 72) 1291 and
// 1261, 896 (fourteen 4096 x 4096 r = 64) 10510 and 10340, 1600 (a hundred 1024 x 1024 r = 72) 2479 and 2333, 3840 (120 of 512 x 2048
// r = 68) 3565 and 2724; 768 (twenty-four 2048 x 2048 r = 64) 3044 and 3075, 640 (forty 1024 x 1024 r = 72) 1400 and 1421.  Long walks, refresh
// r = 76: 16384 x 1024 beside seventy 512 x 512, 37 tiles each, 6508 and 10778, 20000 x 300 (two) beside twenty 1000 x 1000, 4 tiles, 4153 and
// 4243; steps r = 95: those 796 and 1531, 512 and 523, 30000 x 256 beside six 5000 x 512, 7 tiles, 397 and 436, five 11109 x 303 beside five 923 x 378,
// 174 tiles on 86 workgroups, 390 and 403 (refresh 3125 and 3123).
int one_round(const std::vector<Plan>& plan, int side, bool refresh) {
    auto tiles = [side](const Plan& p) { return (int)((side == 0 ? std::max(p.rowsP, p.colsP) : std::min(p.rowsP, p.colsP)) / kGramRows2); };
    int64_t all = 0;
    int longest = 1;
    for (const Plan& p : plan) { all += tiles(p); longest = std::max(longest, tiles(p)); }
    if (all <= 512 + 256 || all > 8 * 512) return 0;
    int lo = 1, hi = std::min<int>(longest, (8 * 512 + (int)plan.size() - 1) / (int)plan.size());
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        int64_t wgs = 0;
        for (const Plan& p : plan) wgs += std::min(tiles(p), mid);
        if (wgs <= 512) lo = mid; else hi = mid - 1;
    }
    const int rounds = (int)((all + 511) / 512);
    return longest <= rounds * lo + (refresh ? longest / 32 : 0) ? lo : 0;
}

Launcher batch_launcher(psgd_ctx* ctx, void* workspace, hipStream_t st) {
    Launcher L{};
    L.ctx = ctx; L.ws = reinterpret_cast<char*>(workspace); L.st = st;
    L.capturing = ctx->prof_on && is_capturing(st);
    L.layers = reinterpret_cast<const LayerDev*>(L.ws + ctx->off_layers_s[ctx->cur_slot]);
    const int nl = ctx->n_layers;
    const int* ids = reinterpret_cast<const int*>(L.ws + ctx->off_ids);
    L.ids_all = ids; L.ids_norm = ids + nl; L.ids_tr = ids + 2 * (size_t)nl;
    L.n_all = nl; L.n_norm = (int)ctx->lists.norm.size(); L.n_tr = (int)ctx->lists.tr.size();
    for (const Plan& p : ctx->plan) geometry(p, L);
    for (int s = 0; s < 2; ++s) L.stream_wgs[s] = ctx->stream_wgs[0][s];
    { static int v = -1; if (v < 0) { const char* e = std::getenv("PSGD_XTAB"); v = (e && e[0] == '0') ? 0 : 1; } L.use_xtab = v == 1; }
    { static int v = -1; if (v < 0) { const char* e = std::getenv("PSGD_XTAB_C"); v = (e && e[0] == '0') ? 0 : 1; } L.use_xtab_c = v == 1; }
    return L;
}

double tol2_of(const psgd_ctx* c) {
    const double t = c->opt.rank_tol > 0.f ? (double)c->opt.rank_tol : 1e-5;
    return t * t;
}

// Most iterations a layer's refresh runs
int iteration_budget(const psgd_ctx* c) { return c->opt.refresh_iters > 0 ? c->opt.refresh_iters : 16; }

// Block subspace iteration + Rayleigh-Ritz for the layers of `L`: leaves P~ (Ritz vectors of the r
// largest singular values) in thin[ROLE_P] and Q = M^T P~ in thin[ROLE_Q].
void refresh_sequence(psgd_ctx* ctx, Launcher& L, bool form_first, bool warm, float* sigma_out, int final_cp,
                      int launch_iters = 0) {
    const int wz = ctx->wz, cpz = ctx->cpz, nbz = cpz / 32;
    const int iters = iteration_budget(ctx);
    const int n_launch = launch_iters > 0 && launch_iters < iters ? launch_iters : iters;
    const double tol2 = tol2_of(ctx);
    L.prof_mute = true;
    const bool tiny = ctx->tiny_refresh && form_first;
    if (tiny) L.note(launch_tiny_iterate(L.layers, L.ids_all, L.n_all, ctx->tiny_lds, tol2, iters, warm ? 1 : 0, ctx->opt.seed, L.st));
    if (!tiny) L.note(launch_init_block(L.layers, L.ids_all, L.n_all, L.max_len(), wz, ROLE_ZQ, ROLE_Q, warm ? 1 : 0,
                             ctx->opt.seed, L.st));
    if (!tiny) L.pack(ROLE_ZQ, cpz, Launcher::PACK_TRANSPOSED);
    for (int it = 0; it < n_launch && !tiny; ++it) {
        // every layer runs its own number of iterations (decided on the device from the Ritz values of
        // its previous refresh); launches past that number find their gate closed and exit at once
        L.gate = make_gate(it, 0, iters, n_launch);
        // Z = orth(M Y);  Y = M^T Z, orthonormalised in the first kOrthYIterations iterations, later only where the factor
        // of Z says that it has to be (see Spread): the span, which is what the iteration is about, does not depend on it,
        // and once the columns of Z have lined up with the singular vectors those of M^T Z are nearly orthogonal (their norms
        // are evened out on the way, see next_scale).  The factorisation and the pass over the thin matrix are half of the
        // serial chain between the products.
        L.prod_orth(true, form_first && it == 0, nbz, ROLE_ZP, wz, tol2, cpz, 0, Launcher::PASS2_DEFERRED);
        L.prod_orth(false, false, nbz, ROLE_ZQ, wz, tol2, cpz, 1, Launcher::PASS2_NEVER, it >= kOrthYIterations);
    }
    L.gate = -1;
    // Rayleigh-Ritz on H = Y^T Y (its partial Gram matrices are the last product's)
    const bool wide = wz > kWideWidth;
    if (wide) L.note(launch_gram_sum(L.layers, L.ids_all, L.n_all, wz, ROLE_ZQ, L.gram_rows_n, L.gram_rows_t, -1, 0, L.st));
    if (!tiny) L.second_pass_deferred(wz, cpz, tol2);
    L.note(launch_jacobi(L.layers, L.ids_all, L.n_all, wz, ROLE_ZQ, wide || tiny ? kOneSlot : kGramRows1, sigma_out, L.st));
    L.note(launch_apply(L.layers, L.ids_all, L.n_all, L.max_lenP(), wz, ctx->rmax, ROLE_ZP, ROLE_P, APPLY_RITZ,
                        final_cp, -1, -2, 0.0, false, 3, 0, L.stream_wgs[0], L.st));
    L.prof_mute = false;
}

}  // namespace

extern "C" {

int psgd_init(psgd_ctx** out, int n_layers, const psgd_layer_desc* layers, int n_workers, const psgd_options* opt) {
    if (!out) return PSGD_E_INVALID_ARG;
    *out = nullptr;
    if (!layers || n_layers < 1 || n_layers > 65535 || n_workers < 1 || n_workers > 4096) return PSGD_E_INVALID_ARG;
    psgd_ctx* c = new (std::nothrow) psgd_ctx();
    if (!c) return PSGD_E_NOMEM;
    {
        static std::atomic<uint64_t> next_serial{1};
        c->serial = next_serial.fetch_add(1);
    }
    c->n_layers = n_layers;
    c->n_workers = n_workers;
    if (opt) c->opt = *opt;
    else { c->opt = psgd_options{}; c->opt.refresh_warm_start = 1; c->opt.refresh_oversample = -1; c->opt.seed = 0x5eed5eedu; }
    int rc = PSGD_OK;
    int rmax = 0;
    c->plan.resize(n_layers);
    for (int l = 0; l < n_layers && rc == PSGD_OK; ++l) {
        psgd_layer_desc d = layers[l];
        if (d.rows < 1 || d.cols < 1 || d.rows > (1 << 24) || d.cols > (1 << 24)) { rc = PSGD_E_SHAPE; break; }
        if (d.r < 1 || d.r > d.rows || d.r > d.cols) { rc = PSGD_E_SHAPE; break; }
        if (d.grad_dtype != PSGD_F32 && d.grad_dtype != PSGD_BF16) { rc = PSGD_E_INVALID_ARG; break; }
        if (d.ld == 0) d.ld = d.cols;
        if (d.ld < d.cols || d.ld % 8 != 0) { rc = PSGD_E_ALIGN; break; }
        // the kernels address a lane's pieces of a 128-row tile with 32-bit byte offsets: 127 * ld * 4 < 2^32
        if (d.ld > kMaxLd) { rc = PSGD_E_SHAPE; break; }
        Plan& p = c->plan[l];
        p.d = d;
        p.transposed = d.rows < d.cols ? 1 : 0;
        p.rowsP = (int)round_up(d.rows, kLenPad);
        p.colsP = (int)round_up(d.cols, kLenPad);
        p.m = (int)(d.rows >= d.cols ? d.rows : d.cols);
        p.n = (int)(d.rows >= d.cols ? d.cols : d.rows);
        (p.transposed ? c->lists.tr : c->lists.norm).push_back(l);
        if (d.r > rmax) rmax = d.r;
    }
    // launch order: the largest layers first (a launch ends with its shortest-lived workgroups)
    auto by_size = [&](int a, int b) {
        return c->plan[a].d.rows * c->plan[a].d.cols > c->plan[b].d.rows * c->plan[b].d.cols;
    };
    if (rc == PSGD_OK) {
        std::stable_sort(c->lists.norm.begin(), c->lists.norm.end(), by_size);
        std::stable_sort(c->lists.tr.begin(), c->lists.tr.end(), by_size);
    }
    if (rc == PSGD_OK) {
        // operand planes: bf16 gradients are compared at 2e-2, two planes (2^-17) are ample; fp32
        // gradients are held to 1e-4 of ||E||, which can be 100x smaller than ||M||: three planes
        bool any_f32 = false;
        for (auto& p : c->plan) any_f32 |= (p.d.grad_dtype == PSGD_F32);
        const int prec = c->opt.precision;
        if (prec != 0 && prec != 2 && prec != 3) rc = PSGD_E_INVALID_ARG;
        c->planes = prec ? prec : (any_f32 ? 3 : 2);
        // M between the passes: stored over E (N*sg + 20 bytes per element over the three kernels) or formed
        // again from G and E in every pass (3*N*sg + 16).  Equal bytes at N*sg = 2 (one bf16 worker), where
        // forming again makes pass 1 read-only -- but the residual then merges three streams and is the slower
        // by more than pass 1 gains (7B-shaped set: 35.4 against 31.6 ms per step), so storing is the default.
        const int pol = c->opt.m_policy;
        if (pol < 0 || pol > 2) rc = PSGD_E_INVALID_ARG;
        if (c->opt.power_iters < 0 || c->opt.power_iters > 64) rc = PSGD_E_INVALID_ARG;
        if (c->opt.refresh_iters < 0 || c->opt.refresh_iters > kMaxRefreshIterations) rc = PSGD_E_INVALID_ARG;
        c->reform_m = pol == 2;
        if (c->opt.lazy_residual != 0 && c->opt.lazy_residual != 1) rc = PSGD_E_INVALID_ARG;
        if (c->opt.q_resident != 0 && c->opt.q_resident != 1) rc = PSGD_E_INVALID_ARG;
        if (c->opt.lazy_residual && c->reform_m) rc = PSGD_E_INVALID_ARG;      // the deferred residual lives in the stored M
        c->lazy = c->opt.lazy_residual == 1;
    }
    if (rc == PSGD_OK) {
        c->rmax = rmax;
        c->cpc = (int)round_up(rmax, 32);
        int over = c->opt.refresh_oversample;
        if (over < 0) over = 8;
        if (c->opt.refresh_oversample < 0) over = rmax / 4 > 8 ? rmax / 4 : 8;
        int nmin = c->plan[0].n, nmax = c->plan[0].n;
        for (auto& p : c->plan) { nmin = std::min(nmin, p.n); nmax = std::max(nmax, p.n); }
        // A block is no wider than its matrix.  One width for all layers where the smallest matrix has room for the largest
        // rank; else each layer's own, the widest as wide as the kernels go if it has to be.
        const int full = (int)round_up(rmax + over, 8);
        c->wz = nmin >= rmax ? std::min(full, nmin) : std::min(std::min(full, nmax), kMaxWidth);
        for (auto& p : c->plan) p.wz = std::min(c->wz, p.n);
        c->cpz = (int)round_up(c->wz, 32);
        c->cpmax = c->cpz > c->cpc ? c->cpz : c->cpc;
        if (c->cpmax > kMaxWidth) rc = PSGD_E_SHAPE;
        if (c->lazy && c->cpc > 128) rc = PSGD_E_SHAPE;
        c->tiny_step = !c->lazy && !c->reform_m && c->opt.power_iters <= 1;
        c->tiny_refresh = true;
        for (const auto& p : c->plan) {
            c->tiny_step = c->tiny_step && tiny_fits(p.d.rows, p.d.cols, p.d.r, n_workers + 1, false);
            c->tiny_refresh = c->tiny_refresh && tiny_fits(p.d.rows, p.d.cols, p.wz, n_workers + 1, true);
            c->tiny_lds = std::max(c->tiny_lds, tiny_lds_bytes(p.d.rows, p.d.cols));
        }
        c->lazy_tr = c->lazy && c->cpc == 32;
        for (int s = 0; s < 2; ++s) { c->stream_wgs[0][s] = one_round(c->plan, s, false); c->stream_wgs[1][s] = one_round(c->plan, s, true); }
    }
    if (rc != PSGD_OK) { delete c; return rc; }
    {
        int64_t m_bytes = 0, tr_bytes = 0;
        bool f32 = false, b16 = false;
        for (auto& p : c->plan) {
            (p.d.grad_dtype == PSGD_F32 ? f32 : b16) = true;
            (p.transposed ? tr_bytes : m_bytes) += p.d.rows * p.d.cols * 4;
        }
        c->grad_kind = f32 && b16 ? 0 : (f32 ? 1 : 2);
        // M that the second pass can find in the 256 MB memory-side cache is stored with plain stores
        c->nt_m = m_bytes > ((int64_t)96 << 20);
        c->nt_read = m_bytes + tr_bytes > ((int64_t)96 << 20);
        if (const char* e = std::getenv("PSGD_NT_M")) c->nt_m = e[0] != '0';     // (measurement knob)
        const int n_norm = (int)c->lists.norm.size();
        if (n_norm >= 32) c->xstride = n_norm + 2;
        // The splits, and with them the workspace.  psgd_compress_static takes what fits its buffer with one split per kind of
        // product, so a context keeps to those where only that fits.
        plan_all(c, false);
        lay_out(c);
        if (c->ws_bytes > (size_t)PSGD_STATIC_WORKSPACE_BYTES) {
            plan_all(c, true);
            lay_out(c);
            if (c->ws_bytes > (size_t)PSGD_STATIC_WORKSPACE_BYTES) {
                plan_all(c, false);
                lay_out(c);
            }
        }
        // XCD table: the row-major layers (positions in the id list `norm`), largest first, each to the XCD with the
        // least work so far
        if (n_norm >= 32) {
            // work = rows x cols decides the deal (the same for both kernels), tiles = what a layer launches
            auto build = [&](std::vector<int>& tab, int& xtiles, auto tiles_of) {
                tab.assign((size_t)16 * c->xstride, 0);
                std::vector<int> order(n_norm);
                for (int i = 0; i < n_norm; ++i) order[i] = i;
                auto work_of = [&](int pos) { const Plan& p = c->plan[c->lists.norm[pos]]; return p.d.rows * p.d.cols; };
                std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return work_of(a) > work_of(b); });
                int64_t work[8] = {0, 0, 0, 0, 0, 0, 0, 0};
                int total[8] = {0, 0, 0, 0, 0, 0, 0, 0}, count[8] = {0, 0, 0, 0, 0, 0, 0, 0};
                for (int pos : order) {
                    int x = 0;
                    for (int k = 1; k < 8; ++k) if (work[k] < work[x]) x = k;
                    tab[(size_t)(8 + x) * c->xstride + count[x]] = pos;
                    total[x] += tiles_of(pos);
                    work[x] += work_of(pos);
                    count[x] += 1;
                    tab[(size_t)x * c->xstride + count[x]] = total[x];
                }
                for (int x = 0; x < 8; ++x) {
                    tab[(size_t)x * c->xstride + c->xstride - 1] = count[x];
                    if (total[x] > xtiles) xtiles = total[x];
                }
            };
            build(c->hXtab, c->xtiles, [&](int pos) { const Plan& p = c->plan[c->lists.norm[pos]]; return (p.rowsP / 32) * p.split[SPLIT_V2][0]; });
            build(c->hXtabC, c->xtiles_c, [&](int pos) { const Plan& p = c->plan[c->lists.norm[pos]]; return ((p.colsP + 255) / 256) * p.split[SPLIT_V2][1]; });
        }
    }
    double bytes = 0.0;
    for (const Plan& p : c->plan) {
        const double sg = p.d.grad_dtype == PSGD_BF16 ? 2.0 : 4.0;
        // two passes separated by the global QR: either M is stored between them (N*sg + 16 bytes
        // per element) or formed twice from the gradients (2*N*sg + 12); the smaller one counts
        const double a = n_workers * sg + 16.0, b = 2.0 * n_workers * sg + 12.0;
        bytes += (double)p.d.rows * (double)p.d.cols * (a < b ? a : b);
        bytes += 4.0 * 4.0 * (double)(p.d.rows + p.d.cols) * p.d.r;
        const double e = (double)p.d.rows * (double)p.d.cols, nsg = n_workers * sg;
        const double thin = 4.0 * (double)(p.d.rows + p.d.cols) * 32.0 * ((p.d.r + 31) / 32);
        const bool deferred = c->lazy && (!p.transposed || c->lazy_tr);
        // (deferred residual: the kept P~ and Q are read as well -- the kept Q not where the pass takes it from the
        // product's own fragments: q_resident, row-major layers)
        const double kept_q = 4.0 * (double)p.d.cols * 32.0 * ((p.d.r + 31) / 32);
        const bool shared_q = deferred && c->opt.q_resident == 1 && !p.transposed;
        if (c->tiny_step) {
            // (one launch: gradients, E and Q read; E, P~, Q and the operand copies of both written.  The other tags are the launches of
            // psgd_compress_finish)
            c->kernel_bytes[0] += e * (nsg + 8.0) + 4.0 * (p.m + 2.0 * p.n) * p.d.r + 64.0 * c->planes * (p.rowsP + p.colsP);
        } else {
            c->kernel_bytes[0] += e * (nsg + 4.0 + (c->reform_m ? 0.0 : 4.0)) + thin * (deferred ? 2.0 : 1.0) - (shared_q ? kept_q : 0.0);
        }
        c->kernel_bytes[1] += e * (c->reform_m ? nsg + 4.0 : 4.0) + thin;
        if (!deferred) c->kernel_bytes[2] += e * (c->reform_m ? nsg + 8.0 : 8.0) + thin;
    }
    c->algo_bytes = bytes;
    // host tables at their final capacity, so that no compute call allocates host memory either
    {
        const size_t nl = (size_t)n_layers, ng = nl * (size_t)n_workers;
        c->hG.reserve(ng);
        for (auto& v : c->hGs) v.reserve(ng);
        c->hE.reserve(nl); c->hQ.reserve(nl); c->hP.reserve(nl);
        c->hOut.reserve(nl); c->hMom.reserve(nl); c->hM2.reserve(nl); c->hX.reserve(nl);
        c->hIds.reserve(3 * nl + 1);
        c->hLayers.reserve(nl + 1);
    }
    *out = c;
    return PSGD_OK;
}

size_t psgd_workspace_bytes(const psgd_ctx* ctx) { return ctx ? ctx->ws_bytes : 0; }

double psgd_algorithmic_bytes(const psgd_ctx* ctx) { return ctx ? ctx->algo_bytes : 0.0; }

double psgd_kernel_bytes(const psgd_ctx* ctx, int tag) {
    return (ctx && tag >= 0 && tag < 3) ? ctx->kernel_bytes[tag] : 0.0;
}

static int bind_common(psgd_ctx* ctx, void* workspace, hipStream_t st, const void* const* G, float* const* E,
                       float* const* Q, float* const* P) {
    if (!ctx || !workspace) return PSGD_E_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(workspace) & 255u) != 0) return PSGD_E_ALIGN;
    const size_t nl = (size_t)ctx->n_layers;
    int rc;
    if (G && (rc = check_table(G, nl * ctx->n_workers)) != PSGD_OK) return rc;
    if (E && (rc = check_table(reinterpret_cast<const void* const*>(E), nl)) != PSGD_OK) return rc;
    if (Q && (rc = check_table(reinterpret_cast<const void* const*>(Q), nl)) != PSGD_OK) return rc;
    if (P && (rc = check_table(reinterpret_cast<const void* const*>(P), nl)) != PSGD_OK) return rc;
    const bool g_changed = sync_table(ctx->hG, G, nl * ctx->n_workers);
    bool changed = false;
    changed |= sync_table(ctx->hE, E, nl);
    changed |= sync_table(ctx->hQ, Q, nl);
    changed |= sync_table(ctx->hP, P, nl);
    return upload_tables(ctx, workspace, st, changed, g_changed);
}

int psgd_workspace_reset(psgd_ctx* ctx) {
    if (!ctx || ctx->pending) return PSGD_E_INVALID_ARG;
    ctx->tables_valid = false;
    ctx->bound_ws = nullptr;
    ctx->outs_ws = nullptr;
    ctx->msgd_ws = nullptr;
    ctx->m2_ws = nullptr;
    ctx->factors_ws = nullptr;
    ctx->iters_gen++;
    return PSGD_OK;
}

int psgd_compress(psgd_ctx* ctx, void* workspace, void* stream, const void* const* G, float* const* E,
                  float* const* Q, float* const* P) {
    if (!ctx || !G || !E || !Q || !P) return PSGD_E_INVALID_ARG;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (ctx->pending && ctx->bound_ws != workspace) return PSGD_E_INVALID_ARG;   // the kept operands live in the old one
    int rc = bind_common(ctx, workspace, st, G, E, Q, P);
    if (rc != PSGD_OK) return rc;
    // Q_{t-1} as a product operand: packed from the caller's buffers, unless they are promised to be what the last
    // call wrote there, whose operand copies are still in place
    const bool q_in_place = ctx->opt.q_resident == 1 && ctx->factors_ws == workspace;
    ctx->factors_ws = nullptr;
    Launcher L = batch_launcher(ctx, workspace, st);
    const int cp = ctx->cpc, nb = cp / 32;
    if (ctx->tiny_step) {
        // (Q_{t-1} from the caller's buffers: where they are promised to be untouched they hold what the copies do)
        const int k = L.prof_begin(PSGD_PROF_SWEEP1);
        L.note(launch_tiny_step(L.layers, L.ids_all, L.n_all, ctx->tiny_lds, tol2_of(ctx), st));
        L.prof_end(k);
        if (L.err != hipSuccess) return fail_hip(ctx, L.err);
        ctx->factors_ws = workspace;
        ctx->factors_kept = false;
        return PSGD_OK;
    }
    if (!q_in_place) L.pack(ROLE_Q, cp, Launcher::PACK_TRANSPOSED);
    // P = M Q_{t-1} (M formed on the way and, unless it is formed again below, stored over E);
    // P~ = QR(P), operand copies of P~;  Q_t = M^T P~, operand copies of Q_t;  K times (Eq. (8)), K = 1 by default
    const bool re = ctx->reform_m;
    const int K = ctx->opt.power_iters > 0 ? ctx->opt.power_iters : 1;
    L.kept_packs = ctx->lazy;
    for (int k = 0; k < K; ++k) {
        L.keep_e = re;
        L.lazy_form = ctx->pending;            // E of the row-major layers is M_{t-1} - (kept P~)(kept Q)^T
        L.lazy_share = q_in_place;
        L.prod_orth(true, k == 0 || re, nb, ROLE_P, ctx->rmax, tol2_of(ctx), cp, 0, Launcher::PASS2_ALWAYS);
        if (k == 0) ctx->pending = false;      // the buffers hold M_t from here on
        L.lazy_form = false;
        L.prod(false, re, nb, ROLE_Q, EPI_PACK);
        L.keep_e = false;
    }
    if (ctx->lazy) {
        L.residual_deferred(nb);                   // owed: E <- M - P~ Q_t^T, applied by the next forming pass
        ctx->pending = L.n_norm > 0 || ctx->lazy_tr;
    } else {
        L.residual(nb, re);                        // E <- M - P~ Q_t^T
    }
    if (L.err != hipSuccess) return fail_hip(ctx, L.err);
    ctx->factors_ws = workspace;                   // the operand copies of P~_t and Q_t are in place
    ctx->factors_kept = ctx->lazy;
    return PSGD_OK;
}

// The built-in workspace of psgd_compress_static: one array per GPU (every device that loads this code object holds its
// own copy at its own address).  In host code the array's name is only a handle for hipGetSymbolAddress; the device
// address it returns, looked up once per device with that device current, is what is passed on.
static __device__ __align__(256) unsigned char g_static_workspace[PSGD_STATIC_WORKSPACE_BYTES];
namespace {
constexpr int kMaxDevices = 64;
struct StaticWorkspace { void* ptr = nullptr; uint64_t owner = 0; };
StaticWorkspace g_static_ws[kMaxDevices];
std::mutex g_static_mutex;
}  // namespace

int psgd_compress_static(psgd_ctx* ctx, void* stream, const void* const* G, float* const* E, float* const* Q,
                         float* const* P) {
    if (!ctx || !G || !E || !Q || !P) return PSGD_E_INVALID_ARG;
    if (ctx->ws_bytes > (size_t)PSGD_STATIC_WORKSPACE_BYTES) return PSGD_E_TOO_LARGE;
    int dev = -1;
    PSGD_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return PSGD_E_INVALID_ARG;
    void* ws = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_static_mutex);
        StaticWorkspace& W = g_static_ws[dev];
        if (!W.ptr) {
            void* p = nullptr;
            PSGD_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(g_static_workspace)));
            if (!p) return fail_hip(ctx, hipErrorInvalidSymbol);
            W.ptr = p;
        }
        ws = W.ptr;
        if (W.owner != ctx->serial) {
            // another context's tables, counters and operand copies are in the buffer (or nothing yet)
            if (ctx->pending && ctx->bound_ws == ws) return PSGD_E_INVALID_ARG;      // its kept operands are gone
            if (ctx->bound_ws == ws) { ctx->tables_valid = false; ctx->iters_gen++; }
            if (ctx->outs_ws == ws) ctx->outs_ws = nullptr;
            if (ctx->msgd_ws == ws) ctx->msgd_ws = nullptr;
            if (ctx->m2_ws == ws) ctx->m2_ws = nullptr;
            if (ctx->factors_ws == ws) ctx->factors_ws = nullptr;
            W.owner = ctx->serial;
        }
    }
    return psgd_compress(ctx, ws, stream, G, E, Q, P);
}

// The two halves of psgd_compress between which a data-parallel job averages P over its workers (and after which
// it averages Q): each worker runs them on its own gradient and error buffer.
int psgd_compress_project(psgd_ctx* ctx, void* workspace, void* stream, const void* const* G, float* const* E,
                          float* const* Q, float* const* P) {
    if (!ctx || !G || !E || !Q || !P) return PSGD_E_INVALID_ARG;
    if (ctx->lazy || ctx->reform_m || ctx->opt.power_iters > 1) return PSGD_E_INVALID_ARG;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    int rc = bind_common(ctx, workspace, st, G, E, Q, P);
    if (rc != PSGD_OK) return rc;
    ctx->factors_ws = nullptr;
    Launcher L = batch_launcher(ctx, workspace, st);
    const int cp = ctx->cpc, nb = cp / 32;
    L.pack(ROLE_Q, cp, Launcher::PACK_TRANSPOSED);
    L.prod(true, true, nb, ROLE_P, EPI_NONE);          // M = mean G + E stored over E;  P = M Q_{t-1}, as it is
    if (L.err != hipSuccess) return fail_hip(ctx, L.err);
    return PSGD_OK;
}

int psgd_compress_finish(psgd_ctx* ctx, void* workspace, void* stream, float* const* E, float* const* Q,
                         float* const* P) {
    if (!ctx || !E || !Q || !P) return PSGD_E_INVALID_ARG;
    if (ctx->lazy || ctx->reform_m || ctx->opt.power_iters > 1) return PSGD_E_INVALID_ARG;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    int rc = bind_common(ctx, workspace, st, nullptr, E, Q, P);
    if (rc != PSGD_OK) return rc;
    Launcher L = batch_launcher(ctx, workspace, st);
    const int cp = ctx->cpc, nb = cp / 32;
    L.orth_given(ROLE_P, ctx->rmax, tol2_of(ctx), cp);  // P~ = QR(P), operand copies of P~
    L.prod(false, false, nb, ROLE_Q, EPI_PACK);         // Q = M^T P~ (this worker's M), operand copies
    L.residual(nb, false);                              // E <- M - P~ Q^T
    if (L.err != hipSuccess) return fail_hip(ctx, L.err);
    ctx->factors_ws = workspace;                        // (copies of P~ and of this worker's Q)
    ctx->factors_kept = false;
    return PSGD_OK;
}

int psgd_flush_residual(psgd_ctx* ctx, void* workspace, void* stream, float* const* E) {
    if (!ctx || !E) return PSGD_E_INVALID_ARG;
    if (!ctx->pending) return PSGD_OK;
    if (ctx->bound_ws != workspace) return PSGD_E_INVALID_ARG;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    int rc = bind_common(ctx, workspace, st, nullptr, E, nullptr, nullptr);
    if (rc != PSGD_OK) return rc;
    Launcher L = batch_launcher(ctx, workspace, st);
    L.prof_mute = true;
    L.residual_owed(ctx->cpc / 32);
    ctx->pending = false;
    if (L.err != hipSuccess) return fail_hip(ctx, L.err);
    return PSGD_OK;
}

int psgd_compress_refresh(psgd_ctx* ctx, void* workspace, void* stream, const void* const* G, float* const* E,
                          float* const* Q, float* const* P) {
    if (!ctx || !G || !E || !Q || !P) return PSGD_E_INVALID_ARG;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (ctx->pending && ctx->bound_ws != workspace) return PSGD_E_INVALID_ARG;   // the kept operands live in the old one
    int rc = bind_common(ctx, workspace, st, G, E, Q, P);
    if (rc != PSGD_OK) return rc;
    ctx->factors_ws = nullptr;
    Launcher L = batch_launcher(ctx, workspace, st);
    for (int s = 0; s < 2; ++s) L.stream_wgs[s] = ctx->stream_wgs[1][s];
    if (ctx->pending) {
        // the subspace iteration forms M from a materialised E: settle what the deferred residual owes first
        L.prof_mute = true;
        L.residual_owed(ctx->cpc / 32);
        L.prof_mute = false;
        ctx->pending = false;
    }
    // how many iterations to launch: the bound fetched behind the last refresh, if that copy has arrived and nothing
    // else has changed the counts since.  (None of this bookkeeping under stream capture: a captured refresh
    // launches the whole budget and fetches nothing.)
    const bool capturing = is_capturing(st);
    int bound = 0;
    if (!capturing && ctx->fetch_last >= 0) {
        psgd_ctx::IterFetch& F = ctx->fetch[ctx->fetch_last];
        if (F.pending && hipEventQuery(F.ev) == hipSuccess) {
            F.pending = false;
            if (F.gen == ctx->iters_gen && F.seq == ctx->refresh_seq) bound = F.h[0];
        }
        (void)hipGetLastError();      // (hipErrorNotReady of the query is not an error)
    }
    const int iters_max = iteration_budget(ctx);
    refresh_sequence(ctx, L, true, ctx->opt.refresh_warm_start != 0, nullptr, ctx->cpc, bound);
    L.residual(ctx->cpc / 32);
    ctx->refresh_seq++;
    ctx->fetch_last = -1;
    if (capturing) ctx->iters_gen++;
    if (ctx->tiny_refresh) {                          // (its one launch knows the counts)
        if (L.err != hipSuccess) return fail_hip(ctx, L.err);
        ctx->factors_ws = workspace;
        ctx->factors_kept = false;
        return PSGD_OK;
    }
    // fetch the bound for the next one (pinned words and events are created on first use; without them every
    // refresh simply launches the whole budget)
    if (!capturing && !ctx->fetch_ready && !ctx->fetch_failed) {
        void* hp = nullptr;
        bool ok = hipHostMalloc(&hp, psgd_ctx::kIterSlots * sizeof(int), hipHostMallocDefault) == hipSuccess;
        for (int k = 0; ok && k < psgd_ctx::kIterSlots; ++k) {
            ctx->fetch[k].h = static_cast<int*>(hp) + k;
            ok = hipEventCreateWithFlags(&ctx->fetch[k].ev, hipEventDisableTiming) == hipSuccess;
            if (!ok) ctx->fetch[k].ev = nullptr;
        }
        if (!ok) {
            for (auto& F : ctx->fetch) { if (F.ev) (void)hipEventDestroy(F.ev); F.ev = nullptr; F.h = nullptr; }
            if (hp) (void)hipHostFree(hp);
            ctx->fetch_failed = true;
        }
        ctx->fetch_ready = ok;
        (void)hipGetLastError();
    }
    if (!capturing && ctx->fetch_ready) {
        int slot = -1;
        for (int k = 0; k < psgd_ctx::kIterSlots && slot < 0; ++k) {
            psgd_ctx::IterFetch& F = ctx->fetch[k];
            if (F.pending && hipEventQuery(F.ev) == hipSuccess) F.pending = false;
            if (!F.pending) slot = k;
        }
        (void)hipGetLastError();
        if (slot >= 0) {
            psgd_ctx::IterFetch& F = ctx->fetch[slot];
            int* d_it = reinterpret_cast<int*>(L.ws + ctx->off_iters) + slot;
            L.note(launch_max_iterations(L.layers, L.ids_all, L.n_all, iters_max, d_it, st));
            L.note(hipMemcpyAsync(F.h, d_it, sizeof(int), hipMemcpyDeviceToHost, st));
            L.note(hipEventRecord(F.ev, st));
            if (L.err == hipSuccess) {
                F.pending = true; F.gen = ctx->iters_gen; F.seq = ctx->refresh_seq;
                ctx->fetch_last = slot;
            }
        }
    }
    if (L.err != hipSuccess) return fail_hip(ctx, L.err);
    ctx->factors_ws = workspace;
    ctx->factors_kept = false;
    return PSGD_OK;
}

int psgd_refresh(psgd_ctx* ctx, void* workspace, void* stream, int layer, const float* M, float* P, float* Q,
                 float* sigma) {
    if (!ctx || !workspace || !M || !P || !Q) return PSGD_E_INVALID_ARG;
    if (layer < 0 || layer >= ctx->n_layers) return PSGD_E_INVALID_ARG;
    if (!aligned16(M) || !aligned16(P) || !aligned16(Q)) return PSGD_E_ALIGN;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    int rc = bind_common(ctx, workspace, st, nullptr, nullptr, nullptr, nullptr);
    if (rc != PSGD_OK) return rc;
    char* ws = reinterpret_cast<char*>(workspace);
    if (is_capturing(st)) return PSGD_E_CAPTURE;       // (every call uploads a descriptor from the host)
    ctx->factors_ws = nullptr;                         // (it rewrites operand copies of this layer)
    const Plan& p = ctx->plan[layer];
    // scratch descriptor: this layer's private regions, the caller's M/P/Q, splits sized for one layer
    LayerDev D;
    build_layer_dev(ctx, ws, layer, ctx->cur_slot, &D);
    D.S = const_cast<float*>(M);
    D.thin[ROLE_P].ptr = P;
    D.thin[ROLE_Q].ptr = Q;
    Plan one = p;
    // (every product of this call is one of the iteration)
    for (int m = 0; m < 2; ++m) {
        D.split[SPLIT_ITER][m] = one.split[SPLIT_ITER][m] = p.split_alone[m];
        if (ctx->n_layers > 1) D.part[m] = reinterpret_cast<float*>(ws + ctx->off_alone[m]);
    }
    ctx->hLayers[ctx->n_layers] = D;
    PSGD_TRY(launch_put(ws + ctx->off_layers_s[ctx->cur_slot] + (size_t)ctx->n_layers * sizeof(LayerDev), &D, sizeof(LayerDev), st));
    // this call rewrites the layer's iteration count: what the host knows about the next batched refresh is void
    ctx->iters_gen++;
    Launcher L{};
    L.ctx = ctx; L.ws = ws; L.st = st;
    L.layers = reinterpret_cast<const LayerDev*>(ws + ctx->off_layers_s[ctx->cur_slot]);
    const int* ids = reinterpret_cast<const int*>(ws + ctx->off_ids) + 3 * (size_t)ctx->n_layers;
    L.ids_all = ids; L.n_all = 1;
    L.ids_norm = ids; L.n_norm = p.transposed ? 0 : 1;
    L.ids_tr = ids; L.n_tr = p.transposed ? 1 : 0;
    geometry(one, L);
    for (int s = 0; s < 2; ++s) L.stream_wgs[s] = one_round({one}, s, true);
    refresh_sequence(ctx, L, false, false, sigma, 0);
    if (L.err != hipSuccess) return fail_hip(ctx, L.err);
    return PSGD_OK;
}

// Factors of a decompress-type call: the caller's P and Q (packed by the call), or, with both tables null, the
// operand copies the last compress-type call left in this workspace.  *packed: whether the copies are in place.
static int bind_factors(psgd_ctx* ctx, void* workspace, hipStream_t st, const float* const* P, const float* const* Q,
                        bool* packed) {
    *packed = !P && !Q;
    if (*packed) {
        if (!workspace || ctx->factors_ws != workspace) return PSGD_E_INVALID_ARG;
        return bind_common(ctx, workspace, st, nullptr, nullptr, nullptr, nullptr);
    }
    if (!P || !Q) return PSGD_E_INVALID_ARG;
    ctx->factors_ws = nullptr;          // the copies will be the caller's P and Q
    return bind_common(ctx, workspace, st, nullptr, nullptr, const_cast<float* const*>(Q), const_cast<float* const*>(P));
}

int psgd_decompress(psgd_ctx* ctx, void* workspace, void* stream, const float* const* P, const float* const* Q,
                    void* const* out, int out_dtype) {
    if (!ctx || !out) return PSGD_E_INVALID_ARG;
    if (out_dtype != PSGD_F32 && out_dtype != PSGD_BF16) return PSGD_E_INVALID_ARG;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    int rc = check_table(reinterpret_cast<const void* const*>(out), (size_t)ctx->n_layers);
    if (rc != PSGD_OK) return rc;
    bool packed = false;
    rc = bind_factors(ctx, workspace, st, P, Q, &packed);
    if (rc != PSGD_OK) return rc;
    char* ws = reinterpret_cast<char*>(workspace);
    if (sync_table(ctx->hOut, out, (size_t)ctx->n_layers) || ctx->outs_ws != workspace) {
        if (is_capturing(st)) { ctx->outs_ws = nullptr; return PSGD_E_CAPTURE; }
        PSGD_TRY(launch_put(ws + ctx->off_outs, ctx->hOut.data(), ctx->hOut.size() * sizeof(void*), st));
    }
    ctx->outs_ws = workspace;
    Launcher L = batch_launcher(ctx, workspace, st);
    const int cp = ctx->cpc, nb = cp / 32;
    if (!packed) L.pack(ROLE_P, cp, Launcher::PACK_OUTER, ROLE_Q);
    // (factors of a compress call with a deferred residual: the layers that defer hold them as their kept copies)
    const bool kept = packed && ctx->factors_kept;
    const int n_kept = !kept ? 0 : ctx->lazy_tr ? L.n_all : L.n_norm;
    const int* ids_kept = ctx->lazy_tr ? L.ids_all : L.ids_norm;
    void* const* outs = reinterpret_cast<void* const*>(ws + ctx->off_outs);
    const int obf = out_dtype == PSGD_BF16 ? 1 : 0;
    if (n_kept > 0) L.note(launch_outer(nb, ctx->planes, true, false, true, L.layers, ids_kept, n_kept, L.outer_tiles(nb), L.outer_rows(nb), outs, obf, st));
    if (!kept) L.note(launch_outer(nb, ctx->planes, true, false, false, L.layers, L.ids_all, L.n_all, L.outer_tiles(nb), L.outer_rows(nb), outs, obf, st));
    else if (!ctx->lazy_tr) L.note(launch_outer(nb, ctx->planes, true, false, false, L.layers, L.ids_tr, L.n_tr, L.outer_tiles(nb), L.outer_rows(nb), outs, obf, st));
    if (L.err != hipSuccess) return fail_hip(ctx, L.err);
    return PSGD_OK;
}

int psgd_decompress_msgd(psgd_ctx* ctx, void* workspace, void* stream, const float* const* P, const float* const* Q,
                         float* const* mom, float* const* X, float mu, float eta) {
    if (!ctx || !mom || !X) return PSGD_E_INVALID_ARG;
    if (!(mu >= 0.f && mu < 1.f) || !(eta == eta)) return PSGD_E_INVALID_ARG;      // Algorithm 2: 0 <= mu < 1
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const size_t nl = (size_t)ctx->n_layers;
    int rc = check_table(reinterpret_cast<const void* const*>(mom), nl);
    if (rc == PSGD_OK) rc = check_table(reinterpret_cast<const void* const*>(X), nl);
    if (rc != PSGD_OK) return rc;
    bool packed = false;
    rc = bind_factors(ctx, workspace, st, P, Q, &packed);
    if (rc != PSGD_OK) return rc;
    char* ws = reinterpret_cast<char*>(workspace);
    const bool changed = sync_table(ctx->hMom, mom, nl) | sync_table(ctx->hX, X, nl);
    if (changed || ctx->msgd_ws != workspace) {
        if (is_capturing(st)) { ctx->msgd_ws = nullptr; return PSGD_E_CAPTURE; }
        PSGD_TRY(launch_put(ws + ctx->off_moms, ctx->hMom.data(), nl * sizeof(void*), st));
        PSGD_TRY(launch_put(ws + ctx->off_xs, ctx->hX.data(), nl * sizeof(void*), st));
    }
    ctx->msgd_ws = workspace;
    Launcher L = batch_launcher(ctx, workspace, st);
    const int cp = ctx->cpc, nb = cp / 32;
    if (!packed) L.pack(ROLE_P, cp, Launcher::PACK_OUTER, ROLE_Q);
    const bool kept = packed && ctx->factors_kept;      // (see psgd_decompress)
    const int n_kept = !kept ? 0 : ctx->lazy_tr ? L.n_all : L.n_norm;
    const int* ids_kept = ctx->lazy_tr ? L.ids_all : L.ids_norm;
    float* const* dm = reinterpret_cast<float* const*>(ws + ctx->off_moms);
    float* const* dx = reinterpret_cast<float* const*>(ws + ctx->off_xs);
    if (n_kept > 0) L.note(launch_msgd(nb, ctx->planes, L.layers, ids_kept, n_kept, L.outer_tiles(nb), L.outer_rows(nb), dm, dx, mu, eta, true, st));
    if (!kept) L.note(launch_msgd(nb, ctx->planes, L.layers, L.ids_all, L.n_all, L.outer_tiles(nb), L.outer_rows(nb), dm, dx, mu, eta, false, st));
    else if (!ctx->lazy_tr) L.note(launch_msgd(nb, ctx->planes, L.layers, L.ids_tr, L.n_tr, L.outer_tiles(nb), L.outer_rows(nb), dm, dx, mu, eta, false, st));
    if (L.err != hipSuccess) return fail_hip(ctx, L.err);
    return PSGD_OK;
}

int psgd_decompress_adam(psgd_ctx* ctx, void* workspace, void* stream, const float* const* P, const float* const* Q,
                         float* const* m1, float* const* m2, float* const* X, int step, float eta, float beta1,
                         float beta2, float eps, float weight_decay) {
    if (!ctx || !m1 || !m2 || !X) return PSGD_E_INVALID_ARG;
    if (step < 1 || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps >= 0.f) ||
        !(eta == eta) || !(weight_decay == weight_decay))
        return PSGD_E_INVALID_ARG;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const size_t nl = (size_t)ctx->n_layers;
    int rc = check_table(reinterpret_cast<const void* const*>(m1), nl);
    if (rc == PSGD_OK) rc = check_table(reinterpret_cast<const void* const*>(m2), nl);
    if (rc == PSGD_OK) rc = check_table(reinterpret_cast<const void* const*>(X), nl);
    if (rc != PSGD_OK) return rc;
    bool packed = false;
    rc = bind_factors(ctx, workspace, st, P, Q, &packed);
    if (rc != PSGD_OK) return rc;
    char* ws = reinterpret_cast<char*>(workspace);
    const bool changed = sync_table(ctx->hMom, m1, nl) | sync_table(ctx->hX, X, nl);
    if (changed || ctx->msgd_ws != workspace) {
        if (is_capturing(st)) { ctx->msgd_ws = nullptr; return PSGD_E_CAPTURE; }
        PSGD_TRY(launch_put(ws + ctx->off_moms, ctx->hMom.data(), nl * sizeof(void*), st));
        PSGD_TRY(launch_put(ws + ctx->off_xs, ctx->hX.data(), nl * sizeof(void*), st));
    }
    ctx->msgd_ws = workspace;
    if (sync_table(ctx->hM2, m2, nl) || ctx->m2_ws != workspace) {
        if (is_capturing(st)) { ctx->m2_ws = nullptr; return PSGD_E_CAPTURE; }
        PSGD_TRY(launch_put(ws + ctx->off_m2s, ctx->hM2.data(), nl * sizeof(void*), st));
    }
    ctx->m2_ws = workspace;
    // bias corrections in double: 1 - beta^t loses nothing for beta close to 1 and small t
    const double bc1 = 1.0 - std::pow((double)beta1, (double)step), bc2 = 1.0 - std::pow((double)beta2, (double)step);
    const float coef[8] = {beta1, beta2, (float)(1.0 - (double)beta1), (float)(1.0 - (double)beta2),
                           (float)((double)eta / bc1), (float)(1.0 / std::sqrt(bc2)), eps,
                           (float)((double)eta * (double)weight_decay)};
    Launcher L = batch_launcher(ctx, workspace, st);
    const int cp = ctx->cpc, nb = cp / 32;
    if (!packed) L.pack(ROLE_P, cp, Launcher::PACK_OUTER, ROLE_Q);
    const bool kept = packed && ctx->factors_kept;      // (see psgd_decompress)
    const int n_kept = !kept ? 0 : ctx->lazy_tr ? L.n_all : L.n_norm;
    const int* ids_kept = ctx->lazy_tr ? L.ids_all : L.ids_norm;
    float* const* d1 = reinterpret_cast<float* const*>(ws + ctx->off_moms);
    float* const* d2 = reinterpret_cast<float* const*>(ws + ctx->off_m2s);
    float* const* dx = reinterpret_cast<float* const*>(ws + ctx->off_xs);
    if (n_kept > 0) L.note(launch_adam(nb, ctx->planes, L.layers, ids_kept, n_kept, L.outer_tiles(nb), L.outer_rows(nb), d1, d2, dx, coef, true, st));
    if (!kept) L.note(launch_adam(nb, ctx->planes, L.layers, L.ids_all, L.n_all, L.outer_tiles(nb), L.outer_rows(nb), d1, d2, dx, coef, false, st));
    else if (!ctx->lazy_tr) L.note(launch_adam(nb, ctx->planes, L.layers, L.ids_tr, L.n_tr, L.outer_tiles(nb), L.outer_rows(nb), d1, d2, dx, coef, false, st));
    if (L.err != hipSuccess) return fail_hip(ctx, L.err);
    return PSGD_OK;
}

int psgd_status(psgd_ctx* ctx, void* workspace, void* stream, int layer, psgd_layer_status* out) {
    if (!ctx || !workspace || !out || layer < 0 || layer >= ctx->n_layers) return PSGD_E_INVALID_ARG;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    PSGD_TRY(hipStreamSynchronize(st));
    char* ws = reinterpret_cast<char*>(workspace);
    const LayerRegion R = layer_region(ctx, ctx->plan[layer]);
    int raw[kStatusWords] = {};
    PSGD_TRY(hipMemcpy(raw, ws + ctx->off_layer[layer] + R.status, sizeof(raw), hipMemcpyDeviceToHost));
    out->rank_deficient = raw[0];
    out->refresh_iters_next = raw[4];
    out->refresh_iters_no_gap = raw[9] < 2 ? 2 : raw[9];
    std::memcpy(&out->sigma_max, &raw[2], sizeof(float));
    std::memcpy(&out->sigma_r, &raw[3], sizeof(float));
    return PSGD_OK;
}

int psgd_copy_bytes(void* stream, void* dst, const void* src, size_t n_bytes) {
    if (!dst || !src || (n_bytes & 15u) || !aligned16(dst) || !aligned16(src)) return PSGD_E_INVALID_ARG;
    hipError_t e = launch_copy(dst, src, n_bytes, reinterpret_cast<hipStream_t>(stream));
    return e == hipSuccess ? PSGD_OK : PSGD_E_HIP;
}

int psgd_last_hip_error(const psgd_ctx* ctx) { return ctx ? ctx->last_hip : 0; }

const char* psgd_strerror(int code) {
    switch (code) {
        case PSGD_OK: return "ok";
        case PSGD_E_INVALID_ARG: return "invalid argument";
        case PSGD_E_SHAPE: return "unsupported shape or rank";
        case PSGD_E_ALIGN: return "leading dimension or pointer alignment";
        case PSGD_E_HIP: return "HIP runtime error";
        case PSGD_E_NOMEM: return "out of host memory";
        case PSGD_E_CAPTURE: return "stream capture: pointer tables not on the device yet (make the same call eagerly once first)";
        case PSGD_E_TOO_LARGE: return "the context needs more workspace than the library's built-in buffer holds";
        default: return "unknown error";
    }
}

int psgd_profile_enable(psgd_ctx* ctx, int max_records) {
    if (!ctx || max_records < 0 || max_records > (1 << 20)) return PSGD_E_INVALID_ARG;
    for (hipEvent_t e : ctx->prof_ev) (void)hipEventDestroy(e);
    ctx->prof_ev.clear();
    ctx->prof_tag.assign((size_t)max_records, 0);
    ctx->prof_used = 0;
    ctx->prof_on = max_records > 0;
    for (int i = 0; i < 2 * max_records; ++i) {
        hipEvent_t e;
        PSGD_TRY(hipEventCreate(&e));
        ctx->prof_ev.push_back(e);
    }
    return PSGD_OK;
}

int psgd_profile_select(psgd_ctx* ctx, int tag_mask) {
    if (!ctx || tag_mask < 0 || tag_mask >= (1 << PSGD_PROF_TAGS)) return PSGD_E_INVALID_ARG;
    ctx->prof_mask = tag_mask;
    return PSGD_OK;
}

int psgd_profile_read(psgd_ctx* ctx, double* total_ms, int* count, int n_tags) {
    if (!ctx || !total_ms || !count || n_tags < 1) return PSGD_E_INVALID_ARG;
    for (int t = 0; t < n_tags; ++t) { total_ms[t] = 0.0; count[t] = 0; }
    for (size_t k = 0; k < ctx->prof_used; ++k) {
        PSGD_TRY(hipEventSynchronize(ctx->prof_ev[2 * k + 1]));
        float ms = 0.f;
        PSGD_TRY(hipEventElapsedTime(&ms, ctx->prof_ev[2 * k], ctx->prof_ev[2 * k + 1]));
        const int t = ctx->prof_tag[k];
        if (t >= 0 && t < n_tags) { total_ms[t] += ms; count[t] += 1; }
    }
    ctx->prof_used = 0;
    return PSGD_OK;
}

void psgd_destroy(psgd_ctx* ctx) {
    if (!ctx) return;
    for (auto& F : ctx->fetch) {
        if (F.pending) (void)hipEventSynchronize(F.ev);
        if (F.ev) (void)hipEventDestroy(F.ev);
    }
    if (ctx->fetch[0].h) (void)hipHostFree(ctx->fetch[0].h);
    for (hipEvent_t e : ctx->prof_ev) (void)hipEventDestroy(e);
    delete ctx;
}

}  // extern "C"
