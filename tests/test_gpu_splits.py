"""Batches of layers of very different sizes and both orientations: every launch cuts its layers' reductions into pieces of
about the same length, so one batch holds layers cut many times, twice, and (where a launch fills the GPU) not at all."""
import numpy as np
import pytest

from oracle import psgd_oracle as orc
from paper_2509_11254_amd import synth
from gpu_harness import Case, back, logical, to_dev_grad, torch_mod

pytestmark = pytest.mark.gpu

MIXED = [(72, 200), (200, 72), (264, 1000), (1000, 264), (64, 64), (70, 2056), (2056, 70), (130, 136), (65, 80)]
TOL = {synth.F32: 1e-4, synth.BF16: 2e-2}


# r = 8: operands 32 wide; r = 33: 64 wide; 24 layers of 1000 rows: row products on 768 workgroups, not split; deferred
# residual: kept operand copies from the row product (width 32) and none for these layers (width 64)
@pytest.mark.parametrize("shapes", [MIXED, [(72, 264)], [(1000, 1032)] * 24], ids=["mixed", "single", "unsplit"])
@pytest.mark.parametrize("r,dtype,lazy", [(8, synth.F32, False), (33, synth.BF16, False), (8, synth.BF16, True), (33, synth.F32, True)])
def test_ssp_steps(shapes, r, dtype, lazy):
    rng = np.random.default_rng(len(shapes) * 100 + r)
    n_workers, steps = 2, 2
    lds = [(c + 7) // 8 * 8 for _, c in shapes]
    sig = [rng.standard_normal((rw, 12)) * 0.7 ** np.arange(12) @ rng.standard_normal((12, cl)) for rw, cl in shapes]

    def grad(s):
        g = (s + 0.05 * rng.standard_normal(s.shape)).astype(np.float32)
        return synth.round_to_bf16(g) if dtype == synth.BF16 else g

    case = Case(shapes, r, n_workers, dtype, lds=lds, lazy_residual=lazy)
    errs = [(0.05 * rng.standard_normal(s)).astype(np.float32) for s in shapes]
    qs = []
    for s in sig:                                            # (a Q of a run under way: near the leading subspace)
        v = np.linalg.svd(logical(s, *s.shape), full_matrices=False)[2][:r].T
        qs.append((v + 0.02 * rng.standard_normal(v.shape)).astype(np.float32))
    q_or = [q.astype(np.float64) for q in qs]
    e_or = [logical(e.astype(np.float64), *e.shape) for e in errs]
    for t in range(steps):
        grads = [[grad(s) for _ in range(n_workers)] for s in sig]
        if t == 0:
            case.upload(grads, errs, qs)
        else:
            case.G = [[to_dev_grad(g, lds[l]) for g in grads[l]] for l in range(len(shapes))]
        case.compress()
        for l, (rw, cl) in enumerate(shapes):
            g = [logical(synth.gradient_as_f64(x), rw, cl) for x in grads[l]]
            m = np.mean(g, axis=0) + e_or[l]
            out = orc.ssp_comp(q_or[l], [m])
            p, q = back(case.P[l]), back(case.Q[l])
            # (bound: that of the parity tests, relative Frobenius)
            assert orc.rel_fro(p @ q.T, out.delta_hat) <= TOL[dtype], (t, l, rw, cl)
            assert np.abs(p.T @ p - np.eye(r)).max() < 2e-5, (t, l, rw, cl)
            # the next step continues from the library's own factors, as its error buffer does
            q_or[l], e_or[l] = q, m - p @ q.T
    if lazy:
        case.comp.flush_residual(case.E)
    for l, (rw, cl) in enumerate(shapes):
        assert orc.rel_fro(logical(back(case.E[l], cl), rw, cl), e_or[l]) <= TOL[dtype], (l, rw, cl)


def _first_layer_errors(shapes, r, seed=5):
    """Errors of layer 0's P~ and Q after one step, against fp64 (relative Frobenius); layer 0 is the same for any shapes[1:]."""
    rng = np.random.default_rng(seed)
    rows, cols = shapes[0]
    m = rng.standard_normal((rows, cols)).astype(np.float32)
    q0 = rng.standard_normal((min(rows, cols), r)).astype(np.float32)
    small = {s: rng.standard_normal(s).astype(np.float32) for s in dict.fromkeys(shapes)}
    case = Case(shapes, r, 1, synth.F32)
    case.upload([[m]] + [[small[s]] for s in shapes[1:]], [np.zeros(s, np.float32) for s in shapes],
                [q0] + [rng.standard_normal((min(s), r)).astype(np.float32) for s in shapes[1:]])
    case.compress()
    p, q, _ = case.outputs(0)
    m64 = m.astype(np.float64)
    return orc.rel_fro(p, orc.ssp_comp(q0.astype(np.float64), [m64]).p_tilde), orc.rel_fro(q, m64.T @ p)


# The error of an fp32 sum grows with the number of its terms.  A matrix's products are cut into no fewer pieces because its
# batch comes near to filling the GPU (224 workgroups of 256, where 160 are cut in two), nor because it holds longer
# matrices beside it; the same pieces give the same errors (a quarter is left for the orders of the sums).
@pytest.mark.parametrize("fewer,more,r,which", [([(4096, 1024)] * 5, [(4096, 1024)] * 7, 100, 0),
                                                ([(2048, 2048)] * 12, [(2048, 2048)] * 8 + [(5632, 2048)] * 4, 16, 1)], ids=["P", "Q"])
def test_errors_do_not_depend_on_the_batch(fewer, more, r, which):
    few, many = _first_layer_errors(fewer, r)[which], _first_layer_errors(more, r)[which]
    assert many <= 1.25 * few, (few, many)


# two planes at r = 112: the step's products run at width 128 and the refresh's iteration at 160, with other splits, in the
# same context and, one after the other, on the same partial sums
@pytest.mark.parametrize("shapes", [[(1000, 520)], [(520, 1000)], [(1000, 520), (264, 1496), (2056, 264)]])
def test_step_and_refresh_at_different_widths(shapes):
    rng = np.random.default_rng(len(shapes))
    r, tol = 112, TOL[synth.BF16]
    ms = [synth.round_to_bf16((np.linalg.qr(rng.standard_normal((s[0], min(s))))[0] * 0.97 ** np.arange(min(s)) @
                               np.linalg.qr(rng.standard_normal((s[1], min(s))))[0].T).astype(np.float32)) for s in shapes]
    case = Case(shapes, r, 1, synth.BF16)
    for refresh in (False, True, False, True):
        case.upload([[m] for m in ms], [np.zeros(s, np.float32) for s in shapes],
                    [rng.standard_normal((min(s), r)).astype(np.float32) for s in shapes])
        q0 = [back(q) for q in case.Q]
        case.compress(refresh=refresh)
        for l, (rows, cols) in enumerate(shapes):
            p, q, e = case.outputs(l)
            m = logical(synth.gradient_as_f64(ms[l]), rows, cols)
            e = logical(e, rows, cols)
            nm = np.linalg.norm(m)
            assert np.abs(p.T @ p - np.eye(r)).max() < 2e-5, (l, refresh)
            assert np.linalg.norm(q - m.T @ p) <= tol * nm and np.linalg.norm(e - (m - p @ q.T)) <= tol * nm, (l, refresh)
            if refresh:
                tail = np.sum(np.linalg.svd(m, compute_uv=False)[r:] ** 2)
                assert abs(np.sum(e ** 2) - tail) <= 1e-4 * nm ** 2, l
            else:
                assert orc.rel_fro(p @ q.T, orc.ssp_comp(q0[l], [m]).delta_hat) <= tol, l


# psgd_refresh splits for one layer: its partial sums are the layer's own region (a context of one layer) or one region for
# all; between steps, on 32 x 256 tiles (r = 24) and at widths 128 and 160, one orientation and both
@pytest.mark.parametrize("shapes", [[(1000, 264)], [(264, 2056)], [(1000, 264), (264, 2056), (520, 520)]])
@pytest.mark.parametrize("r,dtype", [(24, synth.F32), (100, synth.F32), (112, synth.BF16)])
def test_refresh_of_single_layers_between_steps(shapes, r, dtype):
    torch = torch_mod()
    rng = np.random.default_rng(r + len(shapes))
    ms = []
    for s in shapes:
        m = (np.linalg.qr(rng.standard_normal((s[0], min(s))))[0] * 0.95 ** np.arange(min(s)) @
             np.linalg.qr(rng.standard_normal((s[1], min(s))))[0].T).astype(np.float32)
        ms.append(synth.round_to_bf16(m) if dtype == synth.BF16 else m)
    case = Case(shapes, r, 1, dtype)
    for _ in range(2):
        case.upload([[m] for m in ms], [np.zeros(s, np.float32) for s in shapes],
                    [rng.standard_normal((min(s), r)).astype(np.float32) for s in shapes])
        q0 = [back(q) for q in case.Q]
        case.compress()
        for l, (rows, cols) in enumerate(shapes):
            m = logical(synth.gradient_as_f64(ms[l]), rows, cols)
            p, q, _ = case.outputs(l)
            assert orc.rel_fro(p @ q.T, orc.ssp_comp(q0[l], [m]).delta_hat) <= TOL[dtype], l
        for l, (rows, cols) in enumerate(shapes):
            m = logical(synth.gradient_as_f64(ms[l]), rows, cols)
            dense = torch.from_numpy(np.ascontiguousarray(logical(m, rows, cols)).astype(np.float32)).cuda()
            p, q = torch.zeros((max(rows, cols), r), device="cuda"), torch.zeros((min(rows, cols), r), device="cuda")
            case.comp.refresh(l, dense, p, q)
            p, q, nm = back(p), back(q), np.linalg.norm(m)
            assert np.abs(p.T @ p - np.eye(r)).max() < 2e-5, l
            assert np.linalg.norm(q - m.T @ p) <= 2e-5 * nm, l
            tail = np.sum(np.linalg.svd(m, compute_uv=False)[r:] ** 2)
            assert abs(np.linalg.norm(m - p @ q.T) ** 2 - tail) <= 1e-4 * nm ** 2, l


# psgd_compress_static in a context whose workspace fits the built-in one only with its sums as they are planned there
@pytest.mark.parametrize("shapes,r", [([(1024, 4096)], 48), ([(2048, 2048)], 48), ([(1334, 1608)] * 3, 53)])
def test_static_step_equals_step(shapes, r):
    torch = torch_mod()
    rng = np.random.default_rng(r)
    ms = [rng.standard_normal(s).astype(np.float32) for s in shapes]
    qs = [rng.standard_normal((min(s), r)).astype(np.float32) for s in shapes]
    out = []
    for static in (False, True):
        case = Case(shapes, r, 1, synth.F32)
        case.upload([[m] for m in ms], [np.zeros(s, np.float32) for s in shapes], qs)
        (case.comp.compress_static if static else case.comp.compress)(case.G, case.E, case.Q, case.P)
        torch.cuda.synchronize()
        out.append([case.outputs(l) for l in range(len(shapes))])
    assert all(np.array_equal(a, b) for x, y in zip(*out) for a, b in zip(x, y))
