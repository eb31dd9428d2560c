"""Steps and refreshes of layers small enough for one workgroup that holds M in LDS: against the oracle, and against the general
path on the same inputs (which a context takes as a whole when one of its layers is larger)."""
import numpy as np
import pytest

from oracle import psgd_oracle as orc
from paper_2509_11254_amd import psgd, synth
from gpu_harness import Case, back, logical, to_dev_grad, torch_mod
from test_gpu_refresh_loops import _check_refreshed_step

pytestmark = pytest.mark.gpu

# the largest that fits, one 16 x 16 block and less, ragged in both directions, long, both orientations, padded rows
SHAPES = [(256, 128), (16, 16), (5, 3), (130, 129), (129, 130), (450, 56), (40, 560), (176, 181), (33, 70), (64, 24), (128, 256)]
LARGE = (264, 256)


def _inputs(shapes, r, n_workers, dtype, seed, noise_seed=0):
    out = []
    for rows, cols in shapes:
        rng = np.random.default_rng([seed, rows, cols])
        k = min(rows, cols, 12)
        sig = (rng.standard_normal((rows, k)) * 0.6 ** np.arange(k)) @ rng.standard_normal((k, cols))
        rng = np.random.default_rng([seed, rows, cols, noise_seed]) if noise_seed else rng
        g = [(sig + 0.05 * rng.standard_normal((rows, cols))).astype(np.float32) for _ in range(n_workers)]
        g = [synth.round_to_bf16(x) if dtype == synth.BF16 else x for x in g]
        v = np.linalg.svd(logical(sig, rows, cols), full_matrices=False)[2][:r].T
        out.append((g, (0.05 * rng.standard_normal((rows, cols))).astype(np.float32),
                    (v + 0.02 * rng.standard_normal(v.shape)).astype(np.float32)))
    return [list(x) for x in zip(*out)]


def _run(shapes, rs, n_workers, dtype, data, refresh, padded=True, **opts):
    lds = [(c + 7) // 8 * 8 + 8 * (padded and i % 3 == 0) for i, (_, c) in enumerate(shapes)]
    case = Case(shapes, rs, n_workers, dtype, lds=lds, **opts)
    case.upload(*data)
    for e, (_, c) in zip(case.E, shapes):
        assert e.shape[1] == c or bool(torch_mod().isnan(e[:, c:]).all())
    case.compress(refresh=refresh)
    for e, (_, c) in zip(case.E, shapes):                       # the padding is not written
        assert e.shape[1] == c or bool(torch_mod().isnan(e[:, c:]).all())
    return case


@pytest.mark.parametrize("r", [1, 3, 4, 8, 13, 16])
@pytest.mark.parametrize("n_workers,dtype", [(1, synth.F32), (4, synth.F32), (3, synth.BF16)])
def test_step(r, n_workers, dtype):
    rs = [min(r, *s) for s in SHAPES]
    data = _inputs(SHAPES, r, n_workers, dtype, 10 * r + n_workers)
    data[2] = [q[:, :k] for q, k in zip(data[2], rs)]
    case = _run(SHAPES, rs, n_workers, dtype, data, False)
    more = _inputs([LARGE], r, n_workers, dtype, 1)
    general = _run(SHAPES + [LARGE], rs + [r], n_workers, dtype, [a + b for a, b in zip(data, more)], False)
    torch = torch_mod()
    outs = [[torch.zeros_like(e) for e in c.E] for c in (case, general)]
    for c, o in zip((case, general), outs):
        c.comp.decompress(None, None, o, psgd.PSGD_F32)
    for l, (rows, cols) in enumerate(SHAPES):
        m = np.mean([logical(synth.gradient_as_f64(g), rows, cols) for g in data[0][l]], axis=0) + logical(data[1][l].astype(np.float64), rows, cols)
        ref = orc.ssp_comp(data[2][l].astype(np.float64), [m])
        p, q, e = case.outputs(l)
        scale = np.linalg.norm(m)
        # fp32 inputs, products and results, fp64 in between: a few 2^-24 of ||M|| for every type of gradient, times the condition
        # of P = M Q in P~ itself
        tag = (l, rows, cols, r)
        assert np.abs(p.T @ p - np.eye(rs[l])).max() < 2e-6, tag
        assert np.linalg.norm(q - m.T @ p) <= 2e-6 * scale, tag
        # (the update of bf16 gradients is a product of two bf16 planes per factor, 2^-17 of each, and E is what that leaves of M)
        assert np.linalg.norm(logical(e, rows, cols) - (m - p @ q.T)) <= (2e-6 if dtype == synth.F32 else 4 * 2.0 ** -17) * scale, tag
        x = m @ data[2][l].astype(np.float64)
        sv = np.linalg.svd(x / np.linalg.norm(x, axis=0), compute_uv=False)
        if sv[-1] > 1e-3:
            assert np.linalg.norm(p @ q.T - ref.delta_hat) <= 4e-6 / sv[-1] * scale, tag
            tol = (4e-6 if dtype == synth.F32 else 6 * 2.0 ** -17) / sv[-1] * scale
            pg, qg, eg = general.outputs(l)
            assert np.linalg.norm(pg @ qg.T - p @ q.T) <= tol and np.linalg.norm(eg - e) <= tol, tag
        assert np.linalg.norm(logical(back(outs[0][l], cols), rows, cols) - p @ q.T) <= (1e-6 if dtype == synth.F32 else 4 * 2.0 ** -17) * scale, tag
        assert case.comp.status(l).rank_deficient == general.comp.status(l).rank_deficient, tag


# what a step leaves in E and what it lets the update apply are M together, whatever the operand planes
@pytest.mark.parametrize("r", [1, 7, 16])
@pytest.mark.parametrize("n_workers,dtype,precision", [(3, synth.BF16, 0), (1, synth.BF16, 3), (2, synth.F32, 0), (2, synth.F32, 2)])
def test_error_feedback_balances(r, n_workers, dtype, precision):
    torch = torch_mod()
    rs = [min(r, *s) for s in SHAPES]
    data = _inputs(SHAPES, r, n_workers, dtype, 7 * r + n_workers)
    data[2] = [q[:, :k] for q, k in zip(data[2], rs)]
    case = _run(SHAPES, rs, n_workers, dtype, data, False, precision=precision)
    for factors in ((None, None), (case.P, case.Q)):
        out = [torch.zeros_like(e) for e in case.E]
        case.comp.decompress(*factors, out, psgd.PSGD_F32)
        mom, x = [torch.zeros_like(e) for e in case.E], [torch.zeros_like(e) for e in case.E]
        case.comp.decompress_msgd(*factors, mom, x, 0.0, 1.0)
        for l, (rows, cols) in enumerate(SHAPES):
            m = np.mean([synth.gradient_as_f64(g) for g in data[0][l]], axis=0) + data[1][l]
            e = back(case.E[l], cols).astype(np.float64)
            for update in (out[l], mom[l]):
                # five roundings of M (a sum of up to three, a quotient, E added), one of E, and with three planes those of two fp32
                # sums of the update: at most 16 of 2^-24
                assert np.linalg.norm(e + back(update, cols) - m) <= 2.0 ** -20 * np.linalg.norm(m), (l, rows, cols, rs[l])


# block widths up to 16, two refreshes with the budget and a third with the layer's own count
@pytest.mark.parametrize("r", [1, 4, 8])
@pytest.mark.parametrize("n_workers,dtype", [(2, synth.F32), (1, synth.BF16)])
def test_refresh(r, n_workers, dtype):
    rs = [min(r, min(s) - 1) for s in SHAPES]
    data = _inputs(SHAPES, r, n_workers, dtype, 100 * r + n_workers)
    data[2] = [q[:, :k] for q, k in zip(data[2], rs)]
    case = _run(SHAPES, rs, n_workers, dtype, data, True)
    err = data[1]
    for t in range(3):
        if t > 0:
            err = [back(e, c).astype(np.float32) for e, (_, c) in zip(case.E, SHAPES)]
            data = _inputs(SHAPES, r, n_workers, dtype, 100 * r + n_workers, noise_seed=t)
            case.G = [[to_dev_grad(g, e.shape[1]) for g in gl] for gl, e in zip(data[0], case.E)]
            case.compress(refresh=True)
        for l, (rows, cols) in enumerate(SHAPES):
            m = np.mean([logical(synth.gradient_as_f64(g), rows, cols) for g in data[0][l]], axis=0) + logical(err[l].astype(np.float64), rows, cols)
            p, q, e = case.outputs(l)
            _check_refreshed_step(m, p, q, logical(e, rows, cols), rs[l], (t, l, rows, cols, r))


# the most workers whose gradients one workgroup reads, and one more (the general path)
@pytest.mark.parametrize("rows,cols,n_workers", [(256, 128, 96), (256, 128, 97), (128, 256, 97), (64, 24, 260)])
def test_refresh_of_many_workers(rows, cols, n_workers):
    data = _inputs([(rows, cols)], 4, n_workers, synth.F32, n_workers)
    case = _run([(rows, cols)], [4], n_workers, synth.F32, data, True)
    m = np.mean([g.astype(np.float64) for g in data[0][0]], axis=0) + data[1][0]
    p, q, e = case.outputs(0)
    _check_refreshed_step(logical(m, rows, cols), p, q, logical(e, rows, cols), 4, (rows, cols, n_workers))


# a start block out of order (the factorisation of Z asks for an orthonormal Y), one with two columns 1e-6 apart (the second
# CholeskyQR pass), and columns that depend on each other
@pytest.mark.parametrize("rows,cols", [(200, 150), (150, 200)])
@pytest.mark.parametrize("kind", ["ascending", "close", "rank", "zero"])
def test_hard_starts(rows, cols, kind):
    rng = np.random.default_rng(rows)
    n, r = 150, 8
    u, _ = np.linalg.qr(rng.standard_normal((rows, n)))
    v, _ = np.linalg.qr(rng.standard_normal((cols, n)))
    s = {"ascending": 1e-4 ** (np.arange(n) / 16), "close": 0.9 ** np.arange(n), "rank": np.r_[1.0, 0.5, 0.25, np.zeros(n - 3)], "zero": np.zeros(n)}[kind]
    mat = ((u * s) @ v.T).astype(np.float32)
    m = logical(mat.astype(np.float64), rows, cols)
    q0 = np.linalg.svd(m, full_matrices=False)[2][:r].T if kind == "ascending" else rng.standard_normal((n, r))
    q0 = q0[:, ::-1].astype(np.float32) if kind == "ascending" else q0.astype(np.float32)
    if kind == "close":
        q0[:, -1] = q0[:, 0] + np.float32(1e-6) * q0[:, -1]
    data = [[[mat]], [np.zeros((rows, cols), np.float32)], [q0]]
    nm = max(np.linalg.norm(m), 1e-30)
    sv = np.linalg.svd(m, compute_uv=False)
    for refresh, opts in ((False, {}), (True, dict(refresh_iters=4)), (True, dict(refresh_iters=1))):
        case = _run([(rows, cols)], r, 1, synth.F32, data, refresh, rank_tol=1e-7, **opts)
        p, q, e = case.outputs(0)
        g = p.T @ p
        live = np.diag(g) > 0.5
        assert np.abs(g - np.diag(live.astype(float))).max() < 2e-6, (kind, refresh)
        assert np.linalg.norm(q - m.T @ p) <= 2e-6 * nm and np.linalg.norm(logical(e, rows, cols) - (m - p @ q.T)) <= 2e-6 * nm
        if kind in ("ascending", "close"):
            assert live.all() and case.comp.status(0).rank_deficient == 0
        if kind == "zero":
            assert not live.any()
        if refresh and opts["refresh_iters"] == 4 and kind != "close":
            assert abs(np.sum(e ** 2) - np.sum(sv[r:] ** 2)) <= 1e-6 * nm ** 2


# one and two tiles of 16 rows per wave (192 and 193 rows or columns), reductions that end 1, 15, 16, 17 and 31 steps after a
# multiple of 32, large ones
EDGES = [(192, 65), (193, 79), (65, 193), (80, 192), (81, 95), (168, 200), (272, 120), (4, 31), (300, 15), (310, 16), (200, 17), (150, 33)]


@pytest.mark.parametrize("r", [3, 4, 5, 16])
@pytest.mark.parametrize("n_workers,dtype", [(2, synth.F32), (1, synth.BF16)])
def test_step_at_the_edges_of_tiles(monkeypatch, r, n_workers, dtype):
    monkeypatch.setitem(globals(), "SHAPES", EDGES)
    test_step(r, n_workers, dtype)


# the last sizes that fit: with an odd number of 16-byte pieces per column of a thin matrix in LDS, without it, and the first that do not fit
# (the general path)
LAST = [(175, 192), (199, 172), (209, 157), (4, 1905), (177, 189), (246, 137), (128, 265), (29, 853), (176, 200), (172, 199), (206, 171)]


@pytest.mark.parametrize("r", [4, 16])
@pytest.mark.parametrize("n_workers,dtype", [(2, synth.F32), (1, synth.BF16)])
def test_the_last_sizes_that_fit(monkeypatch, r, n_workers, dtype):
    for shape in LAST:
        monkeypatch.setitem(globals(), "SHAPES", [shape])
        test_step(r, n_workers, dtype)
        if r < 16 and min(shape) > 8:
            test_refresh(r, n_workers, dtype)
