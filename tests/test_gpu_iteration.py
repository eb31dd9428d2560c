"""The subspace iteration of the refresh, whose Y = M^T Z is orthonormalised from the second iteration on only where the
factor of Z asks for it: elsewhere its columns are brought to a norm of about one by powers of two, at any scale of the
gradients."""
import numpy as np
import pytest

from oracle import psgd_oracle as orc
from paper_2509_11254_amd import synth
from gpu_harness import Case
from test_gpu_refresh_loops import _check_refreshed_step

pytestmark = pytest.mark.gpu


# block widths 16 (factorised by the apply kernel), 32 and 72 (by finish_kernel or a launch of its own), both orientations,
# odd sizes, reductions split and not; a block as wide as the matrix; more columns than the matrix has rank (fp32 rounding
# noise below 2^-24 sigma_1 is all that the dependent columns hold)
@pytest.mark.parametrize("rows,cols,r,rank", [(333, 203, 4, 60), (203, 333, 24, 60), (1000, 520, 60, 200), (64, 40, 32, 40),
                                              (300, 200, 8, 10)])
@pytest.mark.parametrize("exponent", [0, -90, 40])
def test_refresh_at_any_scale(rows, cols, r, rank, exponent):
    rng = np.random.default_rng(1000 * rows + r)
    u, _ = np.linalg.qr(rng.standard_normal((rows, rank)))
    v, _ = np.linalg.qr(rng.standard_normal((cols, rank)))
    s = 0.9 ** np.arange(rank)
    s[r:] *= 0.5                                                # a gap at the cut
    mat = ((u * s) @ v.T).astype(np.float32)
    ld = (cols + 7) // 8 * 8
    case = Case([(rows, cols)], r, 1, synth.F32, lds=[ld])
    scale = np.float32(2.0) ** np.float32(exponent)
    case.upload([[mat * scale]], [np.zeros((rows, cols), np.float32)],
                [rng.standard_normal((min(rows, cols), r)).astype(np.float32)])
    case.compress(refresh=True)
    p, q, e = case.outputs(0)
    m = mat.astype(np.float64)
    q, e = q / float(scale), e / float(scale)
    if rows < cols:
        m, e = m.T, e.T
    # bounds of _check_refreshed_step: 1e-4 on the subspace, 2e-5 of ||M|| on the exact relations (measured: 1e-6, 1e-7)
    _check_refreshed_step(m, p, q, e, r, (rows, cols, r, exponent))


# A start block that holds the leading right singular vectors in another order than that of their singular values: on the
# way to the right one, columns of Z mix strong and weak directions (ratios up to 1e4 here), and none may be lost.  Block
# widths 16 (factorised by the apply kernel), 32 (by finish_kernel), 40 (a launch of its own) and 184 (beyond the blocked
# factorisation), split and unsplit products, both orientations, two and three operand planes; an outlier over a flat rest.
@pytest.mark.parametrize("r,b", [(8, 16), (24, 32), (32, 40), (144, 184)])
@pytest.mark.parametrize("rows,cols", [(400, 300), (300, 408)])
@pytest.mark.parametrize("order", ["ascending", "permuted", "outlier"])
@pytest.mark.parametrize("planes", [2, 3])
def test_start_block_out_of_order(r, b, rows, cols, order, planes):
    rng = np.random.default_rng(100 * r + rows)
    n = min(rows, cols)
    u, _ = np.linalg.qr(rng.standard_normal((rows, n)))
    v, _ = np.linalg.qr(rng.standard_normal((cols, n)))
    # (two planes carry 2^-17 of sigma_1: nothing asserted here lies below 1e-3)
    if order == "outlier":
        s = np.r_[1e4 if planes == 3 else 1e3, 1.0 + 2.0 * np.exp(-np.arange(n - 1) / (0.5 * r))]
    else:
        s = (1e-4 if planes == 3 else 1e-3) ** (np.arange(n) / b)
    mat = ((u * s) @ v.T).astype(np.float32)
    m = mat.astype(np.float64) if rows >= cols else mat.T.astype(np.float64)
    left, sv, right = np.linalg.svd(m, full_matrices=False)
    perm = rng.permutation(r) if order == "permuted" else np.arange(r)[::-1]
    case = Case([(rows, cols)], r, 1, synth.F32, lds=[(cols + 7) // 8 * 8], refresh_iters=4, precision=planes)
    case.upload([[mat]], [np.zeros((rows, cols), np.float32)], [right[:r].T[:, perm].astype(np.float32)])
    case.compress(refresh=True)
    p, q, e = case.outputs(0)
    if rows < cols:
        e = e.T
    assert case.comp.status(0).rank_deficient == 0
    nm = np.linalg.norm(m)
    # bounds: fp32 storage and 2^-24 / 2^-17 products on the exact relations (as in _check_refreshed_step), the optimum of
    # Eq. (6) to 1e-6 of ||M||^2
    assert np.abs(p.T @ p - np.eye(r)).max() < 2e-6
    assert np.linalg.norm(q - m.T @ p) <= 2e-5 * nm
    assert np.linalg.norm(e - (m - p @ q.T)) <= 2e-5 * nm
    assert abs(np.sum(e ** 2) - np.sum(sv[r:] ** 2)) <= 1e-6 * nm ** 2
    # The subspace, to what the products' rounding leaves of the r-th direction: the start holds the exact vectors in fp32, and
    # an error of 2^-24 (2^-17) sigma_1 in M Y turns it by that over the gap of sigma_r to what is outside the block
    if order != "outlier":
        rounding = 2.0 ** (-24 if planes == 3 else -17) * np.sqrt(r)
        assert orc.sin_theta_max(left[:, :r], p) <= max(4.0 * rounding * sv[0] / (sv[r - 1] - sv[r]), (sv[b] / sv[r - 1]) ** 6)


# The second CholeskyQR pass on Z, made once after the iteration for the layers that ask for it (Z <- Z T, Y <- Y T, the Gram
# matrix of Y anew): one iteration from a start block with two columns 1e-6 apart, whose pivot of 1e-12 leaves an
# orthogonality error of 1e-5 to 1e-2 after the first pass.  Block widths 16, 32, 56 and 120; alone, and in a batch with
# layers that do not ask and keep their bits.
@pytest.mark.parametrize("r", [8, 20, 40, 96])
@pytest.mark.parametrize("shapes", [[(400, 300)], [(300, 408)], [(2000, 264), (300, 408), (400, 300), (264, 1800)]])
def test_second_pass_after_the_iteration(r, shapes):
    rng = np.random.default_rng(r + len(shapes))
    lds = [(c + 7) // 8 * 8 for _, c in shapes]
    ms = [rng.standard_normal(s).astype(np.float32) for s in shapes]
    plain = [np.linalg.qr(rng.standard_normal((min(s), r)))[0].astype(np.float32) for s in shapes]
    close = [q.copy() for q in plain]
    close[0][:, r - 1] = close[0][:, 0] + np.float32(1e-6) * close[0][:, r - 1]
    # one pass on the warm columns in fp64, stored in fp32: what the bound below has to tell from two
    x = ((ms[0] if shapes[0][0] >= shapes[0][1] else ms[0].T) @ close[0]).astype(np.float64)
    d = 1.0 / np.linalg.norm(x, axis=0)
    z = (x @ (d[:, None] * np.linalg.inv(np.linalg.cholesky((x * d).T @ (x * d)).T))).astype(np.float32).astype(np.float64)
    assert np.abs(z.T @ z - np.eye(r)).max() > 4e-6
    out = {}
    for name, qs in (("plain", plain), ("close", close)):
        case = Case(shapes, r, 1, synth.F32, lds=lds, rank_tol=1e-7, refresh_iters=1)
        case.upload([[m] for m in ms], [np.zeros(s, np.float32) for s in shapes], qs)
        case.compress(refresh=True)
        out[name] = [case.outputs(l) for l in range(len(shapes))]
    for l, (rows, cols) in enumerate(shapes):
        if l > 0:
            assert all(np.array_equal(a, b) for a, b in zip(out["close"][l], out["plain"][l])), l
        p, q, e = out["close"][l]
        m = ms[l].astype(np.float64)
        if rows < cols:
            m, e = m.T, e.T
        assert np.abs(p.T @ p - np.eye(r)).max() < 2e-6, l
        assert np.linalg.norm(q - m.T @ p) <= 2e-6 * np.linalg.norm(m), l
        assert np.linalg.norm(e - (m - p @ q.T)) <= 2e-6 * np.linalg.norm(m), l
        # Ritz vectors: Q = M^T P~ has orthogonal columns in falling order (H = Y^T Y of the Y that goes with the final Z)
        h = q.T @ q
        assert np.abs(h - np.diag(np.diag(h))).max() <= 4e-6 * h[0, 0] and np.all(np.diff(np.diag(h)) <= 4e-6 * h[0, 0]), l


# The Rayleigh-Ritz step's rotations, worked out a round ahead or behind the update: widths on both sides of the rule (48, 152 and 160; odd;
# more blocks than threads), with few rows of the eigenvectors per workgroup (one layer) and with many (a batch)
@pytest.mark.parametrize("w,n_layers", [(48, 64), (57, 1), (57, 90), (104, 36), (104, 43), (152, 1), (152, 28), (160, 1), (160, 20), (176, 1)])
def test_ritz_step_of_any_width(w, n_layers):
    rng = np.random.default_rng(100 * w + n_layers)
    rows, cols, r = 240, 57 if w == 57 else 200, w - 8
    u, _ = np.linalg.qr(rng.standard_normal((rows, cols)))
    v, _ = np.linalg.qr(rng.standard_normal((cols, cols)))
    s = 0.97 ** np.arange(cols)
    s[r:] *= 0.3                                                # a gap at the cut
    mats = [((u[rng.permutation(rows)] * s) @ v.T).astype(np.float32) for _ in range(n_layers)]
    case = Case([(rows, cols)] * n_layers, r, 1, synth.F32, lds=[(cols + 7) // 8 * 8] * n_layers, refresh_oversample=8)
    case.upload([[x] for x in mats], [np.zeros((rows, cols), np.float32)] * n_layers,
                [rng.standard_normal((cols, r)).astype(np.float32) for _ in mats])
    case.compress(refresh=True)
    for l in {0, n_layers // 2, n_layers - 1}:
        _check_refreshed_step(mats[l].astype(np.float64), *case.outputs(l), r, (w, n_layers, l))
        st = case.comp.status(l)
        assert abs(st.sigma_max - 1.0) < 1e-5 and abs(st.sigma_r - s[r - 1]) < 1e-5, (w, l, st.sigma_max, st.sigma_r)
