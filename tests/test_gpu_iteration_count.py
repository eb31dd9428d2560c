"""How many iterations a refresh makes and asks for, and what they leave: against as many without an end of their own in fp64."""
import numpy as np
import pytest

from oracle import psgd_oracle as orc
from paper_2509_11254_amd import synth
from gpu_harness import Case

pytestmark = pytest.mark.gpu

SEED = 11


def _spectrum_matrix(rng, rows, cols, s):
    k = len(s)
    u, _ = np.linalg.qr(rng.standard_normal((rows, k)))
    v, _ = np.linalg.qr(rng.standard_normal((cols, k)))
    return ((u * s) @ v.T).astype(np.float32)


def _plain_excess(m, start, r, iters):
    """What `iters` iterations Z = orth(M Y), Y = M^T Z and the Rayleigh-Ritz step leave above the optimum of Eq. (6)."""
    y = start
    for _ in range(iters):
        z, _ = np.linalg.qr(m @ y)
        y = m.T @ z
    theta = np.linalg.svd(y, compute_uv=False)
    return np.sum(np.linalg.svd(m, compute_uv=False)[:r] ** 2) - np.sum(theta[:r] ** 2)


# No gap at the cut: a refresh leaves no more than 16 iterations.  Block widths 16 (in one launch; with
# the factorisation in the apply kernel), 24 (by finish_kernel), 40, 96, 160 (a launch of its own) and 184 (not blocked);
# both orientations, odd sizes, products split and, in a batch, not
@pytest.mark.parametrize("rows,cols,r,b,n_layers", [(200, 150, 8, 16, 1), (150, 200, 8, 16, 1), (520, 333, 8, 16, 1), (333, 520, 8, 16, 1),
                                                    (520, 400, 8, 16, 70), (640, 333, 16, 24, 1), (500, 408, 32, 40, 1), (408, 500, 32, 40, 1),
                                                    (500, 408, 32, 40, 70), (700, 512, 76, 96, 1), (512, 700, 76, 96, 1),
                                                    (900, 640, 128, 160, 1), (640, 520, 144, 184, 1)])
@pytest.mark.parametrize("planes", [2, 3])
def test_no_gap(rows, cols, r, b, n_layers, planes):
    rng = np.random.default_rng(rows + 7 * r)
    n = min(rows, cols)
    # falls by a twentieth from the r-th value to the one after the block, and on at that rate
    s = 0.95 ** (np.arange(n) / (b - r))
    mats = [_spectrum_matrix(rng, rows, cols, s) for _ in range(min(n_layers, 2))]
    mats = [mats[l % len(mats)] for l in range(n_layers)]
    warm = [rng.standard_normal((n, r)).astype(np.float32) for _ in range(min(n_layers, 2))]
    warm = [warm[l % len(warm)] for l in range(n_layers)]
    case = Case([(rows, cols)] * n_layers, r, 1, synth.F32, lds=[(cols + 7) // 8 * 8] * n_layers, precision=planes, seed=SEED)
    case.upload([[x] for x in mats], [np.zeros((rows, cols), np.float32)] * n_layers, warm)
    case.compress(refresh=True)
    for l in {0, n_layers - 1}:
        m = mats[l].astype(np.float64)
        m = m if rows >= cols else m.T
        p, q, e = case.outputs(l)
        norm2 = np.sum(m ** 2)
        start = np.concatenate([warm[l].astype(np.float64), orc.counter_uniform(SEED, l, n, b)[:, r:]], axis=1)
        plain, fewer = _plain_excess(m, start, r, 16), _plain_excess(m, start, r, 14)
        tail = np.sum(np.linalg.svd(m, compute_uv=False)[r:] ** 2)
        excess = np.sum(e ** 2) - tail
        print(rows, cols, r, "excess / ||M||^2", excess / norm2, "plain, 16 iterations", plain / norm2, "14", fewer / norm2)
        # E = M - P~ Q^T is off by 2^-17 (three planes 2^-24) of ||M|| in directions of its own: 2^-16 ||M|| ||E|| at most
        slack = 2.0 ** (-22 if planes == 3 else -16) * norm2
        assert fewer > 1.1 * plain
        assert excess <= 1.05 * plain + slack
        assert np.abs(p.T @ p - np.eye(r)).max() < 2e-6
        assert np.linalg.norm(q - m.T @ p) <= 2e-5 * np.sqrt(norm2)
        assert case.comp.status(l).rank_deficient == 0


# A gap that the iteration crosses long before its budget ends, from a random start: the subspace is what fp32 products leave
# of it.  Also where the columns after the gap have nothing to line up with (rank r, dependent columns) and where one
# direction stands far above the rest.
@pytest.mark.parametrize("rows,cols,r,n_layers", [(200, 150, 8, 1), (640, 333, 8, 1), (333, 640, 8, 70), (500, 408, 32, 1), (700, 512, 76, 1)])
@pytest.mark.parametrize("kind", ["gap", "close_gap", "rank", "outlier"])
def test_ends_when_converged(rows, cols, r, n_layers, kind):
    rng = np.random.default_rng(rows + 7 * r)
    n = min(rows, cols)
    s = np.linspace(2.0, 1.0, n)
    if kind == "rank":
        s = s[:r]
    else:
        s[r:] *= 0.3 if kind == "close_gap" else 0.1
        if kind == "outlier":
            s[0] = 100.0
    mat = _spectrum_matrix(rng, rows, cols, s)
    m = mat.astype(np.float64) if rows >= cols else mat.T.astype(np.float64)
    u, sv, _ = np.linalg.svd(m, full_matrices=False)
    case = Case([(rows, cols)] * n_layers, r, 1, synth.F32, lds=[(cols + 7) // 8 * 8] * n_layers, seed=SEED)
    case.upload([[mat]] * n_layers, [np.zeros((rows, cols), np.float32)] * n_layers, [rng.standard_normal((n, r)).astype(np.float32)] * n_layers)
    for _ in range(2):
        case.compress(refresh=True)
        for l in {0, n_layers - 1}:
            p, q, e = case.outputs(l)
            e = e if rows >= cols else e.T
            # rounding of 2^-24 sigma_1 per product, over the gap sigma_r - sigma_{r+1}
            bound = 64 * 2.0 ** -24 * sv[0] / (sv[r - 1] - (sv[r] if r < len(sv) else 0.0))
            assert orc.sin_theta_max(u[:, :r], p) <= bound, (kind, l)
            assert np.linalg.norm(e - (m - p @ q.T)) <= 2e-6 * np.linalg.norm(m)
        for x in case.E:
            x.zero_()


def _iterate(m, start, iters):
    """Z and Y = M^T Z after `iters` iterations Z = orth(M Y), Y = M^T Z."""
    y = start
    for _ in range(iters):
        z, _ = np.linalg.qr(m @ y)
        y = m.T @ z
    return z, y


def _ritz_vectors(z, y, r):
    return z @ np.linalg.eigh(y.T @ y)[1][:, ::-1][:, :r]


def _start(warm, layer, b):
    n, r = warm.shape
    return np.concatenate([warm.astype(np.float64), orc.counter_uniform(SEED, layer, n, b)[:, r:]], axis=1)


def _tall(x, rows, cols):
    return x.astype(np.float64) if rows >= cols else x.T.astype(np.float64)


# One direction so far above the rest that the factor of Z asks for an orthonormal Y in every iteration (300 at two planes, 5000
# at three), no gap at the cut: no more is left above the optimum than 16 iterations in fp64 leave.  And the iterations that the layer
# asks for are those that its spectrum needs, with and without such a direction, with and without a gap.
@pytest.mark.parametrize("rows,cols,r,b", [(200, 150, 8, 16), (520, 333, 8, 16), (408, 500, 32, 40), (700, 512, 76, 96)])
@pytest.mark.parametrize("planes", [2, 3])
@pytest.mark.parametrize("outlier", [False, True])
@pytest.mark.parametrize("gap", [False, True])
def test_every_iteration_asked_for(rows, cols, r, b, planes, outlier, gap):
    rng = np.random.default_rng(rows + 7 * r)
    n = min(rows, cols)
    s = 0.95 ** (np.arange(n) / (b - r))
    if gap:
        s[r:] *= 0.75
    if outlier:
        s[0] = 300.0 if planes == 2 else 5000.0
    mat = _spectrum_matrix(rng, rows, cols, s)
    warm = rng.standard_normal((n, r)).astype(np.float32)
    case = Case([(rows, cols)], r, 1, synth.F32, lds=[(cols + 7) // 8 * 8], precision=planes, seed=SEED)
    case.upload([[mat]], [np.zeros((rows, cols), np.float32)], [warm])
    case.compress(refresh=True)
    m = _tall(mat, rows, cols)
    sv = np.linalg.svd(m, compute_uv=False)
    z16, y16 = _iterate(m, _start(warm, 0, b), 16)
    plain, fewer = (np.sum(sv[:r] ** 2) - np.sum(np.linalg.svd(_iterate(m, _start(warm, 0, b), k)[1], compute_uv=False)[:r] ** 2) for k in (16, 14))
    # (P~ orthonormal to 64 bits: its rounding times sigma_1 is more than what is looked for)
    p, _ = np.linalg.qr(case.outputs(0)[0])
    excess = np.sum(sv[:r] ** 2) - np.sum((m.T @ p) ** 2)
    # an error of 2^-24 (two planes 2^-17) of sigma_1 in each column of a product
    slack = 4 * r * (2.0 ** (-24 if planes == 3 else -17) * sv[0]) ** 2 + 1e-13 * np.sum(sv ** 2)
    st = case.comp.status(0)
    theta = np.sort(np.linalg.eigvalsh(y16.T @ y16))[::-1]
    rho = theta[b - 1] / theta[r - 1]
    count = int(np.ceil(np.log(1e-5) / np.log(rho))) + 1
    lost = [np.sum((theta[b - 1] / theta[:r]) ** (2 * k) * (theta[:r] - theta[b - 1])) for k in range(2, 65)]
    no_gap = 2 + int(np.argmax(np.array(lost) <= 1e-5 * theta.sum()))
    print(rows, cols, r, "excess", excess, "16 iterations", plain, "14", fewer, "asks for", st.refresh_iters_next, count, st.refresh_iters_no_gap, no_gap)
    assert excess <= 1.05 * plain + slack
    # (by the library's Ritz values: those of the last columns have not settled, or carry the rounding of the products)
    assert abs(st.refresh_iters_next - count) <= max(1, 0.05 * count)
    assert abs(st.refresh_iters_no_gap - no_gap) <= 1


# Blocks of no more columns than the rank (refresh_oversample 0, or a layer of the context as narrow as the rank), a cut after which
# the singular values halve, from random starts: what is outside the block is lost in 16 iterations.  In one launch, factorised by the
# apply kernel, by finish_kernel and by a launch of its own.
@pytest.mark.parametrize("rows,cols,r,narrow", [(200, 150, 8, False), (200, 150, 16, False), (150, 200, 8, False), (520, 333, 8, False),
                                                (333, 520, 24, False), (640, 333, 40, False), (700, 512, 64, False),
                                                (520, 333, 8, True), (333, 520, 24, True)])
@pytest.mark.parametrize("planes", [2, 3])
def test_no_columns_beyond_the_rank(rows, cols, r, narrow, planes):
    rng = np.random.default_rng(rows + 7 * r)
    n, n_layers = min(rows, cols), 4
    mats, warm = [], []
    for _ in range(n_layers):
        s = np.sqrt(np.r_[np.sort(10.0 + rng.random(r - 1))[::-1], 1.0, 0.25 * np.sort(rng.random(n - r))[::-1]])
        mats.append(_spectrum_matrix(rng, rows, cols, s))
        warm.append(rng.uniform(-1, 1, (n, r)).astype(np.float32))
    shapes = [(rows, cols)] * n_layers
    if narrow:
        shapes, mats, warm = shapes + [(100, r)], mats + [rng.standard_normal((100, r)).astype(np.float32)], warm + [np.eye(r, dtype=np.float32)]
    case = Case(shapes, r, 1, synth.F32, lds=[(c + 7) // 8 * 8 for _, c in shapes], precision=planes, seed=SEED,
                refresh_oversample=-1 if narrow else 0)
    case.upload([[x] for x in mats], [np.zeros(s, np.float32) for s in shapes], warm)
    case.compress(refresh=True)
    for l in range(n_layers):
        m = _tall(mats[l], rows, cols)
        u, sv, _ = np.linalg.svd(m, full_matrices=False)
        z, y = _iterate(m, warm[l].astype(np.float64), 16)
        plain = orc.sin_theta_max(u[:, :r], z)
        rounding = 2.0 ** (-24 if planes == 3 else -17) * sv[0] / (sv[r - 1] - sv[r])
        got = orc.sin_theta_max(u[:, :r], case.outputs(l)[0])
        print(rows, cols, r, "layer", l, "sin", got, "16 iterations", plain, "rounding", rounding)
        assert got <= 2 * plain + 16 * rounding, l


# Flat up to the block's last column, and a gap after that one: 16 iterations lose what is outside the block
@pytest.mark.parametrize("rows,cols,r,b", [(200, 150, 8, 16), (520, 333, 8, 16), (333, 520, 32, 40), (640, 333, 64, 80), (700, 512, 128, 160)])
def test_gap_after_the_block(rows, cols, r, b):
    rng = np.random.default_rng(rows + 7 * r)
    n = min(rows, cols)
    s = np.sqrt(np.r_[np.linspace(1.1, 1.0, r), np.full(b - r, 0.94), 0.25 * np.linspace(1.0, 0.1, n - b)])
    mat = _spectrum_matrix(rng, rows, cols, s)
    m = _tall(mat, rows, cols)
    u, sv, _ = np.linalg.svd(m, full_matrices=False)
    warm = rng.uniform(-1, 1, (n, r)).astype(np.float32)
    case = Case([(rows, cols)], r, 1, synth.F32, lds=[(cols + 7) // 8 * 8], seed=SEED)
    case.upload([[mat]], [np.zeros((rows, cols), np.float32)], [warm])
    case.compress(refresh=True)

    def outside(p):
        return np.linalg.norm(p - u[:, :b] @ (u[:, :b].T @ p), 2)

    plain = outside(_ritz_vectors(*_iterate(m, _start(warm, 0, b), 16), r))
    rounding = 2.0 ** -24 * sv[0] / (sv[r - 1] - sv[b])
    got = outside(case.outputs(0)[0])
    print(rows, cols, r, "outside the block", got, "16 iterations", plain, "rounding", rounding)
    assert got <= 2 * plain + 16 * rounding


# A warm start orthogonal to the leading directions: the columns beyond it hold some of them, the others come up from its rounding
# to fp32, and until they have the block grows like one that has converged.  Columns beyond the rank that are fewer than those directions,
# down to one, and the default number.  Factorised in one launch, by the apply kernel, by finish_kernel and by a launch of its own.
@pytest.mark.parametrize("rows,cols,r,over", [(200, 150, 6, 2), (150, 200, 14, 2), (520, 333, 7, 1), (333, 520, 22, 2), (640, 333, 38, 2),
                                              (500, 408, 62, 2), (408, 500, 32, -1), (700, 512, 120, -1)])
def test_start_orthogonal_to_the_leading_directions(rows, cols, r, over):
    rng = np.random.default_rng(rows + 7 * r)
    n, n_layers = min(rows, cols), 3
    s = np.r_[np.linspace(2.0, 1.0, r), 0.3 * np.linspace(1.0, 0.5, n - r)]
    mats = [_spectrum_matrix(rng, rows, cols, s) for _ in range(n_layers)]
    svds = [np.linalg.svd(_tall(x, rows, cols), full_matrices=False) for x in mats]
    case = Case([(rows, cols)] * n_layers, r, 1, synth.F32, lds=[(cols + 7) // 8 * 8] * n_layers, seed=SEED, refresh_oversample=over)
    case.upload([[x] for x in mats], [np.zeros((rows, cols), np.float32)] * n_layers, [v[r:2 * r].T.astype(np.float32) for _, _, v in svds])
    case.compress(refresh=True)
    for l, (u, sv, _) in enumerate(svds):
        got = orc.sin_theta_max(u[:, :r], case.outputs(l)[0])
        # what 16 iterations leave of a direction that rounding holds 2^-25 / sqrt(n) of is below the rounding of a product
        rounding = 2.0 ** -24 * sv[0] / (sv[r - 1] - sv[r])
        print(rows, cols, r, "layer", l, "sin", got, "rounding", rounding)
        assert got <= 16 * rounding, l


# Whether a refresh has ended before its maximum: it leaves the same bits as one with a smaller maximum that it does not reach, and
# others where it has not converged by then
@pytest.mark.parametrize("rows,cols,r", [(200, 150, 8), (640, 333, 8), (333, 640, 24), (500, 408, 32), (700, 512, 76), (640, 520, 144)])
@pytest.mark.parametrize("planes,fewer", [(2, 8), (3, 10)])
@pytest.mark.parametrize("gap", [False, True])
def test_ends_before_its_maximum(rows, cols, r, planes, fewer, gap):
    rng = np.random.default_rng(rows + 7 * r)
    n = min(rows, cols)
    s = np.linspace(2.0, 1.0, n)
    if gap:
        s[r:] *= 0.05               # (8.6 powers of two or more per iteration: 30 and 38 are asked of them)
    mat = _spectrum_matrix(rng, rows, cols, s)
    warm = rng.standard_normal((n, r)).astype(np.float32)
    out = []
    for iters in (fewer, 16, 40):
        case = Case([(rows, cols)], r, 1, synth.F32, lds=[(cols + 7) // 8 * 8], precision=planes, seed=SEED, refresh_iters=iters)
        case.upload([[mat]], [np.zeros((rows, cols), np.float32)], [warm])
        case.compress(refresh=True)
        out.append(case.outputs(0))
    same = [all(np.array_equal(a, b) for a, b in zip(out[0], x)) for x in out[1:]]
    assert same == [gap, gap]
