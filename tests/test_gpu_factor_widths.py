"""The factorisation of the orthonormaliser at the widths where its path changes: 16 x 16 blocks from width 17 on (whole
and cut off), 32 / 33 (factorised by the kernel that adds partial products up / by a launch of its own), the widest that
fits blocked (176) and beyond; with and without dependent columns inside and at the edges of blocks."""
import numpy as np
import pytest

from oracle import psgd_oracle as orc
from paper_2509_11254_amd import synth
from gpu_harness import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [16, 17, 32, 33, 47, 48, 80, 100, 128, 160, 176, 177, 192])
@pytest.mark.parametrize("rows,cols", [(520, 264), (264, 1496)])
@pytest.mark.parametrize("dependent", [False, True])
def test_ssp_step(r, rows, cols, dependent):
    rng = np.random.default_rng(10 * r + rows)
    m = rng.standard_normal((rows, cols)).astype(np.float32)
    q = rng.standard_normal((min(rows, cols), r)).astype(np.float32)
    dep = []
    if dependent:
        dep = sorted({r // 2, min(15, r - 1), r - 1})       # (a zero column, copies of an earlier one)
        q[:, dep[0]] = 0.0
        for j in dep[1:]:
            q[:, j] = 2.0 * q[:, 1]
    case = Case([(rows, cols)], r, 1, synth.F32, refresh_oversample=0)
    case.upload([[m]], [np.zeros((rows, cols), np.float32)], [q])
    case.compress()
    p, q1, e = case.outputs(0)
    ml = m.astype(np.float64)
    if rows < cols:
        ml, e = ml.T, e.T
    out = orc.ssp_comp(q.astype(np.float64), [ml])
    # (cond(M Q) is up to about 60 here: 2^-24 products give a few 1e-6)
    assert orc.rel_fro(p, out.p_tilde) <= 1e-4
    assert orc.rel_fro(q1, out.q) <= 1e-4
    assert orc.rel_fro(e, ml - out.delta_hat) <= 1e-4
    assert case.comp.status(0).rank_deficient == len(dep)
    assert all(np.all(p[:, j] == 0.0) for j in dep)
