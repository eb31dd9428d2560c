"""The subspace iteration of the refresh, whose Y = M^T Z is not orthonormalised from the second iteration on: its
columns are brought to a norm of about one by powers of two instead, at any scale of the gradients."""
import numpy as np
import pytest

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
