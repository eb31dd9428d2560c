"""The eigenvectors of the refresh's Rayleigh-Ritz step at the edges of its kernels: Q = M^T P~ comes out with orthogonal columns of
falling norms, the singular values of M on the span of P~."""
import numpy as np
import pytest

from paper_2509_11254_amd import synth
from gpu_harness import Case

pytestmark = pytest.mark.gpu


# Block widths: below one block of 8 and of 16, 9 and 13 (capped by the matrix), 16, 24, 40 and 48 (256 threads), 56, 80 and 96 (512), 104, 152
# and 160 (1024; the widest in blocks), 168 (the kernel on 2 x 2 blocks), batches whose workgroups hold many rows of V, and a
# batch of layers with widths of their own
@pytest.mark.parametrize("shapes,r", [([(40, 6)], 3), ([(60, 9)], 4), ([(13, 70)], 5), ([(200, 150)], 4), ([(300, 200)], 13), ([(300, 200)], 32),
                                      ([(300, 200)], 38), ([(300, 200)], 42), ([(400, 300)], 64), ([(400, 300)], 76), ([(400, 300)], 80),
                                      ([(400, 300)], 120), ([(500, 400)], 128), ([(500, 400)], 132), ([(200, 150)] * 70, 64),
                                      ([(200, 150)] * 300, 20), ([(300, 200), (120, 90), (70, 200)], 64)])
@pytest.mark.parametrize("spectrum", ["falling", "flat"])
def test_ritz_vectors(shapes, r, spectrum):
    rng = np.random.default_rng(len(shapes) + r)
    mats = []
    for rows, cols in shapes[:3]:
        n = min(rows, cols)
        u, _ = np.linalg.qr(rng.standard_normal((rows, n)))
        v, _ = np.linalg.qr(rng.standard_normal((cols, n)))
        # (down to 1e-3: below 1e-5, the default rank_tol, a direction counts as dependent and its column of P~ is zero)
        mats.append(((u * np.geomspace(1.0, 1e-3 if spectrum == "falling" else 0.9, n)) @ v.T).astype(np.float32))
    mats = [mats[l % len(mats)] for l in range(len(shapes))]
    case = Case(shapes, r, 1, synth.F32, lds=[(cols + 7) // 8 * 8 for _, cols in shapes], seed=5)
    case.upload([[x] for x in mats], [np.zeros(s, np.float32) for s in shapes], [rng.standard_normal((min(s), r)).astype(np.float32) for s in shapes])
    for _ in range(2):
        case.compress(refresh=True)
        for l in {0, 1 % len(shapes), len(shapes) // 2, len(shapes) - 1}:
            p, q, _ = case.outputs(l)
            norms = np.linalg.norm(q, axis=0)
            # rounding of Q's entries to fp32, and what the iteration on H leaves (off-diagonal mass 1e-10 of the diagonal's)
            bound = 2.0 ** -22 * np.outer(norms, norms) + 2e-10 * np.sum(norms ** 2)
            gram = q.T @ q
            assert np.all(np.abs(gram - np.diag(np.diag(gram))) <= bound), l
            assert np.all(norms[1:] <= norms[:-1] * (1 + 2.0 ** -22)), l
            assert np.abs(p.T @ p - np.eye(r)).max() < 2e-6
        for x in case.E:
            x.zero_()
