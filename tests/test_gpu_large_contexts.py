"""Wide products (fp32 gradients, widths from 96 on) in contexts of many elements: steps, refreshes and psgd_refresh of ragged
layers of both orientations beside a large one, at magnitudes from 1e-28 to 1e34, with outliers and with columns of very different
size, against fp64.  (Below 1e-28, the third bf16 plane of the factors that the residual multiplies, 2^-18 of elements of 1e-4 of
this, leaves the normal numbers.)"""
import pytest

from paper_2509_11254_amd import psgd
from gpu_harness import torch_mod

pytestmark = pytest.mark.gpu

# the first makes the context large enough; tiles and reductions that end at every kind of edge, one chunk, many
LAYERS = [(2900, 2900, 2904), (333, 203, 208), (200, 328, 328), (193, 700, 704), (1985, 190, 192), (191, 2049, 2056), (256, 256, 256)]


def _inputs(r, scale, outliers):
    torch = torch_mod()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(r)
    G, E, Q, P = [], [], [], []
    for l, (rows, cols, ld) in enumerate(LAYERS):
        k = min(rows, cols)
        s = 0.93 ** torch.arange(k, device="cuda", dtype=torch.float32)
        u, v = (torch.linalg.qr(torch.randn((x, k), generator=gen, device="cuda"))[0] for x in (rows, cols))
        g, e = (torch.full((rows, ld), float("nan"), device="cuda") for _ in range(2))
        g[:, :cols] = (u * s) @ v.T
        e[:, :cols] = 1e-3 / k ** 0.5 * torch.randn((rows, cols), generator=gen, device="cuda")
        if outliers:
            for i in range(3):
                g[7 * i + l, 5 * i] = 20.0 * (-1) ** i
        g[:, :cols] *= scale
        e[:, :cols] *= scale
        short = v if rows >= cols else u
        G.append([g])
        E.append(e)
        Q.append((short[:, :r] * s[:r] + 0.01 * s[r - 1] / k ** 0.5 * torch.randn((k, r), generator=gen, device="cuda")).contiguous())
        P.append(torch.zeros((max(rows, cols), r), device="cuda"))
    return G, E, Q, P


def _formed(G, E):
    out = []
    for g, e, (rows, cols, ld) in zip(G, E, LAYERS):
        m = g[0][:, :cols].double() + e[:, :cols].double()
        out.append(m if rows >= cols else m.T)
    return out


def _check(M, E, Q, P, scale):
    torch = torch_mod()
    for l, (rows, cols, ld) in enumerate(LAYERS):
        m, p, q = M[l], P[l].double(), Q[l].double()
        e = E[l][:, :cols].double()
        e = e if rows >= cols else e.T
        norm = float((m / scale).norm())
        tag = (l, rows, cols)
        assert float((p.T @ p - torch.eye(p.shape[1], device="cuda", dtype=torch.float64)).abs().max()) < 2e-6, tag
        # fp32 sums (row by row and tighter: test_each_row_to_its_own_size)
        assert float(((q - m.T @ p) / scale).norm()) <= 1e-6 * norm, tag
        assert float(((e - (m - p @ q.T)) / scale).norm()) <= 1e-6 * norm, tag
        assert ld == cols or bool(torch.isnan(E[l][:, cols:]).all()), tag


@pytest.mark.parametrize("scale,outliers", [(1.0, False), (1.0, True), (1e-28, False), (1e34, False), (1e-12, True)])
@pytest.mark.parametrize("r", [70, 100, 128])
def test_step(r, scale, outliers):
    comp = psgd.Compressor([(rows, cols, r, psgd.PSGD_F32, ld) for rows, cols, ld in LAYERS], 1)
    G, E, Q, P = _inputs(r, scale, outliers)
    M = _formed(G, E)
    start = [q.double() for q in Q]
    comp.compress(G, E, Q, P)
    _check(M, E, Q, P, scale)
    torch = torch_mod()
    for l, m in enumerate(M):                                   # the span of M Q, column by column to 2^-23 of ||M|| ||q||
        x = m @ start[l] / scale
        worst = float((torch.linalg.matrix_norm(m / scale, 2) * start[l].norm(dim=0) / x.norm(dim=0)).max())
        x = x / x.norm(dim=0)
        low = float(torch.linalg.svdvals(x)[-1])
        q = torch.linalg.qr(x)[0]
        assert float((q - P[l].double() @ (P[l].double().T @ q)).norm()) <= 2.0 ** -23 * worst * r ** 0.5 / low, l


@pytest.mark.parametrize("scale,outliers", [(1.0, False), (1.0, True), (1e-12, False), (1e12, False)])
@pytest.mark.parametrize("r", [60, 100, 144])
def test_refresh(r, scale, outliers):
    torch = torch_mod()
    comp = psgd.Compressor([(rows, cols, r, psgd.PSGD_F32, ld) for rows, cols, ld in LAYERS], 1)
    G, E, Q, P = _inputs(r, scale, outliers)
    M = _formed(G, E)
    for l, m in list(enumerate(M))[1:3]:                        # an optimal compressor of a given matrix: nothing formed before
        rows, cols, ld = LAYERS[l]
        given = torch.full((rows, ld), float("nan"), device="cuda")
        given[:, :cols] = (m if rows >= cols else m.T).float()
        p, q = torch.zeros_like(P[l]), torch.zeros_like(Q[l])
        comp.refresh(l, given, p, q)
        m32 = given[:, :cols].double() if rows >= cols else given[:, :cols].double().T
        sv = torch.linalg.svdvals(m32 / scale)
        left = m32 / scale - p.double() @ (q.double() / scale).T
        assert float(((q.double() - m32.T @ p.double()) / scale).norm()) <= 1e-6 * float(sv.norm()), l
        assert float((left.norm() ** 2 - (sv[r:] ** 2).sum()).abs()) <= 1e-5 * float((sv ** 2).sum()), l
    for _ in range(2):
        M = _formed(G, E)
        comp.compress_refresh(G, E, Q, P)
        _check(M, E, Q, P, scale)
        for l, m in list(enumerate(M))[1:]:
            sv = torch.linalg.svdvals(m / scale)
            left = (m - P[l].double() @ Q[l].double().T) / scale
            assert float((left.norm() ** 2 - (sv[r:] ** 2).sum()).abs()) <= 1e-5 * float((sv ** 2).sum()), l


def _uneven(r, n_workers, dtype):
    """Gradients and E whose columns (of the matrix with the long side first) span 36 binary orders: three quarters of them of one
    size, the others 2^-8 to 2^-36 of it."""
    torch = torch_mod()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(r)
    G, E, Q, P = [], [], [], []
    for rows, cols, ld in LAYERS:
        k = min(rows, cols)
        d = torch.ones(k, device="cuda")
        d[3::4] = 2.0 ** -(8.0 + 4.0 * (torch.arange(len(d[3::4]), device="cuda") % 8))
        d = d if rows >= cols else d[:, None]
        G.append([torch.zeros((rows, ld), device="cuda", dtype=dtype) for _ in range(n_workers)])
        for g in G[-1]:
            g[:, :cols] = (torch.randn((rows, cols), generator=gen, device="cuda") * d).to(dtype)
        e = torch.zeros((rows, ld), device="cuda")
        e[:, :cols] = 0.01 * torch.randn((rows, cols), generator=gen, device="cuda") * d
        E.append(e)
        Q.append(torch.randn((k, r), generator=gen, device="cuda"))
        P.append(torch.zeros((max(rows, cols), r), device="cuda"))
    return G, E, Q, P


@pytest.mark.parametrize("op", ["compress", "compress_refresh"])
@pytest.mark.parametrize("n_workers,bf16,opts", [(1, False, {}), (2, False, {}), (1, True, {"precision": 3}),
                                                 (1, False, {"lazy_residual": True}),
                                                 (1, False, {"lazy_residual": True, "q_resident": True})])
@pytest.mark.parametrize("r", [70, 128])
def test_each_row_to_its_own_size(r, n_workers, bf16, opts, op):
    """Three planes hold every element of M to 2^-24 of itself, however small it is beside the largest.  So each row of
    Q = M^T P~ is good to fp32 sums over its own column of M, and so is each column of E: K = 6 len / 16 additions of 2^-24 of
    at most ||m_j||, as independent roundings, and some for the operands; in a refresh for each of the block's columns."""
    torch = torch_mod()
    dtype = torch.bfloat16 if bf16 else torch.float32
    comp = psgd.Compressor([(rows, cols, r, psgd.PSGD_BF16 if bf16 else psgd.PSGD_F32, ld) for rows, cols, ld in LAYERS], n_workers, **opts)
    G, E, Q, P = _uneven(r, n_workers, dtype)
    M = []
    for g, e, (rows, cols, ld) in zip(G, E, LAYERS):
        m = sum(x[:, :cols].double() for x in g) / n_workers + e[:, :cols].double()
        M.append(m if rows >= cols else m.T)
    getattr(comp, op)(G, E, Q, P)
    if opts.get("lazy_residual"):
        comp.flush_residual(E)
    for l, (rows, cols, ld) in enumerate(LAYERS):
        m, p, q = M[l], P[l].double(), Q[l].double()
        size = m.norm(dim=0)
        tag = (l, rows, cols)
        columns = 1 if op == "compress" else r + max(8, r // 4)
        bound = 2.0 ** -24 * ((6 * m.shape[0] / 16) ** 0.5 + 4) * columns ** 0.5
        worst = float(((q - m.T @ p).abs().amax(dim=1) / size).max())
        assert worst <= bound, (tag, worst, bound)
        e = E[l][:, :cols].double()
        e = e if rows >= cols else e.T
        bound = 2.0 ** -24 * ((6 * r / 16) ** 0.5 + 4)
        worst = float(((e - (m - p @ q.T)).norm(dim=0) / (size + q.norm(dim=1) * r ** 0.5)).max())
        assert worst <= bound, (tag, worst, bound)
