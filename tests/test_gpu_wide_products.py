"""The products that read a stored M at widths of three and more blocks of 32 columns (128 rows or columns per workgroup, 64 steps of
the reduction at a time, half of them per wave): both orientations, tiles and reductions cut off at every kind of edge, rows with padding
that holds NaN, one chunk, whole walks and split ones."""
import pytest

from paper_2509_11254_amd import psgd
from gpu_harness import torch_mod

pytestmark = pytest.mark.gpu


def matrix(rows, cols, singular_values, gen):
    torch = torch_mod()
    k = min(rows, cols)
    u, v = (torch.linalg.qr(torch.randn((x, k), generator=gen, device="cuda", dtype=torch.float64))[0] for x in (rows, cols))
    return (u * singular_values) @ v.T


@pytest.mark.parametrize("rows,cols,ld", [(129, 127, 136), (1000, 161, 168), (192, 192, 192), (2049, 1999, 2008), (127, 129, 136),
                                          (161, 1023, 1024), (1985, 2081, 2088), (40000, 130, 136), (130, 40000, 40000)])
@pytest.mark.parametrize("r", [66, 100, 125])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_two_power_iterations(rows, cols, ld, r, dtype):
    torch = torch_mod()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows + r)
    bf = dtype == "bf16"
    comp = psgd.Compressor([(rows, cols, r, psgd.PSGD_BF16 if bf else psgd.PSGD_F32, ld)], 1, power_iters=2)
    G, E = (torch.full((rows, ld), float("nan"), device="cuda") for _ in range(2))
    k = min(rows, cols)
    G[:, :cols] = matrix(rows, cols, torch.linspace(2, 1, k, device="cuda", dtype=torch.float64), gen).float()
    E[:, :cols] = 0.2 / (rows + cols) ** 0.5 * torch.randn((rows, cols), generator=gen, device="cuda")
    G = G.bfloat16() if bf else G
    m, n = max(rows, cols), min(rows, cols)
    Q, P = torch.randn((n, r), generator=gen, device="cuda"), torch.zeros((m, r), device="cuda")
    M = G[:, :cols].double() + E[:, :cols].double()
    M = M if rows >= cols else M.T

    def orth(a):
        q, upper = torch.linalg.qr(a)
        return q * torch.sign(torch.diagonal(upper))

    second = M @ (M.T @ orth(M @ Q.double()))                # (this one's columns before they are orthonormalised)
    comp.compress([[G]], [E], [Q], [P])
    # an operand's planes carry 2^-17 or 2^-24 of it (two operands, M itself rounded to fp32), the fp32 sums of a walk of m steps
    # in pieces of 16 a random walk of roundings; what a product is off by goes into P with the condition of its columns, and
    # the first product's with that of both
    rel = 4 * 2.0 ** (-17 if bf else -23) + 2.0 ** -24 * (m / 16) ** 0.5
    assert torch.linalg.norm(Q.double() - M.T @ P.double()) <= rel * torch.linalg.norm(M)
    cond = float(torch.linalg.cond(second))
    assert torch.linalg.norm(P.double() - orth(second)) <= 3 * rel * cond * r ** 0.5
    D = P.double() @ Q.double().T
    assert torch.linalg.norm(E[:, :cols].double() - (M - D if rows >= cols else (M - D).T)) <= rel * torch.linalg.norm(M)


@pytest.mark.parametrize("rows,cols", [(700, 401), (401, 700)])
@pytest.mark.parametrize("r,oversample", [(80, 8), (120, 16), (150, 10), (168, 24)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_refresh(rows, cols, r, oversample, dtype):
    """Every width of the iteration's products, with a gap at the cut: the best approximation of rank r."""
    torch = torch_mod()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows + r)
    bf = dtype == "bf16"
    k = min(rows, cols)
    G = matrix(rows, cols, torch.cat([torch.logspace(0, -1, r, device="cuda"), 1e-2 * torch.ones(k - r, device="cuda")]).double(), gen)
    G = G.bfloat16() if bf else G.float()
    ld = (cols + 7) // 8 * 8
    G = torch.nn.functional.pad(G, (0, ld - cols), value=float("nan"))
    comp = psgd.Compressor([(rows, cols, r, psgd.PSGD_BF16 if bf else psgd.PSGD_F32, ld)], 1, refresh_oversample=oversample)
    E = torch.zeros((rows, ld), device="cuda")
    Q, P = torch.randn((k, r), generator=gen, device="cuda"), torch.zeros((max(rows, cols), r), device="cuda")
    M = G[:, :cols].double()
    M = M if rows >= cols else M.T
    best = float(torch.linalg.svdvals(M)[r:].square().sum())
    comp.compress_refresh([[G]], [E], [Q], [P])
    left = float(E[:, :cols].double().square().sum())
    rel = 4 * 2.0 ** (-17 if bf else -23) + 2.0 ** -24 * (max(rows, cols) / 16) ** 0.5
    assert torch.linalg.norm(Q.double() - M.T @ P.double()) <= rel * torch.linalg.norm(M)
    # (sixteen iterations leave (1e-2 / 0.1)^32 of the rest; then the products' error, to first order with the cut's 1e-2)
    assert abs(left - best) <= 2 * rel * float(torch.linalg.norm(M)) * best ** 0.5 + (rel * float(torch.linalg.norm(M))) ** 2
