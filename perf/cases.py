"""The work that a user of this compressor has it do, as cases that can be timed and compared.

A case is one step of a training loop on a fixed set of weight matrices: the gradients are compressed with error
feedback (psgd_compress, psgd_compress_refresh, or the two halves between which a data-parallel job exchanges P), and the
compressed update is used (reconstructed, or fed to the fused momentum-SGD or Adam step).  Inputs are those of a run
under way: gradients with a shared low-rank signal and fresh noise per worker, an error buffer that holds what earlier steps
did not send, a Q that spans roughly the leading subspace, optimizer state of the size the updates have.

Keys of a case:
  layers   "ROWSxCOLS[/LD][*COUNT],..." in storage order; rows < cols is a layer stored as the transpose
  r        compression rank;  n_workers: gradients averaged per layer;  dtype: "f32" or "bf16" gradients
  op       "step" (SSP-Comp), "refresh" (SVD-Comp) or "halves" (project + finish, one worker of a data-parallel job)
  update   "f32" / "bf16" (psgd_decompress into that type), "msgd" or "adam" (fused optimizer step)
  factors  "kept" (the update takes the factors the compress call left in the workspace) or "given" (P and Q passed)
  lazy     deferred residual;  signal, decay: rank and decay of the gradients' common signal;  noise: noise / signal norm
"""
import math

import torch

from paper_2509_11254_amd import psgd

BLOCK_1B = "2048x2048*4,5632x2048*2,2048x5632"      # q, k, v, o, gate, up, down as stored
BLOCK_7B = "4096x4096*4,11008x4096*3"


def _repeat(block, count):
    out = []
    for item in block.split(","):
        shape, _, n = item.partition("*")
        out.append("%s*%d" % (shape, int(n or 1) * count))
    return ",".join(out)


def _case(layers, r, n_workers, dtype, op, update, factors="kept", lazy=False, signal=64, decay=0.9, noise=0.01):
    return {"layers": layers, "r": r, "n_workers": n_workers, "dtype": dtype, "op": op, "update": update,
            "factors": factors, "lazy": lazy, "signal": signal, "decay": decay, "noise": noise}


def listed():
    named = {
        # the smallest use: one 256 x 128 variable; launches and host work are all there is to it
        "linear_256x128_f32": _case("256x128", 4, 4, "f32", "step", "f32", signal=8, decay=0.5, noise=0.1),
        # its refresh, due every few steps on such problems (tau = 5)
        "linear_256x128_f32_refresh": _case("256x128", 4, 4, "f32", "refresh", "f32", signal=8, decay=0.5, noise=0.1),
        # odd sizes, padded rows, both orientations, momentum SGD: the layers of a small mixed model
        "ragged_f32_msgd": _case("333x203/208,1000x264,264x1000,200x328,520x328,130x129/136,1000x40,64x24", 8, 2, "f32",
                                 "step", "msgd", signal=16, decay=0.8),
        # one large dense matrix, eight fp32 workers: the common single-matrix step
        "dense_4096_f32_n8": _case("4096x4096", 8, 8, "f32", "step", "f32", signal=32, decay=0.8),
        # its refresh (tau = 10)
        "dense_4096_f32_n8_refresh": _case("4096x4096", 8, 8, "f32", "refresh", "f32", signal=32, decay=0.8),
        # a few transformer blocks in fp32 at a low rank with momentum SGD; the "down" matrices are stored transposed
        "blocks_1b_two_f32_msgd": _case(_repeat(BLOCK_1B, 2), 16, 2, "f32", "step", "msgd"),
        # all matrices of a 1B-shaped model, four bf16 workers on the GPU, deferred residual
        "blocks_1b_all_bf16_n4": _case(_repeat(BLOCK_1B, 22), 32, 4, "bf16", "step", "f32", lazy=True),
        # one GPU's share of a data-parallel job on 7B-shaped blocks: two halves around the exchange, then Adam on the
        # averaged factors
        "blocks_7b_two_halves_adam": _case(_repeat(BLOCK_7B, 2), 64, 1, "bf16", "halves", "adam", factors="given"),
        # the refresh of a 7B-shaped block
        "blocks_7b_one_bf16_refresh": _case(BLOCK_7B, 64, 1, "bf16", "refresh", "f32", signal=128, decay=0.95),
        # a refresh at every step on one wide, high-rank matrix (tau = 1)
        "dense_8192_f32_r128_refresh": _case("8192x8192", 128, 1, "f32", "refresh", "f32", signal=256, decay=0.95),
        # the plain step at a high rank on bf16 gradients, update written in bf16
        "dense_8192_bf16_r128": _case("8192x8192", 128, 1, "bf16", "step", "bf16", signal=256, decay=0.95),
        # the largest: all 224 matrices of a 7B-shaped model, bf16, deferred residual
        "blocks_7b_all_bf16": _case(_repeat(BLOCK_7B, 32), 64, 1, "bf16", "step", "f32", lazy=True),
    }
    return [dict(case, name=name) for name, case in named.items()]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: a single matrix of any size or a batch of blocks, any rank, type and option."""
    dtype = rng.choice(["f32", "bf16"])
    op = rng.choice(["step", "step", "step", "refresh", "halves"])
    update = rng.choice(["f32", "bf16", "msgd", "adam"])
    if rng.random() < 0.5:
        rows, cols = _log_int(rng, 64, 8192), _log_int(rng, 64, 8192)
        if rng.random() < 0.5:
            rows, cols = max(64, rows // 64 * 64), max(64, cols // 64 * 64)
        ld = (cols + 7) // 8 * 8 + (8 * rng.randrange(1, 4) if rng.random() < 0.25 else 0)
        layers = "%dx%d/%d" % (rows, cols, ld) if ld != cols else "%dx%d" % (rows, cols)
        n_workers = rng.choice([1, 1, 2, 3, 4, 8, 16]) if rows * cols <= 1 << 24 else rng.choice([1, 2, 4])
        r = min(_log_int(rng, 2, 128), min(rows, cols) // 2)
    else:
        hidden = 8 * _log_int(rng, 32, 512)
        inter = 8 * int(hidden * rng.uniform(2.0, 4.0) / 8)
        n_workers = rng.choice([1, 1, 1, 2, 4])
        most = (2.5e9 if op != "refresh" else 4e8) / (hidden * (4 * hidden + 3 * inter)) / n_workers
        count = max(1, min(_log_int(rng, 1, 32), int(most)))
        down = "%dx%d" % ((hidden, inter) if rng.random() < 0.5 else (inter, hidden))
        layers = _repeat("%dx%d*4,%dx%d*2,%s" % (hidden, hidden, inter, hidden, down), count)
        r = min(_log_int(rng, 4, 64), hidden // 2)
    if op == "halves":
        n_workers = 1
    lazy = op == "step" and rng.random() < 0.5
    factors = "given" if op == "halves" else rng.choice(["kept", "given"])
    return _case(layers, r, n_workers, dtype, op, update, factors=factors, lazy=lazy, signal=2 * r,
                 decay=round(0.5 ** (8.0 / (2 * r)), 4))


def _shapes(case):
    out = []
    for item in case["layers"].split(","):
        shape, _, count = item.partition("*")
        shape, _, ld = shape.partition("/")
        rows, cols = (int(x) for x in shape.split("x"))
        out += [(rows, cols, int(ld or cols))] * int(count or 1)
    return out


def _buckets(sizes, dtype, most=4):
    """One tensor per layer, cut from at most `most` flat buffers (as a job that exchanges buckets keeps them)."""
    flats, views = [], []
    per = -(-len(sizes) // most)
    for i in range(0, len(sizes), per):
        part = sizes[i:i + per]
        offs = [0]
        for rows, ld in part:
            offs.append(offs[-1] + (rows * ld + 63) // 64 * 64)
        flat = torch.zeros(offs[-1], dtype=dtype, device="cuda")
        flats.append(flat)
        views += [flat[o:o + rows * ld].view(rows, ld) for o, (rows, ld) in zip(offs, part)]
    return flats, views


def prepare(case, seed):
    shapes, r, bf16 = _shapes(case), case["r"], case["dtype"] == "bf16"
    comp = psgd.Compressor([(rows, cols, r, psgd.PSGD_BF16 if bf16 else psgd.PSGD_F32, ld) for rows, cols, ld in shapes],
                           case["n_workers"], lazy_residual=case["lazy"],
                           q_resident=case["op"] == "step" and case["factors"] == "kept")
    return dict(_inputs(case, seed), comp=comp)


def _inputs(case, seed):
    shapes, r, n, sk = _shapes(case), case["r"], case["n_workers"], case["signal"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def randn(*size):
        return torch.randn(size, generator=gen, device="cuda")

    bf16 = case["dtype"] == "bf16"
    state = {"case": dict(case), "t": 100}
    full = [(rows, ld) for rows, cols, ld in shapes]
    state["E_flat"], E = _buckets(full, torch.float32)
    state["P_flat"], P = _buckets([(max(rows, cols), r) for rows, cols, ld in shapes], torch.float32)
    state["Q_flat"], Q = _buckets([(min(rows, cols), r) for rows, cols, ld in shapes], torch.float32)
    if case["update"] in ("msgd", "adam"):
        state["X_flat"], X = _buckets(full, torch.float32)
        state["M1_flat"], M1 = _buckets(full, torch.float32)
        if case["update"] == "adam":
            state["M2_flat"], M2 = _buckets(full, torch.float32)
    else:
        state["O_flat"], out = _buckets(full, torch.bfloat16 if case["update"] == "bf16" else torch.float32)
        state["out"] = out
    scale = case["decay"] ** torch.arange(sk, device="cuda", dtype=torch.float32)
    size = float(scale.square().sum().sqrt())
    G = []
    for l, (rows, cols, ld) in enumerate(shapes):
        k = min(sk, rows, cols)
        u, v = randn(rows, k) / rows ** 0.5, randn(cols, k) / cols ** 0.5
        signal = (u * scale[:k]) @ v.T
        sigma = case["noise"] * size / (rows * cols) ** 0.5
        per_worker = []
        for _ in range(n):
            g = torch.zeros((rows, ld), dtype=torch.bfloat16 if bf16 else torch.float32, device="cuda")
            g[:, :cols] = torch.add(signal, randn(rows, cols), alpha=sigma)
            per_worker.append(g)
        G.append(per_worker)
        # what earlier steps did not send: of the size of a step's noise
        E[l][:, :cols] = sigma * randn(rows, cols)
        # Q of the step before: the signal's short-side factor, a little off
        short = v if rows >= cols else u
        q = torch.zeros_like(Q[l])
        q[:, :min(k, r)] = short[:, :min(k, r)] * scale[:min(k, r)]
        Q[l].copy_(q + 0.02 * float(scale[min(k, r) - 1]) / Q[l].shape[0] ** 0.5 * randn(*q.shape))
        if case["update"] in ("msgd", "adam"):
            rms = size / (rows * cols) ** 0.5
            X[l][:, :cols] = 0.02 * randn(rows, cols)
            M1[l][:, :cols] = rms * randn(rows, cols)
            if case["update"] == "adam":
                M2[l][:, :cols] = (rms * (1.0 + 0.2 * randn(rows, cols))).square()
    state.update(G=G, E=E, P=P, Q=Q)
    if case["update"] in ("msgd", "adam"):
        state.update(X=X, M1=M1)
        if case["update"] == "adam":
            state["M2"] = M2
    return state


def run(state):
    case, comp = state["case"], state["comp"]
    G, E, P, Q = state["G"], state["E"], state["P"], state["Q"]
    if case["op"] == "refresh":
        comp.compress_refresh(G, E, Q, P)
    elif case["op"] == "halves":
        comp.compress_project(G, E, Q, P)       # (the job averages P here, and Q below)
        comp.compress_finish(E, Q, P)
    else:
        comp.compress(G, E, Q, P)
    fp, fq = (P, Q) if case["factors"] == "given" else (None, None)
    out = {"E": state["E_flat"]}                # (deferred residual: M, as documented, until it is settled)
    if case["op"] != "refresh":
        # (a refresh's singular vectors have free signs: what it gives is in E and in the update)
        out.update(P=state["P_flat"], Q=state["Q_flat"])
    if case["update"] == "msgd":
        comp.decompress_msgd(fp, fq, state["M1"], state["X"], 0.9, 1e-3)
        out.update(X=state["X_flat"], M1=state["M1_flat"])
    elif case["update"] == "adam":
        state["t"] += 1
        comp.decompress_adam(fp, fq, state["M1"], state["M2"], state["X"], state["t"], 1e-3, weight_decay=0.01)
        out.update(X=state["X_flat"], M1=state["M1_flat"], M2=state["M2_flat"])
    else:
        comp.decompress(fp, fq, state["out"], psgd.PSGD_BF16 if case["update"] == "bf16" else psgd.PSGD_F32)
        out["update"] = state["O_flat"]
    return out


def exact(case, seed):
    """The first pass on a new state in 64 bits (the flat buffers' padding stays zero); None for the largest sets."""
    shapes, r = _shapes(case), case["r"]
    if sum(rows * cols for rows, cols, ld in shapes) > 450e6:
        return None
    state = _inputs(case, seed)
    full = [(rows, ld) for rows, cols, ld in shapes]
    flat, view = {}, {}
    for key, sizes in (("E", full), ("P", [(max(rows, cols), r) for rows, cols, ld in shapes]),
                       ("Q", [(min(rows, cols), r) for rows, cols, ld in shapes]), ("update", full),
                       ("X", full), ("M1", full), ("M2", full)):
        if key in ("E", "P", "Q") or key in state or (key == "update" and "out" in state):
            flat[key], view[key] = _buckets(sizes, torch.float64)
    for l, (rows, cols, ld) in enumerate(shapes):
        m = sum(g[:, :cols].double() for g in state["G"][l]) / case["n_workers"] + state["E"][l][:, :cols].double()
        tall = m if rows >= cols else m.T
        p = _leading(tall, r, case["signal"]) if case["op"] == "refresh" else _orth(tall @ state["Q"][l].double())
        q = tall.T @ p
        d = p @ q.T if rows >= cols else q @ p.T
        view["P"][l].copy_(p)
        view["Q"][l].copy_(q)
        view["E"][l][:, :cols] = m if case["lazy"] else m - d
        if case["update"] == "msgd":
            m1 = 0.9 * state["M1"][l][:, :cols].double() + d
            view["M1"][l][:, :cols] = m1
            view["X"][l][:, :cols] = state["X"][l][:, :cols].double() - 1e-3 * m1
        elif case["update"] == "adam":
            t, x = state["t"] + 1, state["X"][l][:, :cols].double()
            m1 = 0.9 * state["M1"][l][:, :cols].double() + 0.1 * d
            m2 = 0.999 * state["M2"][l][:, :cols].double() + 0.001 * d * d
            view["M1"][l][:, :cols] = m1
            view["M2"][l][:, :cols] = m2
            step = (m1 / (1 - 0.9 ** t)) / ((m2 / (1 - 0.999 ** t)).sqrt() + 1e-8)
            view["X"][l][:, :cols] = x - 1e-3 * (step + 0.01 * x)
        else:
            view["update"][l][:, :cols] = d
    if case["op"] == "refresh":
        del flat["P"], flat["Q"]
    return flat


def _orth(a):
    """The Q factor with R's diagonal positive."""
    q, upper = torch.linalg.qr(a)
    return q * torch.sign(torch.diagonal(upper))


def _leading(a, r, signal):
    """The r leading left singular vectors; by block iteration where a whole decomposition would take long (the block
    holds all of the signal, and the singular values after it are the noise's)."""
    n = a.shape[1]
    if n <= 512:
        return torch.linalg.svd(a, full_matrices=False)[0][:, :r]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    y = torch.randn((n, min(n, signal + 64)), generator=gen, device="cuda", dtype=torch.float64)
    for _ in range(50):
        z = _orth(a @ y)
        y = a.T @ z
    return z @ torch.linalg.eigh(y.T @ y)[1].flip(1)[:, :r]


def work(case):
    """Each gradient, error buffer and optimizer state read once and each result written once; the products that the
    step is made of at its rank (a refresh: one product each way, whatever iterations its spectrum asks for)."""
    shapes, r = _shapes(case), case["r"]
    per = case["n_workers"] * (2 if case["dtype"] == "bf16" else 4) + 8
    per += {"f32": 4, "bf16": 2, "msgd": 16, "adam": 24}[case["update"]]
    elems = sum(rows * cols for rows, cols, ld in shapes)
    thin = sum(4.0 * r * (max(rows, cols) + 2 * min(rows, cols)) for rows, cols, ld in shapes)
    return {"bytes": per * elems + thin, "flops": 4 * 2.0 * elems * r}


def tolerance(case):
    """About four times the distance to the same step in fp64 over these ranges, largest over a case's outputs.  It is that
    of the error buffer, which is the small difference of M and its projection (two bf16 planes per operand for bf16
    gradients: 3.2e-4 and at most 5.7e-3; three for fp32: 3.3e-6 and 4.5e-5, and 3e-5 and 3.5e-4 where a refresh cuts a
    slowly falling spectrum), or of the rounding of a bf16 update (1.7e-3)."""
    rel, most = (1.3e-3, 2.4e-2) if case["dtype"] == "bf16" else (1.2e-4, 1.5e-3) if case["op"] == "refresh" else (1.5e-5, 2e-4)
    if case["update"] == "bf16":
        rel, most = max(rel, 7e-3), max(most, 2e-2)
    return {"rel": rel, "max": most}
