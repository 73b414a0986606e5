"""Workloads of the M-FAC library for performance measurement.

Three families, over the sizes at which the library is used:

  window cases   the sliding window: a step (`Window.replace`, alone, with
                 extra queries, or refactoring on every replace), a sequence of
                 known gradients, plain IHVPs, the restore of a checkpoint;
  optim cases    `MFAC.step` on the parameters of a network;
  static cases   the pruning step (precompute, inverse diagonal, keep-mask, OBS
                 correction) in both precision modes, and IHVPs on a finished
                 precompute.

Gradients follow the distributions of the benchmark workloads: log-normal
per-coordinate scales times normal entries over sqrt(d), or plain normal
entries over sqrt(d). `exact` is the textbook evaluation in 64 bits (Woodbury
over the m x m Gram matrix).
"""

import math

import torch

from paper_2107_03356_amd import StaticBlocks, Window
from paper_2107_03356_amd.optim import MFAC

DEV = "cuda:0"
POOL = 4              # distinct new gradients a window case cycles through
STATIC_SCALE_D = 4_194_304   # static gradients keep the entry scale of a 4.19M-weight network
THETA_STD = 0.05


def listed():
    return [
        # the smallest window: a few dense layers' worth of weights, where a
        # step is launches and latency
        dict(name="step_tiny", kind="step", d=4096, m=16, lam=1e-3, dist="gauss", q=0, period=-1),
        # a whole optimizer step on a CIFAR ResNet-20 (59 parameter tensors)
        dict(name="optim_resnet20", kind="optim", d=269_722, m=512, lam=1e-4, dist="gauss", net="resnet20"),
        # a mid-size network's step, coefficient phase and passes both visible
        dict(name="step_d1m_m256", kind="step", d=1_048_576, m=256, lam=1e-4, dist="lognormal", q=0, period=-1),
        # ResNet18-sized window, 8 extra vectors preconditioned with each step
        dict(name="step_resnet18_q8", kind="step", d=11_200_000, m=1024, lam=1e-5, dist="lognormal", q=8, period=-1),
        # IHVPs for a batch of vectors; odd d, so that no row but the first is
        # 16-byte aligned, and m no multiple of a tile
        dict(name="ihvp_odd_n4", kind="ihvp", d=777_777, m=300, lam=1e-4, dist="lognormal", n=4),
        # the most conservative coefficient policy: full refactor on each replace
        dict(name="step_refactor_m1024", kind="step", d=262_144, m=1024, lam=1e-5, dist="lognormal", q=0, period=0),
        # resuming an optimizer of a WRN-40-2: rows back into the window, Gram
        # matrix, factor, first IHVP
        dict(name="restore_wrn40_2", kind="restore", d=2_255_156, m=512, lam=1e-4, dist="gauss"),
        # eight gradients known in advance, entered one after another
        dict(name="seq_wrn40_2_n8", kind="seq", d=2_255_156, m=512, lam=1e-4, dist="gauss", n=8),
        # the pruning step of a 4.19M-weight network, fp32 matrix cores with
        # the exact keep-mask
        dict(name="prune_fast_4m", kind="prune", d=4_194_304, m=1024, lam=1e-4, dist="lognormal", block=2048,
             fast=True),
        # the same in the library's default mode (fp64) on a quarter of it
        dict(name="prune_fp64_1m", kind="prune", d=1_048_576, m=1024, lam=1e-4, dist="lognormal", block=2048,
             fast=False),
        # a small network in many narrow blocks, sizes that no tile divides
        dict(name="prune_small", kind="prune", d=60_000, m=100, lam=1e-4, dist="lognormal", block=100, fast=True),
        # IHVPs on the finished precompute
        dict(name="static_ihvp_4m", kind="static_ihvp", d=4_194_304, m=1024, lam=1e-4, dist="lognormal", block=2048,
             n=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any kind, sizes log-uniform over its range (odd ones
    among them), capped at the largest listed window or gradient matrix."""
    kind = rng.choice(["step", "step", "step", "ihvp", "seq", "restore", "optim", "prune", "prune", "static_ihvp"])
    lam = rng.choice([1e-5, 1e-4, 1e-3])
    dist = rng.choice(["gauss", "lognormal"])
    if kind in ("prune", "static_ihvp"):
        block = rng.choice([64, 100, 256, 500, 1024, 2048, 4096, 0])
        m = _log_int(rng, 64, 1024)
        cap = 1.5e9 if kind == "prune" else 4.2e9   # entries of G
        if block == 0:                              # one block over all coordinates
            block = 4 * _log_int(rng, 4_000, min(1_000_000, int(cap / m) // 4))
            d = block
        else:
            m = min(m, 4 * block)                   # more gradients than a few block widths add nothing
            d = block * _log_int(rng, max(1, 16_000 // block), max(2, int(min(4e6, cap / m)) // block))
        case = dict(kind=kind, d=d, m=m, lam=max(lam, 1e-4), dist=dist, block=block)
        if kind == "prune":
            case["fast"] = rng.random() < 0.6 and block <= 4096
        else:
            case["n"] = rng.randint(1, 4)
        return case
    m = _log_int(rng, 16, 1024)
    d = _log_int(rng, 4096, 11_000_000)
    if rng.random() < 0.5:
        d = d // 4 * 4
    case = dict(kind=kind, d=d, m=m, lam=lam, dist=dist)
    if kind == "step":
        case["q"] = rng.choice([0, 0, 0, 1, 3, 8])
        case["period"] = rng.choice([-1, -1, -1, 0])
    elif kind == "ihvp":
        case["n"] = rng.choice([1, 1, 2, 4, 9])
    elif kind == "seq":
        case["n"] = rng.randint(2, 8)
        case["d"] = min(d, 4_000_000)
    elif kind == "restore":
        case["d"] = min(d, 4_000_000)
    elif kind == "optim":
        case["net"] = "mlp"
        width = _log_int(rng, 24, 1200)
        case["width"] = width
        case["d"] = sum(math.prod(s) for s in _mlp_shapes(width))
    return case


# ---------------------------------------------------------------- inputs


def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + stream) & 0x7FFF_FFFF_FFFF_FFFF)
    return g


def _scales(case, seed):
    """Per-coordinate entry scale (fp32): s_j / sqrt(d)."""
    d = case["d"]
    sd = max(d, STATIC_SCALE_D) if "block" in case else d
    s = torch.full((d,), 1.0 / math.sqrt(sd), device=DEV)
    if case["dist"] == "lognormal":
        s *= torch.exp(torch.randn(d, generator=_gen(seed, 0), device=DEV))
    return s


def _vectors(case, seed, stream, n, scales):
    """n gradient-like vectors (n x d fp32)."""
    v = torch.randn((n, case["d"]), generator=_gen(seed, stream), device=DEV)
    return v.mul_(scales)


def _row_chunks(case, seed, scales):
    """The window's (or G's) m rows in chunks of at most 2 GB: (first, rows)."""
    d, m = case["d"], case["m"]
    step = max(1, min(m, (1 << 29) // d))
    for r in range(0, m, step):
        yield r, _vectors(case, seed, 1000 + r, min(step, m - r), scales)


def _resnet20_shapes():
    shapes = [(16, 3, 3, 3), (16,), (16,)]
    cin = 16
    for cout in (16, 32, 64):
        for _ in range(3):
            shapes += [(cout, cin, 3, 3), (cout,), (cout,), (cout, cout, 3, 3), (cout,), (cout,)]
            cin = cout
    return shapes + [(10, 64), (10,)]


def _mlp_shapes(width):
    return [(width, 784), (width,), (width, width), (width,), (10, width), (10,)]


OPT_LR, OPT_WD = 1e-3, 5e-4


def _opt_inputs(case, seed, scales):
    """Weights and gradients of the network's parameters, as flat vectors."""
    w = torch.randn(case["d"], generator=_gen(seed, 5), device=DEV) * 0.05
    g = _vectors(case, seed, 6, 1, scales)[0]
    return w, g


def _split(flat, shapes):
    out, off = [], 0
    for s in shapes:
        n = math.prod(s)
        out.append(flat[off:off + n].view(s))
        off += n
    return out


def _theta(case, seed):
    return torch.randn(case["d"], generator=_gen(seed, 4), device=DEV) * THETA_STD


def _fill(win, case, seed, scales):
    for r, rows in _row_chunks(case, seed, scales):
        win.set_rows(r, rows)
    win.rebuild()


def prepare(case, seed):
    kind, d, m = case["kind"], case["d"], case["m"]
    sc = _scales(case, seed)
    st = dict(case=case)
    if kind in ("step", "ihvp", "seq"):
        q = {"step": case.get("q", 0), "ihvp": case.get("n", 1) - 1, "seq": 0}[kind]
        win = Window(d, m, case["lam"], max_queries=q, device=DEV)
        _fill(win, case, seed, sc)
        if case.get("period", -1) >= 0:
            win.set_refactor_period(case["period"])
        st.update(win=win, t=0)
        if kind == "step":
            st["g"] = [_vectors(case, seed, 10 + t, 1, sc)[0] for t in range(POOL)]
            st["X"] = _vectors(case, seed, 20, q, sc) if q else None
            st["y"] = torch.empty(d, device=DEV)
            st["Y"] = torch.empty((q, d), device=DEV) if q else None
        else:
            st["X"] = _vectors(case, seed, 20, case["n"], sc)
            st["Y"] = torch.empty_like(st["X"])
    elif kind == "restore":
        st["rows"] = torch.cat([rows for _, rows in _row_chunks(case, seed, sc)])
        st["x"] = _vectors(case, seed, 20, 1, sc)[0]
        st["y"] = torch.empty(d, device=DEV)
        st["win"] = Window(d, m, case["lam"], device=DEV)
    elif kind == "optim":
        shapes = _resnet20_shapes() if case["net"] == "resnet20" else _mlp_shapes(case["width"])
        w, g = _opt_inputs(case, seed, sc)
        params = [torch.nn.Parameter(p.clone()) for p in _split(w, shapes)]
        for p, gp in zip(params, _split(g, shapes)):
            p.grad = gp.clone()
        opt = MFAC(params, lr=OPT_LR, m=m, damp=case["lam"], weight_decay=OPT_WD)
        _fill(opt.window, case, seed, sc)
        st.update(opt=opt, params=params)
    else:
        G = torch.cat([rows for _, rows in _row_chunks(case, seed, sc)])
        if kind == "prune":
            st["G0"], st["theta"] = G, _theta(case, seed)
            # the fp64 mode overwrites its G: it works on a copy
            st["G"] = G if case["fast"] else torch.empty_like(G)
        else:
            st["sb"] = StaticBlocks(G, case["block"], case["lam"])
            st["X"] = _vectors(case, seed, 20, case["n"], sc)
            st["Y"] = torch.empty_like(st["X"])
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "step":
        g = st["g"][st["t"] % POOL]
        st["t"] += 1
        if st["X"] is None:
            return st["win"].replace(g, y_out=st["y"])
        return st["win"].replace(g, y_out=st["y"], X=st["X"], Y=st["Y"])
    if kind == "ihvp":
        return st["win"].ihvp(st["X"], st["Y"])
    if kind == "seq":
        return st["win"].replace_seq(st["X"], st["Y"])
    if kind == "restore":
        win = st["win"]
        win.set_rows(0, st["rows"])
        win.rebuild()
        win.set_head(0, case["m"])
        return win.ihvp(st["x"], st["y"])
    if kind == "optim":
        st["opt"].step()
        return [p.data for p in st["params"]] + [st["opt"].preconditioned()]
    if kind == "static_ihvp":
        return st["sb"].ihvp(st["X"], st["Y"])
    if not case["fast"]:
        st["G"].copy_(st["G0"])
    sb = StaticBlocks(st["G"], case["block"], case["lam"], fp32=case["fast"])
    diag = sb.inv_diag(fp64=True)
    mask, _ = sb.obs_mask(st["theta"], case["d"] // 2, scores=False)
    delta = sb.obs_update(st["theta"], mask)
    sb.close()
    return [diag, mask, delta]


def work(case):
    """Each input read once and each output written once; the operations of the
    textbook evaluation (a multiplication and an addition each one)."""
    kind, d, m = case["kind"], float(case["d"]), float(case["m"])
    chol = 2.0 * m ** 3 / 3.0       # factor and triangular inverse
    if kind == "step":
        # the window is read for G x and again for G^T c, which depends on all of it
        nv = 1 + case["q"]
        return dict(bytes=4 * d * (2 * m + 2 * nv) + 4 * d, flops=4 * m * d * nv + (chol if case["period"] == 0 else 0))
    if kind == "ihvp":
        return dict(bytes=4 * d * (2 * m + 2 * case["n"]), flops=4 * m * d * case["n"])
    if kind == "seq":
        # one read per gradient, and one more for the first
        return dict(bytes=4 * d * ((case["n"] + 1) * m + 3 * case["n"]), flops=4 * m * d * case["n"])
    if kind == "restore":
        return dict(bytes=4 * d * (3 * m + 2), flops=m * m * d + chol + 4 * m * d)
    if kind == "optim":
        return dict(bytes=4 * d * (2 * m + 5), flops=4 * m * d)
    B = float(case["block"])
    if kind == "static_ihvp":
        return dict(bytes=4 * d * (2 * m + 2 * case["n"]), flops=4 * m * d * case["n"])
    # Gram (lower half) and triangular W, factor and inverse per block, W twice for the correction
    return dict(bytes=4 * d * m + 8 * d + 4 * d + d + 4 * d, flops=2 * m * m * d + chol * (d / B) + 4 * m * d)


def tolerance(case):
    """About four times what is seen against the 64-bit evaluation: 2.5e-8 to
    5e-8 (the fp32 rounding of the outputs) where sums run in fp64; 8e-7 where
    more than four vectors are fused into a pass, whose per-lane sums are fp32;
    the fp32 matrix products of the fast static mode, 6e-9 to 6e-8 on
    well-conditioned blocks, more on wide ones. Keep-masks are exact in either mode."""
    if case["kind"] == "prune" and case["fast"]:
        return {"rel": 1e-6, "differ": 0.0}
    if case["kind"] in ("step", "ihvp") and max(case.get("q", 0) + 1, case.get("n", 1)) > 4:
        return {"rel": 4e-6}
    return {"rel": 2e-7, "differ": 0.0}


# ---------------------------------------------------------------- 64-bit evaluation


def _cols(d, m):
    """Column ranges of at most 2 GB in fp64 over m rows."""
    step = max(1, (1 << 28) // m)
    for c in range(0, d, step):
        yield slice(c, min(d, c + step))


class _ExactWindow:
    """F^-1 x of the window G (fp32 rows, m x d) in fp64: Woodbury over A = G G^T + m lam I."""

    def __init__(self, G, lam):
        self.G, self.lam, self.m = G, lam, G.shape[0]
        self.K = torch.zeros((self.m, self.m), dtype=torch.float64, device=DEV)
        for c in _cols(G.shape[1], self.m):
            g = G[:, c].double()
            self.K += g @ g.T

    def replace(self, k, g):
        self.G[k] = g
        p = self.products(g[None])[:, 0]
        self.K[k, :] = p
        self.K[:, k] = p

    def products(self, X):
        P = torch.zeros((self.m, X.shape[0]), dtype=torch.float64, device=DEV)
        for c in _cols(self.G.shape[1], self.m):
            P += self.G[:, c].double() @ X[:, c].double().T.contiguous()
        return P

    def _solve(self, P):
        A = self.K.cpu() + self.m * self.lam * torch.eye(self.m, dtype=torch.float64)
        return torch.cholesky_solve(P.cpu(), torch.linalg.cholesky(A)).to(DEV)

    def _combine(self, C):
        Y = torch.empty((C.shape[1], self.G.shape[1]), dtype=torch.float64, device=DEV)
        for c in _cols(self.G.shape[1], self.m):
            Y[:, c] = C.T.contiguous() @ self.G[:, c].double()
        return Y

    def inserted(self, k):
        """F^-1 g for the g in slot k: m G^T A^-1 e_k."""
        e = torch.zeros((self.m, 1), dtype=torch.float64)
        e[k] = 1.0
        return self.m * self._combine(self._solve(e))[0]

    def ihvp(self, X):
        return (X.double() - self._combine(self._solve(self.products(X)))) / self.lam


def _exact_blocks(G, case):
    """A_b^-1 G_b per block, in fp64: yields (first coordinate, G_b, Z_b) for a few blocks at a time."""
    B, m, lam = case["block"], case["m"], case["lam"]
    nb = case["d"] // B
    step = max(1, (1 << 28) // (m * max(m, min(B, 1 << 20))))
    eye = torch.eye(m, dtype=torch.float64, device=DEV)
    for b0 in range(0, nb, step):
        n = min(step, nb - b0)
        A = torch.empty((n, m, m), dtype=torch.float64, device=DEV)
        for i in range(n):
            A[i] = m * lam * eye
            for c in _cols(B, m):
                g = G[:, (b0 + i) * B:(b0 + i + 1) * B][:, c].double()
                A[i] += g @ g.T
        # inverse of an SPD matrix by its factor's inverse (one triangular solve)
        Linv = torch.linalg.solve_triangular(torch.linalg.cholesky(A), eye.expand(n, m, m), upper=False)
        for i in range(n):
            Ainv = Linv[i].T.contiguous() @ Linv[i]
            for c in _cols(B, m):
                g = G[:, (b0 + i) * B:(b0 + i + 1) * B][:, c].double()
                yield (b0 + i) * B + c.start, g, Ainv, i == n - 1


def _exact_static(case, seed):
    lam, d, B = case["lam"], case["d"], case["block"]
    if d // B > 4096 or case["m"] ** 2 * d > 6e12:
        return None
    sc = _scales(case, seed)
    G = torch.cat([rows for _, rows in _row_chunks(case, seed, sc)])
    if case["kind"] == "static_ihvp":
        X = _vectors(case, seed, 20, case["n"], sc).double()
        return _static_apply(G, case, X)
    diag = torch.empty(d, dtype=torch.float64, device=DEV)
    for j, g, Ainv, _ in _exact_blocks(G, case):
        diag[j:j + g.shape[1]] = (1.0 - (g * (Ainv @ g)).sum(0)) / lam
    theta = _theta(case, seed).double()
    score = theta * theta / (2.0 * diag)
    keep = torch.zeros(d, dtype=torch.uint8, device=DEV)
    keep[torch.sort(score, descending=True, stable=True).indices[:d // 2]] = 1
    x = torch.where(keep.bool(), torch.zeros_like(theta), theta / diag)
    return [diag, keep, -_static_apply(G, case, x[None])[0]]


def _static_apply(G, case, X):
    lam, B = case["lam"], case["block"]
    P = torch.zeros((X.shape[0], case["d"] // B, case["m"]), dtype=torch.float64, device=DEV)
    for j, g, _, _ in _exact_blocks_plain(G, case):
        P[:, j // B] += X[:, j:j + g.shape[1]] @ g.T.contiguous()
    Y = torch.empty_like(X)
    for j, g, Ainv, _ in _exact_blocks(G, case):
        Y[:, j:j + g.shape[1]] = (X[:, j:j + g.shape[1]] - P[:, j // B] @ Ainv @ g) / lam
    return Y


def _exact_blocks_plain(G, case):
    B = case["block"]
    for b in range(case["d"] // B):
        for c in _cols(B, case["m"]):
            yield b * B + c.start, G[:, b * B:(b + 1) * B][:, c].double(), None, False


def exact(case, seed):
    kind = case["kind"]
    if kind in ("prune", "static_ihvp"):
        return _exact_static(case, seed)
    sc = _scales(case, seed)
    G = torch.empty((case["m"], case["d"]), device=DEV)
    for r, rows in _row_chunks(case, seed, sc):
        G[r:r + rows.shape[0]] = rows
    E = _ExactWindow(G, case["lam"])
    if kind == "step":
        E.replace(0, _vectors(case, seed, 10, 1, sc)[0])
        y = E.inserted(0)
        return [y, E.ihvp(_vectors(case, seed, 20, case["q"], sc))] if case["q"] else y
    if kind == "ihvp":
        return E.ihvp(_vectors(case, seed, 20, case["n"], sc))
    if kind == "seq":
        out = []
        for t, g in enumerate(_vectors(case, seed, 20, case["n"], sc)):
            E.replace(t, g)
            out.append(E.inserted(t))
        return torch.stack(out)
    if kind == "restore":
        return E.ihvp(_vectors(case, seed, 20, 1, sc))[0]
    w, g = _opt_inputs(case, seed, sc)
    E.replace(0, g + OPT_WD * w)
    y = E.inserted(0)
    shapes = _resnet20_shapes() if case["net"] == "resnet20" else _mlp_shapes(case["width"])
    return _split(w.double() - OPT_LR * y, shapes) + [y]
