"""Performance cases: the work that programs have this library do, through its
public entry points, over the range of sizes and options it is used with.

listed() names the cases, draw() gives more of the same ranges, prepare()
makes what a program holds before the call (inputs on the GPU from a seed, the
plan, batch or server it keeps), run() is one pass, work() the bytes and
floating-point operations a pass cannot do without, exact() the same outputs
in 64 bits by plain NumPy where that takes seconds.

Inputs follow the library's scene model: every pixel is a draw from
CN(0, A (x) B + I) with A of rank r_a and B of rank r_b at 30 dB clutter to
noise, plus moving targets of 0-15 dB.  Ranks match the plan, as in use (a
plan's rank is set from the scene), and plans with r_a > 1 run a fixed number
of LR-Kron iterations.
"""
import math

import numpy as np
import torch

import paper_1604_03622_amd as kstap

CNR = 1000.0


def listed():
    return [
        # the smallest frame (one tile of a detector's test chip): launch and latency
        dict(name="frame_tiny", kind="frame", p=3, q=8, n=64, r_a=1, r_b=3, H=64, W=64, precision="fp32"),
        # a ragged region of interest, larger temporal rank
        dict(name="frame_ragged", kind="frame", p=3, q=12, n=128, r_a=1, r_b=6, H=187, W=233, precision="fp32"),
        # the headline workload: one full SAR frame resident in HBM
        dict(name="frame_full", kind="frame", p=3, q=16, n=200, r_a=1, r_b=4, H=2048, W=2048, precision="fp32"),
        # the mixed path: split-BF16 covariance with FP64 solves
        dict(name="frame_mixed", kind="frame", p=3, q=16, n=200, r_a=1, r_b=4, H=1024, W=1024, precision="bf16x3"),
        # FP32 covariance with FP64 solves, for frames with strong returns
        dict(name="frame_fp64_solves", kind="frame", p=3, q=16, n=200, r_a=1, r_b=4, H=512, W=512,
             precision="fp32_f64"),
        # more channels and pulses than one wavefront's covariance holds
        dict(name="frame_wide", kind="frame", p=5, q=24, n=256, r_a=1, r_b=4, H=512, W=512, precision="fp32"),
        # a 16-bin Doppler bank with the enhancement image and the bin map
        dict(name="frame_bank", kind="variants", p=3, q=16, n=200, r_a=1, r_b=4, H=768, W=768, precision="fp32",
             nbank=16, passes=1),
        # two registered passes stacked in the channels: change detection
        dict(name="frame_multipass", kind="variants", p=6, q=16, n=200, r_a=2, r_b=3, H=256, W=256, precision="fp32",
             nbank=0, passes=2),
        # uneven tiles of several classes in one reusable batch
        dict(name="batch_tiles", kind="batch", tiles=12, largest=512, scene=1),
        # intermediates (U_A, U_B, eta) of a detection list
        dict(name="probe_list", kind="probe", p=3, q=16, n=200, r_a=1, r_b=4, H=128, W=128, precision="fp32",
             npix=600),
        # one large covariance from five snapshots, with its q x q time factor
        dict(name="lrkron_large", kind="lrkron", p=3, q=2500, n=5, r_a=1),
        # frames that arrive in host memory, through the continuous-batching server
        dict(name="served_frames", kind="served", frames=6, smallest=128, largest=448, scene=1),
    ]


NARROW = [(2, 8, 4), (2, 16, 4), (3, 8, 4), (3, 8, 8), (3, 12, 4), (3, 12, 8), (3, 16, 4), (3, 16, 8), (4, 8, 4),
          (4, 16, 4)]
MIXED = [(3, 8, 4), (3, 8, 8), (3, 12, 4), (3, 12, 8), (3, 16, 4), (3, 16, 8)]
SOLVES = [(3, 8, 4), (3, 16, 4)]
WIDE = [(5, 24, 4), (6, 16, 4)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frame", "frame", "frame", "frame", "wide", "variants", "batch", "probe", "lrkron", "served"])
    if kind == "lrkron":
        p = rng.choice([2, 3, 6])
        return dict(kind="lrkron", p=p, q=_log(rng, 25, 2500 if p < 6 else 1250), n=rng.randint(3, 8), r_a=1)
    if kind == "batch":
        return dict(kind="batch", tiles=rng.randint(3, 12), largest=_log(rng, 96, 512), scene=rng.randint(0, 999))
    if kind == "served":
        return dict(kind="served", frames=rng.randint(2, 6), smallest=64, largest=_log(rng, 128, 448),
                    scene=rng.randint(0, 999))
    precision = rng.choice(["fp32", "fp32", "bf16x3", "fp32_f64"])
    if kind == "wide":
        precision = rng.choice(["fp32", "bf16x3"])
        p, q, rbm = rng.choice(WIDE)
        top = 384
    else:
        if kind in ("variants", "probe"):
            precision = "fp32"
        p, q, rbm = rng.choice({"fp32": NARROW, "bf16x3": MIXED, "fp32_f64": SOLVES}[precision])
        top = 1200 if kind == "frame" else 640 if kind == "variants" else 256
    r_a = 1 if p < 4 or kind == "probe" or rng.random() < 0.6 else 2
    c = dict(kind="frame" if kind == "wide" else kind, p=p, q=q, n=rng.randint(max(61, p * q), 256), r_a=r_a,
             r_b=rng.randint(2, 4) if rbm == 4 else rng.randint(5, 6), H=_log(rng, 40, top), W=_log(rng, 40, top),
             precision=precision)
    if kind == "variants":
        c.update(nbank=rng.choice([0, 0, 7, 16]), passes=1)
    if kind == "probe":
        c["npix"] = _log(rng, 40, 1500)
    return c


# ------------------------------------------------------------------- inputs
def _basis(rs, d, r):
    g = rs.standard_normal((d, r)) + 1j * rs.standard_normal((d, r))
    return np.linalg.qr(g)[0]


def _frame(c, seed, device):
    """One scene [p, H, W, q]: Kronecker clutter of ranks (r_a, r_b), unit
    noise, moving targets (all-ones temporal signature)."""
    p, q, H, W, ra, rb = c["p"], c["q"], c["H"], c["W"], c["r_a"], c["r_b"]
    rs = np.random.default_rng([seed, p, q, H, W])
    la, lb = rs.uniform(0.5, 1.0, ra), rs.uniform(0.5, 1.0, rb)
    K = c.get("passes", 1)
    if K > 1:   # pass k's own rank-one spatial factor in its block of channels, coherence 0.9 across the passes
        ua = np.zeros((p, K), complex)
        for k in range(K):
            ua[k * (p // K):(k + 1) * (p // K), k:k + 1] = _basis(rs, p // K, 1)
        wa = ua @ np.linalg.cholesky(0.9 * np.ones((K, K)) + 0.1 * np.eye(K))
    else:
        wa = _basis(rs, p, ra) * np.sqrt(la)
    wb = _basis(rs, q, rb) * np.sqrt(lb)
    root = np.kron(wa, wb)                                        # [pq, ra rb]
    root *= math.sqrt(CNR * p * q / np.sum(np.abs(root) ** 2))
    gen = torch.Generator(device=device)
    gen.manual_seed(int(rs.integers(1 << 40)))
    x = torch.randn((p, H, W, q), dtype=torch.complex64, device=device, generator=gen)
    z = torch.randn((H * W, root.shape[1]), dtype=torch.complex64, device=device, generator=gen)
    rt = torch.from_numpy(root.T.astype(np.complex64)).to(device)
    for i in range(p):
        x[i] += (z @ rt[:, i * q:(i + 1) * q].contiguous()).reshape(H, W, q)
    nt = max(1, round(H * W * 200 / 2048 ** 2))
    rows, cols = rs.integers(0, H, nt), rs.integers(0, W, nt)
    amp = np.sqrt(10.0 ** (rs.uniform(0, 15, nt) / 10)) * np.exp(2j * np.pi * rs.random(nt))
    steer = amp[:, None] * np.exp(1j * rs.uniform(0, 2 * np.pi, nt)[:, None] * np.arange(p))
    add = torch.from_numpy(np.repeat(steer.T.astype(np.complex64)[:, :, None], q, 2)).to(device)
    for t in range(nt):
        x[:, int(rows[t]), int(cols[t]), :] += add[:, t]
    return x


def _options(c):
    o = dict(r_a=c["r_a"], r_b=c["r_b"], precision=c["precision"])
    if c["r_a"] > 1:
        o.update(eps=0.0, max_iter=4)
    if c["kind"] == "variants":
        o.update(nbank=c["nbank"], passes=c["passes"])
    return o


def _plan(c):
    return kstap.Plan(c["p"], c["q"], c["n"], **_options(c))


def _members(c):
    """The frames of a batch or of a served stream, largest side varied over
    the range, the classes that uneven streams mix."""
    rs = np.random.default_rng([7, c["scene"], c["largest"]])
    out = []
    for k in range(c["tiles"] if c["kind"] == "batch" else c["frames"]):
        lo = 96 if c["kind"] == "batch" else c["smallest"]
        side = [int(round(math.exp(v))) for v in rs.uniform(math.log(min(lo, c["largest"])), math.log(c["largest"]), 2)]
        if k == 0:
            side = [c["largest"], c["largest"]]
        q = int(rs.choice([8, 12, 16] if c["kind"] == "batch" else [8, 16]))
        out.append(dict(kind="frame", p=3, q=q, n=int(rs.choice([64, 128, 200, 256])), r_a=1,
                        r_b=int(rs.integers(2, 7)) if c["kind"] == "batch" else 3, H=side[0], W=side[1],
                        precision="fp32"))
    return out


def _pixels(c, seed):
    """A detection list: valid and a few border pixels."""
    rs = np.random.default_rng([seed, 11])
    return np.stack([rs.integers(4, c["H"] - 4, c["npix"]), rs.integers(4, c["W"] - 4, c["npix"])], 1).astype(np.int32)


def _snapshots(c, seed, device):
    rs = np.random.default_rng([seed, c["p"], c["q"], 5])
    u = _basis(rs, c["p"], 1) * math.sqrt(CNR * c["p"])
    n, p, q = c["n"], c["p"], c["q"]
    cn = lambda s: (rs.standard_normal(s) + 1j * rs.standard_normal(s)) / math.sqrt(2.0)  # noqa: E731
    X = u[None] * cn((n, 1, q)) + cn((n, p, q))
    return torch.from_numpy(X.astype(np.complex64)).to(device)


def prepare(case, seed):
    c, dev = case, "cuda"
    if c["kind"] == "lrkron":
        return dict(case=c, X=_snapshots(c, seed, dev))
    if c["kind"] == "batch":
        tiles = []
        for k, m in enumerate(_members(c)):
            x = _frame(m, seed * 1000 + k, dev)
            tiles.append((_plan(m), x, torch.empty((m["H"], m["W"]), dtype=torch.float32, device=dev),
                          torch.empty((m["H"], m["W"]), dtype=torch.uint8, device=dev)))
        return dict(case=c, tiles=tiles, batch=kstap.Batch(tiles))
    if c["kind"] == "served":
        frames = [(_plan(m), _frame(m, seed * 1000 + k, dev).cpu().pin_memory()) for k, m in enumerate(_members(c))]
        return dict(case=c, frames=frames, server=kstap.Server(1 << 30))
    st = dict(case=c, plan=_plan(c), x=_frame(c, seed, dev))
    if c["kind"] == "probe":
        st["pix"] = _pixels(c, seed)
    return st


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "frame":
        T, D = kstap.run(state["plan"], state["x"])
        return dict(T=T, D=D)
    if kind == "variants":
        return {k: v for k, v in kstap.run_ex(state["plan"], state["x"]).items() if v is not None}
    if kind == "batch":
        state["batch"].launch()
        return [dict(T=t[2], D=t[3]) for t in state["tiles"]]
    if kind == "probe":
        out = kstap.probe(state["plan"], state["x"], state["pix"])
        return {k: out[k] for k in ("T", "eta", "iters", "U_A", "U_B")}
    if kind == "lrkron":
        out = kstap.lrkron(state["X"], r_a=c["r_a"], eps=1e-4)
        return {k: out[k] for k in ("A", "B", "stats")}
    tickets = [state["server"].submit(plan, x) for plan, x in state["frames"]]
    return [dict(zip(("T", "D"), state["server"].wait(t)[:2])) for t in tickets]


# ------------------------------------------------------------ training stencil
def _stencil(n):
    w = 10
    while w * w - 9 < n:
        w += 2
    cand = [(a, b) for a in range(-(w // 2), w - w // 2) for b in range(-(w // 2), w - w // 2)
            if not (abs(a) <= 1 and abs(b) <= 1)]
    cand.sort(key=lambda t: (t[0] * t[0] + t[1] * t[1], t[0], t[1]))
    return np.array(cand[:n])


def _region(c):
    s = _stencil(c["n"])
    return (max(0, -s[:, 0].min()), c["H"] - max(0, s[:, 0].max()), max(0, -s[:, 1].min()),
            c["W"] - max(0, s[:, 1].max()))


def _frame_work(c, pixels=None):
    """Every sample read once, every output written once; the covariance of a
    pixel from its neighbour's by the vectors that enter and leave (4 pq
    (pq + 1) flops per vector, the Hermitian half), a probe's from all n; two
    LR-Kron half-step pairs over the Hermitian half of the covariance."""
    pq = c["p"] * c["q"]
    r0, r1, c0, c1 = _region(c)
    npx = max(0, r1 - r0) * max(0, c1 - c0)
    st = {tuple(t) for t in _stencil(c["n"]).tolist()}
    vec = 2 * sum((a, b + 1) not in st for a, b in st)
    samples = pq * c["H"] * c["W"]
    out = 5 * c["H"] * c["W"]
    if pixels is not None:
        npx, vec = pixels, c["n"]
        samples = min(samples, pixels * (c["n"] + 1) * pq)
        out = pixels * (12 + 8 * (c["p"] * c["r_a"] + c["q"] * c["r_b"]))
    return dict(bytes=8 * samples + out, flops=npx * (4.0 * vec * pq * (pq + 1) + 2 * 8 * pq * (pq + 1)))


def work(case):
    c = case
    if c["kind"] == "lrkron":
        n, p, q = c["n"], c["p"], c["q"]
        return dict(bytes=8 * (n * p * q + q * q + p * p) + 32, flops=8.0 * n * p * q * q + 8.0 * (n * p) ** 2 * q)
    if c["kind"] in ("batch", "served"):
        w = [_frame_work(m) for m in _members(c)]
        return {k: sum(v[k] for v in w) for k in ("bytes", "flops")}
    w = _frame_work(c, c["npix"] if c["kind"] == "probe" else None)
    if c["kind"] == "variants":
        w["bytes"] += c["H"] * c["W"] * (5 + (8 * c["passes"] - 4 if c["passes"] > 1 else 0))
    return w


# ------------------------------------------------------- the same in 64 bits
MOST = 1.6e10   # px n (pq)^2 of a frame that NumPy evaluates within seconds


def _cost(c, px=None):
    r0, r1, c0, c1 = _region(c)
    px = max(0, r1 - r0) * max(0, c1 - c0) if px is None else px
    return px * (c["n"] + 40.0) * (c["p"] * c["q"]) ** 2


def _covariance(x, rows, cols, n):
    s = _stencil(n)
    v = x[:, rows[:, None] + s[None, :, 0], cols[:, None] + s[None, :, 1], :]      # [p, N, n, q]
    v = torch.from_numpy(np.ascontiguousarray(v.transpose(1, 0, 3, 2)).reshape(rows.size, -1, n).astype(np.complex128))
    return (torch.bmm(v, v.conj().transpose(1, 2).contiguous()) / n).numpy()


def _top(M, r):
    lam, V = np.linalg.eigh((M + M.conj().swapaxes(-1, -2)) / 2)
    return lam[..., ::-1][..., :r], V[..., ::-1][..., :r]


def _lr_kron(R, p, r_a, eps, min_iter, max_iter):
    """R [N, p, p, q, q] (block (i, j) of the covariance): the spatial factor,
    its top basis, the unnormalised time factor, eta and the iterations."""
    N = R.shape[0]
    rn = np.sqrt(np.sum(np.abs(R) ** 2, (1, 2, 3, 4)))
    A = R.mean((3, 4))
    U = np.zeros((N, p, r_a), complex)
    eta, prev, its, on = np.zeros(N), np.full(N, np.inf), np.zeros(N, int), np.arange(N)
    half = lambda A, R: np.einsum("nij,nijkl->nkl", A.conj(), R, optimize=True) / np.sum(np.abs(A) ** 2, (1, 2))[:, None, None]  # noqa: E731,E501
    while on.size:
        r = R[on]
        b = half(A[on], r)
        a = np.einsum("nijkl,nkl->nij", r, b.conj(), optimize=True) / np.sum(np.abs(b) ** 2, (1, 2))[:, None, None]
        lam, u = _top(a, r_a)
        a = np.einsum("nia,na,nja->nij", u, lam, u.conj())
        e = np.sqrt(np.sum(np.abs(r - a[:, :, :, None, None] * b[:, None, None]) ** 2, (1, 2, 3, 4))) / rn[on]
        A[on], U[on] = a, u
        its[on] += 1
        stop = (its[on] >= max_iter) | ((its[on] >= min_iter) & (eps > 0) & (np.abs(e - prev[on]) <= eps))
        eta[on], prev[on] = e, e
        on = on[~stop]
    return A, U, half(A, R), eta, its


def _statistic(c, X, U, V, b):
    """||F_A X conj(F_B b)||^2 / (b^H F_B b) and F_A X conj(F_B b)."""
    g = b - np.einsum("nka,na->nk", V, np.einsum("nka,k->na", V.conj(), b))
    z = np.einsum("nik,nk->ni", X, g.conj())
    z = z - np.einsum("nia,na->ni", U, np.einsum("nia,ni->na", U.conj(), z))
    den = np.real(np.sum(b.conj() * g, 1))
    return np.sum(np.abs(z) ** 2, 1) / den, z / np.sqrt(den)[:, None]


def _pixels_exact(c, x, rows, cols):
    p, q = c["p"], c["q"]
    o = _options(c)
    step = max(1, int(4e7 / (c["n"] * p * q)))
    parts = []
    for k in range(0, rows.size, step):
        r, cc = rows[k:k + step], cols[k:k + step]
        S = _covariance(x, r, cc, c["n"])
        R = S.reshape(-1, p, q, p, q).transpose(0, 1, 3, 2, 4)
        A, U, B, eta, its = _lr_kron(R, p, c["r_a"], o.get("eps", 1e-6), 2, o.get("max_iter", 50))
        V = _top(B, c["r_b"])[1]
        X = x[:, r, cc, :].transpose(1, 0, 2).astype(np.complex128)
        bank = o.get("nbank", 0)
        best = None
        for m in range(max(1, bank)):
            b = np.exp(2j * np.pi * ((m * np.arange(q)) % bank) / bank) if bank else np.ones(q, complex)
            t, z = _statistic(c, X, U, V, b)
            sar = np.abs(np.einsum("nk,k->n", X[:, 0], b.conj())) ** 2 / q
            new = (t, z, t / sar, np.full(t.size, m))
            if best is None:
                best = new
            else:
                up = t > best[0]
                best = tuple(np.where(up[:, None] if u.ndim == 2 else up, u, v) for u, v in zip(new, best))
        parts.append(best + (eta, its))
    return [np.concatenate(v) for v in zip(*parts)] if parts else None


def _gamma_tail(k, pfa):
    lo, hi = 0.0, 200.0
    for _ in range(200):
        t = (lo + hi) / 2
        sf = math.exp(-t) * sum(t ** i / math.factorial(i) for i in range(k))
        lo, hi = (t, hi) if sf > pfa else (lo, t)
    return lo


def _frame_exact(c, seed):
    if _cost(c) > MOST:
        return None
    x = _frame(c, seed, "cuda").cpu().numpy()
    H, W = c["H"], c["W"]
    r0, r1, c0, c1 = _region(c)
    rr, cc = np.meshgrid(np.arange(r0, r1), np.arange(c0, c1), indexing="ij")
    out = dict(T=np.zeros((H, W)), D=None)
    K = c.get("passes", 1)
    if c["kind"] == "variants":
        out.update(E=np.zeros((H, W)), bin=None)
        if K > 1:
            out.update(T_pass=np.zeros((K, H, W)), C=np.zeros((K - 1, H, W)))
    if not rr.size or r1 <= r0 or c1 <= c0:
        return out
    rr, cc = rr.ravel(), cc.ravel()
    T, z, E, m, _, _ = _pixels_exact(c, x, rr, cc)
    out["T"][rr, cc] = T
    if c["kind"] == "variants":
        out["E"][rr, cc] = E
        if K > 1:
            e = np.sum(np.abs(z.reshape(z.shape[0], K, -1)) ** 2, 2).T
            out["T_pass"][:, rr, cc] = e
            out["C"][:, rr, cc] = np.sqrt(e[1:]) - np.sqrt(e[:1])
    return out


def exact(case, seed):
    c = case
    if c["kind"] in ("frame", "variants"):
        return _frame_exact(c, seed)
    if c["kind"] in ("batch", "served"):   # the tiles and frames that fit in the time
        out, left = [], MOST
        for k, m in enumerate(_members(c)):
            fits = _cost(m) <= left
            left -= _cost(m) if fits else 0.0
            out.append(_frame_exact(m, seed * 1000 + k) if fits else dict(T=None, D=None))
        return out
    if c["kind"] == "probe":
        if _cost(c, c["npix"]) > MOST:
            return None
        pix = _pixels(c, seed).astype(np.int64)
        r0, r1, c0, c1 = _region(c)
        ok = (pix[:, 0] >= r0) & (pix[:, 0] < r1) & (pix[:, 1] >= c0) & (pix[:, 1] < c1)
        T, eta = np.zeros(c["npix"]), np.zeros(c["npix"])
        if ok.any():
            t, _, _, _, e, _ = _pixels_exact(c, _frame(c, seed, "cuda").cpu().numpy(), pix[ok, 0], pix[ok, 1])
            T[ok], eta[ok] = t, e
        return dict(T=T, eta=eta, iters=None, U_A=None, U_B=None)   # a basis is exact up to a rotation
    # R(S) = (1/n) sum_m conj(X_m) (x) X_m, without forming the covariance
    X = _snapshots(c, seed, "cpu").numpy().astype(np.complex128)
    n, p, q = X.shape
    s = X.sum(2)
    A = np.einsum("mi,mj->ij", s, s.conj()) / (n * q * q)
    G = np.einsum("mik,njk->mnij", X, X.conj(), optimize=True)
    rn = math.sqrt(np.sum(np.abs(np.einsum("mnii->mn", G)) ** 2)) / n
    prev, it = math.inf, 0
    while True:
        na = np.sum(np.abs(A) ** 2)
        Y = np.einsum("mik,ij->mjk", X, A.conj()) / (n * na)      # B = sum_m Y_m^T conj(X_m)
        b2 = np.real(np.einsum("mnij,mnij->", np.einsum("mik,njk->mnij", Y, Y.conj(), optimize=True), G.conj()))
        P = np.einsum("mjk,nik->mnji", Y.conj(), X, optimize=True)
        a = np.einsum("mnji,mnjl->il", P, np.conj(np.einsum("nik,mjk->mnji", X, X.conj(), optimize=True))) / (n * b2)
        lam, u = _top(a, c["r_a"])
        new = (u * lam) @ u.conj().T
        r2 = rn ** 2 - 2 * b2 * np.real(np.sum(new.conj() * a)) + np.sum(np.abs(new) ** 2) * b2
        eta = math.sqrt(max(r2, 0.0)) / rn
        A, it = new, it + 1
        if it >= 50 or (it >= 2 and abs(eta - prev) <= 1e-4):
            break
        prev = eta
    B = np.einsum("mjk,mjl->kl", np.einsum("mik,ij->mjk", X, A.conj()) / (n * np.sum(np.abs(A) ** 2)), X.conj(),
                  optimize=True)
    return dict(A=A, B=B, stats=np.array([eta, it, rn, math.sqrt(b2)]))
