"""The library's work, case by case: what a program that uses it has it do.

The sizes are those of the repository's own workloads (``synth.make_config``): Si-like (8 k x
64 q, 24 bands, 4 occupied, N_MB 620), ZnO-like (60 bands, 18 occupied, N_MB 820-1400, 144 q),
SrTiO3-like (100 bands, 20 occupied, N_MB 2002-2600, 216 q), the oracle-sized one (8 q, 16
bands, 8 occupied, N_MB 300) and a ragged one. The ZnO- and SrTiO3-like cases take some of the
workload's k points (an evaluation is a loop or one launch over all of them), so that a state
fits the card several times over. Inputs are drawn on the GPU from the seed alone: a Hermitian
positive definite v(q) with the spectrum of the workloads (multipole strengths 1-10, 4 pi /
|q+G|^2 for the plane waves) and Gaussian projections M with a slow decay over the basis index.

A case's "call" is one of
  all      ``matrix_all`` over every k, then ``energy_device``: one outer iteration;
  per_k    ``matrix(k)`` for every k, then ``energy_device``: M streamed k by k;
  setup    a new context (Cholesky of every v(q)) and V(0): the start of a self-consistency cycle;
  back     ``back_transform`` of every V(k) to the LAPW basis;
  predict  the learned extrapolator's prediction of V between exact evaluations.
"""
import math

import numpy as np
import torch

import paper_1003_0524_amd as lib

DEVICE = "cuda:0"


# --------------------------------------------------------------------------- cases
def _system(name, call, precision, **kw):
    case = {"name": name, "call": call, "precision": precision, "mdtype": "c128", "inversion": False,
            "n_k": 1, "n_q": 8, "n_occ": 4, "bands_lo": 24, "bands_hi": 24, "channels": "even", "n_ch": 0,
            "mt": 0, "lmax": 0, "nrad_top": 0, "pw_lo": 100, "pw_hi": 100, "shape_seed": 0}
    case.update(kw)
    return case


def listed():
    si = dict(n_k=8, n_q=64, n_occ=4, bands_lo=24, bands_hi=24, channels="falling", n_ch=50, lmax=4, nrad_top=10,
              pw_lo=260, pw_hi=260)
    zno = dict(n_q=144, n_occ=18, bands_lo=60, bands_hi=60, n_ch=100, mt=455, pw_lo=272, pw_hi=844)
    sto = dict(n_q=108, n_occ=20, bands_lo=100, bands_hi=100, n_ch=180, mt=1200, pw_lo=622, pw_hi=1220)
    return [
        # the smallest call: one k of the oracle-sized system in the default precision, where
        # launches and latency count
        _system("small fp64", "per_k", "fp64", n_k=1, n_q=8, n_occ=8, bands_lo=16, bands_hi=16, channels="falling",
                n_ch=50, lmax=4, nrad_top=3, pw_lo=150, pw_hi=150),
        # odd sizes in every dimension: uneven bands per k, plane waves per q, channels of 0-6
        # multipole-free functions
        _system("ragged fp32", "all", "fp32", n_k=3, n_q=6, n_occ=5, bands_lo=13, bands_hi=37, channels="random",
                n_ch=23, nrad_top=7, pw_lo=37, pw_hi=130, shape_seed=7),
        # one outer iteration of the Si-like workload: the default (FP64) and the fastest mode
        _system("si fp64", "all", "fp64", **si),
        _system("si bf16x3", "all", "bf16x3", **si),
        # the same crystal with its inversion symmetry used (real v, real bands packed in pairs)
        _system("si real bf16x3", "all", "bf16x3", **dict(si, inversion=True)),
        # ZnO-like: the FP64 form with complex128 M streamed per k (one k), the reduced-precision
        # forms with complex64 M resident
        _system("zno fp64", "per_k", "fp64", **dict(zno, n_k=1)),
        _system("zno bf16x3", "all", "bf16x3", mdtype="c64", **dict(zno, n_k=2)),
        _system("zno bf16x6", "all", "bf16x6", mdtype="c64", **dict(zno, n_k=2, n_q=72)),
        # SrTiO3-like: the headline workload, two of its k points on half of its q mesh
        _system("sto bf16x3", "all", "bf16x3", mdtype="c64", **dict(sto, n_k=2)),
        # the start of a self-consistency cycle on the ZnO-like system: v(q) prepared, first V(k)
        _system("zno setup", "setup", "bf16x3", mdtype="c64", **dict(zno, n_k=1)),
        # V(k) of a 100-band system in a basis of 2000 LAPW functions
        _system("back 2000", "back", "fp64", n_k=1, n_q=2, n_occ=8, bands_lo=100, bands_hi=100, n_ch=8, mt=24,
                pw_lo=60, pw_hi=60, n_g=2000),
        # prediction of V for 21 k of 60 bands (whole eigenbasis out, density matrices of 144 k')
        _system("predict zno", "predict", "fp64", n_k=21, n_q=2, n_occ=8, bands_lo=60, bands_hi=60, n_ch=8, mt=24,
                pw_lo=60, pw_hi=60, n_p=144, n_blk=60),
    ]


def _between(rng, lo, hi):
    """An integer of [lo, hi], spread over the logarithm where the range spans a factor of ten."""
    if lo > 0 and hi > 10 * lo:
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))
    return rng.randint(lo, hi)


def draw(rng):
    kind = rng.choice(["small", "si", "zno", "zno fp64", "sto", "setup", "back", "predict"])
    seed = rng.randrange(1 << 30)
    mixed = ["fp32", "bf16x3", "bf16x6"]
    if kind == "small":
        lo = rng.randint(3, 20)
        pw = rng.randint(30, 100)
        c = _system("", rng.choice(["all", "per_k"]), rng.choice(["fp64"] + mixed), n_k=rng.randint(1, 3),
                    n_q=rng.randint(3, 10), n_occ=rng.randint(1, 9), bands_lo=lo, bands_hi=lo + rng.randint(0, 24),
                    channels="random", n_ch=rng.randint(0, 50), nrad_top=rng.randint(2, 8), pw_lo=pw,
                    pw_hi=pw + rng.randint(0, 80), shape_seed=seed)
    elif kind == "si":
        pw = rng.randint(150, 280)
        nb = rng.randint(10, 30)
        c = _system("", "all", rng.choice(["fp64"] + mixed), inversion=rng.random() < 0.4, n_k=rng.randint(2, 8),
                    n_q=_between(rng, 8, 64), n_occ=rng.randint(3, 8), bands_lo=nb, bands_hi=nb,
                    channels="falling", n_ch=rng.choice([25, 50]), lmax=4, nrad_top=rng.randint(5, 10), pw_lo=pw,
                    pw_hi=pw + rng.randint(0, 60), shape_seed=seed)
    elif kind in ("zno", "zno fp64", "setup"):
        n_ch = rng.choice([50, 75, 100])
        pw = rng.randint(200, 420)
        nb = rng.randint(40, 72)
        c = _system("", "all", rng.choice(mixed), mdtype="c64", n_k=rng.randint(1, 2), n_q=_between(rng, 12, 108),
                    n_occ=rng.randint(9, 19), bands_lo=nb, bands_hi=nb, n_ch=n_ch,
                    mt=int(n_ch * rng.uniform(2.5, 5.0)), pw_lo=pw, pw_hi=pw + rng.randint(0, 420), shape_seed=seed)
        if kind == "zno fp64":
            c.update(call="per_k", precision="fp64", mdtype="c128", n_k=1)
        elif kind == "setup":
            c.update(call="setup", precision=rng.choice(["fp64"] + mixed), n_k=1, n_occ=rng.randint(4, 10))
    elif kind == "sto":
        nb = rng.randint(80, 120)
        pw = rng.randint(500, 800)
        c = _system("", "all", rng.choice(mixed), mdtype="c64", n_k=rng.randint(1, 2), n_q=_between(rng, 10, 64),
                    n_occ=rng.randint(10, 20), bands_lo=nb, bands_hi=nb, n_ch=180, mt=rng.randint(700, 1250), pw_lo=pw,
                    pw_hi=pw + rng.randint(0, 420), shape_seed=seed)
    elif kind == "back":
        nb = rng.randint(8, 120)
        c = _system("", "back", "fp64", n_k=1, n_q=2, n_occ=4, bands_lo=nb, bands_hi=nb, n_ch=8, mt=24, pw_lo=60,
                    pw_hi=60, n_g=_between(rng, 150, 2500), shape_seed=seed)
    else:
        nb = rng.randint(16, 60)
        c = _system("", "predict", "fp64", n_k=rng.randint(4, 21), n_q=2, n_occ=4, bands_lo=nb, bands_hi=nb, n_ch=8,
                    mt=24, pw_lo=60, pw_hi=60, n_p=_between(rng, 8, 144), n_blk=rng.randint(8, nb), shape_seed=seed)
    del c["name"]
    return c


# --------------------------------------------------------------------------- shapes and inputs
class _Shape:
    """The sizes of a case (bands per k, channels, plane waves per q); the same for every seed."""

    def __init__(self, c):
        rng = np.random.default_rng([c["shape_seed"], 11])
        self.n_k, self.n_q, self.n_occ = c["n_k"], c["n_q"], c["n_occ"]
        self.n_bands = [int(x) for x in rng.integers(c["bands_lo"], c["bands_hi"] + 1, size=self.n_k)]
        self.n_bands[-1] = c["bands_hi"]
        n = c["n_ch"]
        if c["channels"] == "falling":           # n_rad(l) = top - l on whole atoms (top itself: the same on every l)
            per = (c["lmax"] + 1) ** 2
            fall = 1 if c["nrad_top"] > c["lmax"] else 0
            of_l = [c["nrad_top"] - fall * l for l in range(c["lmax"] + 1) for _ in range(2 * l + 1)]
            self.ch_nrad = [of_l[i % per] for i in range(n)]
        elif c["channels"] == "random":
            self.ch_nrad = [int(x) for x in rng.integers(1, c["nrad_top"] + 1, size=n)]
        else:                                    # `mt` multipole-free functions spread evenly
            self.ch_nrad = [1 + c["mt"] // n + (1 if i < c["mt"] % n else 0) for i in range(n)]
        self.n_ch = n
        self.n_pw = [int(x) for x in rng.integers(c["pw_lo"], c["pw_hi"] + 1, size=self.n_q)]
        self.n_s = sum(self.ch_nrad) - n
        self.n_d = [n + p for p in self.n_pw]
        self.n_mb = [self.n_s + d for d in self.n_d]
        self.n_cols = (self.n_occ + 1) // 2 if c["inversion"] else self.n_occ    # columns n'' of M

    def m_elems(self, k):
        return sum(self.n_cols * self.n_bands[k] * n for n in self.n_mb)


def _gen(seed, *key):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(np.random.default_rng([seed, *key]).integers(1 << 62)))
    return g


def _coulomb(c, s, seed):
    """(E on the GPU, D, C): v(q) in its block-sparse form, Hermitian positive definite."""
    rng = np.random.default_rng([seed, 1])
    m_c = rng.uniform(1.0, 10.0, size=s.n_ch)
    real = c["inversion"]
    D, C = [], []
    for ch, b in enumerate(s.ch_nrad):
        x = rng.standard_normal((b - 1, b - 1)) + (0 if real else 1j) * rng.standard_normal((b - 1, b - 1))
        d = (x @ x.conj().T / max(1, b - 1) + np.eye(b - 1)) * rng.uniform(0.5, 2.0)
        d = 0.5 * (d + d.conj().T)
        v = rng.standard_normal(b - 1) + (0 if real else 1j) * rng.standard_normal(b - 1)
        if b > 1:
            v = v * math.sqrt(np.linalg.eigvalsh(d)[0] * m_c[ch] / 8.0) / np.linalg.norm(v)
        D.append(d)
        C.append(v)
    # E = S^1/2 (1 + H/2) S^1/2, |H| < 1, S = multipole strengths and 4 pi / |q+G|^2
    n = max(s.n_d)
    g = _gen(seed, 2)
    dt = torch.float64 if real else torch.complex128
    h = torch.randn((n, n), generator=g, dtype=dt, device=DEVICE)
    h = (h + h.conj().T) / (3.0 * math.sqrt(n))
    E = []
    for q in range(s.n_q):
        nd = s.n_d[q]
        G = (1.0 + 0.3 * torch.arange(1, s.n_pw[q] + 1, dtype=torch.float64, device=DEVICE)) ** (1.0 / 3.0)
        G = G * (0.8 + 0.2 * (q + 1) / s.n_q)
        st = torch.cat([torch.from_numpy(m_c).to(DEVICE), 4.0 * math.pi / G ** 2]).sqrt()
        if real:
            ph = 1.0 - 2.0 * torch.randint(0, 2, (nd,), generator=g, device=DEVICE).to(torch.float64)
        else:
            ph = torch.polar(torch.ones(nd, dtype=torch.float64, device=DEVICE),
                             2 * math.pi * torch.rand(nd, generator=g, dtype=torch.float64, device=DEVICE))
        a = ph * st
        e = 0.5 * a[:, None] * h[:nd, :nd] * a.conj()[None, :]
        e.diagonal().add_(st * st)
        E.append(0.5 * (e + e.conj().T))
    return E, D, C


def _m(c, s, seed, k):
    """M(k): the q blocks in order, [n''][n][I] each."""
    dt = torch.complex64 if c["mdtype"] == "c64" else torch.complex128
    out = torch.empty(s.m_elems(k), dtype=dt, device=DEVICE)
    g = _gen(seed, 3, k)
    at = 0
    for q in range(s.n_q):
        rows, n = s.n_cols * s.n_bands[k], s.n_mb[q]
        blk = out[at:at + rows * n].view(rows, n)
        torch.view_as_real(blk).normal_(generator=g)
        blk *= torch.exp(-0.1 * torch.arange(n, device=DEVICE) / n)
        if c["inversion"] and s.n_occ % 2:       # the last column holds one real band
            torch.view_as_real(blk.view(s.n_cols, s.n_bands[k], n)[-1])[..., 1] = 0
        at += rows * n
    return out


def _context(c, s, blocks):
    E, D, C = blocks
    return lib.Exchange(s.n_bands, s.n_pw, s.ch_nrad, s.n_occ, E, D, C, precision=c["precision"],
                        inversion=c["inversion"])


IN_DIM, HIDDEN, SKETCH_SEED = 64, 256, 0x5EED5EED


def _network(c, s, seed):
    out = s.n_k * c["n_blk"] ** 2
    g = _gen(seed, 5)
    parts = []
    for rows, cols in ((HIDDEN, IN_DIM), (HIDDEN, HIDDEN), (out, HIDDEN)):
        parts.append((torch.rand((rows, cols), generator=g, device=DEVICE) * 2 - 1) / math.sqrt(cols))
        parts.append(0.1 * torch.randn(rows, generator=g, device=DEVICE))
    return parts


def _densities(c, s, seed):
    """Density matrices of n_p k points at the anchor and now, and the anchor's V(k) with its eigenvectors."""
    g = _gen(seed, 6)
    nb = s.n_bands[0]

    def hermitian(n, m):
        x = torch.randn((n, m, m), generator=g, dtype=torch.complex128, device=DEVICE)
        return (x + x.conj().transpose(1, 2)).contiguous() / (2 * math.sqrt(m))

    p0 = hermitian(c["n_p"], nb)
    p1 = p0 + 0.01 * hermitian(c["n_p"], nb)
    v = [hermitian(1, m)[0] * 3.0 - 5.0 * torch.eye(m, dtype=torch.complex128, device=DEVICE) for m in s.n_bands]
    z = torch.cat([torch.linalg.eigh(x)[1].T.reshape(-1) for x in v])        # columns, k after k
    return p1.reshape(-1), p0.reshape(-1), v, z


def prepare(case, seed):
    c, s = case, _Shape(case)
    state = {"case": c, "shape": s}
    blocks = _coulomb(c, s, seed)
    if c["call"] == "setup":
        state.update(blocks=blocks, M=_m(c, s, seed, 0))
        return state
    ex = _context(c, s, blocks)
    state["ex"] = ex
    if c["call"] in ("all", "per_k"):
        state["M"] = [_m(c, s, seed, k) for k in range(s.n_k)]
        state["e"] = torch.zeros(1, dtype=torch.float64, device=DEVICE)
        if c["call"] == "all":
            ex.matrix_all(state["M"])             # a context chooses its kernels on its first call
    elif c["call"] == "back":
        for k in range(s.n_k):
            ex.matrix(k, _m(c, s, seed, k))
        g = _gen(seed, 4)
        state["Z"] = [torch.randn((nb, c["n_g"]), generator=g, dtype=torch.complex128, device=DEVICE).T
                      for nb in s.n_bands]
    else:
        ex.nn_init(IN_DIM, HIDDEN, s.n_k * c["n_blk"] ** 2, 1)
        ex.nn_set_params(torch.cat([p.reshape(-1) for p in _network(c, s, seed)]))
        p1, p0, v, z = _densities(c, s, seed)
        state.update(P=p1, P_anchor=p0, V_anchor=[x.T.contiguous().view(-1) for x in v], Z=z)
    torch.cuda.synchronize()
    return state


def run(state):
    c, s = state["case"], state["shape"]
    call = c["call"]
    if call == "setup":
        ex = _context(c, s, state["blocks"])
        v = ex.matrix(0, state["M"])
        ex.close()
        return {"V": [v]}
    ex = state["ex"]
    if call == "back":
        return {"V": [ex.back_transform(k, state["Z"][k]) for k in range(s.n_k)]}
    if call == "predict":
        x, norm = ex.nn_features(state["P"], state["P_anchor"], IN_DIM, SKETCH_SEED)
        y = ex.nn_predict(x.view(1, IN_DIM)).view(s.n_k, c["n_blk"] ** 2)
        outs = [torch.empty_like(v) for v in state["V_anchor"]]
        ex.nn_expand(state["V_anchor"], state["Z"], c["n_blk"], y, float(norm.item()), outs)
        return {"x": x, "norm": norm, "y": y, "V": [o.view(nb, nb).T for o, nb in zip(outs, s.n_bands)]}
    if call == "all":
        V = ex.matrix_all(state["M"])
    else:
        V = [ex.matrix(k, m) for k, m in enumerate(state["M"])]
    ex.energy_device(state["e"])
    return {"V": V, "E": state["e"]}


# --------------------------------------------------------------------------- floors and 64-bit values
def work(case):
    c, s = case, _Shape(case)
    if c["call"] == "back":
        n, g = s.n_bands, c["n_g"]
        return {"bytes": sum(16.0 * (g * b + b * b + g * g) for b in n),
                "flops": sum(8.0 * g * b * b + 4.0 * g * (g + 1) * b for b in n)}
    if c["call"] == "predict":
        out = s.n_k * c["n_blk"] ** 2
        par = HIDDEN * (IN_DIM + HIDDEN + out + 2) + out
        b, nk, m = s.n_bands[0], s.n_k, c["n_blk"]
        return {"bytes": 32.0 * c["n_p"] * b * b + 4.0 * (par + 2 * out) + 32.0 * nk * b * b + 16.0 * nk * b * m,
                "flops": 4.0 * IN_DIM * c["n_p"] * b * b + 2.0 * par + nk * 8.0 * (b * m * m + b * b * m)}
    msz = 8.0 if c["mdtype"] == "c64" else 16.0
    per = 2.0 if c["inversion"] else 4.0         # flops of a multiply-add of a packed / complex column, per factor entry
    nbytes = sum(16.0 * d * d for d in s.n_d)
    flops = 0.0
    for k, b in enumerate(s.n_bands):
        nbytes += msz * s.m_elems(k) + 16.0 * b * b
        sp = sum(per * (r - 1) * r for r in s.ch_nrad)
        for q in range(s.n_q):
            r = s.n_cols * b
            flops += per * s.n_d[q] ** 2 * r + sp * r + (per * b * (b + 1) * s.n_mb[q] * s.n_cols)
    if c["call"] == "setup":
        flops += sum((4.0 / 3.0) * d ** 3 for d in s.n_d)
    return {"bytes": nbytes, "flops": flops}


def _sketch(n_real, dp):
    """x_i = sum_j S_ij v_j / |v|, S_ij = -+1/sqrt(m) by the top bit of SplitMix64 output i n_real + j."""
    def shr(z, k):
        return (z >> k) & ((1 << (64 - k)) - 1)

    def i64(u):
        return u - (1 << 64) if u >= 1 << 63 else u

    norm = dp.norm()
    x = torch.empty(IN_DIM, dtype=torch.float64, device=DEVICE)
    for i in range(IN_DIM):
        n = torch.arange(i * n_real + 1, (i + 1) * n_real + 1, dtype=torch.int64, device=DEVICE)
        z = n * i64(0x9E3779B97F4A7C15) + SKETCH_SEED
        z = (z ^ shr(z, 30)) * i64(0xBF58476D1CE4E5B9)
        z = (z ^ shr(z, 27)) * i64(0x94D049BB133111EB)
        z = z ^ shr(z, 31)
        x[i] = torch.where(z < 0, -dp, dp).sum() / math.sqrt(IN_DIM) / norm
    return x, norm


def exact(case, seed):
    c, s = case, _Shape(case)
    if c["call"] == "predict":
        p1, p0, v, z = _densities(c, s, seed)
        dp = torch.view_as_real(p1).reshape(-1) - torch.view_as_real(p0).reshape(-1)
        x, norm = _sketch(dp.numel(), dp)
        w1, b1, w2, b2, w3, b3 = (t.double() for t in _network(c, s, seed))
        y = w3 @ torch.tanh(w2 @ torch.tanh(w1 @ x + b1) + b2) + b3
        m, at, V = c["n_blk"], 0, []
        yk = y.view(s.n_k, m, m)
        for k, nb in enumerate(s.n_bands):
            B = z[at:at + nb * nb].view(nb, nb).T[:, :m]
            at += nb * nb
            up = torch.triu(yk[k])
            im = torch.tril(yk[k], -1).T
            h = torch.complex(up + torch.triu(up, 1).T, im - im.T)
            V.append(v[k] + norm * (B @ h @ B.conj().T))
        return {"x": x, "norm": norm.view(1), "y": y.view(s.n_k, m * m), "V": V}
    E, D, C = _coulomb(c, s, seed)
    # the q-independent part: channel blocks D_c and their couplings C_c to the multipole functions
    mt = torch.zeros((s.n_s + s.n_ch,) * 2, dtype=torch.complex128)
    o = 0
    for ch, b in enumerate(s.ch_nrad):
        e, j = o + b - 1, s.n_s + ch
        mt[o:e, o:e] = torch.from_numpy(np.asarray(D[ch], np.complex128))
        mt[o:e, j] = torch.from_numpy(np.asarray(C[ch], np.complex128))
        mt[j, o:e] = mt[o:e, j].conj()
        o = e
    mt = mt.to(DEVICE)
    Vs = []
    for k in range(s.n_k):
        M = _m(c, s, seed, k)
        nb = s.n_bands[k]
        V = torch.zeros((nb, nb), dtype=torch.complex128, device=DEVICE)
        at = 0
        for q in range(s.n_q):
            n = s.n_mb[q]
            v = torch.zeros((n, n), dtype=torch.complex128, device=DEVICE)
            v[:mt.shape[0], :mt.shape[0]] = mt
            v[s.n_s:, s.n_s:] = E[q].to(torch.complex128)
            A = M[at:at + s.n_cols * nb * n].view(s.n_cols * nb, n).to(torch.complex128)
            at += A.numel()
            W = (A @ v.T).view(s.n_cols, nb, n)
            A = A.view(s.n_cols, nb, n)
            for j in range(s.n_cols):
                V -= (A[j].conj() @ W[j].T) / s.n_q
        if c["inversion"]:
            V = torch.complex(V.real, torch.zeros_like(V.real))
        Vs.append(V)
        if c["call"] == "setup":
            break
    if c["call"] == "back":
        g = _gen(seed, 4)
        Z = [torch.randn((nb, c["n_g"]), generator=g, dtype=torch.complex128, device=DEVICE).T for nb in s.n_bands]
        return {"V": [z @ V @ z.conj().T for z, V in zip(Z, Vs)]}
    if c["call"] == "setup":
        return {"V": Vs}
    occ = [V.diagonal()[:s.n_occ].real.sum() for V in Vs]
    return {"V": Vs, "E": (sum(occ) / s.n_k).view(1)}
