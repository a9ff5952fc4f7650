"""Workloads timed through the public entry points of ``paper_2509_23018_amd``.

Each case is one call (or one forward and backward) that a GW program makes:
chi0 in its precisions and on its three frequency axes, its adjoint through
autograd, several q-points in one call, the static subspace (Diag, and
chi_BB'(z) in a given basis), eps^-1, the GPP self-energy matrix, pseudobands
and batches of small Hermitian eigenproblems.

* ``listed()``: the named cases; ``draw(rng)``: another one of the same ranges;
* ``prepare(case, seed)``: inputs on the GPU, drawn from the seed;
* ``run(state)``: one pass; ``work(case)``: its bytes and operations;
* ``exact(case, seed)``: the outputs of ``run`` from plain torch and numpy in
  double precision.

Inputs follow the benchmark recipes: complex Gaussian bands of unit norm on
the grid, valence energies uniform in [-0.4, 0] Ha, conduction energies in
[0.05, 1.1] Ha, complete G-spheres in a cubic cell of 10 bohr.
"""
import math
import random

import numpy as np
import torch

import paper_2509_23018_amd as gw

CELL = 10.0
VOLUME = CELL ** 3
SPIN = 2.0
C128 = torch.complex128


# ---------------------------------------------------------------- cases

def listed():
    return [
        dict(name="chi0 16^3 static", op="chi0", n1=16, n2=16, n3=16, nv=4, nc=28, r2=10,
             axis="static", nz=1, precision="fp64", slices=0),
        dict(name="chi0 48^3 real axis", op="chi0", n1=48, n2=48, n3=48, nv=64, nc=960, r2=61,
             axis="real", nz=4, precision="fp64", slices=0),
        dict(name="chi0 72^3 imaginary axis", op="chi0", n1=72, n2=72, n3=72, nv=4, nc=960, r2=126,
             axis="imag", nz=8, precision="fp64", slices=0),
        dict(name="chi0 48^3 split bf16", op="chi0", n1=48, n2=48, n3=48, nv=16, nc=960, r2=61,
             axis="real", nz=4, precision="split_bf16", slices=3),
        dict(name="chi0 gradient 32^3", op="grad", n1=32, n2=32, n3=32, nv=32, nc=480, r2=42,
             axis="static", nz=1),
        dict(name="8 q-points 40^3", op="batch", nq=8, n1=40, n2=40, n3=40, nv=12, nc_lo=75,
             nc_hi=225, ng_lo=200, ng_hi=2000, nz=8, graph=True),
        dict(name="chi_BB' 48^3 from kept M", op="subspace", n1=48, n2=48, n3=48, nv=16, nc=480,
             r2=61, axis="imag", nz=8, n_eig=201, kept=True),
        dict(name="Diag 1189", op="diag", ng=1189, n_eig=119),
        dict(name="epsinv 2007 x 4", op="epsinv", ng=2007, nz=4),
        dict(name="GPP 64 x 739", op="gpp", nb=64, ns=48, ng=739, ne=16),
        dict(name="pseudobands 48^3", op="bands", nr=48 ** 3, nb=960, keep=64, slices=6, n_xi=4),
        dict(name="heev 24 of 48", op="heev", n=48, batch=24),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid_of(rng, lo=12, hi=72):
    n = rng.choice([k for k in (12, 16, 18, 20, 24, 27, 30, 32, 36, 40, 45, 48, 54, 60, 64, 72)
                    if lo <= k <= hi])
    m = [n, n, n]
    if rng.random() < 0.3:                       # an elongated cell
        m[rng.randrange(3)] += rng.choice([2, 4, 6])
    radius = rng.uniform(0.14, 0.24) * n
    return m, max(2, int(radius * radius))


def draw(rng):
    op = rng.choice(["chi0", "chi0", "chi0", "grad", "batch", "subspace", "diag", "epsinv", "gpp",
                     "bands", "heev"])
    if op in ("chi0", "grad", "subspace"):
        n, r2 = _grid_of(rng, hi=40 if op == "grad" else 72)
        c = dict(op=op, n1=n[0], n2=n[1], n3=n[2], nv=_logint(rng, 1, 64),
                 nc=_logint(rng, 4, 960), r2=r2)
        c["axis"] = rng.choice(["static", "real", "imag"])
        c["nz"] = 1 if c["axis"] == "static" else rng.randint(1, 8)
        if op == "chi0":
            c["precision"], c["slices"] = rng.choice(
                [("fp64", 0), ("fp64", 0), ("fp64", 0), ("fp32", 0), ("split_bf16", 3),
                 ("split_bf16", 4), ("split_fp16x9", 4), ("split_fp16", 3)])
        ng = len(_gsphere(c["r2"], n))
        if op == "subspace":
            c["n_eig"] = max(1, int(ng * rng.uniform(0.08, 0.22)))
            c["kept"] = rng.random() < 0.5
        cap = {"chi0": 3e12, "grad": 3e11, "subspace": 1.5e12}[op]
        while c["nv"] * c["nc"] > 4 and work(c)["flops"] > cap:
            key = "nv" if c["nv"] > 4 and rng.random() < 0.5 else "nc"
            c[key] = max(1, c[key] * 3 // 4)
        return c
    if op == "batch":
        n, _ = _grid_of(rng, lo=16, hi=40)
        lo = _logint(rng, 40, 300)
        most = int(2.0 * (0.24 * min(n)) ** 3)   # G that the grid holds well
        return dict(op="batch", nq=rng.randint(2, 10), n1=n[0], n2=n[1], n3=n[2],
                    nv=rng.randint(2, 16), nc_lo=_logint(rng, 8, 75), nc_hi=_logint(rng, 80, 225),
                    ng_lo=min(lo, most), ng_hi=min(most, lo * rng.randint(2, 8)),
                    nz=rng.randint(1, 8), graph=rng.random() < 0.5)
    if op == "diag":
        ng = _logint(rng, 150, 1500)
        return dict(op="diag", ng=ng, n_eig=max(4, int(ng * rng.uniform(0.08, 0.2))))
    if op == "epsinv":
        ng, nz = _logint(rng, 57, 2200), rng.randint(1, 8)
        while ng ** 3 * nz > 4 * 2007 ** 3:
            nz -= 1
        return dict(op="epsinv", ng=ng, nz=nz)
    if op == "gpp":
        c = dict(op="gpp", nb=_logint(rng, 2, 128), ns=_logint(rng, 4, 130),
                 ng=_logint(rng, 60, 1400), ne=_logint(rng, 1, 32))
        while c["nb"] > 1 and work(c)["flops"] > 1e12:
            c["nb"] = c["nb"] * 3 // 4
        return c
    if op == "bands":
        n = rng.choice([20, 24, 27, 32, 36, 40, 48])
        slices = rng.randint(2, 6)
        keep = rng.randint(0, 64)
        return dict(op="bands", nr=n ** 3, nb=keep + rng.randint(16 * 2 ** slices - 16, 900),
                    keep=keep, slices=slices, n_xi=rng.choice([1, 2, 3, 4, 8]))
    n = _logint(rng, 4, 300)
    return dict(op="heev", n=n, batch=rng.randint(1, max(1, min(64, int(6e6 / n ** 2.5)))))


# ---------------------------------------------------------------- inputs

def _gsphere(r2, n):
    """All integer g with |g|^2 <= r2 that the grid holds, by (|g|^2, g)."""
    r = math.isqrt(r2)
    ax = np.arange(-r, r + 1)
    g = np.stack(np.meshgrid(ax, ax, ax, indexing="ij"), -1).reshape(-1, 3)
    n2 = (g * g).sum(1)
    nn = np.asarray(n)
    ok = (n2 <= r2) & np.all((g >= -(nn // 2)) & (g <= (nn + 1) // 2 - 1), axis=1)
    g, n2 = g[ok], n2[ok]
    return np.ascontiguousarray(g[np.lexsort((g[:, 2], g[:, 1], g[:, 0], n2))], dtype=np.int32)


def _gsphere_shifted(q, count, n):
    """The count g of the grid with the smallest |q + g|^2."""
    r = int(math.ceil((3.0 * count / (4.0 * math.pi)) ** (1.0 / 3.0))) + 3
    ax = np.arange(-r, r + 1)
    g = np.stack(np.meshgrid(ax, ax, ax, indexing="ij"), -1).reshape(-1, 3)
    nn = np.asarray(n)
    g = g[np.all((g >= -(nn // 2)) & (g <= (nn + 1) // 2 - 1), axis=1)]
    k2 = ((g + np.asarray(q)[None, :]) ** 2).sum(1)
    order = np.lexsort((g[:, 2], g[:, 1], g[:, 0], k2))[:count]
    return np.ascontiguousarray(g[order], dtype=np.int32)


def _frequencies(axis, nz):
    if axis == "static":
        return np.zeros(nz, dtype=np.complex128)
    if axis == "real":
        return np.linspace(0.0, 1.0, nz) + 0.005j
    x, _ = np.polynomial.legendre.leggauss(nz)
    return 1j * (1.0 + x) / (1.0 - x)


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(gen, *shape):
    return torch.randn(shape, generator=gen, device="cuda", dtype=C128)


def _uniform(gen, n, lo, hi):
    return lo + (hi - lo) * torch.rand(n, generator=gen, device="cuda", dtype=torch.float64)


def _problem(gen, n, nv, nc, gvec, z):
    """Bands of unit norm on the grid on average (dV sum |psi|^2 = 1)."""
    nr = n[0] * n[1] * n[2]
    return gw.Chi0Problem(
        n=n, volume=VOLUME, psi_v=_normal(gen, nv, nr).mul_(VOLUME ** -0.5),
        psi_c=_normal(gen, nc, nr).mul_(VOLUME ** -0.5), e_v=_uniform(gen, nv, -0.4, 0.0),
        e_c=_uniform(gen, nc, 0.05, 1.1), gvec=gvec, z=z)


def _one_problem(case, seed):
    n = (case["n1"], case["n2"], case["n3"])
    gen = _generator(seed)
    return gen, _problem(gen, n, case["nv"], case["nc"], _gsphere(case["r2"], n),
                         _frequencies(case["axis"], case["nz"]))


def _batch_shapes(case):
    """(nc, ng, q) of every problem: uneven sizes, shuffled."""
    r = random.Random(case["nq"])
    nq, last = case["nq"], max(1, case["nq"] - 1)
    a, b = list(range(nq)), list(range(nq))
    r.shuffle(a)
    r.shuffle(b)
    out = []
    for k in range(nq):
        nc = round(case["nc_lo"] + (case["nc_hi"] - case["nc_lo"]) * a[k] / last)
        ng = round(case["ng_lo"] * (case["ng_hi"] / case["ng_lo"]) ** (b[k] / last))
        out.append((nc, ng, [r.choice((-0.375, -0.125, 0.125, 0.375)) for _ in range(3)]))
    return out


def _batch_problems(case, seed):
    gen = _generator(seed)
    n = (case["n1"], case["n2"], case["n3"])
    z = _frequencies("imag", case["nz"])
    return [_problem(gen, n, case["nv"], nc, _gsphere_shifted(q, ng, n), z)
            for nc, ng, q in _batch_shapes(case)]


def _coulomb(ng):
    """v_G = 4 pi / |G|^2 of the ng smallest G of the cell, the head excluded."""
    r = int(math.ceil((3.0 * ng / (4.0 * math.pi)) ** (1.0 / 3.0))) + 2
    g = _gsphere(r * r, (4 * r, 4 * r, 4 * r))[:ng]
    g2 = (g.astype(np.float64) ** 2).sum(1) * (2.0 * math.pi / CELL) ** 2
    v = np.zeros(ng)
    v[g2 > 0] = 4.0 * math.pi / g2[g2 > 0]
    return v


def _static_chi(gen, ng, nz):
    """Hermitian negative semidefinite matrices whose head and wings vanish and
    which fall off with |G|, as chi0 on the imaginary axis."""
    v = torch.from_numpy(_coulomb(ng)).cuda()
    g2 = torch.where(v > 0, 4.0 * math.pi / v.clamp_min(1e-300), torch.zeros_like(v))
    d = torch.sqrt(g2 / (1.0 + g2) / (1.0 + 0.05 * g2))
    out = torch.empty((nz, ng, ng), dtype=C128, device="cuda")
    for w in range(nz):
        x = _normal(gen, ng, 3 * ng).mul_(d[:, None])
        out[w] = (x @ x.conj().T).mul_(-0.05 / (1.0 + w) / (3 * ng))
    return 0.5 * (out + out.conj().transpose(1, 2)), v


def _gpp_inputs(case, seed):
    gen = _generator(seed)
    nb, ns, ng, ne = case["nb"], case["ns"], case["ng"], case["ne"]
    rng = np.random.default_rng(seed)
    e_n = np.sort(rng.uniform(-0.5, 1.5, nb))
    x = _normal(gen, ng, ng).mul_(2.0 ** 0.5)
    wt = _uniform(gen, ng * ng, 0.3, 2.0).reshape(ng, ng)
    return dict(m=_normal(gen, nb, ns, ng).mul_(ng ** -0.5), e_n=e_n,
                occupied=(e_n < 0.0).astype(np.int32),
                energies=(np.linspace(-0.5, 1.0, ne) if ne > 1 else np.array([0.25])) + 0.01j,
                omega2=0.5 * (x + x.conj().T).contiguous(), wtilde=(0.5 * (wt + wt.T)).contiguous(),
                vcoul=_uniform(gen, ng, 0.1, 2.0))


def _bands_inputs(case, seed):
    """Bands in energy order: the lowest kept, the rest in slices that double."""
    gen = _generator(seed)
    nb, keep, ns = case["nb"], case["keep"], case["slices"]
    psi = _normal(gen, nb, case["nr"]).mul_(VOLUME ** -0.5)
    rng = np.random.default_rng(seed)
    e = rng.uniform(0.05, 1.1, nb)
    order = np.argsort(e)
    size = [16 * 2 ** k for k in range(ns)]
    size[-1] = nb - keep - sum(size[:-1])
    at = np.concatenate([[0], np.cumsum(size)]) + keep
    slices = [order[at[k]:at[k + 1]] for k in range(ns)]
    return dict(psi=psi, e=torch.from_numpy(e).cuda(), keep=order[:keep], slices=slices,
                n_xi=case["n_xi"], theta=[rng.random((case["n_xi"], len(s))) for s in slices])


def prepare(case, seed):
    op = case["op"]
    if op == "chi0":
        _, p = _one_problem(case, seed)
        return dict(op=op, problem=p, kw=dict(precision=case["precision"], n_slices=case["slices"]))
    if op == "grad":
        gen, p = _one_problem(case, seed)
        ng = len(p.gvec)
        w = _normal(gen, case["nz"], ng, ng)
        leaves = [t.requires_grad_(True) for t in (p.psi_v, p.psi_c, p.e_v, p.e_c)]
        return dict(op=op, problem=p, leaves=leaves,
                    grad=(0.5 * (w + w.conj().transpose(1, 2))).contiguous())
    if op == "batch":
        return dict(op=op, problems=_batch_problems(case, seed),
                    flags=gw.GW_FLAG_GRAPH if case["graph"] else 0)
    if op == "subspace":
        gen, p = _one_problem(case, seed)
        ng = len(p.gvec)
        basis = torch.linalg.qr(_normal(gen, ng, case["n_eig"]))[0].contiguous()
        weight = torch.from_numpy(_coulomb(ng) ** 0.5).cuda()
        s = dict(op=op, problem=p, basis=basis, weight=weight, m=None)
        if case["kept"]:
            one = gw.Chi0Problem(n=p.n, volume=p.volume, psi_v=p.psi_v, psi_c=p.psi_c, e_v=p.e_v,
                                 e_c=p.e_c, gvec=p.gvec, z=np.zeros(1, dtype=np.complex128))
            s["m"] = gw.gw_chi0_keep_m(one)[1]
        return s
    if op == "diag":
        chi, v = _static_chi(_generator(seed), case["ng"], 1)
        return dict(op=op, chi=chi[0].contiguous(), weight=torch.sqrt(v), n_eig=case["n_eig"])
    if op == "epsinv":
        chi, v = _static_chi(_generator(seed), case["ng"], case["nz"])
        return dict(op=op, chi=chi.contiguous(), vcoul=v)
    if op == "gpp":
        return dict(op=op, **_gpp_inputs(case, seed))
    if op == "bands":
        return dict(op=op, **_bands_inputs(case, seed))
    x = _normal(_generator(seed), case["batch"], case["n"], case["n"])
    return dict(op=op, a=(0.5 * (x + x.conj().transpose(1, 2))).contiguous())


# ---------------------------------------------------------------- one pass

def run(s):
    op = s["op"]
    if op == "chi0":
        return gw.gw_chi0(s["problem"], **s["kw"])
    if op == "grad":
        p = s["problem"]
        chi = gw.chi0(*s["leaves"], p.gvec, p.z, p.n, p.volume)
        grads = torch.autograd.grad(chi, s["leaves"], grad_outputs=s["grad"])
        return [chi.detach(), *grads]
    if op == "batch":
        return gw.gw_chi0(s["problems"], flags=s["flags"])
    if op == "subspace":
        if s["m"] is not None:
            return gw.gw_chi0_from_m(s["problem"], s["m"], s["basis"], weight=s["weight"])
        return gw.gw_chi0_subspace(s["problem"], s["basis"], weight=s["weight"])
    if op == "diag":
        basis, ev, _ = gw.gw_subspace_basis(s["chi"], s["n_eig"], weight=s["weight"])
        return [ev, basis]
    if op == "epsinv":
        return gw.gw_epsinv(s["chi"], s["vcoul"])
    if op == "gpp":
        return gw.gw_gpp_sigma(s["m"], s["e_n"], s["occupied"], s["energies"], s["omega2"],
                               s["wtilde"], s["vcoul"])
    if op == "bands":
        return list(gw.gw_pseudobands(s["psi"], s["e"], s["keep"], s["slices"], s["n_xi"],
                                      s["theta"]))
    return list(gw.gw_heev(s["a"]))


# ---------------------------------------------------------------- cost

def _chi0_work(nr, nv, nc, ng, nz, real_delta, ncol=None):
    """FFT and contraction of nv nc pairs (a Hermitian chi: half its entries)."""
    ncol = ncol or ng
    pairs = nv * nc
    entries = ncol * (ncol + 1) / 2 if real_delta else ncol * ncol
    flops = pairs * (8.0 * entries * nz + 5.0 * nr * math.log2(nr))
    return flops, 16.0 * ((nv + nc) * nr + nz * ncol * ncol)


def work(case):
    op = case["op"]
    if op in ("chi0", "grad", "subspace"):
        n = (case["n1"], case["n2"], case["n3"])
        nr, ng = n[0] * n[1] * n[2], len(_gsphere(case["r2"], n))
        nv, nc, nz = case["nv"], case["nc"], case["nz"]
        real_delta = case["axis"] != "real"
        if op == "subspace":
            flops, data = _chi0_work(nr, nv, nc, ng, nz, real_delta, case["n_eig"])
            flops += 8.0 * nv * nc * ng * case["n_eig"]
            if case["kept"]:
                flops -= nv * nc * 5.0 * nr * math.log2(nr)
                data += 16.0 * (nv * nc * ng - (nv + nc) * nr)
            return dict(flops=flops, bytes=data + 16.0 * ng * case["n_eig"])
        flops, data = _chi0_work(nr, nv, nc, ng, nz, real_delta)
        if op == "grad":   # g_M = M (W or W + W^H), the inverse transform, the band sums
            flops += nv * nc * (8.0 * ng * ng * nz * (1 if real_delta else 2)
                                + 5.0 * nr * math.log2(nr) + 16.0 * nr)
            data *= 2
        return dict(flops=flops, bytes=data)
    if op == "batch":
        nr = case["n1"] * case["n2"] * case["n3"]
        w = [_chi0_work(nr, case["nv"], nc, ng, case["nz"], True)
             for nc, ng, _ in _batch_shapes(case)]
        return dict(flops=sum(x[0] for x in w), bytes=sum(x[1] for x in w))
    if op == "diag":       # one product with chi, one Ritz matrix and one rotation of the block
        ng, k = case["ng"], case["n_eig"]
        return dict(flops=8.0 * ng * k * (ng + 2.0 * k) + 72.0 * k ** 3,
                    bytes=16.0 * (ng * ng + ng * k))
    if op == "epsinv":
        return dict(flops=8.0 * case["ng"] ** 3 * case["nz"], bytes=32.0 * case["ng"] ** 2 * case["nz"])
    if op == "gpp":
        nb, ns, ng, ne = case["nb"], case["ns"], case["ng"], case["ne"]
        return dict(flops=nb * ne * 8.0 * (ns * ng * ng + ng * ns * ns),
                    bytes=16.0 * (nb * ns * ng + 1.5 * ng * ng + ne * ns * ns))
    if op == "bands":
        mixed, nr = case["nb"] - case["keep"], case["nr"]
        out = case["keep"] + case["slices"] * case["n_xi"]
        return dict(flops=8.0 * mixed * case["n_xi"] * nr, bytes=16.0 * (case["nb"] + out) * nr)
    return dict(flops=72.0 * case["n"] ** 3 * case["batch"], bytes=48.0 * case["n"] ** 2 * case["batch"])


# ---------------------------------------------------------------- double precision

def _exact_m(p, v0, v1):
    """M of the pairs of valence bands v0..v1 with every conduction band."""
    n = tuple(p.n)
    rho = (p.psi_v[v0:v1, None, :].conj() * p.psi_c[None, :, :]).reshape(-1, *n)
    f = torch.fft.ifftn(rho, dim=(1, 2, 3)).reshape(rho.shape[0], -1)
    g = np.asarray(p.gvec, dtype=np.int64) % np.asarray(n)
    at = torch.from_numpy((g[:, 0] * n[1] + g[:, 1]) * n[2] + g[:, 2]).to(f.device)
    return f[:, at] * p.volume


def _exact_delta(p, v0, v1, z):
    de = (p.e_v[v0:v1, None] - p.e_c[None, :]).reshape(-1)
    return 1.0 / (de + complex(z)) + 1.0 / (de - complex(z))


def _valence_blocks(p, most=3e9):
    nr = p.psi_c.shape[1]
    step = max(1, int(most / (16.0 * nr * max(1, p.psi_c.shape[0]))))
    return [(a, min(a + step, p.psi_v.shape[0])) for a in range(0, p.psi_v.shape[0], step)]


def _exact_chi(p, cols=None):
    ng = len(p.gvec) if cols is None else cols.shape[1]
    chi = torch.zeros((len(p.z), ng, ng), dtype=C128, device="cuda")
    for a, b in _valence_blocks(p):
        m = _exact_m(p, a, b)
        m = m if cols is None else m @ cols
        mh = m.conj().T.contiguous()
        for w, z in enumerate(p.z):
            chi[w] += SPIN * (mh @ (_exact_delta(p, a, b, z)[:, None] * m))
    return chi


def _exact_grad(s):
    p = s["problem"]
    out = [torch.zeros_like(t) for t in s["leaves"]]
    chi = torch.zeros((len(p.z), len(p.gvec), len(p.gvec)), dtype=C128, device="cuda")
    for a, b in _valence_blocks(p, 1e9):
        m = _exact_m(p, a, b)
        part = torch.stack([SPIN * (m.conj().T @ (_exact_delta(p, a, b, z)[:, None] * m))
                            for z in p.z])
        for o, g in zip(out, torch.autograd.grad(part, s["leaves"], grad_outputs=s["grad"])):
            o += g
        chi += part.detach()
    return [chi, *out]


def _exact_gpp(s):
    m, nb, ne = s["m"], s["m"].shape[0], len(s["energies"])
    out = torch.zeros((ne, m.shape[1], m.shape[1]), dtype=C128, device="cuda")
    top = s["omega2"] * s["vcoul"][None, :] / (2.0 * s["wtilde"])
    for k in range(nb):
        sn = -1.0 if s["occupied"][k] else 1.0
        left, right = m[k].conj().contiguous(), m[k].T.contiguous()
        for i, e in enumerate(s["energies"]):
            pole = complex(e) - float(s["e_n"][k]) - sn * s["wtilde"]
            out[i] += left @ (top / pole) @ right
    return out


def _exact_bands(s):
    psi, n_xi = s["psi"], s["n_xi"]
    out, e = [psi[torch.from_numpy(s["keep"]).cuda()]], [s["e"].cpu().numpy()[s["keep"]]]
    for idx, th in zip(s["slices"], s["theta"]):
        phase = torch.from_numpy(np.exp(2j * np.pi * th)).cuda() / math.sqrt(n_xi)
        out.append(phase @ psi[torch.from_numpy(idx).cuda()])
        e.append(np.full(n_xi, s["e"].cpu().numpy()[idx].mean()))
    return [torch.cat(out), torch.from_numpy(np.concatenate(e))]


def exact(case, seed):
    op = case["op"]
    if op == "chi0":
        return _exact_chi(_one_problem(case, seed)[1])
    if op == "batch":
        return [_exact_chi(p) for p in _batch_problems(case, seed)]
    if op == "subspace":
        gen, p = _one_problem(case, seed)
        ng = len(p.gvec)
        basis = torch.linalg.qr(_normal(gen, ng, case["n_eig"]))[0]
        return _exact_chi(p, torch.from_numpy(_coulomb(ng) ** 0.5).cuda()[:, None] * basis)
    s = prepare(case, seed)
    if op == "grad":
        return _exact_grad(s)
    if op == "diag":       # eigenvectors carry a phase of their own: values only
        w = s["weight"].cpu().numpy()
        a = w[:, None] * s["chi"].cpu().numpy() * w[None, :]
        return [torch.from_numpy(np.linalg.eigvalsh(a)[:case["n_eig"]]), None]
    if op == "epsinv":
        v = s["vcoul"].cpu().numpy()
        eps = np.eye(case["ng"])[None] - v[None, :, None] * s["chi"].cpu().numpy()
        return torch.from_numpy(np.linalg.inv(eps))
    if op == "gpp":
        return _exact_gpp(s)
    if op == "bands":
        return _exact_bands(s)
    return [torch.from_numpy(np.linalg.eigvalsh(s["a"].cpu().numpy())), None]
