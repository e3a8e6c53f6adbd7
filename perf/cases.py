"""Measured cases of the framework, through its public entry points.

A case is a dict of plain values; `prepare` builds what a program has in hand
before the call (a bound context, network parameters, training data), `run` is
one pass, `work` the bytes and operations such a pass cannot do without and
`exact` the same results in 64 bits from plain torch.

Kinds:
  solve    CCD of one or more pure-neutron-matter problems from the MBPT2 start
           (or, with learned=True, from the network's) until the energy's
           remaining change is below 2e-8, then the amplitudes (a checkpoint)
  twist    the same on a mesh of twisted boundary conditions, and its averages
  mbpt3    third-order energies of neutron matter, diagram by diagram
  nuclear  sweeps of symmetric nuclear matter (protons and neutrons), then the
           amplitudes
  forward  the warm-start network on a buffer of amplitude features
  grad     its loss and gradient over a data set
  train    Adam steps of a training run in progress
  dense    CCD of a small model space given by its matrix elements
"""
import functools
import math

import numpy as np
import torch

from paper_1611_06765_amd import ccd, inputs

MINNESOTA = ((200.0, 1.487), (-178.0, 0.639), (-91.85, 0.465))  # (V, kappa) of the R, T and S channels
HBAR2_OVER_M = 41.47
PRECISIONS = {"fp64": ccd.CCD_PREC_FP64, "fp32": ccd.CCD_PREC_FP32, "bf16": ccd.CCD_PREC_BF16}
MIXED_TOL = {"fp64": 0.0, "fp32": 1e-4, "bf16": 1e-2}  # MeV, where a mixed-precision phase hands over to FP64
SWEEPS = 25  # sweeps that a solve takes from the MBPT2 start at ordinary densities


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the paper's pairing model, its published table: the smallest call there is
        dict(name="pairing_8_states", kind="dense", model="pairing", size=4, holes=4),
        # one small box: a quick look, or one point of a scan run as separate programs; latency only
        dict(name="pnm14_n4", kind="solve", n=14, nmax2=4, count=1, precision="fp64", learned=False),
        # the equation of state: 66 neutrons at ten densities as one batch
        dict(name="pnm66_n20_x10", kind="solve", n=66, nmax2=20, count=10, precision="fp64", learned=False),
        # one solve in the largest basis the paper's tables use
        dict(name="pnm66_n36", kind="solve", n=66, nmax2=36, count=1, precision="fp64", learned=False),
        # the same with BF16 contractions and FP64 refinement
        dict(name="pnm66_n36_bf16", kind="solve", n=66, nmax2=36, count=1, precision="bf16", learned=False),
        # boxes of different sizes and cutoffs in one context (a finite-size and cutoff study)
        dict(name="pnm_mixed_x12", kind="solve", n=0, nmax2=36, count=12, precision="fp64", learned=False),
        # held-out densities from the network's start
        dict(name="pnm66_n36_learned_x3", kind="solve", n=66, nmax2=36, count=3, precision="fp64", learned=True),
        # twist averaging on two points per direction
        dict(name="pnm66_n20_twist8", kind="twist", n=66, nmax2=20, mesh=2),
        # symmetric nuclear matter: a small box and the largest one of the benchmark
        dict(name="snm28_n4", kind="nuclear", n=28, nmax2=4, sweeps=16),
        dict(name="snm108_n20", kind="nuclear", n=108, nmax2=20, sweeps=16),
        # the network on every amplitude of one n^2 <= 36 problem
        dict(name="network_forward", kind="forward", rows=1037776, precision="bf16"),
        # part of an epoch at the trainer's default batch
        dict(name="network_train", kind="train", rows=335492, batch=4096, steps=32),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve"] * 6 + ["twist", "mbpt3", "nuclear", "nuclear", "nuclear", "forward", "forward",
                                       "grad", "train", "train", "dense"])
    if kind == "solve":
        n = rng.choice([2, 14, 38, 54, 66, 66, 0])
        nmax2 = rng.randint(max(1, {2: 1, 14: 2, 38: 4, 54: 5, 66: 6}.get(n, 12)), 36)
        small = nmax2 * nmax2 * max(n, 40) <= 66 * 22 * 22
        return dict(kind=kind, n=n, nmax2=nmax2, count=_log_int(rng, 1, 10 if small else 3),
                    precision=rng.choice(["fp64", "fp64", "fp64", "fp32", "bf16"]), learned=rng.random() < 0.15)
    if kind == "twist":
        return dict(kind=kind, n=rng.choice([14, 38, 54, 66]), nmax2=rng.randint(8, 20), mesh=rng.choice([1, 2]))
    if kind == "mbpt3":
        return dict(kind=kind, n=rng.choice([14, 38, 54, 66]), nmax2=rng.randint(8, 30), count=rng.randint(1, 3))
    if kind == "nuclear":
        n = rng.choice([4, 28, 28, 108])
        nmax2 = rng.choice([4, 6, 9, 10, 12, 14, 16, 17, 20] if n < 108 else [12, 14, 16, 18, 20])
        return dict(kind=kind, n=n, nmax2=nmax2, sweeps=rng.randint(8, 16))
    if kind == "forward":
        return dict(kind=kind, rows=_log_int(rng, 100, 1037776), precision=rng.choice(["bf16", "fp32"]))
    if kind == "grad":
        return dict(kind=kind, rows=_log_int(rng, 300, 335492))
    if kind == "train":
        batch = _log_int(rng, 256, 16384)
        return dict(kind=kind, rows=max(batch, _log_int(rng, 20000, 335492)), batch=batch, steps=rng.randint(8, 32))
    if rng.random() < 0.15:  # two neutrons, n^2 <= 1
        return dict(kind=kind, model="plane waves", size=1, holes=2)
    size = rng.randint(4, 9)
    return dict(kind=kind, model="pairing", size=size, holes=rng.choice([2, 4, 6] if size <= 6 else [2, 4]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _problems(case, seed):
    """(N, nmax2, rho) of every problem: densities from the seed, sizes from the case alone."""
    rng = np.random.default_rng(seed)
    lo = 0.06 if case["kind"] in ("twist", "mbpt3") else 0.02
    rho = np.sort(rng.uniform(lo, 0.20, size=case["count"]))
    if case["count"] == 1:
        rho = rng.uniform(0.08, 0.20, size=1)
    if case["n"]:
        return [(case["n"], case["nmax2"], float(r)) for r in rho]
    # every N of the list in turn, cutoffs spread evenly from 12 up to nmax2
    sizes = [14, 38, 54, 66]
    span = np.linspace(12, case["nmax2"], case["count"]).round().astype(int) if case["count"] > 1 else [case["nmax2"]]
    return [(sizes[k % 4], int(span[(5 * k) % case["count"]]), float(r)) for k, r in enumerate(rho)]


def _nuclear_density(case, seed):
    # the iteration with linear mixing converges from these densities up
    lo, hi = {4: (0.10, 0.20), 28: (0.20, 0.24), 108: (0.14, 0.20)}[case["n"]]
    return float(np.random.default_rng(seed).uniform(lo, hi))


def _network(seed, scale):
    """Network parameters: the initial draw, its output layer scaled so that the predictions are as small
    as a trained network's."""
    p = inputs.mlp_init(seed % 100003)
    p[inputs.OFF_W3:inputs.OFF_B3] *= scale
    return p


def _rows(n, seed):
    """Features of n amplitudes and their targets, with the ranges and zeros of real ones (float32, on the GPU)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    u = lambda lo, hi: lo + (hi - lo) * torch.rand(n, generator=g, device="cuda")  # noqa: E731
    rho = 0.02 + 0.18 * torch.randint(0, 24, (n,), generator=g, device="cuda") / 23.0
    ku = 2.0 * math.pi * (rho / 66.0) ** (1.0 / 3.0)
    q = [0.5 * ku * torch.randint(0, 120, (n,), generator=g, device="cuda").sqrt() for _ in range(2)]
    v = torch.where(u(0, 1) < 0.5, torch.zeros((), device="cuda"), u(-0.3, 0.3))
    cols = [rho / 0.16, q[0], q[1], u(-0.5, 0.3), u(-0.5, 0.3), u(0.3, 2.5), u(0.3, 2.5), v]
    feat = torch.stack(cols, dim=1).to(torch.float32).contiguous()
    target = (0.02 * torch.sin(3.0 * feat[:, 1] - feat[:, 2]) * (feat[:, 7] + 0.1 * feat[:, 5])).contiguous()
    return feat, target


def _dense(case, seed):
    """h, v and the holes of a dense model space."""
    rng = np.random.default_rng(seed)
    if case["model"] == "pairing":
        h, v = inputs.pairing_hamiltonian(float(rng.uniform(0.1, 0.7)), n_levels=case["size"])
        return h, v, case["holes"]
    m = _Matter(2, case["size"], float(rng.uniform(0.04, 0.12)), species=1, device="cpu")
    every = torch.arange(m.ns)
    return m.tkin.numpy(), m.element(every, every, every, every).numpy(), 2


def prepare(case, seed):
    kind, stream = case["kind"], torch.cuda.current_stream().cuda_stream
    if kind == "solve":
        specs = _problems(case, seed)
        s = dict(kind=kind, precision=case["precision"], net=None,
                 ctx=ccd.Context([ccd.problem(*p) for p in specs], stream=stream).bind())
        if case["learned"]:
            s["net"] = torch.tensor(_network(seed, 0.1), device="cuda")
        return s
    if kind == "twist":
        (n, nmax2, rho), = _problems(dict(case, count=1), seed)
        theta, weight = ccd.twist_mesh(case["mesh"])
        probs = [ccd.problem(n, nmax2, rho, twist=t) for t in theta]
        return dict(kind=kind, ctx=ccd.Context(probs, stream=stream).bind(), weight=weight)
    if kind == "mbpt3":
        return dict(kind=kind, ctx=ccd.Context([ccd.problem(*p) for p in _problems(case, seed)], stream=stream).bind())
    if kind == "nuclear":
        p = ccd.nm_problem(case["n"], case["nmax2"], _nuclear_density(case, seed))
        return dict(kind=kind, ctx=ccd.NMContext(p, stream=stream).bind(), sweeps=case["sweeps"])
    if kind == "dense":
        h, v, holes = _dense(case, seed)
        return dict(kind=kind, h=h, v=v, holes=holes, stream=stream)
    feat, target = _rows(case["rows"], seed)
    s = dict(kind=kind, feat=feat, target=target, params=torch.tensor(_network(seed, 1.0), device="cuda"))
    if kind == "forward":
        s["precision"] = PRECISIONS[case["precision"]]
    if kind == "train":  # a run in progress: moments of earlier steps, the order of the next ones
        m, v = _moments(seed)
        s["adam"] = ccd.AdamState(s["params"])
        s["adam"].m.copy_(m)
        s["adam"].v.copy_(v)
        s["adam"].step.value = 1000
        s["order"] = _order(case, seed)
        s["batch"] = case["batch"]
        s["work"] = ccd.mlp_work_buffer(case["batch"], "cuda")
    return s


def _moments(seed):
    g = torch.Generator(device="cuda").manual_seed(seed + 1)
    n = inputs.N_PARAM
    return (1e-3 * torch.randn(n, generator=g, device="cuda"),
            1e-4 * (0.2 + torch.rand(n, generator=g, device="cuda")))


def _order(case, seed):
    rng = np.random.default_rng(seed)
    want = case["batch"] * case["steps"]
    rounds = -(-want // case["rows"])
    order = np.concatenate([rng.permutation(case["rows"]) for _ in range(rounds)])[:want]
    return torch.from_numpy(order.astype(np.int32)).cuda()


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    kind = s["kind"]
    if kind == "solve":
        ctx = s["ctx"]
        if s["net"] is None:
            ctx.reset_amplitudes()
        else:
            ctx.warm_start(s["net"])
        r = ctx.iterate(mixing=0.5, tol_rel=2e-8, max_iter=200, check_every=8, stop_rule=1, history=True,
                        precision=PRECISIONS[s["precision"]], mixed_tol=MIXED_TOL[s["precision"]], refine_sweeps=1)
        return {"sweeps": r["sweeps"], "history": r["history"], "energies": [ctx.energy(p) for p in range(ctx.n)],
                "amplitudes": [ctx.get_amplitudes(p) for p in range(ctx.n)]}
    if kind == "twist":
        ctx = s["ctx"]
        ctx.reset_amplitudes()
        r = ctx.iterate(mixing=0.5, tol_rel=2e-8, max_iter=200, check_every=8, stop_rule=1, history=True)
        return {"sweeps": r["sweeps"], "history": r["history"], "average": ctx.twist_average(s["weight"]),
                "energies": [ctx.energy(p) for p in range(ctx.n)],
                "amplitudes": [ctx.get_amplitudes(p) for p in range(ctx.n)]}
    if kind == "mbpt3":
        return s["ctx"].mbpt3()
    if kind == "nuclear":
        r = s["ctx"].iterate(mixing=0.5, max_iter=s["sweeps"])
        return {"history": r["history"], "amplitudes": s["ctx"].get_amplitudes()}
    if kind == "forward":
        return ccd.mlp_forward(s["params"], s["feat"], s["precision"])
    if kind == "grad":
        loss, grad = ccd.mlp_loss_grad(s["params"], s["feat"], s["target"])
        return {"loss": loss, "grad": grad}
    if kind == "train":
        loss = ccd.mlp_train(s["params"], s["adam"], s["feat"], s["target"], s["order"], s["batch"], 1e-3,
                             work=s["work"])
        return {"loss": loss, "params": s["params"], "m": s["adam"].m, "v": s["adam"].v}
    r = ccd.dense_solve(s["h"], s["v"], s["holes"], mixing=0.7, tol=1e-9, max_iter=60, stream=s["stream"])
    history = np.full(60, np.nan)
    history[:r["sweeps"]] = r["history"]
    return {"e_ref": r["e_ref"], "e_mbpt2": r["e_mbpt2"], "e_ccd": r["e_ccd"], "sweeps": r["sweeps"], "history": history}


# ---------------------------------------------------------------------------
# bytes and operations
# ---------------------------------------------------------------------------
@functools.lru_cache(maxsize=None)
def _counts(n, nmax2, species):
    """(amplitudes, operations of one CCD sweep in blocks of conserved momentum, spin and isospin)."""
    st = _states(nmax2, species)
    holes, parts = st[:n], st[n:]
    base = np.array([1, 64, 64 ** 2, 64 ** 3, 64 ** 3 * 8], dtype=np.int64)

    def keys(x, y, sign, upper):
        k = (x[:, None, :] + sign * y[None, :, :]).astype(np.int64) @ base
        return k[np.triu_indices(len(x), 1)] if upper else k.reshape(-1)

    hk, hc = np.unique(keys(holes, holes, 1, True), return_counts=True)
    pk, pc = np.unique(keys(parts, parts, 1, True), return_counts=True)
    npp = dict(zip(pk.tolist(), pc.tolist()))
    nhh = dict(zip(hk.tolist(), hc.tolist()))
    amps = sum(c * npp.get(k, 0) for k, c in nhh.items())
    # pp ladder over momentum pairs (half the rows), hh ladder and chi_klij
    flops = sum(2.0 * (npp.get(k, 0) / 2.0) ** 2 * c + 4.0 * npp.get(k, 0) * c * c for k, c in nhh.items())
    xk, xc = np.unique(keys(parts, holes, -1, False), return_counts=True)
    nph = dict(zip(xk.tolist(), xc.tolist()))
    # two terms of every pair of cross channels {Q, -Q} in three products
    flops += sum(3.0 * c * c * nph.get(-k, 0) for k, c in nph.items())
    return amps, flops


def work(case):
    kind = case["kind"]
    if kind in ("solve", "twist", "mbpt3", "nuclear"):
        if kind == "nuclear":
            specs, species, sweeps = [(case["n"], case["nmax2"])], 2, case["sweeps"]
        elif kind == "twist":
            specs, species, sweeps = [(case["n"], case["nmax2"])] * case["mesh"] ** 3, 1, SWEEPS
        else:
            specs, species = [p[:2] for p in _problems(case, 0)], 1
            sweeps = 4 if kind == "mbpt3" else SWEEPS
        counts = [_counts(n, m, species) for n, m in specs]
        # a sweep reads the amplitudes and writes the new ones
        return {"bytes": sweeps * sum(16.0 * a for a, _ in counts), "flops": sweeps * sum(f for _, f in counts)}
    if kind == "dense":
        n, nh = (2 * case["size"], case["holes"]) if case["model"] == "pairing" else (14 if case["size"] == 1 else 38, 2)
        m = float(nh * nh * (n - nh) ** 2)
        per = m * (2.0 * (n - nh) ** 2 + 4.0 * nh * nh + 12.0 * nh * (n - nh))
        return {"bytes": 8.0 * n ** 4 + 16.0 * m * 20, "flops": 20 * per}
    w = inputs.WIDTH
    layer = 4 * (2.0 * w * w + 2.0 * w * inputs.N_IN + 2.0 * w)  # four swap variants of an amplitude
    if kind == "forward":
        return {"bytes": 36.0 * case["rows"], "flops": layer * case["rows"]}
    if kind == "grad":
        return {"bytes": 36.0 * case["rows"] + 8.0 * inputs.N_PARAM, "flops": 3 * layer * case["rows"]}
    rows = case["batch"] * case["steps"]
    return {"bytes": 40.0 * rows + 24.0 * inputs.N_PARAM * case["steps"], "flops": 3 * layer * rows}


# ---------------------------------------------------------------------------
# the same in 64 bits, from the equations
# ---------------------------------------------------------------------------
def _states(nmax2, species):
    """(n_x, n_y, n_z, 2 s_z, 2 t_z) of every plane wave up to the cutoff, shell by shell."""
    r = math.isqrt(nmax2)
    out = []
    for shell in range(nmax2 + 1):
        for x in range(-r, r + 1):
            for y in range(-r, r + 1):
                for z in range(-r, r + 1):
                    if x * x + y * y + z * z == shell:
                        out += [(x, y, z, s, t) for s in (-1, 1) for t in ((-1, 1) if species == 2 else (1,))]
    return np.array(out)


class _Matter:
    """Nucleons in a box with the Minnesota interaction: kinetic energies and antisymmetrised elements."""

    def __init__(self, n, nmax2, rho, species, device="cuda"):
        self.st = torch.from_numpy(_states(nmax2, species)).to(device)
        self.ns, self.n = len(self.st), n
        self.box = (n / rho) ** (1.0 / 3.0)
        k = 2.0 * math.pi / self.box
        self.tkin = 0.5 * HBAR2_OVER_M * k * k * (self.st[:, :3] ** 2).sum(1).to(torch.float64)
        m = torch.arange(4 * nmax2 + 1, dtype=torch.float64, device=device)
        self.table = [v / self.box ** 3 * (math.pi / kp) ** 1.5 * torch.exp(-k * k * m / (4.0 * kp))
                      for v, kp in MINNESOTA]

    def _direct(self, p, q, r, s):
        # <pq|v|rs> of v = (V_R + (1 + P_s) V_T / 2 + (1 - P_s) V_S / 2) (1 - P_s P_t) / 2, with the exchange
        # operators P_s and P_t of spin and isospin, before antisymmetrisation
        d2 = ((p[..., :3] - r[..., :3]) ** 2).sum(-1)
        same = lambda a, b, c: a[..., c] == b[..., c]  # noqa: E731
        ds, xs = same(p, r, 3) & same(q, s, 3), same(p, s, 3) & same(q, r, 3)
        dt, xt = same(p, r, 4) & same(q, s, 4), same(p, s, 4) & same(q, r, 4)
        f = lambda a: a.to(torch.float64)  # noqa: E731
        one, ps, pt, pst = f(ds & dt), f(xs & dt), f(ds & xt), f(xs & xt)
        w = [t[d2.clamp(max=len(t) - 1)] for t in self.table]
        return 0.5 * (w[0] * (one - pst) + 0.5 * w[1] * (one + ps - pst - pt) + 0.5 * w[2] * (one - ps - pst + pt))

    def element(self, p, q, r, s):
        """<pq||rs> on the outer product of four index lists."""
        out = torch.zeros(len(p), len(q), len(r), len(s), dtype=torch.float64, device=self.st.device)
        for i in range(len(p)):  # one p at a time keeps the index arrays small
            a = self.st[p[i]].view(1, 1, 1, 5)
            b, c, d = self.st[q].view(-1, 1, 1, 5), self.st[r].view(1, -1, 1, 5), self.st[s].view(1, 1, -1, 5)
            keep = ((a + b)[..., :3] == (c + d)[..., :3]).all(-1)
            idx = keep.nonzero(as_tuple=True)
            B, C, D = self.st[q][idx[0]], self.st[r][idx[1]], self.st[s][idx[2]]
            A = self.st[p[i]].expand_as(B)
            out[i][idx] = self._direct(A, B, C, D) - self._direct(A, B, D, C)
        return out

    def canonical(self):
        """Indices (i, j, a, b) of the amplitudes in the library's order: blocks by isospin, spin and momentum."""
        st = self.st.cpu().numpy()
        hh, pp = {}, {}
        key = lambda p, q: tuple((st[p] + st[q])[[4, 3, 0, 1, 2]].tolist())  # noqa: E731
        for i in range(self.n):
            for j in range(i + 1, self.n):
                hh.setdefault(key(i, j), []).append((i, j))
        for a in range(self.n, self.ns):
            for b in range(a + 1, self.ns):
                k = key(a, b)
                if k in hh:
                    pp.setdefault(k, []).append((a, b))
        out = [(i, j, a, b) for k in sorted(hh) for a, b in pp.get(k, ()) for i, j in hh[k]]
        return torch.tensor(out, device=self.st.device)


class _Ccd:
    """CCD amplitude iteration (eq. ccd3) on dense blocks, t[i, j, a, b]."""

    def __init__(self, element, tkin, n):
        ns, dev = len(tkin), tkin.device
        o, v = torch.arange(n, device=dev), torch.arange(n, ns, device=dev)
        every = torch.arange(ns, device=dev)
        eps = tkin.clone()
        for p in range(ns):
            one = every[p:p + 1]
            eps[p] += torch.diagonal(element(one, o, one, o)[0, :, 0, :]).sum()
        diag = element(o, o, o, o)
        self.e_ref = float(tkin[:n].sum() + 0.5 * torch.diagonal(diag.reshape(n * n, n * n)).sum())
        self.oooo, self.vvvv = diag, element(v, v, v, v)
        self.oovv = element(o, o, v, v)
        self.ovvo = element(o, v, v, o)
        self.den = eps[:n].view(-1, 1, 1, 1) + eps[:n].view(-1, 1, 1) - eps[n:].view(-1, 1) - eps[n:].view(1, -1)
        self.no, self.nv = n, ns - n
        self.t = self.oovv / self.den

    def energy(self):
        return float(0.25 * (self.oovv * self.t).sum())

    def sweep(self, mixing):
        o, v, t, w = self.no, self.nv, self.t, self.oovv
        mat = lambda x, r, c: x.reshape(r, c)  # noqa: E731
        r = w.clone()
        r += 0.5 * mat(mat(t, o * o, v * v) @ mat(self.vvvv, v * v, v * v).T, o * o, v * v).reshape(o, o, v, v)
        chi = self.oooo.permute(2, 3, 0, 1).reshape(o * o, o * o) \
            + 0.5 * mat(t, o * o, v * v) @ mat(w, o * o, v * v).T  # [ij][kl]
        r += 0.5 * (chi @ mat(t, o * o, v * v)).reshape(o, o, v, v)
        tp = t.permute(0, 2, 1, 3).reshape(o * v, o * v)  # [ia][kc]
        wp = w.permute(0, 2, 1, 3).reshape(o * v, o * v)  # [kc][ld]
        ring = (tp @ self.ovvo.permute(0, 2, 3, 1).reshape(o * v, o * v)).reshape(o, v, o, v).permute(0, 2, 1, 3)
        r += ring - ring.transpose(0, 1) - ring.transpose(2, 3) + ring.transpose(0, 1).transpose(2, 3)
        quad = (tp @ wp @ tp).reshape(o, v, o, v).permute(0, 2, 1, 3)  # t_ik^ac w_klcd t_ld^jb
        r += quad - quad.transpose(0, 1)
        # sum_kcd w_klcd t_ik^dc and sum_klc w_klcd t_lk^ac
        hole = mat(t.permute(0, 1, 3, 2), o, o * v * v) @ mat(w.permute(1, 0, 2, 3), o, o * v * v).T  # [i][l]
        part = mat(t.permute(2, 1, 0, 3), v, o * o * v) @ mat(w.permute(3, 0, 1, 2), v, o * o * v).T  # [a][d]
        x = (hole @ mat(t, o, o * v * v)).reshape(o, o, v, v)  # t_lj^ab
        r -= 0.5 * (x - x.transpose(0, 1))
        y = torch.tensordot(t, part, dims=([2], [1])).permute(0, 1, 3, 2)  # t_ij^db [a][d]
        r -= 0.5 * (y - y.transpose(2, 3))
        self.t = mixing * r / self.den + (1.0 - mixing) * t

    def at(self, idx):
        return self.t[idx[:, 0], idx[:, 1], idx[:, 2] - self.no, idx[:, 3] - self.no]


def _solve(c, mixing, tol, tol_rel, rule, max_iter):
    """The stop rules of the iteration: rule 1 also bounds the geometric tail, in two sweeps in a row."""
    hist, old, prev, streak = [], c.energy(), 0.0, 0
    for _ in range(max_iter):
        c.sweep(mixing)
        e = c.energy()
        hist.append(e)
        de, thr = abs(e - old), tol + tol_rel * abs(e)
        stop = de < thr
        if rule:
            r = de / prev if prev > 0.0 else 1.0
            streak = streak + 1 if stop and r < 1.0 and de * r < thr * (1.0 - r) else 0
            stop = streak >= 2
        old, prev = e, de
        if stop and (tol > 0.0 or tol_rel > 0.0):
            break
    return hist


def _net64(flat):
    p = flat.to(torch.float64)
    w = inputs.WIDTH
    return [p[:inputs.OFF_B1].reshape(w, 8)[:, :7], p[inputs.OFF_B1:inputs.OFF_W2],
            p[inputs.OFF_W2:inputs.OFF_B2].reshape(w, w), p[inputs.OFF_B2:inputs.OFF_W3], p[inputs.OFF_W3:inputs.OFF_B3]]


def _variants(f):
    """The network's inputs for the four swaps (none, a b, i j, both) of each amplitude: [rows, 4, 7]."""
    rho, q, x, i, j, a, b, v = f.to(torch.float64).unbind(1)
    swaps = [(rho, q, i, j, a, b, v), (rho, x, i, j, b, a, -v), (rho, x, j, i, a, b, -v), (rho, q, j, i, b, a, v)]
    return torch.stack([torch.stack(c, 1) for c in swaps], 1)


def _predict64(net, f):
    w1, b1, w2, b2, w3 = net
    h = torch.relu(_variants(f) @ w1.T + b1)
    g = torch.relu(h @ w2.T + b2) @ w3
    return 0.25 * (g[:, 0] - g[:, 1] - g[:, 2] + g[:, 3])


def _grad64(flat, feat, target, scale):
    """Loss sum scale (y - y*)^2 / 2 and its gradient in the flat layout."""
    p = flat.to(torch.float64).clone().requires_grad_(True)
    loss = 0.0
    for k in range(0, len(feat), 65536):
        y = _predict64(_net64(p), feat[k:k + 65536])
        part = 0.5 * scale * ((y - target[k:k + 65536].to(torch.float64)) ** 2).sum()
        part.backward()
        loss += float(part.detach())
    return loss, p.grad


def exact(case, seed):
    kind = case["kind"]
    if kind == "dense":
        h, v, holes = _dense(case, seed)
        vt = torch.from_numpy(np.ascontiguousarray(v))
        c = _Ccd(lambda p, q, r, s: vt[p][:, q][:, :, r][:, :, :, s], torch.from_numpy(h), holes)
        e2 = c.energy()
        hist = _solve(c, 0.7, 1e-9, 0.0, 0, 60)
        return {"e_ref": c.e_ref, "e_mbpt2": e2, "e_ccd": hist[-1], "sweeps": len(hist),
                "history": np.array(hist + [math.nan] * (60 - len(hist)))}
    if kind == "nuclear":
        if len(_states(case["nmax2"], 2)) > 140:
            return None  # too large for dense blocks
        m = _Matter(case["n"], case["nmax2"], _nuclear_density(case, seed), species=2)
        c = _Ccd(m.element, m.tkin, m.n)
        hist = []
        for _ in range(case["sweeps"]):
            c.sweep(0.5)
            hist.append(c.energy())
        return {"history": np.array(hist), "amplitudes": c.at(m.canonical()).cpu().numpy()}
    if kind == "solve":
        specs = _problems(case, seed)
        if case["learned"] or case["precision"] != "fp64" or len(specs) > 4 or \
                any(len(_states(m, 1)) > 110 for _, m, _ in specs):
            return None  # too large for dense blocks, or a start or handover of its own
        out = {"sweeps": [], "history": [], "energies": [], "amplitudes": []}
        for n, nmax2, rho in specs:
            m = _Matter(n, nmax2, rho, species=1)
            c = _Ccd(m.element, m.tkin, n)
            e2 = c.energy()
            hist = _solve(c, 0.5, 0.0, 2e-8, 1, 200)
            out["sweeps"].append(len(hist))
            out["history"].append(hist + [math.nan] * (200 - len(hist)))
            out["energies"].append((c.e_ref, e2, hist[-1]))
            out["amplitudes"].append(c.at(m.canonical()).cpu().numpy())
        return dict(out, sweeps=np.array(out["sweeps"], dtype=np.int32), history=np.array(out["history"]))
    if kind not in ("forward", "grad", "train"):
        return None
    feat, target = _rows(case["rows"], seed)
    flat = torch.tensor(_network(seed, 1.0), device="cuda")
    if kind == "forward":
        net = _net64(flat)
        return torch.cat([_predict64(net, feat[k:k + 65536]) for k in range(0, len(feat), 65536)])
    if kind == "grad":
        loss, grad = _grad64(flat, feat, target, 1.0 / len(feat))
        return {"loss": loss, "grad": grad}
    m, v = (x.to(torch.float64) for x in _moments(seed))
    order, p, total = _order(case, seed).long(), flat.to(torch.float64), 0.0
    for s in range(case["steps"]):
        rows = order[s * case["batch"]:(s + 1) * case["batch"]]
        loss, g = _grad64(p, feat[rows], target[rows], 1.0 / case["batch"])
        total += loss
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        k = 1001 + s
        p = p - 1e-3 * (m / (1.0 - 0.9 ** k)) / (torch.sqrt(v / (1.0 - 0.999 ** k)) + 1e-8)
    return {"loss": total / case["steps"], "params": p, "m": m, "v": v}
