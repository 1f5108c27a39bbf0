"""Timed cases of the library: what its users have it do, through the public
Python entry points, over the sizes that the drivers, the tests and the
benchmark of this repository run.

A case is a dict of plain values with a "kind":

  step       one lattice context advanced and observed (growth runs, the
             oracle-sized workload, the storage forms, the scheme's options)
  batch      many lattices advanced together (the stability sweep, the paper's
             three 72^2 cells), then amplitudes and observables
  init       tpl_init: the forced base state on a column, copied and perturbed
  corrected  a coarse lattice stepped with an attached correction network
  mlp        the network's own calls on a snapshot of coarse nodes
  pair       one training pair of the network: restriction of a fine state,
             features, coarse steps, targets

listed(), draw(rng), prepare(case, seed), run(state), work(case) and
exact(case, seed) are described at each function.
"""
import math

import numpy as np
import torch

import paper_2201_10132_amd as P
from paper_2201_10132_amd import inputs
from paper_2201_10132_amd.learned import standardisation

FP64, FP32, BF16 = 0, 1, 2


# ---------------------------------------------------------------------------
# The cases.

def _step(name, nx, ny, nq, precision, steps, *, periods=1, Re=20.0, Wi=0.5, beta=0.8,
          perturbation=1e-4, inplace=0, gradients=0, spring_shift=0, qe_model=1, pre_steps=300,
          observe="amplitude"):
    return dict(name=name, kind="step", nx=nx, ny=ny, nq=nq, precision=precision, steps=steps,
                periods=periods, Re=Re, Wi=Wi, beta=beta, perturbation=perturbation,
                inplace=inplace, gradients=gradients, spring_shift=spring_shift,
                qe_model=qe_model, pre_steps=pre_steps, observe=observe)


def listed():
    return [
        # the smallest call: one step of a 16^2 lattice and its diagnostics,
        # as an interactive check or a test does it; all latency
        _step("step_16_fp64_1", 16, 16, 6, FP64, 1, observe="diagnostics"),
        # the 64^2 workload that the oracle also runs, sampled every 20 steps
        # (the growth runs sample the amplitude)
        _step("step_64_fp64_20", 64, 64, 16, FP64, 20, perturbation=1e-3),
        # the benchmark's FP64 lattice (1024 columns, four periods of 256
        # rows, 16 Q-points) at half its height
        _step("step_1024x512_fp64_4", 1024, 512, 16, FP64, 4, periods=2, Re=60.0, Wi=1.0,
              beta=0.7),
        # the same flow at full size in the BF16 storage form
        _step("step_1024_bf16_4", 1024, 1024, 16, BF16, 4, periods=4, Re=60.0, Wi=1.0, beta=0.7),
        # a ragged FP32 lattice with the spring term from psi at the beads
        _step("step_500x300_fp32_shift_6", 500, 300, 16, FP32, 6, periods=1, Re=40.0, Wi=1.0,
              beta=0.7, spring_shift=1),
        # an FP64 lattice held in one array (in place), same-step gradients
        _step("step_256_fp64_inplace_samestep_6", 256, 256, 16, FP64, 6, periods=1, Re=40.0,
              Wi=1.0, beta=0.7, inplace=1, gradients=1),
        # the paper's three 72^2 cells on 32 Q-points, between two samples
        dict(name="batch_72_nq32_fp64_40", kind="batch", set="cells", count=3, first=0, nq=32,
             precision=FP64, steps=40, diagnostics=True, pre_steps=100),
        # a stability sweep of 48 seeded lattices (128..512), FP32, 6 Q-points
        dict(name="batch_sweep48_fp32_6", kind="batch", set="sweep", count=48, first=0, nq=6,
             precision=FP32, steps=6, diagnostics=False, pre_steps=100),
        # start of a run: the forced base state by a column pre-run
        dict(name="init_256_fp64_nq8_1000", kind="init", nx=256, ny=256, nq=8, precision=FP64,
             periods=4, Re=50.0, Wi=1.0, beta=0.7, perturbation=1e-4, pre_steps=1000),
        # the learned correction's coarse lattice, ten corrected steps
        # (between two evaluations against the fine run)
        dict(name="corrected_256_nq8_10", kind="corrected", nx=256, ny=256, nq=8, periods=4,
             Re=50.0, Wi=0.8, beta=0.7, steps=10),
        # one Adam step on one snapshot of that lattice
        dict(name="mlp_train_65536", kind="mlp", op="train", rows=65536, nin=54, nout=5),
        # one training pair: restriction of a 1024^2 fine state, features,
        # four coarse steps, targets
        dict(name="pair_1024_256_nq8", kind="pair", nx=1024, ny=1024, factor=4, nq=8, periods=4,
             Re=50.0, Wi=0.8, beta=0.7, steps=4),
    ]


# bytes that a drawn case may move at most (the largest listed ones move about
# as much)
_MOST_BYTES = 150e9
_MOST_STATE = 40e9


def _size(rng, lo, hi, multiple=0):
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if multiple:
        return max(multiple, n // multiple * multiple)
    return n


def draw(rng):
    """One more case of the ranges that the listed ones stand for."""
    kind = rng.choice(["step", "step", "step", "batch", "init", "corrected", "mlp", "pair"])
    while True:
        if kind == "step":
            precision = rng.choice([FP64, FP64, FP32, BF16])
            option = rng.choice(["", "", "", "inplace", "gradients", "spring_shift", "qe2"])
            if precision == BF16 and option in ("inplace", "gradients", "spring_shift"):
                option = ""
            inplace = int(option == "inplace")
            nx = _size(rng, 64, 1024, 64) if inplace else _size(rng, 16, 1100)
            ny = _size(rng, 16, 1100)
            nq = rng.choice([6, 8, 10, 12, 16])
            c = _step("", nx, ny, nq, precision, 2 * rng.randint(1, 10),
                      periods=max(1, round(ny / 256)), Re=rng.uniform(15.0, 60.0),
                      Wi=rng.uniform(0.4, 1.2), beta=rng.uniform(0.6, 0.85), inplace=inplace,
                      gradients=int(option == "gradients"),
                      spring_shift=int(option == "spring_shift"),
                      qe_model=2 if option == "qe2" else 1,
                      observe=rng.choice(["amplitude", "amplitude", "diagnostics"]))
            if _state_bytes(c) > _MOST_STATE:
                continue
        elif kind == "batch":
            if rng.random() < 0.4:
                c = dict(kind="batch", set="cells", count=rng.randint(1, 3), first=0,
                         nq=rng.choice([16, 20, 24, 32]), precision=FP64,
                         steps=rng.randint(5, 40), diagnostics=True, pre_steps=100)
            else:
                c = dict(kind="batch", set="sweep", count=rng.randint(2, 40),
                         first=rng.choice([0, 8, 16, 64, 100]), nq=rng.choice([6, 6, 8]),
                         precision=FP32, steps=rng.randint(2, 12), diagnostics=False,
                         pre_steps=100)
        elif kind == "init":
            ny = _size(rng, 32, 1024)
            c = dict(kind="init", nx=_size(rng, 16, 512), ny=ny, nq=rng.choice([6, 8, 12, 16]),
                     precision=rng.choice([FP64, FP32]), periods=max(1, round(ny / 256)),
                     Re=rng.uniform(15.0, 60.0), Wi=rng.uniform(0.4, 1.2),
                     beta=rng.uniform(0.6, 0.85), perturbation=1e-4,
                     pre_steps=rng.randint(200, 1500))
        elif kind == "corrected":
            n = _size(rng, 96, 320)
            c = dict(kind="corrected", nx=n, ny=_size(rng, 128, 320), nq=8, periods=2,
                     Re=rng.uniform(20.0, 60.0), Wi=rng.uniform(0.4, 1.2), beta=0.7,
                     steps=rng.randint(2, 20))
        elif kind == "mlp":
            c = dict(kind="mlp", op=rng.choice(["train", "grads", "forward"]),
                     rows=_size(rng, 1000, 150000), nin=rng.choice([54, 54, 54, 33]),
                     nout=rng.choice([5, 5, 5, 9]))
        else:
            m = rng.choice([2, 4])
            n = _size(rng, 64, 256, 2)
            c = dict(kind="pair", nx=m * n, ny=m * _size(rng, 96, 256, 2), factor=m, nq=8,
                     periods=2, Re=rng.uniform(20.0, 60.0), Wi=rng.uniform(0.4, 1.2), beta=0.7,
                     steps=rng.randint(1, 8))
        if work(c)["bytes"] <= _MOST_BYTES:
            c.pop("name", None)
            return c


# ---------------------------------------------------------------------------
# What a user's program has in hand, and one pass.

def _params(c, **more):
    d = dict(nq=c["nq"], pre_steps=c.get("pre_steps", 300), precision=c.get("precision", FP64))
    for k in ("inplace", "gradients", "spring_shift", "qe_model"):
        if c.get(k):
            d[k] = c[k]
    d.update(more)
    if d.get("qe_model") == 2:
        d.update(tau_ratio_p=0.5)
    return d


def _context(c, **more):
    return P.Tpl(c["nx"], c["ny"], c["Re"], c["Wi"], c["beta"], periods=c["periods"],
                 **_params(c, **more))


def _instances(c, seed):
    if c["set"] == "cells":  # the paper's cells: Re 3.5, beta 0.5, Wi 0.1 / 2.5 / 5
        return [dict(nx=72, ny=72, periods=4, Re=3.5, beta=0.5, u0=0.01, Wi=w, seed=seed + i,
                     perturbation=1e-3) for i, w in enumerate((2.5, 0.1, 5.0)[:c["count"]])]
    # the sweep's instances, without the two (62, 214) that diverge
    out = [d for i, d in enumerate(inputs.c4_instances(c["first"] + c["count"] + 2))
           if i not in (62, 214)]
    return [dict(d, seed=seed + i) for i, d in
            enumerate(out[c["first"]:c["first"] + c["count"]])]


def _observed(n):
    return torch.empty((P.TPL_NFIELDS, n), dtype=torch.float64, device="cuda")


class _Lattice:
    """One context whose state lives in torch tensors (tpl_adopt_buffers)."""

    def __init__(self, c, seed):
        self.c = c
        t = self.t = _context(c)
        sizes = [int(t.query(k)) for k in ("bytes_XS", "bytes_XP", "bytes_PSI", "bytes_FLD")]
        self.bufs = [torch.empty(n, dtype=torch.uint8, device="cuda") for n in sizes]
        t.adopt_buffers([b.data_ptr() for b in self.bufs], sizes)
        t.init(seed=seed, perturbation=c["perturbation"])
        self.steps = 24 if c["inplace"] else 2
        t.step(self.steps)  # past the first call's choice of a launch shape
        self.obs = _observed(c["nx"] * c["ny"])

    def state(self):
        """The current solvent and polymer populations and psi, as stored."""
        c, nqd, h = self.c, self.t.nqd, self.steps & 1
        real = torch.float64 if c["precision"] == FP64 else torch.float32
        pops = torch.bfloat16 if c["precision"] == BF16 else real
        shape = (c["ny"], c["nx"])
        ip = bool(c["inplace"])
        xs = self.bufs[0].view(real).view(1 if ip else 2, 9, *shape)[0 if ip else h]
        xp = self.bufs[1].view(pops).view(1 if ip else 2, -1, nqd, *shape)[0 if ip else h]
        psi = self.bufs[2].view(real).view(2, nqd, *shape)[h]
        # the BF16 form's planes 0 and 25 are the two halves of FP32 values
        return xs, (xp[1:25] if c["precision"] == BF16 else xp), psi


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "step":
        return dict(case=c, lattice=_Lattice(c, seed))
    if kind == "batch":
        insts = _instances(c, seed)
        b = P.Batch(insts, precision=c["precision"], nq=c["nq"], pre_steps=c["pre_steps"])
        b.init()
        b.step(2)
        ns = [d["nx"] * d["ny"] for d in insts]
        return dict(case=c, batch=b, insts=[b.instance(i) for i in range(len(ns))],
                    obs=[_observed(n) for n in ns])
    if kind == "init":
        return dict(case=c, t=_context(c), seed=seed, obs=_observed(c["nx"] * c["ny"]))
    if kind == "corrected":
        t = _context(dict(c, perturbation=1e-2))
        t.init(seed=seed, perturbation=1e-2)
        n = c["nx"] * c["ny"]
        x = torch.empty((2, n, 54), dtype=torch.float32, device="cuda")
        for snapshot in x:
            t.step(_APART)
            t.features_device(snapshot.data_ptr(), snapshot.numel())
        net = P.Mlp(54, 64, 5, seed=seed)
        net.set_norm(*_norms(x))
        t.attach(net, 0.05)
        t.step(2)
        return dict(case=c, t=t, net=net, obs=_observed(n))
    if kind == "mlp":
        g = torch.Generator(device="cuda").manual_seed(seed)
        x, y, scale, shift = _mlp_data(c, g)
        net = P.Mlp(c["nin"], 64, c["nout"], seed=seed)
        net.set_norm(shift.cpu().numpy(), scale.cpu().numpy(),
                     *(v.cpu().numpy() for v in (y.mean(0), y.std(0))))
        return dict(case=c, net=net, x=x, y=y, out=torch.empty_like(y))
    fine = _context(c)
    fine.init(seed=seed, perturbation=1e-2)
    m = c["factor"]
    small = dict(c, nx=c["nx"] // m, ny=c["ny"] // m)
    coarse = [_context(small, pre_steps=0) for _ in range(2)]
    for t in coarse:
        t.init(0, 0.0)
    n = small["nx"] * small["ny"]
    return dict(case=c, fine=fine, a=coarse[0], b=coarse[1], obs=_observed(n),
                X=torch.empty((n, 54), dtype=torch.float32, device="cuda"),
                T=torch.empty((n, 5), dtype=torch.float32, device="cuda"))


_APART = 50  # coarse steps between the snapshots that the inputs' statistics come from


def _norms(x):
    """Input statistics of the snapshots; outputs of the size of a coarse
    lattice's error per step."""
    xm, xs, _, _ = standardisation(torch, x, x[..., :5])
    return xm, xs, np.zeros(5), np.array([1e-8, 1e-8, 1e-9, 1e-9, 1e-9])


def _mlp_data(c, g):
    """Snapshot-like inputs: offset, correlated fields of different scales."""
    dev, n = g.device, c["rows"]
    base = torch.randn((n, 6), generator=g, device=dev, dtype=torch.float32)
    mix = torch.randn((6, c["nin"]), generator=g, device=dev, dtype=torch.float32) / 6 ** 0.5
    z = base @ mix + 0.3 * torch.randn((n, c["nin"]), generator=g, device=dev,
                                       dtype=torch.float32)
    scale = torch.exp(torch.rand(c["nin"], generator=g, device=dev) * 4 - 4)
    shift = torch.randn(c["nin"], generator=g, device=dev)
    proj = torch.randn((c["nin"], c["nout"]), generator=g, device=dev) / c["nin"] ** 0.5
    y = 1e-4 * torch.tanh(z @ proj) + 2e-5 * torch.randn((n, c["nout"]), generator=g, device=dev)
    return (z * scale + shift).contiguous(), y.contiguous(), scale, shift


_DIAG = ("mass_S", "mass_P", "mom_x", "mom_y", "amplitude", "enstrophy", "qrms", "min_psi")


def _diag(t):
    d = t.diagnostics()
    return np.array([d[k] for k in _DIAG])


def run(state):
    c, kind = state["case"], state["case"]["kind"]
    if kind == "step":
        s = state["lattice"]
        s.t.step(c["steps"])
        s.steps += c["steps"]
        seen = _diag(s.t) if c["observe"] == "diagnostics" else s.t.amplitude()
        s.t.moments_device(s.obs.data_ptr(), s.obs.numel())
        xs, xp, psi = s.state()
        return dict(XS=xs, XP=xp, psi=psi, observables=s.obs, seen=seen)
    if kind == "batch":
        state["batch"].step(c["steps"])
        out = dict(amplitudes=state["batch"].amplitudes(), status=state["batch"].status())
        if c["diagnostics"]:
            out["diagnostics"] = np.stack([_diag(t) for t in state["insts"]])
        for t, o in zip(state["insts"], state["obs"]):
            t.moments_device(o.data_ptr(), o.numel())
        out["observables"] = state["obs"]
        return out
    if kind == "init":
        t, o = state["t"], state["obs"]
        t.init(seed=state["seed"], perturbation=c["perturbation"])
        t.moments_device(o.data_ptr(), o.numel())
        return dict(observables=o, amplitude=t.amplitude())
    if kind == "corrected":
        t, o = state["t"], state["obs"]
        t.step(c["steps"])
        t.moments_device(o.data_ptr(), o.numel())
        return dict(observables=o)
    if kind == "mlp":
        net, x, y = state["net"], state["x"], state["y"]
        if c["op"] == "train":
            loss = net.train_step(x.data_ptr(), y.data_ptr(), c["rows"], 1e-3)
            return dict(loss=loss, params=net.get_params())
        if c["op"] == "grads":
            grad, loss = net.grads(x.data_ptr(), y.data_ptr(), c["rows"])
            return dict(loss=loss, grad=grad)
        net.forward(x.data_ptr(), state["out"].data_ptr(), c["rows"])
        return dict(y=state["out"])
    a, b, X, T, o = state["a"], state["b"], state["X"], state["T"], state["obs"]
    a.restrict_from(state["fine"])
    b.restrict_from(state["fine"])
    b.moments_device(o.data_ptr(), o.numel())
    a.features_device(X.data_ptr(), X.numel())
    a.step(c["steps"])
    a.targets_device(o.data_ptr(), T.data_ptr(), T.numel())
    return dict(features=X, targets=T, observables=o)


# ---------------------------------------------------------------------------
# What a pass cannot do without.

def _disk(nq):
    r = 0.5 * nq
    return [(a + 0.5 - r, b + 0.5 - r) for b in range(nq) for a in range(nq)
            if (a + 0.5 - r) ** 2 + (b + 0.5 - r) ** 2 < r * r]


def _node_bytes(c):
    """Populations and recorded psi of one r-node, stored once."""
    nqd = len(_disk(c["nq"]))
    real, pop = {FP64: (8, 200), FP32: (4, 100), BF16: (4, 52)}[c.get("precision", FP64)]
    return 9 * real + nqd * (pop + real)


def _state_bytes(c):
    copies = 1 if c.get("inplace") else 2
    return copies * c["nx"] * c["ny"] * (_node_bytes(c) + 144)


def _step_work(c, nodes, steps):
    """Each step reads and writes every population, the recorded psi and the
    mixture velocity; same-step gradients read the populations once more
    (the neighbours' psi is needed before any node collides)."""
    nqd, b = len(_disk(c["nq"])), _node_bytes(c)
    one = 2 * b + 2 * 16 + (b if c.get("gradients") else 0)
    return dict(bytes=nodes * steps * one, flops=nodes * steps * (nqd * 300 + 300))


def work(case):
    c, kind = case, case["kind"]
    n = c.get("nx", 0) * c.get("ny", 0)
    seen = 8 * P.TPL_NFIELDS
    if kind == "step":
        w = _step_work(c, n, c["steps"])
        w["bytes"] += n * seen
        return w
    if kind == "batch":
        n = sum(d["nx"] * d["ny"] for d in _instances(c, 0))
        w = _step_work(c, n, c["steps"])
        w["bytes"] += n * seen
        return w
    if kind == "init":
        w = _step_work(dict(c, precision=FP64), c["ny"], c["pre_steps"])
        w["bytes"] += n * (2 * _node_bytes(c) + seen)
        return w
    if kind == "corrected":
        w = _step_work(c, n, c["steps"])
        w["bytes"] += n * seen
        w["flops"] += n * c["steps"] * 2 * (54 * 64 + 64 * 64 + 64 * 5)
        return w
    if kind == "mlp":
        mac = c["nin"] * 64 + 64 * 64 + 64 * c["nout"]
        f = c["rows"] * 2 * mac * (1 if c["op"] == "forward" else 3)
        return dict(bytes=4 * c["rows"] * (c["nin"] + c["nout"]), flops=f)
    nc = n // c["factor"] ** 2
    w = _step_work(c, nc, c["steps"])
    w["bytes"] += 2 * n * _node_bytes(c) + 2 * nc * _node_bytes(c) + nc * (seen + 4 * 59)
    return w


# ---------------------------------------------------------------------------
# The same outputs from plain torch in 64 bits.

_C9 = [(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)]
_W9 = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4
_CP = [(0, 0, 0, 0)]
for _a, _b in ((0, 1), (0, 2), (0, 3), (1, 2), (1, 3), (2, 3)):
    for _s, _t in ((1, 1), (1, -1), (-1, 1), (-1, -1)):
        _v = [0, 0, 0, 0]
        _v[_a], _v[_b] = _s, _t
        _CP.append(tuple(_v))
_WP = [1 / 3] + [1 / 36] * 24


class _Scheme:
    """The scheme as separate whole-array operations, fields [..., ny, nx]."""

    def __init__(self, c, nx=None, tau_ratio_p=None, u0=0.05):
        self.nx, self.ny = nx or c["nx"], c["ny"]
        self.model = c.get("qe_model") or 1
        ratio = tau_ratio_p or (0.5 if self.model == 2 else 1.0)
        nq, phi, b, cs2 = c["nq"], 0.01, 25.0, 1 / 3
        self.kf = 2 * math.pi * c["periods"] / self.ny
        l = 1 / self.kf
        nu = u0 * l / c["Re"]
        lam = c["Wi"] * l / u0
        self.G = (1 - c["beta"]) * nu / lam
        self.sigma = 0.5 * nq / math.sqrt(b)
        s2 = self.sigma ** 2
        relax, flux = 3 * c["beta"] * nu, s2 / (2 * cs2 * lam)
        if self.model == 2:
            self.t2S = self.t1S = relax
            self.t1P, self.t2P = flux, flux / ratio
            self.tJS, self.tJP = self.t1S, self.t1P
        else:
            self.t1S, self.t2S, self.t2P, self.t1P = relax, 1.0, flux, ratio * flux
            self.tJS, self.tJP = self.t2S, self.t2P
        self.DQ = cs2 * flux
        self.F0 = nu * u0 * self.kf ** 2
        self.shift, self.same = c.get("spring_shift", 0), c.get("gradients", 0)
        self.rhoS0, self.rhoP0 = 1 - phi, phi
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        disk = _disk(nq)
        at = {q: i for i, q in enumerate(disk)}
        cap = min(0.2, 2 - 2 / (2 * self.t1P + 1))
        force, weight = [], []
        for qx, qy in disk:
            r2 = qx * qx + qy * qy
            f = 1 / s2 / (1 - r2 / (b * s2))
            drift = self.DQ * f * math.sqrt(r2)
            f *= min(1.0, cap / drift)
            force.append((f * qx, f * qy))
            weight.append((1 - r2 / (b * s2)) ** (0.5 * b))
        planes = []
        for k, v in enumerate(_CP):
            star = _CP.index((v[0], v[1], -v[2], -v[3]))
            for i, (qx, qy) in enumerate(disk):
                j = at.get((qx - v[2], qy - v[3]))
                planes.append(k * len(disk) + j if j is not None else star * len(disk) + i)
        t = lambda v: torch.tensor(v, dtype=torch.float64, device=self.dev)  # noqa: E731
        self.nqd, self.disk = len(disk), disk
        self.planes = torch.tensor(planes, device=self.dev).view(25, -1)
        self.Q, self.F = t(disk).T[:, :, None, None], t(force).T[:, :, None, None]
        self.peq = t(weight)[:, None, None] / sum(weight)
        self.meq = 0.5 * float((self.peq * (self.Q * self.F).sum(0)).sum())
        self.kappa = self.G * self.tJP / (self.rhoP0 * self.meq)
        y = torch.arange(self.ny, dtype=torch.float64, device=self.dev)
        self.force = (self.F0 * torch.sin(self.kf * y))[:, None].expand(self.ny, self.nx)
        self.source = None

    def rest(self):
        one = torch.ones((self.ny, self.nx), dtype=torch.float64, device=self.dev)
        self.XS = torch.stack([w * self.rhoS0 * one for w in _W9])
        self.psi = self.rhoP0 * self.peq * one
        self.XP = torch.stack([w * self.psi for w in _WP])
        self.U = torch.zeros((2, self.ny, self.nx), dtype=torch.float64, device=self.dev)
        self.rhoS, self.rhoP = self.XS.sum(0), self.psi.sum(0)

    def d(self, f, axis):  # axis 0: x, 1: y
        return 0.5 * (torch.roll(f, -1, -1 - axis) - torch.roll(f, 1, -1 - axis))

    def spring(self, psi):
        if not self.shift:
            return self.Q[0] * self.d(psi, 0) + self.Q[1] * self.d(psi, 1)
        out = torch.empty_like(psi)
        for q, (qx, qy) in enumerate(self.disk):
            v = 0.0
            for sign in (1, -1):
                ax, ay = sign * 0.5 * qx, sign * 0.5 * qy
                ix, iy = math.floor(ax), math.floor(ay)
                fx, fy = ax - ix, ay - iy
                for jx, wx in ((ix, 1 - fx), (ix + 1, fx)):
                    for jy, wy in ((iy, 1 - fy), (iy + 1, fy)):
                        v = v + sign * wx * wy * torch.roll(psi[q], (-jy, -jx), (0, 1))
            out[q] = v
        return out

    def pull(self):
        gS = torch.stack([torch.roll(self.XS[i], (c[1], c[0]), (0, 1))
                          for i, c in enumerate(_C9)])
        flat = self.XP.view(25 * self.nqd, self.ny, self.nx)
        gP = torch.empty_like(self.XP)
        for k, v in enumerate(_CP):
            gP[k] = torch.roll(flat[self.planes[k]], (v[1], v[0]), (1, 2))
        return gS, gP

    def mixture(self, gS, rhoS, rhoP, JP, S, Fb):
        aS, aP = 1 / (2 * self.tJS + 1), 1 / (2 * self.tJP + 1)
        JS = torch.stack([sum(c[a] * gS[i] for i, c in enumerate(_C9) if c[a])
                          for a in (0, 1)])
        U = ((JS + 0.5 * Fb) * aS + (JP + S / (2 * self.tJP)) * aP) / (rhoS * aS + rhoP * aP)
        return U, JS

    def step(self):
        gS, gP = self.pull()
        Fb = torch.stack([self.force, torch.zeros_like(self.force)])
        if self.source is not None:
            Fb = Fb + self.source
        rhoS, psi = gS.sum(0), gP.sum(0)
        J = [sum(v[a] * gP[k] for k, v in enumerate(_CP) if v[a]) for a in range(4)]
        rhoP, JP = psi.sum(0), torch.stack([J[0].sum(0), J[1].sum(0)])
        psi_rec, U_rec = self.psi, self.U
        if self.same:
            psi_rec = psi
        s = self.kappa * self.spring(psi_rec)
        sx, sy = s * self.F[0], s * self.F[1]
        S = torch.stack([sx.sum(0), sy.sum(0)])
        U, JS = self.mixture(gS, rhoS, rhoP, JP, S, Fb)
        if self.same:
            U_rec = U
        K = [[self.d(U_rec[a], b) for b in (0, 1)] for a in (0, 1)]
        # solvent
        v = U + self.tJS * Fb / rhoS
        aS, aP = 1 / (2 * self.tJS + 1), 1 / (2 * self.tJP + 1)
        bS, rS = 1 / (2 * self.t1S + 1), self.t1S / self.t2S

        def quad(rho, u, i):
            cu = _C9[i][0] * u[0] + _C9[i][1] * u[1]
            return _W9[i] * rho * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * (u * u).sum(0))

        new = []
        if self.model == 2:
            pS = 1 / (2 * self.t2S + 1)
            D = [[None, None], [None, None]]
            for a in (0, 1):
                for b in (0, 1):
                    Pab = sum(c[a] * c[b] * gS[i] for i, c in enumerate(_C9) if c[a] * c[b])
                    eq = rhoS * ((1 / 3 if a == b else 0) + v[a] * v[b])
                    D[a][b] = (1 - pS) * Pab + pS * eq - (rhoS / 3 if a == b else 0)
        else:
            us = (2 * self.tJS * JS + rhoS * U + self.tJS * Fb) * aS / rhoS
        for i, c in enumerate(_C9):
            fe = quad(rhoS, v, i)
            if self.model == 2:
                h = sum(D[a][b] * (c[a] * c[b] - (1 / 3 if a == b else 0))
                        for a in (0, 1) for b in (0, 1))
                fs = _W9[i] * (rhoS + 3 * rhoS * (c[0] * v[0] + c[1] * v[1]) + 4.5 * h)
            else:
                fs = quad(rhoS, us, i)
            new.append((1 - 2 * bS) * gS[i] + 2 * bS * ((1 - rS) * fs + rS * fe))
        # polymer
        E = [psi * U[0] + sx, psi * U[1] + sy,
             psi * (K[0][0] * self.Q[0] + K[0][1] * self.Q[1] - self.DQ * self.F[0]),
             psi * (K[1][0] * self.Q[0] + K[1][1] * self.Q[1] - self.DQ * self.F[1])]
        bP, rP = 1 / (2 * self.t1P + 1), self.t1P / self.t2P
        if self.model == 2:
            pP = 1 / (2 * self.t2P + 1)
            D = {}
            for a in range(4):
                for b in range(a, 4):
                    Pab = sum(w[a] * w[b] * gP[k] for k, w in enumerate(_CP) if w[a] * w[b])
                    D[a, b] = (1 - pP) * Pab + ((pP - 1) * psi / 3 if a == b else 0)
            trace = (D[0, 0] + D[1, 1] + D[2, 2] + D[3, 3]) / 3
            A = E
        else:
            A = [(1 - rP) * (2 * self.tJP * J[a] + E[a]) * aP + rP * E[a] for a in range(4)]
        for k, w in enumerate(_CP):
            t = psi + 3 * sum(w[a] * A[a] for a in range(4) if w[a]) if any(w) else psi.clone()
            if self.model == 2:
                h = -trace
                for a in range(4):
                    for b in range(a, 4):
                        if w[a] * w[b]:
                            h = h + (1 if a == b else 2) * w[a] * w[b] * D[a, b]
                t = t + (1 - rP) * 4.5 * h
            gP[k] *= 1 - 2 * bP
            gP[k] += 2 * bP * _WP[k] * t
        self.XS, self.XP, self.psi, self.U = torch.stack(new), gP, psi, U
        self.rhoS, self.rhoP = rhoS, rhoP

    def observables(self):
        s2, m = self.sigma ** 2, self.rhoP0 * self.meq
        rows = [self.rhoS + self.rhoP, self.U[0], self.U[1], self.rhoP]
        tot = self.psi.sum(0)
        rows += [(self.psi * self.Q[a] * self.Q[b]).sum(0) / tot / s2
                 for a, b in ((0, 0), (0, 1), (1, 1))]
        rows += [self.G * ((self.psi * self.Q[a] * self.F[b]).sum(0) / m - float(a == b))
                 for a, b in ((0, 0), (0, 1), (1, 1))]
        return torch.stack(rows).view(10, -1)

    def amplitude(self, u0=0.05):
        d = self.U - self.U.mean(2, keepdim=True)
        return math.sqrt(float((d * d).sum()) / (self.nx * self.ny)) / u0

    def diagnostics(self, u0=0.05):
        w = self.d(self.U[1], 0) - self.d(self.U[0], 1)
        mom = [float(sum(c[a] * self.XS[i].sum() for i, c in enumerate(_C9)))
               + float(sum(v[a] * self.XP[k].sum() for k, v in enumerate(_CP))) for a in (0, 1)]
        q = math.sqrt(float((self.psi * (self.Q ** 2).sum(0)).sum() / self.psi.sum()))
        return np.array([float(self.rhoS.sum()), float(self.rhoP.sum()), *mom,
                         self.amplitude(u0), 0.5 * float((w * w).sum()),
                         q / (self.sigma * 5.0), float(self.psi.min())])


def _started(c, seed, perturbation, **kw):
    """tpl_init: the column's forced state on every column, perturbed."""
    col = _Scheme(c, nx=1, **kw)
    col.rest()
    for _ in range(c.get("pre_steps", 300)):
        col.step()
    s = _Scheme(c, **kw)
    for name in ("XS", "XP", "psi", "U", "rhoS", "rhoP"):
        v = getattr(col, name)
        setattr(s, name, v.expand(*v.shape[:-1], s.nx).contiguous())
    gen = inputs.splitmix64(seed)
    u01 = lambda: inputs.uniform01(gen)  # noqa: E731
    X = torch.arange(s.nx, dtype=torch.float64, device=s.dev)[None, :]
    Y = torch.arange(s.ny, dtype=torch.float64, device=s.dev)[:, None]
    du = torch.zeros_like(s.U)
    for kx in range(-8, 9):
        if not kx:
            continue
        for ky in range(-8, 9):
            r1, r2, r3 = u01(), u01(), u01()
            a = math.sqrt(-2 * math.log(1 - r1)) * math.cos(2 * math.pi * r2)
            th = 2 * math.pi * (kx * X / s.nx + ky * Y / s.ny) + 2 * math.pi * r3
            du[0] -= a * torch.sin(th) * (2 * math.pi * ky / s.ny)
            du[1] += a * torch.sin(th) * (2 * math.pi * kx / s.nx)
    du *= perturbation * kw.get("u0", 0.05) / math.sqrt(float((du * du).sum(0).mean()))
    rho = s.XS.sum(0)
    for i, e in enumerate(_C9):
        s.XS[i] += 3 * _W9[i] * rho * (e[0] * du[0] + e[1] * du[1])
    pop = s.XP.sum(0)
    for k, v in enumerate(_CP):
        if v[0] or v[1]:
            s.XP[k] += 3 / 36 * pop * (v[0] * du[0] + v[1] * du[1])
    s.U = s.U + du
    return s, col


def _features(s):
    o = s.observables().float().view(10, s.ny, s.nx)[[0, 1, 2, 4, 5, 6]]
    cols = [torch.roll(o, (-dy, -dx), (1, 2)) for dy in (-1, 0, 1) for dx in (-1, 0, 1)]
    return torch.stack(cols).view(54, -1).T.contiguous()


def _net64(theta, x, nin, nout):
    """The network on standardised inputs, from the flat parameters."""
    at, parts = 0, []
    for shape in ((64, nin), (64,), (64, 64), (64,), (nout, 64), (nout,)):
        n = math.prod(shape)
        parts.append(theta[at:at + n].view(*shape))
        at += n
    h = torch.nn.functional.gelu(x @ parts[0].T + parts[1])
    h = torch.nn.functional.gelu(h @ parts[2].T + parts[3])
    return h @ parts[4].T + parts[5]


def _theta0(nin, nout, seed):
    gen = inputs.splitmix64(seed)
    out = []
    for rows, fan in ((64, nin), (64, 64), (nout, 64)):
        a = 1 / math.sqrt(fan)
        out += [np.float32(a * (2 * inputs.uniform01(gen) - 1)) for _ in range(rows * fan)]
        out += [np.float32(0)] * rows
    return torch.tensor(np.array(out, dtype=np.float64))


def _restricted(f, m):
    """Full weighting: coarse node (X, Y) averages fine nodes around (mX, mY)."""
    h, out = m // 2, 0.0
    for j in range(-h, h + 1):
        for i in range(-h, h + 1):
            w = (0.5 if abs(j) == h else 1.0) * (0.5 if abs(i) == h else 1.0)
            out = out + w * torch.roll(f, (-j, -i), (-2, -1))[..., ::m, ::m]
    return out / (m * m)


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "step":
        s, col = _started(c, seed, c["perturbation"])
        for _ in range((24 if c["inplace"] else 2) + c["steps"]):
            s.step()
        seen = s.diagnostics() if c["observe"] == "diagnostics" else s.amplitude()
        obs = s.observables()
        if c["precision"] == FP64:
            return dict(XS=s.XS, XP=s.XP, psi=s.psi, observables=obs, seen=seen)
        # stored as deviations from the base state rounded to FP32
        for name in ("XS", "XP", "psi"):
            v = getattr(s, name)
            v -= getattr(col, name).float().double()
        xp = s.XP[1:] if c["precision"] == BF16 else s.XP
        return dict(XS=s.XS, XP=xp, psi=s.psi, observables=obs, seen=seen)
    if kind == "batch":
        insts = _instances(c, seed)
        if sum(d["nx"] * d["ny"] for d in insts) * c["steps"] * len(_disk(c["nq"])) > 3e9:
            return None
        out = dict(amplitudes=[], status=None, diagnostics=[], observables=[])
        for d in insts:
            s, _ = _started(dict(c, **{k: d[k] for k in ("nx", "ny", "periods", "Re", "Wi",
                                                        "beta")}), d["seed"], d["perturbation"],
                            u0=d["u0"])
            for _ in range(2 + c["steps"]):
                s.step()
            out["amplitudes"].append(s.amplitude(d["u0"]))
            out["diagnostics"].append(s.diagnostics(d["u0"]))
            out["observables"].append(s.observables())
        out["amplitudes"] = np.array(out["amplitudes"])
        out["diagnostics"] = np.stack(out["diagnostics"]) if c["diagnostics"] else None
        return out
    if kind == "init":
        s, _ = _started(c, seed, c["perturbation"])
        return dict(observables=s.observables(), amplitude=s.amplitude())
    if kind == "corrected":
        s, _ = _started(c, seed, 1e-2)
        seen = []
        for _ in range(2):
            for _ in range(_APART):
                s.step()
            seen.append(_features(s))
        xm, xs, ym, ys = (torch.tensor(np.float32(v), device=s.dev)
                          for v in _norms(torch.stack(seen)))
        theta = _theta0(54, 5, seed).to(s.dev)
        for _ in range(2 + c["steps"]):
            x = ((_features(s) - xm) / xs).double()
            y = (_net64(theta, x, 54, 5) * ys.double() + ym.double()).T.view(5, s.ny, s.nx)
            mean = y[:2].mean((1, 2), keepdim=True)
            s.source = torch.stack([y[0] + s.d(y[2], 0) + s.d(y[3], 1),
                                    y[1] + s.d(y[3], 0) + s.d(y[4], 1)]) - mean
            s.step()
        return dict(observables=s.observables())
    if kind == "mlp":
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        x, y, scale, shift = _mlp_data(c, torch.Generator(device=dev).manual_seed(seed))
        ym, ys = y.mean(0), y.std(0)
        z, t = ((x - shift) / scale).double(), ((y.double() - ym.double()) / ys.double())
        theta = _theta0(c["nin"], c["nout"], seed).to(dev).requires_grad_(True)
        o = _net64(theta, z, c["nin"], c["nout"])
        if c["op"] == "forward":
            return dict(y=o.detach() * ys.double() + ym.double())
        loss = ((o - t) ** 2).mean()
        g, = torch.autograd.grad(loss, theta)
        if c["op"] == "grads":
            return dict(loss=loss.item(), grad=g)
        # one Adam step from zero moments
        new = theta.detach() - 1e-3 * g / (g.abs() + 1e-8)
        return dict(loss=loss.item(), params=new)
    m = c["factor"]
    s, _ = _started(c, seed, 1e-2)
    small = dict(c, nx=c["nx"] // m, ny=c["ny"] // m)
    r = _Scheme(small)
    for name in ("XS", "psi", "U"):
        setattr(r, name, _restricted(getattr(s, name), m))
    r.XP = torch.stack([_restricted(v, m) for v in s.XP])
    r.rhoS, r.rhoP = r.XS.sum(0), r.XP.sum((0, 1))
    obs, feat = r.observables(), _features(r)
    for _ in range(c["steps"]):
        r.step()
    after = r.observables()

    def stress(o):
        return torch.stack([o[0] * o[1], o[0] * o[2], o[7], o[8], o[9]]).T

    return dict(features=feat, targets=stress(obs) - stress(after), observables=obs)
