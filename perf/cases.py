"""The work that programs have this library do, as cases to be timed: LB steps
of single boxes, batches and semidilute solutions, the sampling loop of a
production run, an adjoint window under autograd, and a checkpoint.

A case is a dict of plain values:
  work       "steps"       step(steps), then a frame of the trajectory (the bead positions)
             "fluid"       step(steps), then the observables (mode variances of a fluid)
             "sample"      step(steps), then observables, bead positions and velocities
             "window"      adjoint.LBWindow over T steps and its backward pass
             "checkpoint"  the whole state exported and imported again
  boxes      boxes in the batch; box b has the Philox key (seed, b)
  L, N       edge and beads of every box; L = 0: each box draws its own from
             {16, 24, 32, 48, 64} and {8, 16, 32, 64}, N <= L
  chain_len  beads per chain (0: one chain of N beads)
  fluid      "lj" (kT = 1e-4, 10 MD substeps a step), "warm" (kT = 1e-2, rates
             1.25 / 0.8 / 1.4) or "paper" (Sec. II.E of arXiv:0903.5067: kT =
             1.2, 2 MD substeps)
  therm      modes thermalized: 0 none, 1 stress, 2 all
  fp64       populations in FP64 (else FP32 deviations)
  steps      LB steps of one pass; graph: steps per HIP graph (0: direct launches)
  warm       LB steps taken in prepare(), from the fluid at rest
  T, k       window length and checkpoint interval ("window")

Outputs are the whole updated state (populations and beads, as views of the
buffers that the caller of the library owns) and whatever the calls return.
exact() is an independent statement of the method in FP64 torch operations.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_0903_5067_amd as lbm
from paper_0903_5067_amd import adjoint

SQRT12 = 3.4641016151377544
FLUIDS = {
    "lj": dict(rho0=1.0, omega_s=1.0, omega_b=1.0, omega_g=1.0, kT=1e-4, tau_lb=0.1, md_dt=0.01, md_substeps=10,
               mass=1.0, zeta=20.0, k_fene=30.0, r0_fene=1.5, eps_wca=1.0, sigma_wca=1.0),
    "paper": dict(rho0=0.864, omega_s=1.0 / (3.0 * 2.8 * 0.02 + 0.5), omega_b=1.0 / (3.0 * 2.8 * 0.02 + 0.5),
                  omega_g=1.0, kT=1.2, tau_lb=0.02, md_dt=0.01, md_substeps=2, mass=1.0, zeta=20.8, k_fene=7.0,
                  r0_fene=2.0, eps_wca=1.0, sigma_wca=1.0),
}
FLUIDS["warm"] = dict(FLUIDS["lj"], kT=1e-2, omega_s=1.25, omega_b=0.8, omega_g=1.4)


def _case(work, boxes, L, N, fluid="lj", chain_len=0, therm=2, fp64=False, steps=20, graph=20, warm=20, T=0, k=0):
    return dict(work=work, boxes=boxes, L=L, N=N, chain_len=chain_len, fluid=fluid, therm=therm, fp64=fp64,
                steps=steps, graph=graph, warm=warm, T=T, k=k)


def listed():
    return [
        # the smallest box: a first run or a convergence check in FP64, where launches and latency count
        dict(name="small_fp64", **_case("steps", 1, 16, 16, fp64=True)),
        # mode variances of a fluid-only box, sampled every step: one collide and one pass of sums per call
        dict(name="fluid_modes", **_case("fluid", 1, 64, 0, fluid="warm", steps=1, graph=0)),
        # one 64-bead chain in a 64^3 box: bound by the chain's serial substeps
        dict(name="single_chain", **_case("steps", 1, 64, 64)),
        # production loop of the single-chain study: 128 boxes advanced one LJ time, then sampled
        dict(name="ensemble_sample", **_case("sample", 128, 15, 32, fluid="paper", steps=50, graph=50)),
        # finite-size sweep: 256 boxes of uneven size in one batch
        dict(name="sweep", **_case("steps", 256, 0, 0)),
        # a 512-bead chain in a box of ordinary size, steps launched directly
        dict(name="long_chain", **_case("steps", 1, 96, 512, graph=0)),
        # semidilute solution: 64 boxes of 32 chains of 32 beads, above the overlap concentration
        dict(name="semidilute", **_case("steps", 64, 20, 1024, fluid="paper", chain_len=32)),
        # the largest single box, 1024-bead chain, bound by HBM
        dict(name="large_box", **_case("steps", 1, 256, 1024)),
        # the same box in FP64 storage
        dict(name="large_box_fp64", **_case("steps", 1, 256, 1024, fp64=True, steps=10, graph=10)),
        # gradient of a velocity-autocorrelation loss over a 200-step window
        dict(name="window", **_case("window", 1, 32, 32, steps=0, graph=0, T=200, k=20)),
        # checkpoint of a 64^3 box and resume from it
        dict(name="checkpoint", **_case("checkpoint", 1, 64, 64, steps=0, graph=0)),
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["single", "single", "fluid", "sample", "batch", "sweep", "long", "semidilute", "large",
                       "window", "checkpoint"])
    therm = rng.choice([2, 2, 2, 1])
    fp64 = rng.random() < 0.3
    graph = rng.choice([0, 20])
    steps = 2 * _spread(rng, 1, 20)
    warm = 2 * rng.randint(5, 12)
    if kind == "single":
        L = _spread(rng, 10, 120)
        return _case("steps", 1, L, min(_spread(rng, 4, 256), L * L // 4), therm=therm, fp64=fp64, steps=steps,
                     graph=graph, warm=warm)
    if kind == "fluid":
        return _case("fluid", 1, _spread(rng, 16, 160), 0, fluid="warm", therm=therm, fp64=fp64,
                     steps=rng.choice([1, 2, 10]), graph=0, warm=warm)
    if kind == "sample":
        return _case("sample", _spread(rng, 8, 128), rng.randint(10, 25), rng.choice([16, 24, 32, 33]),
                     fluid="paper", therm=therm, steps=50, graph=50, warm=warm)
    if kind == "batch":
        L = _spread(rng, 10, 40)
        return _case("steps", _spread(rng, 2, 128), L, min(_spread(rng, 4, 128), L * L // 4),
                     therm=therm, fp64=fp64, steps=steps, graph=graph, warm=warm)
    if kind == "sweep":
        return _case("steps", _spread(rng, 16, 256), 0, 0, therm=therm, steps=20, graph=20, warm=warm)
    if kind == "long":
        return _case("steps", 1, _spread(rng, 40, 160), rng.randint(257, 1024), therm=therm, fp64=fp64, steps=steps,
                     graph=graph, warm=warm)
    if kind == "semidilute":
        n, M = rng.choice([(16, rng.randint(20, 60)), (32, rng.randint(12, 32)), (64, rng.randint(6, 16))])
        return _case("steps", _spread(rng, 4, 64), rng.randint(16, 24), n * M, fluid="paper", chain_len=n,
                     therm=therm, fp64=fp64, steps=20, graph=graph, warm=warm)
    if kind == "large":
        return _case("steps", 1, _spread(rng, 128, 240), rng.choice([0, 64, 300, 1000]), therm=therm, fp64=fp64,
                     steps=10, graph=rng.choice([0, 10]), warm=10)
    if kind == "window":
        L = rng.randint(12, 36)
        T = rng.randint(40, 160)
        return _case("window", rng.choice([1, 1, 2]), L, rng.choice([8, 20, 32, 64]), therm=therm, fp64=fp64,
                     steps=0, graph=0, warm=warm, T=T, k=rng.randint(8, 24))
    L = _spread(rng, 12, 72)
    return _case("checkpoint", 1, L, min(_spread(rng, 4, 200), L * L // 4), therm=therm, fp64=fp64, steps=0, graph=0,
                 warm=warm)


# ------------------------------------------------------------------- inputs
def _sizes(case, seed):
    if case["L"]:
        return [(case["L"], case["N"])] * case["boxes"]
    # the same table for every seed, as a study has one: only the chains and the noise differ
    rng = np.random.default_rng([3, case["boxes"]])
    Ls = rng.choice([16, 24, 32, 48, 64], size=case["boxes"])
    return [(int(L), int(rng.choice([n for n in (8, 16, 32, 64) if n <= L]))) for L in Ls]


def _boxes(case, seed):
    return [dict(FLUIDS[case["fluid"]], L=L, N=N, chain_len=case["chain_len"] if N else 0, therm=case["therm"],
                 seed=int(seed) & 0x7FFFFFFF, box_id=b) for b, (L, N) in enumerate(_sizes(case, seed))]


def _walks(n_boxes, N, n, L, gen, dev, bond=0.97, near=0.9):
    """Self-avoiding walks, n_boxes boxes side by side, float64 [n_boxes, N, 3]: a box's
    beads form chains of n, bond 0.97, no two beads closer than 0.9 (minimum image).  A
    single chain starts at the box centre, one of several at a uniform random point; a
    chain that cannot grow takes back its last eight beads."""
    x = torch.zeros(n_boxes, N, 3, dtype=torch.float64, device=dev)
    row, bead, tries = torch.arange(n_boxes, device=dev), torch.arange(N, device=dev), 24
    at = torch.zeros(n_boxes, dtype=torch.int64, device=dev)       # beads placed
    failed = torch.zeros_like(at)
    for _ in range(40 * N):
        k = at.clamp(max=N - 1)
        d = torch.randn(n_boxes, tries, 3, dtype=torch.float64, device=dev, generator=gen)
        start = L * torch.rand(n_boxes, tries, 3, dtype=torch.float64, device=dev, generator=gen) if n < N else \
            torch.full_like(d, 0.5 * L)
        grown = x[row, (k - 1).clamp(min=0), None] + bond * d / d.norm(dim=-1, keepdim=True)
        cand = torch.where((k % n == 0)[:, None, None], start, grown)
        r = cand[:, :, None] - x[:, None]
        r2 = (r - L * torch.round(r / L)).square().sum(-1).masked_fill_((bead >= k[:, None])[:, None], 4.0)
        ok = r2.amin(-1) >= near * near
        put = ok.any(1) & (at < N)
        x[row, k] = torch.where(put[:, None], cand[row, ok.to(torch.int8).argmax(1)], x[row, k])
        failed = torch.where(put, torch.zeros_like(failed), failed + 1)
        at = torch.where(put, at + 1, torch.where((failed % 8 == 7) & (at < N), torch.maximum(at - 8, at // n * n), at))
        if bool((at >= N).all()):
            return x
    raise RuntimeError("the walks could not be grown")


def _chains(case, seed):
    """Initial beads of all boxes in order, float64 [sum N, 3] on the host, or None."""
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    sizes = _sizes(case, seed)
    parts = [None] * len(sizes)
    for L, N in sorted(set(sizes)):
        at = [b for b, s in enumerate(sizes) if s == (L, N)]
        got = _walks(len(at), N, case["chain_len"] or N, L, gen, dev).cpu().numpy() if N else None
        for j, b in enumerate(at):
            parts[b] = got[j] if N else np.zeros((0, 3))
    x = np.concatenate(parts)
    return x if len(x) else None


def _theta(case, seed):
    """(omega_shear, omega_bulk, zeta) per box, a little off the fluid's own, and the VACF aimed at."""
    rng = np.random.default_rng([int(seed), 7])
    p = FLUIDS[case["fluid"]]
    th = np.array([[p["omega_s"], p["omega_b"], p["zeta"]]] * case["boxes"]) * rng.uniform(0.9, 1.1, (case["boxes"], 3))
    target = 3.0 * p["kT"] * np.exp(-0.2 * np.arange(min(20, case["T"] // 2)))
    return torch.from_numpy(th), torch.from_numpy(target)


def prepare(case, seed):
    boxes = _boxes(case, seed)
    s = lbm.LBSystem(boxes, precision=lbm.FP64 if case["fp64"] else lbm.FP32_DEV, bead_x0=_chains(case, seed),
                     hist_steps=1 if case["work"] == "sample" else 0)
    if case["work"] != "window":
        s.set_launch(batched=True, graph_steps=case["graph"])
    s.step(case["warm"])
    s.synchronize()
    st = {"case": case, "s": s, "taken": case["warm"]}
    if case["work"] == "window":
        st["theta"], st["target"] = _theta(case, seed)
        s.window_forward(case["T"], case["k"])      # the workspace that such a program keeps
        s.window_rewind()
    else:
        st["out"] = [_views(s, 0), _views(s, 1)]
    return st


def _views(s, which):
    """The state buffer's arrays: two population buffers (the current one is
    `which`), then bead x, v, F and coupling force, each 256-byte aligned."""
    esz, dt = (8, torch.float64) if s.precision == lbm.FP64 else (4, torch.float32)
    elems = sum(-(-int(b["L"]) ** 3 // 1024) * 19 * 1024 for b in s.boxes)
    up = lambda v: (v + 255) // 256 * 256  # noqa: E731
    at = which * up(elems * esz)
    out = {"pops": s.state[at:at + elems * esz].view(dt)}
    at = 2 * up(elems * esz)
    for key in ("x", "v", "f", "fc") if s.n_beads else ():
        out[key] = s.state[at:at + 24 * s.n_beads].view(torch.float64).view(-1, 3)
        at += up(24 * s.n_beads)
    return out


def run(st):
    case, s = st["case"], st["s"]
    work = case["work"]
    if work == "window":
        theta = st["theta"].clone().requires_grad_(True)
        vh = adjoint.LBWindow.apply(theta, s, case["T"], case["k"])
        loss = adjoint.vacf_loss(vh, st["target"])
        loss.backward()
        s.window_rewind()               # the next pass of a fit starts from the same state
        return {"v": vh.detach(), "loss": loss.detach(), "grad": theta.grad}
    if work == "checkpoint":
        saved = s.export_state()
        s.import_state(saved)
        return {"n": [b["n"] for b in saved["boxes"]], "step": saved["step"],
                "beads": [{k: b[k] for k in ("x", "v", "f", "fc")} for b in saved["boxes"]]}
    s.step(case["steps"])
    st["taken"] += case["steps"]
    out = dict(st["out"][st["taken"] & 1])
    if work == "steps":
        if s.n_beads:
            out["at_x"] = s.bead_positions()
        return out
    obs = s.observables()
    for key in ("mass", "neg", "mode_sq", "com", "rg2", "re2")[:6 if work == "sample" else 3]:
        out["obs_" + key] = np.array([o[key] for o in obs])
    if work == "sample":
        out["at_x"] = s.bead_positions()
        out["at_v"] = s.velocity_history(obs[0]["step"] - 1)
    return out


def work(case):
    """Bytes: every population read once and written once in each LB step (38
    values a node), once read for sums, once read and written as FP64 for a
    checkpoint; in a window a step takes the forward, its replay with the
    store, and the reverse (read the state, read and write the FP64 adjoint).
    Flops: ~300 a node for the collision, ~400 for its adjoint, ~350 a bead
    and MD substep."""
    nodes = sum(L ** 3 for L, _ in _sizes(case, 0))
    beads = sum(N for _, N in _sizes(case, 0))
    esz = 8 if case["fp64"] else 4
    sub = FLUIDS[case["fluid"]]["md_substeps"]
    if case["work"] == "window":
        return {"bytes": case["T"] * nodes * 19 * (5.0 * esz + 16.0),
                "flops": case["T"] * (nodes * 1000.0 + beads * sub * 1200.0)}
    if case["work"] == "checkpoint":
        return {"bytes": nodes * 19 * (2.0 * esz + 16.0), "flops": nodes * 38.0}
    passes = case["steps"] * 38.0 + (0.0 if case["work"] == "steps" else 19.0)
    return {"bytes": nodes * passes * esz + case["steps"] * beads * 192.0,
            "flops": case["steps"] * (nodes * 300.0 + beads * sub * 350.0)}


# ---------------------------------------------------- the method in 64 bits
C = np.array([[0, 0, 0], [1, 0, 0], [-1, 0, 0], [0, 1, 0], [0, -1, 0], [0, 0, 1], [0, 0, -1],
              [1, 1, 0], [1, -1, 0], [-1, 1, 0], [-1, -1, 0], [1, 0, 1], [1, 0, -1], [-1, 0, 1], [-1, 0, -1],
              [0, 1, 1], [0, 1, -1], [0, -1, 1], [0, -1, -1]])


def _modes():
    """Mode matrix [19, 19] (mass, momentum, bulk, five shear, nine ghost), norms and weights."""
    x, y, z = C.T.astype(float)
    c2 = x * x + y * y + z * z
    w = np.where(c2 == 0, 1 / 3, np.where(c2 == 1, 1 / 18, 1 / 36))
    e = np.stack([np.ones(19), x, y, z, c2 - 1, 3 * x * x - c2, y * y - z * z, x * y, y * z, x * z,
                  (3 * c2 - 5) * x, (3 * c2 - 5) * y, (3 * c2 - 5) * z, (y * y - z * z) * x, (z * z - x * x) * y,
                  (x * x - y * y) * z, 3 * c2 * c2 - 6 * c2 + 1, (2 * c2 - 3) * (3 * x * x - c2),
                  (2 * c2 - 3) * (y * y - z * z)])
    return e, (w * e * e).sum(1), w


def _philox(c, k0, k1):
    """Philox4x32-10 of counters c (four int64 tensors of 32-bit words)."""
    m32 = 0xFFFFFFFF
    c = list(c)
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & m32) ^ c[1] ^ k0, p1 & m32, ((p0 >> 32) & m32) ^ c[3] ^ k1, p0 & m32]
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    return c


def _unit(w):
    """Unit-variance uniform variate of the top 24 bits of a word."""
    return (((w >> 8) * 2 + 1 - (1 << 24)).to(torch.float64)) * (SQRT12 * 2.0 ** -25)


class _Reference:
    """All boxes of a case in FP64: deviations p [19, nodes] as collided (not
    yet moved), beads x, v, f, fc [boxes, most beads, 3]."""

    def __init__(self, case, seed):
        self.dev = dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
        self.case, self.par = case, FLUIDS[case["fluid"]]
        self.sizes, self.seed = _sizes(case, seed), int(seed) & 0x7FFFFFFF
        i64 = lambda v: torch.as_tensor(v, dtype=torch.int64, device=dev)  # noqa: E731
        Ls, Ns = [s[0] for s in self.sizes], [s[1] for s in self.sizes]
        V = i64([L ** 3 for L in Ls])
        self.off = torch.cumsum(V, 0) - V
        box = torch.repeat_interleave(i64(range(len(Ls))), V)
        self.box = box.to(torch.int32)
        self.local = (torch.arange(int(V.sum()), device=dev) - self.off[box]).to(torch.int32)
        self.L = i64(Ls)
        self.c = i64(C)
        e, b, w = _modes()
        f64 = lambda v: torch.as_tensor(v, dtype=torch.float64, device=dev)  # noqa: E731
        self.e, self.b, self.w = f64(e), f64(b), f64(w)
        self.p = torch.zeros(19, int(V.sum()), dtype=torch.float64, device=dev)
        self.nb, self.nmax = Ns, max(Ns)
        self.t = 0
        th = [self.par["omega_s"], self.par["omega_b"], self.par["zeta"]]
        self.theta = f64([th] * len(Ls))
        if self.nmax:
            x0 = _chains(case, seed)
            x = np.zeros((len(Ls), self.nmax, 3))
            x += np.arange(self.nmax)[None, :, None] * 50.0     # padding, masked below
            at = 0
            for k, N in enumerate(Ns):
                x[k, :N] = x0[at:at + N]
                at += N
            self.x = f64(x)
            self.mask = torch.arange(self.nmax, device=dev)[None] < i64(Ns)[:, None]
            n = case["chain_len"] or 1 << 30
            bead = torch.arange(self.nmax, device=dev)
            self.bond = self.mask[:, 1:] & ((bead[1:] % n) != 0)[None]
            self.v = torch.zeros_like(self.x)
            self.fc = torch.zeros_like(self.x)
            self.f = self._conservative(self.x)

    def _conservative(self, x):
        p = self.par
        Ld = self.L.to(torch.float64)[:, None, None, None]
        d = x[:, :, None] - x[:, None]
        d = d - Ld * torch.round(d / Ld).detach()
        r2 = d.square().sum(-1)
        pair = self.mask[:, :, None] & self.mask[:, None] & ~torch.eye(self.nmax, dtype=torch.bool, device=self.dev)
        near = pair & (r2 < 2.0 ** (1 / 3) * p["sigma_wca"] ** 2)
        r2 = torch.where(near, r2, torch.ones_like(r2))
        s6 = (p["sigma_wca"] ** 2 / r2) ** 3
        g = torch.where(near, 24.0 * p["eps_wca"] * s6 * (2.0 * s6 - 1.0) / r2, torch.zeros_like(r2))
        F = (g[..., None] * d).sum(2)
        if self.nmax > 1:
            d = x[:, 1:] - x[:, :-1]
            r2 = torch.where(self.bond, d.square().sum(-1), torch.zeros_like(d[..., 0]))
            g = torch.where(self.bond, p["k_fene"] / (1.0 - r2 / p["r0_fene"] ** 2), torch.zeros_like(r2))
            pull = g[..., None] * d
            zero = torch.zeros_like(x[:, :1])
            F = F + torch.cat([pull, zero], 1) - torch.cat([zero, pull], 1)
        return F

    def _couple(self, p, x, v, f, theta):
        """MD substeps of one LB step in the frozen fluid; returns the beads and the node impulses."""
        q, dev = self.par, self.dev
        dt, h = q["md_dt"], 0.5 * q["md_dt"] / q["mass"]
        Lb = self.L[:, None, None]
        zeta = theta[:, 2][:, None, None]
        amp = torch.sqrt(2.0 * q["kT"] * zeta / dt)
        corner = torch.tensor([[k & 1, (k >> 1) & 1, k >> 2] for k in range(8)], device=dev)
        bead = torch.arange(self.nmax, device=dev)[None]
        bid = torch.arange(len(self.sizes), device=dev)[:, None]
        dirs = torch.arange(19, device=dev)[:, None, None, None]
        cf = self.c.to(torch.float64)
        keep = self.mask[:, :, None].to(torch.float64)
        dp = torch.zeros(3, p.shape[1], dtype=torch.float64, device=dev)
        fc = torch.zeros_like(x)
        for s in range(q["md_substeps"]):
            v = v + f * h * keep
            x = x + v * dt
            F = self._conservative(x)
            base = torch.floor(x.detach()).to(torch.int64)
            fr = x - base
            node = torch.remainder(base[:, :, None] + corner, Lb[..., None])             # [B, N, 8, 3]
            g = torch.where(corner.bool(), fr[:, :, None], 1.0 - fr[:, :, None])
            w = g[..., 0] * g[..., 1] * g[..., 2]
            src = torch.remainder(node[None] - self.c[:, None, None, None], Lb[None, ..., None])
            at = src[..., 0] + Lb[None] * (src[..., 1] + Lb[None] * src[..., 2]) + self.off[:, None, None]
            d = p[dirs, at]                                                              # [19, B, N, 8]
            j = torch.einsum("ibnk,ic->bnkc", d, cf)
            u = j / (q["rho0"] + d.sum(0))[..., None] / q["tau_lb"]
            ub = (w[..., None] * u).sum(2)
            wd = _philox((bead.expand(len(self.sizes), -1), torch.full_like(bead, self.t),
                          torch.full_like(bead, (1 << 16) | s), torch.zeros_like(bead)), self.seed, bid)
            fc = (-zeta * (v - ub) + amp * torch.stack([_unit(a) for a in wd[:3]], -1)) * keep
            f = F + fc
            v = v + f * h * keep
            hand = -w[..., None] * fc[:, :, None] * dt * q["tau_lb"]
            here = (node[..., 0] + Lb * (node[..., 1] + Lb * node[..., 2]) + self.off[:, None, None]).reshape(-1)
            dp = dp.index_add(1, here, hand.reshape(-1, 3).T)
        return x, v, f, fc, dp

    def _collide(self, p, dp, theta, a, b):
        """Post-collision deviations of flat nodes a..b-1."""
        q = self.par
        box, r = self.box[a:b].to(torch.int64), self.local[a:b].to(torch.int64)
        L, off = self.L[box], self.off[box]
        x, y, z = r % L, (r // L) % L, r // (L * L)
        rows = []
        for i in range(19):
            s = [torch.remainder(v - int(C[i, k]), L) if C[i, k] else v for k, v in enumerate((x, y, z))]
            rows.append(p[i, off + s[0] + L * (s[1] + L * s[2])])
        m = self.e @ torch.stack(rows)
        rho = q["rho0"] + m[0]
        f = dp[:, a:b] if dp is not None else torch.zeros(3, b - a, dtype=torch.float64, device=self.dev)
        u = (m[1:4] + 0.5 * f) / rho
        gs, gb, gg = 1.0 - theta[:, 0], 1.0 - theta[:, 1], 1.0 - q["omega_g"]
        gs, gb = (g[box] if len(self.sizes) > 1 else g[0] for g in (gs, gb))
        uu, uf = u * u, 2.0 * u * f
        e6 = [uu.sum(0), 2 * uu[0] - uu[1] - uu[2], uu[1] - uu[2], u[0] * u[1], u[1] * u[2], u[0] * u[2]]
        s6 = [uf.sum(0), 2 * uf[0] - uf[1] - uf[2], uf[1] - uf[2], u[0] * f[1] + u[1] * f[0],
              u[1] * f[2] + u[2] * f[1], u[0] * f[2] + u[2] * f[0]]
        out = [m[0], m[1] + f[0], m[2] + f[1], m[3] + f[2]]
        gam = [gb] + [gs] * 5 + [torch.full((), gg, dtype=torch.float64, device=self.dev)] * 9
        for k in range(4, 10):
            eq = rho * e6[k - 4]
            out.append(eq + gam[k - 4] * (m[k] - eq) + 0.5 * (1.0 + gam[k - 4]) * s6[k - 4])
        out += [gg * m[k] for k in range(10, 19)]
        if self.case["therm"]:
            mu = 3.0 * q["kT"] * q["tau_lb"] ** 2
            amp = torch.sqrt(mu * rho)
            zero = torch.zeros_like(r)
            for blk in range(4 if self.case["therm"] > 1 else 2):
                wd = _philox((r, zero + self.t, zero, zero + blk), self.seed, box)
                for j in range(4):
                    k = 4 + 4 * blk + j
                    if k > (18 if self.case["therm"] > 1 else 9):
                        break
                    out[k] = out[k] + amp * torch.sqrt((1.0 - gam[k - 4] ** 2) * self.b[k]) * _unit(wd[j])
        M = torch.stack(out) / self.b[:, None]
        return self.w[:, None] * (self.e.T @ M)

    def _step(self, p, x, v, f, theta):
        fc = dp = None
        if self.nmax:
            x, v, f, fc, dp = self._couple(p, x, v, f, theta)
        n, chunk = p.shape[1], 1 << 21
        if n <= chunk:
            return self._collide(p, dp, theta, 0, n), x, v, f, fc
        new = torch.empty_like(p)
        for a in range(0, n, chunk):
            new[:, a:a + chunk] = self._collide(p, dp, theta, a, min(n, a + chunk))
        return new, x, v, f, fc

    def steps(self, n):
        for _ in range(n):
            x, v, f = (self.x, self.v, self.f) if self.nmax else (None, None, None)
            self.p, self.x, self.v, self.f, self.fc = self._step(self.p, x, v, f, self.theta)
            self.t += 1

    def beads(self, a):
        return a[self.mask]

    def moved(self):
        """Populations where they arrive, n_i(r) - w_i rho0, [19, nodes]."""
        box, r = self.box.to(torch.int64), self.local.to(torch.int64)
        L, off = self.L[box], self.off[box]
        x, y, z = r % L, (r // L) % L, r // (L * L)
        out = torch.empty_like(self.p)
        for i in range(19):
            s = [torch.remainder(v - int(C[i, k]), L) for k, v in enumerate((x, y, z))]
            out[i] = self.p[i, off + s[0] + L * (s[1] + L * s[2])]
        return out

    def packed(self):
        """The library's storage order: per box, tiles of 1024 nodes, 19 planes a tile, zeros after the last node."""
        parts, at = [], 0
        for L, _ in self.sizes:
            V = L ** 3
            tiles = -(-V // 1024)
            q = torch.zeros(19, tiles * 1024, dtype=torch.float64, device=self.dev)
            q[:, :V] = self.p[:, at:at + V]
            parts.append(q.view(19, tiles, 1024).permute(1, 0, 2).reshape(-1))
            at += V
        return torch.cat(parts)


def exact(case, seed):
    with torch.no_grad():
        R = _Reference(case, seed)
        R.steps(case["warm"])
    if case["work"] == "window":
        return _exact_window(R, case, seed)
    with torch.no_grad():
        R.steps(case["steps"])
        out = {}
        if case["work"] == "checkpoint":
            L, N = R.sizes[0]
            n = R.moved() + (R.w * R.par["rho0"])[:, None]
            return {"n": [n.view(19, L, L, L)], "step": None,
                    "beads": [{k: R.beads(getattr(R, k)) for k in ("x", "v", "f", "fc")}]}
        out["pops"] = R.packed()
        for k in ("x", "v", "f", "fc") if R.nmax else ():
            out[k] = R.beads(getattr(R, k))
        if case["work"] == "steps":
            if R.nmax:
                out["at_x"] = out["x"]
            return out
        d, V = R.moved(), [L ** 3 for L, _ in R.sizes]
        m = R.e @ d
        per = [(m[:, a:a + n], d[:, a:a + n]) for a, n in zip(np.cumsum([0] + V[:-1]).tolist(), V)]
        base = (R.w * R.par["rho0"])[:, None]
        out["obs_mass"] = torch.stack([R.par["rho0"] * q.shape[1] + q[0].sum() for q, _ in per])
        out["obs_neg"] = None       # a count: an FP32 population within rounding of zero may fall either way
        out["obs_mode_sq"] = torch.stack([q.square().sum(1) for q, _ in per])
        if case["work"] == "sample":
            x = R.x                 # one chain a box, all of N beads
            com = x.mean(1)
            out["obs_com"] = com
            out["obs_rg2"] = (x - com[:, None]).square().sum(-1).mean(1)
            out["obs_re2"] = (x[:, -1] - x[:, 0]).square().sum(-1)
            out["at_x"], out["at_v"] = out["x"], out["v"]
        return out


def _exact_window(R, case, seed):
    from torch.utils.checkpoint import checkpoint
    theta, target = _theta(case, seed)
    theta = theta.to(R.dev).requires_grad_(True)
    p, x, v, f = R.p, R.x, R.v, R.f
    t0, vs = R.t, []

    def one(t, p, x, v, f, theta):
        R.t = t                     # the noise of that step, also when it is run again in the backward pass
        return R._step(p, x, v, f, theta)[:4]

    for t in range(case["T"]):
        p, x, v, f = checkpoint(one, t0 + t, p, x, v, f, theta, use_reentrant=False)
        vs.append(R.beads(v))
    vh = torch.stack(vs)
    loss = adjoint.vacf_loss(vh, target.to(R.dev))
    loss.backward()
    return {"v": vh.detach(), "loss": loss.detach(), "grad": theta.grad.cpu()}
