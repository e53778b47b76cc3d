"""The work a user of ldrop has it do, as a fixed set of timed cases.

Every case is one pass through the Python binding of libldrop (System,
Ensemble) on a seeded droplet of the repository's own recipes
(workloads.config_small / medium / large / learned / ensemble), at the
recipes' sizes or at odd sizes in between.  listed() are the cases that are
followed; draw() gives more of the same ranges.

Kinds of case:

direct    a chunk of steps of the all-pairs droplet, then the positions are
          read back: the frame loop of a simulation with a live view (the
          paper's use), from a thousand NPs to the headline's 250 000.
ensemble  the same for many independent droplets stepped together.
paper     the same for the paper's own truncated, inertial scheme.
learned   the same for the learned far field with a given set of weights.
grads     loss and gradients of the learned field's network for one batch
          (a training iteration driven from Python).
analysis  the post-processing of a stored frame: RDF and radial
          concentration, both fractal dimensions, sub-aggregates.
surface   the post-processing of a frame with NPs gathered in patches on the
          droplet's surface: surface count, surface fractal dimension, labels.
"""
import math

import numpy as np
import torch

from paper_2501_04456_amd import ldrop
from paper_2501_04456_amd import workloads as W

DT = 5e-4                 # the medium and large recipes' step
KICK = 0.05               # random velocity of the paper scheme (bench.py's default)
RANGE_FACTOR = 4.0        # the paper's 4 (r_i + r_j)
R_MAX, N_BINS = 10.0, 200  # RDF window (bench.py's analysis)
CONTACT = 1.1
GRID, BLOCK, HIDDEN = 32, 5, 128


def listed():
    return [
        # the small recipe: a thousand NPs, launch-bound steps, a frame every 10
        {"name": "direct small 1000", "kind": "direct", "recipe": "small", "n": 1000, "steps": 10},
        # the size the paper shows in real time (5000 NPs), two charged types
        {"name": "direct medium 5000", "kind": "direct", "recipe": "medium", "n": 5000, "steps": 10},
        # the medium recipe
        {"name": "direct medium 32768", "kind": "direct", "recipe": "medium", "n": 32768, "steps": 5},
        # the headline: three types, a fifth of the NPs uncharged
        {"name": "direct large 250000", "kind": "direct", "recipe": "large", "n": 250000, "steps": 2},
        # a parameter scan over a few small droplets
        {"name": "ensemble 12", "kind": "ensemble", "drops": 12, "n_min": 500, "n_max": 2000,
         "steps": 10},
        # the ensemble recipe: 256 droplets of 500 to 8000 NPs
        {"name": "ensemble 256", "kind": "ensemble", "drops": 256, "n_min": 500, "n_max": 8000,
         "steps": 5},
        # the paper's own scheme at the paper's size, and on the headline droplet
        {"name": "paper 5000", "kind": "paper", "recipe": "medium", "n": 5000, "steps": 10},
        {"name": "paper 250000", "kind": "paper", "recipe": "large", "n": 250000, "steps": 10},
        # the learned far field at its recipe's size
        {"name": "learned 250000", "kind": "learned", "recipe": "medium", "n": 250000, "steps": 2},
        # one training batch of its network
        {"name": "grads 8192", "kind": "grads", "rows": 8192},
        # post-processing of a frame of the headline droplet
        {"name": "analysis 250000", "kind": "analysis", "recipe": "large", "n": 250000},
        # post-processing of a smaller frame with surface aggregates (odd size)
        {"name": "surface 30011", "kind": "surface", "n": 30011, "n_surf": 6007},
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["direct", "direct", "direct", "ensemble", "ensemble", "paper", "paper",
                       "learned", "grads", "analysis", "surface"])
    if kind == "direct":
        recipe = rng.choice(["small", "medium", "large"])
        n = _size(rng, 400, 120000)
        return {"kind": kind, "recipe": recipe, "n": n, "steps": 2 if n > 40000 else rng.randint(2, 12)}
    if kind == "ensemble":
        lo = _size(rng, 300, 1000)
        return {"kind": kind, "drops": _size(rng, 4, 128), "n_min": lo, "n_max": lo * rng.randint(2, 6),
                "steps": rng.randint(2, 8)}
    if kind == "paper":
        return {"kind": kind, "recipe": rng.choice(["medium", "large"]), "n": _size(rng, 2000, 200000),
                "steps": rng.randint(4, 12)}
    if kind == "learned":
        return {"kind": kind, "recipe": rng.choice(["medium", "large"]), "n": _size(rng, 60000, 200000),
                "steps": rng.randint(1, 3)}
    if kind == "grads":
        return {"kind": kind, "rows": _size(rng, 1000, 8000)}
    if kind == "analysis":
        return {"kind": kind, "recipe": rng.choice(["small", "medium", "large"]),
                "n": _size(rng, 2000, 200000)}
    n = _size(rng, 5000, 100000)
    return {"kind": "surface", "n": n, "n_surf": max(500, int(n * rng.uniform(0.1, 0.4)))}


# ---- inputs ------------------------------------------------------------------

RECIPES = {"small": W.config_small, "medium": W.config_medium, "large": W.config_large}


def _droplet(case, seed):
    """The recipe's droplet of n NPs: positions and noise from the seed, the
    radius drying to three quarters over the first 4000 steps."""
    w = RECIPES[case["recipe"]](n=case["n"], seed=seed)
    w.dt = DT
    w.radius = W.Radius(kind=W.RADIUS_LINEAR, R0=w.radius.R0, R1=0.75 * w.radius.R0, T=4000 * DT)
    if case["kind"] == "paper":      # the paper's spring: within one NP radius of the surface
        w.params.wall_band = 1
        w.params.wall_offset = [0.5 * s for s in w.params.sigma]
    return w


def _drops(case, seed):
    """Droplets of the ensemble recipe: sizes spread evenly over the logarithm
    (the same for every seed), compositions and positions from the seed."""
    rng = np.random.default_rng([seed, 11])
    m, sigma = case["drops"], [1.0, 1.5]
    sizes = np.exp(np.linspace(math.log(case["n_min"]), math.log(case["n_max"]), m)).round().astype(int)
    drops = []
    for d, n in enumerate(np.roll(sizes[::-1], m // 3)):
        n = int(n)
        n0 = int(round(n * rng.uniform(0.2, 0.8)))
        typ = np.repeat(np.arange(2, dtype=np.int32), [n0, n - n0])
        R0 = (float(np.sum(np.asarray(sigma)[typ] ** 3)) / (8.0 * 1e-3)) ** (1.0 / 3.0)
        p = W.Params(sigma=sigma, eps=[1.0, 2.0], mass=[s ** 3 for s in sigma], gamma=list(sigma),
                     k_wall=[50.0, 50.0], wall_offset=[0.0, 0.0])
        R = W.Radius(kind=W.RADIUS_LINEAR, R0=R0, R1=0.75 * R0, T=4000 * DT)
        pos = W.sample_positions(typ, sigma, R0, int(rng.integers(1 << 40)))
        drops.append(W.Workload("drop", n, typ, np.where(typ == 0, 1.0, -1.0), pos, p, R, DT, 1,
                                int(rng.integers(1 << 40))))
    return drops


def _surface(case, seed):
    sigma = [1.0, 1.5]
    R0 = 300.0 * (case["n"] / 250000.0) ** (1.0 / 3.0)
    x, t = W.surface_clusters(case["n_surf"], case["n"] - case["n_surf"], R0, sigma, seed,
                              n_centres=max(4, case["n_surf"] // 125), spread=4.0)
    p = W.config_medium(n=100, with_positions=False).params
    return W.Workload("surface", case["n"], t.astype(np.int32), np.zeros(case["n"]),
                      x.astype(np.float32), p, W.Radius(kind=W.RADIUS_CONST, R0=R0), DT, 1, seed)


def _net(seed):
    """Weights of the network (K = 4 BLOCK^3 + 3 inputs, two hidden layers),
    unit-variance fan-in scaling, and their packed form."""
    rng = np.random.default_rng([seed, 12])
    K, H = 4 * BLOCK ** 3 + 3, HIDDEN
    Kp = (K + 31) // 32 * 32
    w = {"W1": rng.standard_normal((K, H)) / math.sqrt(K), "b1": 0.1 * rng.standard_normal(H),
         "W2": rng.standard_normal((H, H)) / math.sqrt(H), "b2": 0.1 * rng.standard_normal(H),
         "W3": rng.standard_normal((H, 3)) / math.sqrt(H), "b3": 0.1 * rng.standard_normal(3)}
    w = {k: v.astype(np.float32) for k, v in w.items()}
    W1, W3, b3 = np.zeros((Kp, H), np.float32), np.zeros((H, 16), np.float32), np.zeros(16, np.float32)
    W1[:K], W3[:, :3], b3[:3] = w["W1"], w["W3"], w["b3"]
    return w, np.concatenate([v.ravel() for v in (W1, w["b1"], w["W2"], w["b2"], W3, b3)])


OUT_SCALE = 0.01          # of the order of the recipe's trained residual


def _batch(case, seed):
    rng = np.random.default_rng([seed, 13])
    K = 4 * BLOCK ** 3 + 3
    X = rng.standard_normal((case["rows"], K)).astype(np.float32)
    X[:, -3:] = rng.random((case["rows"], 3)) - 0.5
    return X, rng.standard_normal((case["rows"], 3)).astype(np.float32)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "ensemble":
        return {"kind": kind, "ens": ldrop.Ensemble(_drops(case, seed)), "steps": case["steps"]}
    if kind == "grads":
        s = ldrop.System.from_workload(W.config_small(seed=seed))
        s.ff_enable(grid=GRID, block=BLOCK, hidden=HIDDEN, near_mode=ldrop.NEAR_BLOCK)
        s.ff_set_weights(_net(seed)[1], 1.0, 1.0)
        X, T = _batch(case, seed)
        return {"kind": kind, "sys": s, "X": X, "T": T}
    w = _surface(case, seed) if kind == "surface" else _droplet(case, seed)
    s = ldrop.System.from_workload(w)
    if kind == "paper":
        s.paper_enable(range_factor=RANGE_FACTOR, kick=KICK)
    if kind == "learned":
        s.ff_enable(grid=GRID, block=BLOCK, hidden=HIDDEN, near_mode=ldrop.NEAR_BLOCK)
        s.ff_set_weights(_net(seed)[1], s.ff_weights()[1], OUT_SCALE)
        s.ff_mode(1)
    return {"kind": kind, "sys": s, "steps": case.get("steps", 0)}


def run(state):
    kind = state["kind"]
    if kind == "ensemble":
        state["ens"].step(state["steps"], DT)
        return state["ens"].positions64()
    s = state["sys"]
    if kind in ("direct", "learned"):
        s.step(state["steps"], DT)
        return s.positions64()
    if kind == "paper":
        s.step(state["steps"], DT)
        return {"x": s.positions64(), "v": s.velocities()}
    if kind == "grads":
        loss, g = s.ff_grads(state["X"], state["T"])
        return {"loss": loss, "grads": g}
    if kind == "analysis":
        counts, cc, g, cbar = s.rdf(R_MAX, N_BINS)
        rg, df, dbox, scales, boxes = s.fractal()
        return {"counts": counts.astype(np.int64), "ccounts": cc.astype(np.int64), "g": g,
                "cbar": cbar, "R_g": rg, "D_f": df, "D_box": dbox, "scales": scales,
                "boxes": boxes, "aggregates": s.aggregates(CONTACT, labels=True)}
    return {"n_surf": s.surface_count(), "fractal": s.surface_fractal(labels=True),
            "aggregates": s.aggregates(CONTACT)}


# ---- work that cannot be left out ---------------------------------------------

# one unordered pair: 3 differences, 5 for r^2, 1 root, 4 for the two weights,
# 12 for the two sums
PAIR = 25
STATE = 2 * 24 + 4 + 4    # a step: FP64 position in and out, type, index


def _sphere_pairs(n, R0, r):
    """Unordered pairs closer than r among n NPs uniform in a ball of R0."""
    return 0.5 * n * n * (r / R0) ** 3


def work(case):
    kind = case["kind"]
    if kind == "grads":
        K = 4 * BLOCK ** 3 + 3
        net = K * HIDDEN + HIDDEN * HIDDEN + HIDDEN * 3
        return {"bytes": 4.0 * (case["rows"] * (K + 3) + 2 * net), "flops": 6.0 * net * case["rows"]}
    if kind == "ensemble":
        sizes = np.exp(np.linspace(math.log(case["n_min"]), math.log(case["n_max"]), case["drops"]))
        return {"bytes": float(STATE * sizes.sum() * case["steps"]),
                "flops": float(PAIR * 0.5 * (sizes ** 2).sum() * case["steps"])}
    n = case["n"]
    if kind == "surface":
        return {"bytes": 28.0 * n + 12.0 * n, "flops": 60.0 * n}
    w = RECIPES[case["recipe"]](n=n, with_positions=False)
    charged, R0 = int(np.count_nonzero(w.charge)), w.radius.R0
    if kind == "analysis":
        return {"bytes": 28.0 * n + 4.0 * n, "flops": 10.0 * _sphere_pairs(n, R0, R_MAX) + 60.0 * n}
    if kind == "direct":
        flops = PAIR * 0.5 * charged * charged
    elif kind == "paper":
        flops = 40.0 * _sphere_pairs(n, R0, RANGE_FACTOR * float(np.mean(np.asarray(w.params.sigma)[w.type])))
    else:
        near = 0.5 * charged * charged * BLOCK ** 3 * 6.0 / (math.pi * GRID ** 3)
        flops = PAIR * near + 2.0 * n * (HIDDEN * HIDDEN + 6 * HIDDEN)
    vel = 48 if kind == "paper" else 0
    return {"bytes": float((STATE + vel) * n * case["steps"]), "flops": float(flops * case["steps"])}


# ---- the same outputs in 64 bits, in plain torch and numpy ---------------------

def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _normals(n, step, seed):
    """Philox4x32-10 at counter (i, step, 0, 0) with the seed as key, then the
    three normals of the documented Box-Muller map."""
    M = np.uint64(0xFFFFFFFF)
    c = [np.arange(n, dtype=np.uint64), np.full(n, step, np.uint64), np.zeros(n, np.uint64),
         np.zeros(n, np.uint64)]
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & M,
             (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), p0 & M]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    u = [((v >> np.uint64(9)).astype(np.float64) + 0.5) * 2.0 ** -23 for v in c]
    a, b = np.sqrt(-2.0 * np.log(u[0])), np.sqrt(-2.0 * np.log(u[2]))
    return np.stack([a * np.cos(2 * np.pi * u[1]), a * np.sin(2 * np.pi * u[1]),
                     b * np.cos(2 * np.pi * u[3])], 1)


class _Droplet:
    """A droplet's state and parameters as FP64 tensors."""

    def __init__(self, w):
        d = _dev()
        f = lambda v: torch.as_tensor(np.asarray(v, np.float64), device=d)  # noqa: E731
        p = w.params
        self.p, self.w, self.t, self.k = p, w, 0.0, 0
        self.x = f(w.pos)
        self.typ = torch.as_tensor(w.type.astype(np.int64), device=d)
        self.q = f(w.charge) * math.sqrt(p.kT * p.bjerrum)
        s = f(p.sigma)
        self.sig, self.sij = s, 0.5 * (s[:, None] + s[None, :])
        self.eij = torch.sqrt(f(p.eps)[:, None] * f(p.eps)[None, :])
        self.mass, self.gamma, self.kw, self.off = (f(v)[self.typ] for v in
                                                    (p.mass, p.gamma, p.k_wall, p.wall_offset))

    def radius(self, t):
        r = self.w.radius
        return r.R0 + (r.R1 - r.R0) * min(1.0, t / r.T)

    def ext(self, R):
        x, p = self.x, self.p
        r = x.norm(dim=1)
        on = r > R - self.off
        if p.wall_band:
            h = 0.5 * self.sig[self.typ]
            on &= (r > R - h) & (r < R + h)
        F = torch.where(on, -self.kw * (r - (R - self.off)) / r, torch.zeros_like(r))[:, None] * x
        F = F + self.mass[:, None] * torch.as_tensor(p.gravity, dtype=x.dtype, device=x.device)
        return F + (self.mass * p.omega ** 2)[:, None] * x

    def lj(self, i, j, cut, coulomb=False):
        """LJ forces (with the Coulomb term of the same pairs) on i from the
        pairs (i, j) closer than cut sigma_ij."""
        d = self.x[i] - self.x[j]
        r2 = (d * d).sum(1)
        s = self.sij[self.typ[i], self.typ[j]]
        keep = r2 < (cut * s) ** 2
        i, j, d, r2, s = i[keep], j[keep], d[keep], r2[keep], s[keep]
        s6 = (s * s / r2) ** 3
        g = 24.0 * self.eij[self.typ[i], self.typ[j]] * (2.0 * s6 * s6 - s6) / r2
        if coulomb:
            g = g + self.q[i] * self.q[j] / (r2 * r2.sqrt())
        return torch.zeros_like(self.x).index_add_(0, i, g[:, None] * d)

    def _rows(self):
        n = len(self.x)
        b = max(1, min(n, (1 << 28) // n))
        return [slice(k, min(n, k + b)) for k in range(0, n, b)]

    def near_pairs(self, reach):
        """Ordered pairs (i, j), i != j, closer than reach."""
        x, got = self.x, []
        for s in self._rows():
            r2 = torch.zeros((s.stop - s.start, len(x)), dtype=x.dtype, device=x.device)
            for c in range(3):
                d = x[s, c][:, None] - x[None, :, c]
                r2.addcmul_(d, d)
            i, j = torch.nonzero(r2 < reach * reach, as_tuple=True)
            i = i + s.start
            got.append((i[i != j], j[i != j]))
        return torch.cat([g[0] for g in got]), torch.cat([g[1] for g in got])

    def direct(self):
        """All-pairs Coulomb and truncated LJ."""
        x, q, F = self.x, self.q, torch.empty_like(self.x)
        rhs = torch.cat([q[:, None], q[:, None] * x], 1)
        reach, ii, jj = self.p.lj_cut * float(self.sij.max()), [], []
        for s in self._rows():
            r2 = torch.zeros((s.stop - s.start, len(x)), dtype=x.dtype, device=x.device)
            for c in range(3):
                d = x[s, c][:, None] - x[None, :, c]
                r2.addcmul_(d, d)
            del d
            own = torch.arange(s.start, s.stop, device=x.device)
            r2[own - s.start, own] = math.inf
            i, j = torch.nonzero(r2 < reach * reach, as_tuple=True)
            ii.append(i + s.start)
            jj.append(j)
            w = r2.rsqrt_().pow_(3) @ rhs
            F[s] = q[s, None] * (x[s] * w[:, :1] - w[:, 1:])
        return F + self.lj(torch.cat(ii), torch.cat(jj), self.p.lj_cut)

    def overdamped(self, F):
        mu, p = 1.0 / self.gamma, self.p
        F = F + self.ext(self.radius(self.t + DT))
        xi = torch.as_tensor(_normals(len(self.x), self.k, self.w.seed), device=self.x.device)
        self.x = self.x + (mu * DT)[:, None] * F + torch.sqrt(2.0 * p.kT * mu * DT)[:, None] * xi
        self.t, self.k = self.t + DT, self.k + 1


def _exact_paper(D, steps):
    v = torch.zeros_like(D.x)
    i, j = D.near_pairs(RANGE_FACTOR * float(D.sij.max()) + 2.0)
    for _ in range(steps):
        F = D.lj(i, j, RANGE_FACTOR, coulomb=True) + D.ext(D.radius(D.t + DT))
        v = v + DT * (F - D.gamma[:, None] * v) / D.mass[:, None]
        u = torch.as_tensor(_normals(len(D.x), D.k, D.w.seed), device=v.device)
        v = v + KICK * u / u.norm(dim=1, keepdim=True)
        D.x = D.x + DT * v
        D.t, D.k = D.t + DT, D.k + 1
    return {"x": D.x, "v": v}


def _silu(z):
    return z * torch.sigmoid(z)


def _expansion(R, Q, P):
    """Field, gradient and second gradient of monopoles Q and dipoles P at
    distance R = target - source: E [.., 3], J [.., 3, 3], H [.., 3, 3, 3],
    summed over the sources (axis 1)."""
    I = torch.eye(3, dtype=R.dtype, device=R.device)
    r2 = (R * R).sum(-1)
    i2 = 1.0 / r2
    i3 = i2 * i2.sqrt()
    i5, pr = i3 * i2, (R * P).sum(-1)
    i7 = i5 * i2
    i9 = i7 * i2
    es = lambda f, *v: torch.einsum(f, *v)  # noqa: E731
    E = ((Q * i3 + 3.0 * pr * i5)[..., None] * R - i3[..., None] * P).sum(1)
    a = -3.0 * Q * i5 - 15.0 * pr * i7
    RR = es("tsa,tsb->tsab", R, R).flatten(2)
    PR = es("tsa,tsb->tsab", P, R)
    J = (a[..., None] * RR).sum(1).view(-1, 3, 3) + (3.0 * i5[..., None, None]
                                                     * (PR + PR.transpose(2, 3))).sum(1)
    J += (Q * i3 + 3.0 * pr * i5).sum(1)[:, None, None] * I
    b = 15.0 * Q * i7 + 105.0 * pr * i9
    H = es("tsa,tsb->tab", b[..., None] * R, RR).view(-1, 3, 3, 3)
    l = (a[..., None] * R + 3.0 * i5[..., None] * P).sum(1)
    m = es("tsa,tsb->tab", -15.0 * i7[..., None] * P, RR).view(-1, 3, 3, 3)
    H = H + m + m.permute(0, 2, 1, 3) + m.permute(0, 2, 3, 1)
    H = H + es("ta,bc->tabc", l, I) + es("tb,ac->tabc", l, I) + es("tc,ab->tabc", l, I)
    return E, J, H


def _learned(D, net, sq):
    """Near Coulomb over the 5^3 block, LJ, the far cells' expansion and the
    network."""
    x, q, G, half, dev = D.x, D.q, GRID, BLOCK // 2, D.x.device
    m = x.float().abs().max().item()
    L = float(np.float32(m) * np.float32(1.0009765625))
    h = 2.0 * L / G
    cell = torch.clamp(torch.floor((x + L) / h), 0, G - 1).long()
    off = x - (-L + (cell + 0.5) * h)
    flat = (cell[:, 2] * G + cell[:, 1]) * G + cell[:, 0]
    mom = torch.zeros((G ** 3, 4), dtype=x.dtype, device=dev)
    mom.index_add_(0, flat, torch.cat([q[:, None], q[:, None] * off], 1))
    F = torch.zeros_like(x)
    # near part, slab by slab
    order = torch.argsort(flat)
    first = torch.searchsorted(cell[order, 2].contiguous(), torch.arange(G + 1, device=dev)).tolist()
    reach, ii, jj = D.p.lj_cut * float(D.sij.max()), [], []
    for k in range(G):
        src = order[first[max(0, k - half)]:first[min(G, k + half + 1)]]
        rhs = torch.cat([q[src, None], q[src, None] * x[src]], 1)
        tgt = order[first[k]:first[k + 1]]
        for t in tgt.split(max(1, (1 << 26) // max(1, len(src)))) if len(tgt) else []:
            r2 = torch.zeros((len(t), len(src)), dtype=x.dtype, device=dev)
            far = torch.zeros((len(t), len(src)), dtype=torch.bool, device=dev)
            for c in range(3):
                d = x[t, c][:, None] - x[None, src, c]
                r2.addcmul_(d, d)
                far |= (cell[t, c][:, None] - cell[None, src, c]).abs() > half
            r2[t[:, None] == src[None, :]] = math.inf
            i, j = torch.nonzero(r2 < reach * reach, as_tuple=True)
            ii.append(t[i])
            jj.append(src[j])
            r2[far] = math.inf
            w = r2.rsqrt_().pow_(3) @ rhs
            F[t] = q[t, None] * (x[t] * w[:, :1] - w[:, 1:])
    F = F + D.lj(torch.cat(ii), torch.cat(jj), D.p.lj_cut)
    # the field of the cells outside the block, expanded about each occupied cell
    occ = torch.unique(flat)
    ijk = torch.stack([occ % G, (occ // G) % G, occ // (G * G)], 1)
    E, J, H = [], [], []
    for s in range(0, len(occ), 128):
        sep = ijk[s:s + 128, None, :] - ijk[None, :, :]
        out = (sep.abs().amax(-1) > half).to(x.dtype)
        Q, P = mom[occ, 0] * out, mom[occ, 1:] * out[..., None]
        R = torch.where(out[..., None] > 0, h * sep.to(x.dtype), torch.ones((), dtype=x.dtype, device=dev))
        for to, v in zip((E, J, H), _expansion(R, Q, P)):
            to.append(v)
    E, J, H = torch.cat(E), torch.cat(J), torch.cat(H)
    at = torch.searchsorted(occ, flat)
    field = E[at] + torch.einsum("pab,pb->pa", J[at], off)
    field += 0.5 * torch.einsum("pabc,pb,pc->pa", H[at], off, off)
    # the network
    pad = torch.zeros((G + 2 * half,) * 3 + (4,), dtype=x.dtype, device=dev)
    scaled = mom / torch.as_tensor([sq] + 3 * [sq * h], dtype=x.dtype, device=dev)
    pad[half:half + G, half:half + G, half:half + G] = scaled.view(G, G, G, 4)
    z = torch.zeros((len(occ), HIDDEN), dtype=x.dtype, device=dev)
    for k in range(BLOCK ** 3):
        dx, dy, dz = k % BLOCK, (k // BLOCK) % BLOCK, k // BLOCK ** 2
        z += pad[ijk[:, 2] + dz, ijk[:, 1] + dy, ijk[:, 0] + dx] @ net["W1"][4 * k:4 * k + 4]
    a1 = _silu(z[at] + (off / h) @ net["W1"][-3:] + net["b1"])
    y = _silu(a1 @ net["W2"] + net["b2"]) @ net["W3"] + net["b3"]
    return F + q[:, None] * (field + OUT_SCALE * y)


def _exact_analysis(D):
    x, n, w = D.x, len(D.x), D.w
    dr = R_MAX / N_BINS
    r = np.arange(N_BINS + 1) * dr
    dV = 4.0 / 3.0 * math.pi * (r[1:] ** 3 - r[:-1] ** 3)
    V = 4.0 / 3.0 * math.pi * w.radius.R0 ** 3
    i, j = D.near_pairs(R_MAX)
    keep = i < j
    hist = lambda d: torch.bincount(torch.floor(d / dr).long()[d < R_MAX],  # noqa: E731
                                    minlength=N_BINS)[:N_BINS].cpu().numpy()
    counts = hist((x[i[keep]] - x[j[keep]]).norm(dim=1))
    g = (2.0 * counts / n) / ((n - 1.0) * dV / V)
    cbar = (hist(x.norm(dim=1)) / n) / (dV / V)
    rg = float((x - x.mean(0)).square().sum(1).mean().sqrt())
    sig = np.asarray(w.params.sigma)[w.type]
    df = math.log(n / 1.593) / math.log(2.0 * rg / float(sig.mean()))
    lo, e, lx, ly = x.min(0).values, float(sig.min()), [], []
    while e <= rg:
        b = torch.floor((x - lo) / e).long()
        m = int(b.max()) + 1
        lx.append(math.log(e))
        ly.append(math.log(len(torch.unique((b[:, 2] * m + b[:, 1]) * m + b[:, 0]))))
        e *= 2.0
    dbox = -float(np.polyfit(lx[1:], ly[1:], 1)[0]) if len(lx) >= 3 else None
    return {"counts": None, "ccounts": None, "g": g, "cbar": cbar, "R_g": rg, "D_f": df,
            "D_box": dbox, "scales": None, "boxes": None, "aggregates": None}


def _exact_surface(D):
    x, R = D.x, D.w.radius.R0
    on = ((x.norm(dim=1) - R).abs() < 0.5 * D.sig[D.typ]).nonzero()[:, 0]
    S = _Droplet(D.w.replace(pos=D.w.pos[on.cpu().numpy()], type=D.w.type[on.cpu().numpy()],
                             charge=D.w.charge[on.cpu().numpy()]))
    i, j = S.near_pairs(CONTACT * float(S.sij.max()))
    touch = (S.x[i] - S.x[j]).norm(dim=1) < CONTACT * S.sij[S.typ[i], S.typ[j]]
    i, j = i[touch], j[touch]
    lab = torch.arange(len(on), device=x.device)
    while True:          # smallest label over contacts, then over labels
        new = lab.scatter_reduce(0, i, lab[j], "amin")
        new = torch.minimum(new, new[new])
        if torch.equal(new, lab):
            break
        lab = new
    ids, size = torch.unique(lab, return_counts=True)
    best = ids[size == size.max()].min()
    mem = lab == best
    u = S.x[mem] / S.x[mem].norm(dim=1, keepdim=True)
    c = u.sum(0) / u.sum(0).norm()
    ang = torch.atan2(torch.linalg.cross(u, c.expand_as(u)).norm(dim=1), u @ c)
    rg = float((R * ang).square().mean().sqrt())
    d, m = float(S.sig[S.typ][mem].mean()), int(mem.sum())
    df = math.log(m / (math.pi / math.sqrt(3.0))) / math.log(2.0 * rg / d) if m > 1 else None
    return {"n_surf": None, "aggregates": None,
            "fractal": {"components": None, "largest": None, "label": None, "R_g": rg, "d": d,
                        "D_f": df, "labels": None}}


def exact(case, seed):
    kind = case["kind"]
    if kind == "ensemble":
        out = []
        for w in _drops(case, seed):
            D = _Droplet(w)
            for _ in range(case["steps"]):
                D.overdamped(D.direct())
            out.append(D.x)
        return torch.cat(out)
    if kind == "grads":
        X, T = (torch.as_tensor(v, dtype=torch.float64, device=_dev()) for v in _batch(case, seed))
        net = {k: torch.as_tensor(v, dtype=torch.float64, device=_dev()).requires_grad_()
               for k, v in _net(seed)[0].items()}
        y = _silu(_silu(X @ net["W1"] + net["b1"]) @ net["W2"] + net["b2"]) @ net["W3"] + net["b3"]
        loss = (y - T).square().mean()
        loss.backward()
        g = {k: v.grad for k, v in net.items()}
        pad = torch.nn.functional.pad
        Kp = (len(g["W1"]) + 31) // 32 * 32
        flat = torch.cat([pad(g["W1"], (0, 0, 0, Kp - len(g["W1"]))).ravel(), g["b1"],
                          g["W2"].ravel(), g["b2"], pad(g["W3"], (0, 13)).ravel(), pad(g["b3"], (0, 13))])
        return {"loss": loss.item(), "grads": flat}
    D = _Droplet(_surface(case, seed) if kind == "surface" else _droplet(case, seed))
    if kind == "paper":
        return _exact_paper(D, case["steps"])
    if kind == "analysis":
        return _exact_analysis(D)
    if kind == "surface":
        return _exact_surface(D)
    net = {k: torch.as_tensor(v, dtype=torch.float64, device=_dev()) for k, v in _net(seed)[0].items()}
    sq = float(D.q.abs().max().float())
    for _ in range(case["steps"]):
        D.overdamped(D.direct() if kind == "direct" else _learned(D, net, sq))
    return D.x
