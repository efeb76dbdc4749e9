"""Timed workloads of the reweighting library, through its public entry points.

A case is a dict of plain values:
  kind    "reweight" (Process.reweight), "kpoly" (Process.reweight_kpoly),
          "surrogate" (Process.reweight_surrogate) or "step" (one forward and
          backward pass of the surrogate network, Process.surrogate_fwd_bwd)
  proc    process name; prec: "mixed" or "fp64"
  events  events of the batch ("step": sample rows)
  points  new parameter points beside the base point
  weights True: the caller has input weights; False: unit weights
  alphas  True: the points change alpha_s together with kappa (g g processes)

Inputs are made on the GPU from the seed: massive RAMBO phase space with the
usual generator cuts (the recipes of the repository's own samples), kappa
uniform in [0.8, 1.2], alpha uniform in [0.5, 1.5] alpha_0.
"""
import itertools
import math

import numpy as np
import torch

DEV = "cuda"
MT, ALPHAS, ALPHA = 173.0, 0.118, 1 / 132.5
# external particles, incoming and outgoing gluons, colour flows, helicity configurations that do not vanish
PROCS = {
    "gg_tt": dict(ng=2, flows=2, hel=16, sqrt_s=None, masses=(MT, MT), pt=0.0, dr=0.0, eta=None),
    "gg_ttg": dict(ng=3, flows=6, hel=32, sqrt_s=1500.0, masses=(MT, MT, 0.0), pt=20.0, dr=0.0, eta=None),
    "gg_ttgg": dict(ng=4, flows=24, hel=64, sqrt_s=1500.0, masses=(MT, MT, 0.0, 0.0), pt=20.0, dr=0.4, eta=None),
    "gg_ttggg": dict(ng=5, flows=120, hel=128, sqrt_s=2000.0, masses=(MT, MT, 0.0, 0.0, 0.0), pt=20.0, dr=0.4,
                     eta=None),
    "ee_5a": dict(ng=0, flows=1, hel=64, sqrt_s=1000.0, masses=(0.0,) * 5, pt=10.0, dr=0.4, eta=2.5),
}
# operations of the diagrams of one helicity configuration, without the colour sum
CHAIN_FLOPS = {"gg_tt": 700, "gg_ttg": 3800, "gg_ttgg": 24600, "gg_ttggg": 250000, "ee_5a": 3278}
MLP_FLOPS = 2 * (64 * 256 + 3 * 256 * 256)   # one row through the network


def _case(name, kind, proc, prec, events, points=16, weights=False, alphas=False):
    return dict(name=name, kind=kind, proc=proc, prec=prec, events=events, points=points, weights=weights,
                alphas=alphas)


def listed():
    return [
        # a handful of events per request: a generator that reweights while it runs, an analysis of a small selection
        _case("ttgg mixed 1000", "reweight", "gg_ttgg", "mixed", 1000),
        # a scan over one event file of 10^4 events with its weights, alpha_s and kappa both varied
        _case("ttgg mixed 10007", "reweight", "gg_ttgg", "mixed", 10007, weights=True, alphas=True),
        # a production sample
        _case("ttgg mixed 1M", "reweight", "gg_ttgg", "mixed", 1 << 20),
        # the reference precision on a validation sample
        _case("ttgg fp64 20011", "reweight", "gg_ttgg", "fp64", 20011),
        # lower multiplicities of the same merged sample
        _case("ttg mixed 262147", "reweight", "gg_ttg", "mixed", 262147, weights=True),
        _case("tt mixed 1M", "reweight", "gg_tt", "mixed", 1 << 20),
        # the highest multiplicity, one small batch in either precision
        _case("ttggg mixed 6001", "reweight", "gg_ttggg", "mixed", 6001),
        _case("ttggg fp64 700", "reweight", "gg_ttggg", "fp64", 700),
        # the electroweak coupling scan of 10^5 events of e+ e- -> 5 photons
        _case("5 photons 100000", "reweight", "ee_5a", "mixed", 100000),
        # many points of one coupling: the polynomial form
        _case("ttgg kpoly 200003", "kpoly", "gg_ttgg", "mixed", 200003, weights=True),
        # serving the learned factor with its exact audit
        _case("ttgg surrogate 1M", "surrogate", "gg_ttgg", "mixed", 1 << 20),
        # one gradient of the network at the batch it is trained with
        _case("network step 16384", "step", "gg_ttgg", "mixed", 16384),
    ]


# smallest and largest batch of the drawn cases, by (kind, proc, prec), and how often each is drawn
RANGES = [
    (("reweight", "gg_ttgg", "mixed"), (50, 400000), 5),
    (("reweight", "gg_ttgg", "fp64"), (20, 100000), 2),
    (("reweight", "gg_ttg", "mixed"), (100, 1500000), 2),
    (("reweight", "gg_tt", "mixed"), (100, 4000000), 1),
    (("reweight", "gg_ttggg", "mixed"), (20, 9000), 2),
    (("reweight", "gg_ttggg", "fp64"), (10, 2000), 1),
    (("reweight", "ee_5a", "mixed"), (500, 1000000), 2),
    (("kpoly", "gg_ttgg", "mixed"), (500, 1000000), 2),
    (("surrogate", "gg_ttgg", "mixed"), (5000, 1500000), 1),
    (("step", "gg_ttgg", "mixed"), (1024, 65536), 1),
]


def draw(rng):
    (kind, proc, prec), (lo, hi), _ = rng.choices(RANGES, weights=[w for _, _, w in RANGES])[0]
    points = 16 if rng.random() < 0.5 else rng.choice([1, 2, 3, 5, 8, 12, 24, 40, 64])
    if kind == "surrogate":
        points = min(points, 40)
    # the cost grows with events times points
    hi = max(lo + 1, int(hi * min(1.0, 17.0 / (points + 1))))
    n = int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    if kind == "step":
        n, points = max(1024, n // 64 * 64), 16
    elif rng.random() < 0.6:
        n |= 1
    gluons = proc != "ee_5a" and kind in ("reweight", "kpoly")
    c = _case(None, kind, proc, prec, n, points, kind != "step" and rng.random() < 0.5,
              gluons and rng.random() < 0.3)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs

def _rng(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 16 + stream)
    return g


def _u(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)


def _rambo(g, n, sqrt_s, masses):
    """Massive RAMBO in the centre-of-mass frame: [n_out, 4, n]."""
    k = len(masses)
    c, phi = 2 * _u(g, k, n) - 1, 2 * math.pi * _u(g, k, n)
    e = -torch.log((_u(g, k, n) * _u(g, k, n)).clamp_min(1e-300))
    s = torch.sqrt((1 - c * c).clamp_min(0))
    q = torch.stack([e, e * s * torch.cos(phi), e * s * torch.sin(phi), e * c], 1)
    Q = q.sum(0)
    M = torch.sqrt(Q[0] ** 2 - (Q[1:] ** 2).sum(0))
    b, x, gam = -Q[1:] / M, sqrt_s / M, Q[0] / M
    bq = (b[None] * q[:, 1:]).sum(1)
    p = torch.empty_like(q)
    p[:, 0] = x * (gam * q[:, 0] + bq)
    p[:, 1:] = x * (q[:, 1:] + b[None] * (q[:, 0] + bq / (1 + gam))[:, None])
    m2 = torch.tensor(masses, device=DEV, dtype=torch.float64)[:, None] ** 2
    if sum(masses) > 0:
        pp = (p[:, 1:] ** 2).sum(1)
        xi = torch.full((n,), math.sqrt(1 - (sum(masses) / sqrt_s) ** 2), device=DEV, dtype=torch.float64)
        for _ in range(12):
            en = torch.sqrt(m2 + xi ** 2 * pp)
            xi = xi - (en.sum(0) - sqrt_s) / (xi * pp / en).sum(0)
        p[:, 0] = torch.sqrt(m2 + xi ** 2 * pp)
        p[:, 1:] *= xi
    return p


def _accepted(p, pt_min, dr_min, eta_max):
    ok = torch.ones(p.shape[2], dtype=torch.bool, device=DEV)
    if p.shape[0] == 0:
        return ok
    pt = torch.hypot(p[:, 1], p[:, 2])
    eta, phi = torch.asinh(p[:, 3] / pt), torch.atan2(p[:, 2], p[:, 1])
    ok &= (pt > pt_min).all(0)
    if eta_max is not None:
        ok &= (eta.abs() < eta_max).all(0)
    for i, j in itertools.combinations(range(p.shape[0]), 2):
        d = (phi[i] - phi[j]).abs()
        d = torch.minimum(d, 2 * math.pi - d)
        ok &= (eta[i] - eta[j]) ** 2 + d ** 2 > dr_min ** 2
    return ok


def _events(proc, n, seed):
    """Momenta [n_ext, 4, n] float64 on the GPU."""
    P, g = PROCS[proc], _rng(seed, 0)
    out = torch.zeros(2 + len(P["masses"]), 4, n, device=DEV, dtype=torch.float64)
    if P["sqrt_s"] is None:   # two-body, log-uniform in the energy
        rs = torch.exp(math.log(350.0) + _u(g, n) * (math.log(2000.0) - math.log(350.0)))
        c, phi = 2 * _u(g, n) - 1, 2 * math.pi * _u(g, n)
        s, e = torch.sqrt((1 - c * c).clamp_min(0)), 0.5 * rs
        p = torch.sqrt(e * e - MT * MT)
        out[2] = torch.stack([e, p * s * torch.cos(phi), p * s * torch.sin(phi), p * c])
        out[3] = torch.stack([e, -out[2, 1], -out[2, 2], -out[2, 3]])
        half = e
    else:
        done, first = 0, 0 if proc == "ee_5a" else 2
        while done < n:
            m = int(min((n - done) * 1.6 + 256, 1 << 21))
            p = _rambo(g, m, P["sqrt_s"], P["masses"])
            p = p[:, :, _accepted(p[first:], P["pt"], P["dr"], P["eta"])][:, :, : n - done]
            out[2:, :, done:done + p.shape[2]] = p
            done += p.shape[2]
        half = 0.5 * P["sqrt_s"]
    out[0, 0] = out[0, 3] = out[1, 0] = half
    out[1, 3] = -out[0, 3]
    return out


def _points(case, seed):
    r = np.random.default_rng([int(seed), 1])
    u = r.random(case["points"])
    if case["proc"] == "ee_5a":
        return [{"alpha": float(ALPHA * (0.5 + x))} for x in u]
    a = ALPHAS * (0.9 + 0.2 * r.random(case["points"])) if case["alphas"] else np.full(case["points"], ALPHAS)
    return [{"kappa_ttg": float(k), "alphas": float(x)} for k, x in zip(np.sort(0.8 + 0.4 * u), a)]


def _weights(case, seed):
    return 0.5 + _u(_rng(seed, 2), case["events"]) if case["weights"] else None


def _network(seed):
    """Float32 parameters of the surrogate: hidden layers of unit gain, an output near the mean slope
    d log|M|^2 / d kappa of the sample."""
    r = np.random.default_rng([int(seed), 3])
    out = []
    for k in (64, 256, 256, 256):
        w = r.normal(0.0, math.sqrt(2.0 / min(k, 53)), (256, k))
        w[:, 53:] *= k != 64
        out += [w, r.normal(0.0, 0.05, 256)]
    return np.concatenate([x.reshape(-1) for x in out + [r.normal(0.0, 0.02, 256), np.array([5.0])]]).astype(
        np.float32)


def _features(mom):
    """[n, 53] float64 features of g g -> t tbar g g events (column 24, kappa, left at zero)."""
    rs = mom[0, 0] + mom[1, 0]
    cols = [mom[i, m] * 2.0 / rs for i in range(6) for m in range(4)] + [torch.zeros_like(rs)]
    v = []
    for i, j in itertools.combinations(range(6), 2):
        if (i, j) != (0, 1):
            d = mom[i, 0] * mom[j, 0] - (mom[i, 1:] * mom[j, 1:]).sum(0)
            v.append(2.0 * d / rs ** 2)
    return torch.stack(cols + v + [torch.log(x.clamp_min(1e-12)) for x in v], 1)


def _samples(case, seed):
    """Rows of a training batch: features, kappa - 1, targets (float32, on the GPU)."""
    m = case["events"]
    x = _features(_events(case["proc"], m, seed))
    g = _rng(seed, 4)
    kd = 0.4 * _u(g, m) - 0.2
    x[:, 24] = kd / 0.2
    y = kd * (5.0 + 0.5 * torch.randn(m, generator=g, device=DEV, dtype=torch.float64))
    return x.float().contiguous(), kd.float(), y.float()


def prepare(case, seed):
    import paper_2312_07440_amd as mg

    p = mg.Process(case["proc"], case["prec"])
    if case["kind"] in ("surrogate", "step"):
        p.set_surrogate_params(_network(seed))
    if case["kind"] == "step":
        return dict(kind="step", p=p, rows=_samples(case, seed))
    p.set_params(_points(case, seed))
    return dict(kind=case["kind"], p=p, mom=_events(case["proc"], case["events"], seed), w=_weights(case, seed))


def run(state):
    p = state["p"]
    if state["kind"] == "reweight":
        return p.reweight(state["mom"], w_in=state["w"])
    if state["kind"] == "kpoly":
        return p.reweight_kpoly(state["mom"], w_in=state["w"])
    if state["kind"] == "surrogate":
        w, stats, fell_back = p.reweight_surrogate(state["mom"], w_in=state["w"], max_audit_error=10.0)
        return {"weights": w, "stats": stats, "fell_back": fell_back}
    pred, grad, loss = p.surrogate_fwd_bwd(*state["rows"])
    return {"pred": pred, "grad": grad, "loss": loss}


def work(case):
    n, pts, P = case["events"], case["points"], PROCS[case["proc"]]
    if case["kind"] == "step":
        return {"bytes": 4.0 * n * (53 + 3) + 8.0 * 214273, "flops": 3.0 * n * MLP_FLOPS}
    b = 32.0 * n * (2 + len(P["masses"])) + 8.0 * n * pts + (8.0 * n if case["weights"] else 0.0)
    # every diagram once per event and helicity configuration, the colour sum at every point
    colour = P["hel"] * (2 * P["flows"] ** 2 + 4 * P["flows"])
    f = n * (P["hel"] * CHAIN_FLOPS[case["proc"]] + (pts + 1) * colour)
    if case["kind"] == "surrogate":
        f = 0.01 * f + 1.0 * n * pts * MLP_FLOPS
    return {"bytes": b, "flops": float(f)}


# ------------------------------------------------------- values in 64 bits
#
# g g -> t tbar + n g by the recursion over colour-ordered words (Berends and
# Giele, Nucl. Phys. B306 (1988) 759), every power of kappa apart, linear
# polarisations and any complete pair of top spinors (both sums over
# helicities do not depend on the basis), the colour matrix as explicit sums
# over Gell-Mann matrices.

def _gellmann():
    t = np.zeros((8, 3, 3), complex)
    for k, (i, j) in enumerate([(0, 1), (0, 2), (1, 2)]):
        t[2 * k, i, j] = t[2 * k, j, i] = 1
        t[2 * k + 1, i, j], t[2 * k + 1, j, i] = -1j, 1j
    t[6], t[7] = np.diag([1, -1, 0]), np.diag([1, 1, -2]) / math.sqrt(3)
    return t / 2


def _colour(ng):
    """CF[s, r] = sum over colours of (T^s)_ij conj((T^r)_ij) for the ng! orders s, r."""
    t = W = _gellmann()
    for _ in range(ng - 1):
        W = np.tensordot(W, t, (-1, 1))                  # [a.., i, b, j]
        W = np.moveaxis(W, -2, -3)                       # [a.., b, i, j]
    words = list(itertools.permutations(range(ng)))
    flat = {}

    def rel(s, r):
        key = tuple(s.index(x) for x in r)
        if key not in flat:   # the matrices in the order of r, with the colour of each gluon where s has it
            V = np.transpose(W, [key.index(i) for i in range(ng)] + [ng, ng + 1])
            flat[key] = float(np.vdot(V, W).real)
        return flat[key]

    return words, np.array([[rel(s, r) for r in words] for s in words])


def _dot(a, b):
    return a[0] * b[0] - a[1] * b[1] - a[2] * b[2] - a[3] * b[3]


def _row_slash(a, J):
    """Row spinor times slashed vector, chiral representation."""
    p, m, t, s = J[0] + J[3], J[0] - J[3], J[1] + 1j * J[2], J[1] - 1j * J[2]
    return [a[2] * p + a[3] * t, a[2] * s + a[3] * m, a[0] * m - a[1] * t, a[1] * p - a[0] * s]


def _slash_col(J, v):
    p, m, t, s = J[0] + J[3], J[0] - J[3], J[1] + 1j * J[2], J[1] - 1j * J[2]
    return [m * v[2] - s * v[3], p * v[3] - t * v[2], p * v[0] + s * v[1], t * v[0] + m * v[1]]


def _add(a, b):
    return b if a is None else [x + y for x, y in zip(a, b)]


def _kappa_coefficients(mom, ng, words, cf):
    """[2 ng - 1, n]: coefficients of kappa^2 .. kappa^(2 ng) of sum_h J^+ CF J at unit g_s."""
    n, hel = mom.shape[2], 1 << (ng + 2)
    c = lambda x: x[None].to(torch.complex128)   # noqa: E731
    h = torch.arange(hel, device=mom.device)
    bit = lambda k: ((h >> k) & 1).bool()[:, None]   # noqa: E731
    zero = torch.zeros(hel, n, dtype=torch.complex128, device=mom.device)
    gl = [0, 1] + list(range(4, ng + 2))
    J, P = {}, {}
    for i, g in enumerate(gl):
        k = mom[g]
        kt, ka = torch.hypot(k[1], k[2]), torch.sqrt((k[1:] ** 2).sum(0))
        safe = torch.where(kt > 0, kt, torch.ones_like(kt))
        cp, sp = torch.where(kt > 0, k[1] / safe, torch.ones_like(kt)), k[2] / safe
        e1, e2 = [k[3] / ka * cp, k[3] / ka * sp, -kt / ka], [-sp, cp, torch.zeros_like(sp)]
        J[(i,)] = [zero] + [torch.where(bit(i), c(a), c(b)) for a, b in zip(e1, e2)]
        P[(i,)] = [(x if g < 2 else -x)[None] for x in k]
    for m in range(2, ng + 1):
        for w in itertools.permutations(range(ng), m):
            P[w] = [sum(x) for x in zip(P[w[:1]], P[w[1:]])]
            acc = None
            for a in range(1, m):
                u, v = w[:a], w[a:]
                A, B, p, q = J[u], J[v], P[u], P[v]
                ab, ad, bd = _dot(A, B), _dot(A, [x + 2 * y for x, y in zip(p, q)]), _dot(B, [2 * x + y for x, y in zip(p, q)])
                acc = _add(acc, [-(ab * (p[i] - q[i]) + ad * B[i] - bd * A[i]) for i in range(4)])
                for b in range(a + 1, m):
                    X, Y, Z = J[w[:a]], J[w[a:b]], J[w[b:]]
                    xy, xz, yz = _dot(X, Y), _dot(X, Z), _dot(Y, Z)
                    acc = _add(acc, [2 * Y[i] * xz - Z[i] * xy - X[i] * yz for i in range(4)])
            J[w] = [x / _dot(P[w], P[w]) for x in acc]
    pt, pb = [x[None] for x in mom[2]], [x[None] for x in mom[3]]
    one = torch.ones_like(pt[0]).to(torch.complex128)
    up = [torch.where(bit(ng), one, 0 * one), torch.where(bit(ng), 0 * one, one)]
    ub = [x / torch.sqrt(2 * (pt[0] + MT)) for x in _add(_row_slash(up + up, pt), [MT * x for x in up + up])]
    dn = [torch.where(bit(ng + 1), one, 0 * one), torch.where(bit(ng + 1), 0 * one, one)]
    dn = dn + [-x for x in dn]
    v = [(x - MT * y) / torch.sqrt(2 * (pb[0] + MT)) for x, y in zip(_slash_col(pb, dn), dn)]
    psi = {(): {0: ub}}
    for m in range(1, ng):
        for w in itertools.permutations(range(ng), m):
            q = [a - b for a, b in zip(pt, P[w])]
            den, d = _dot(q, q) - MT * MT, {}
            for a in range(m):
                for k, s in psi[w[:a]].items():
                    x = _row_slash(s, J[w[a:]])
                    y = _row_slash(x, q)
                    d[k + 1] = _add(d.get(k + 1), [-(y[i] + MT * x[i]) / den for i in range(4)])
            psi[w] = d
    amp = {k: [zero] * len(words) for k in range(1, ng + 1)}
    for f, w in enumerate(words):
        for a in range(ng):
            for k, s in psi[w[:a]].items():
                x = _row_slash(s, J[w[a:]])
                amp[k + 1][f] = amp[k + 1][f] + sum(x[i] * v[i] for i in range(4))
    CF = torch.tensor(cf, device=mom.device, dtype=torch.complex128)
    amp = {k: torch.stack(x).reshape(len(words), -1) for k, x in amp.items()}
    out = torch.zeros(2 * ng - 1, n, dtype=torch.float64, device=mom.device)
    for b in amp:
        z = CF @ amp[b]
        for a in amp:
            out[a + b - 2] += (amp[a].conj() * z).real.sum(0).reshape(hel, n).sum(0)
    return out


def _exact_ratio(case, mom, points):
    """|M_k|^2 / |M_base|^2, [points, n]."""
    n = mom.shape[2]
    if case["proc"] == "ee_5a":
        r = torch.tensor([(q["alpha"] / ALPHA) ** 5 for q in points], device=mom.device, dtype=torch.float64)
        return r[:, None].expand(-1, n).clone()
    ng = PROCS[case["proc"]]["ng"]
    words, cf = _colour(ng)
    out = torch.empty(len(points), n, dtype=torch.float64, device=mom.device)
    step = {2: 1 << 17, 3: 1 << 15, 4: 1 << 12, 5: 512}[ng]
    for e in range(0, n, step):
        c = _kappa_coefficients(mom[:, :, e:e + step].contiguous(), ng, words, cf)
        base = c.sum(0)
        for i, q in enumerate(points):
            k, me = q["kappa_ttg"], torch.zeros_like(base)
            for j in range(c.shape[0]):
                me += c[j] * k ** (j + 2)
            out[i, e:e + step] = me / base * (q["alphas"] / ALPHAS) ** ng
    return out


def _layers(par):
    out, o = [], 0
    for k in (64, 256, 256, 256):
        out.append((par[o:o + 256 * k].reshape(256, k), par[o + 256 * k:o + 256 * k + 256]))
        o += 256 * k + 256
    return out, par[o:o + 256], par[o + 256]


def _forward(x, par):
    layers, w5, b5 = _layers(par)
    a = torch.nn.functional.pad(x, (0, 64 - x.shape[1]))
    for W, b in layers:
        a = torch.nn.functional.silu(a @ W.T + b)
    return a @ w5 + b5


def exact(case, seed):
    par = torch.tensor(_network(seed), device=DEV, dtype=torch.float64) if case["kind"] in ("surrogate", "step") else None
    if case["kind"] == "step":
        x, kd, y = (t.double() for t in _samples(case, seed))
        par.requires_grad_(True)
        pred = kd * _forward(x, par)
        loss = ((pred - y) ** 2).mean()
        loss.backward()
        # input columns 53 .. 63 of the first layer are unused
        return {"pred": pred.detach(), "grad": par.grad, "loss": loss.detach()}
    most = {"gg_tt": 1 << 20, "gg_ttg": 300000, "gg_ttgg": 40000, "gg_ttggg": 1500, "ee_5a": 1 << 20}
    if case["events"] > most[case["proc"]]:
        return None
    mom, w, pts = _events(case["proc"], case["events"], seed), _weights(case, seed), _points(case, seed)
    if case["kind"] == "surrogate":
        return None   # most events carry the network's value, about 1 % the exact one, chosen by the library
    r = _exact_ratio(case, mom, pts)
    return r if w is None else r * w
