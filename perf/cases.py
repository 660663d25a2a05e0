"""The work a user of the library has it do, as cases that can be timed.

Four ways a program uses a ``Problem``: gradients for an optimiser of its own
(``grad``: ``loss_and_grad``; ``static``: the allocation-free entry point;
``autograd``: ``DDPLoss`` under torch), training with the built-in Adam and a
checkpoint at the end (``train``: ``step`` then ``get_state``), and the
stitched solution at points it chooses (``eval``).

Sizes are those of the repository's workloads (``workloads.py``), scaled, or a
grid of boxes with widths, depths and counts of its own.  The shape of a case
(widths, depths, counts, cells) is fixed by the case; points, targets and
parameters come from the seed.
"""
import functools
import math

import numpy as np
import torch

from paper_2104_10013_amd import ddpinn, workloads as W

DEVICE = "cuda"


# ---------------------------------------------------------------------------
# the cases


def listed():
    return [
        # the smallest training run: 4 subdomains, 20-wide networks, 4000
        # points, 100 Adam steps (the paper's first example); latency bound
        {"name": "train_poisson_2x2", "do": "train", "workload": "c1_cpinn_poisson", "scale": 1.0, "steps": 100},
        # the benchmark: 16 uneven subdomains, widths 20..80, 143k points
        {"name": "train_poisson_4x4", "do": "train", "workload": "c2_xpinn_poisson", "scale": 1.0, "steps": 20},
        # the same problem driven by a torch optimiser through autograd
        {"name": "autograd_poisson_4x4", "do": "autograd", "workload": "c2_xpinn_poisson", "scale": 1.0},
        # 8 strips, six hidden layers of 50 (a padded width), cPINN fluxes
        {"name": "grad_burgers_strips", "do": "grad", "workload": "c3_cpinn_burgers", "scale": 1.0},
        # three outputs, 60-wide networks, 90k points
        {"name": "grad_navier_stokes_3x3", "do": "grad", "workload": "c4_xpinn_kovasznay", "scale": 1.0},
        # the largest: two networks per cell, widths 20..100, 170k points
        {"name": "grad_inverse", "do": "grad", "workload": "c5_xpinn_inverse_diffusion", "scale": 1.0},
        # tanh / sin / cos networks with trainable slopes
        {"name": "grad_inverse_adaptive", "do": "grad", "workload": "c5_table4_adaptive", "scale": 1.0},
        # many equal narrow networks (20 x 5), 80k points, space-time boxes
        {"name": "train_burgers_space_time", "do": "train", "workload": "burgers_st_xpinn_4x4", "scale": 1.0,
         "steps": 20},
        # odd everything: widths 9..112, depths 1..6, ragged counts, cPINN
        # Navier-Stokes fluxes
        {"name": "grad_ragged_boxes", "do": "grad", "pde": W.PDE_NS2D, "method": W.METHOD_CPINN, "nx": 3, "ny": 2,
         "w_lo": 9, "w_hi": 112, "d_lo": 1, "d_hi": 6, "n_res": 7013, "n_bnd": 37, "n_iface": 67, "shape": 5,
         "act": "tanh", "adaptive": False},
        # a probe of the solution at a few points between training steps
        {"name": "eval_few_points", "do": "eval", "workload": "c1_cpinn_poisson", "scale": 0.1, "points": 5},
        # the reporting grid of the benchmark problem (201 x 201)
        {"name": "eval_grid_poisson", "do": "eval", "workload": "c2_xpinn_poisson", "scale": 0.1, "points": 40401},
        # a fine grid of a three-output solution, as for plotting
        {"name": "eval_fine_navier_stokes", "do": "eval", "workload": "c4_xpinn_kovasznay", "scale": 0.1,
         "points": 1002001},
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


_DRAWN_WORKLOADS = ("c1_cpinn_poisson", "c2_xpinn_poisson", "c3_cpinn_burgers", "c4_xpinn_kovasznay",
                    "c5_xpinn_inverse_diffusion", "c5_table4_adaptive", "burgers_st_cpinn_8x1",
                    "burgers_st_xpinn_4x4", "burgers_st_hybrid_4x4", "ns_cpinn_kovasznay")


def draw(rng):
    do = rng.choice(("grad", "grad", "grad", "autograd", "static", "train", "train", "eval", "eval"))
    if rng.random() < 0.5:
        case = {"do": do, "workload": rng.choice(_DRAWN_WORKLOADS), "scale": round(_log_uniform(rng, 0.03, 1.0), 4)}
    else:
        w_lo = rng.randint(8, 96)
        d_lo = rng.randint(1, 6)
        nx, ny = rng.randint(1, 5), rng.randint(1, 4)
        case = {"do": do, "pde": rng.choice((W.PDE_POISSON2D, W.PDE_BURGERS1D, W.PDE_NS2D)),
                "method": rng.choice((W.METHOD_CPINN, W.METHOD_XPINN)), "nx": nx, "ny": ny,
                "w_lo": w_lo, "w_hi": rng.randint(w_lo, 112), "d_lo": d_lo, "d_hi": rng.randint(d_lo, 7),
                "n_res": int(_log_uniform(rng, 200, 90000)), "n_bnd": rng.randint(1, 120),
                "n_iface": rng.randint(1, 250), "shape": rng.randint(0, 10 ** 6),
                "act": rng.choice(("tanh", "tanh", "tanh", "sin", "mixed")), "adaptive": rng.random() < 0.3}
    if do == "train":
        case["steps"] = rng.choice((1, 5, 20))
    if do in ("grad", "train") and rng.random() < 0.15:
        case["per_subdomain"] = True
    if do == "eval":
        case["points"] = int(_log_uniform(rng, 1, 1000000))
        if "workload" in case:
            case["scale"] = 0.1
        else:
            case["n_res"] = min(case["n_res"], 2000)
    # at most the largest listed case's work
    most = work(listed()[5])["flops"]
    while do != "eval" and work(case)["flops"] > most:
        if "scale" in case:
            case["scale"] = round(case["scale"] * 0.8, 4)
        elif case.get("steps", 1) > 1:
            case["steps"] = 1
        else:
            case["n_res"] = int(case["n_res"] * 0.8)
    return case


# ---------------------------------------------------------------------------
# the problem of a case


def _key(case):
    return tuple(sorted((k, v) for k, v in case.items() if k not in ("name", "do", "steps", "points", "per_subdomain")))


@functools.lru_cache(maxsize=8)
def _base(key):
    """The problem whose shape (widths, depths, counts, cells) the case has."""
    case = dict(key)
    if "workload" in case:
        return W.make_problem(case["workload"], seed=0, scale=case["scale"])
    return _boxes(case, 0)


def _boxes(case, seed):
    rng = np.random.default_rng(case["shape"])
    n = case["nx"] * case["ny"]
    d_out = W.PDE_DOUT[case["pde"]]
    widths = [[2] + [int(rng.integers(case["w_lo"], case["w_hi"] + 1))] * int(rng.integers(case["d_lo"], case["d_hi"] + 1))
              + [d_out] for _ in range(n)]
    share = rng.uniform(0.3, 1.7, n)
    counts = [max(1, int(round(case["n_res"] * s / share.sum()))) for s in share]
    coef = {W.PDE_POISSON2D: (), W.PDE_BURGERS1D: (0.01 / math.pi,), W.PDE_NS2D: (40.0,)}[case["pde"]]
    prob = W.custom_box_problem(case["method"], case["pde"], case["nx"], case["ny"], widths, counts, case["n_bnd"],
                                case["n_iface"], seed=seed, coef=coef)
    acts = ("tanh", "sin", "cos") if case["act"] == "mixed" else (case["act"],)
    if case["adaptive"] or acts != ("tanh",):
        W.with_activations(prob, acts, adaptive=case["adaptive"])
    return prob


def _problem(case, seed):
    """Points, targets and parameters of the seed in the shape of the case.
    The parameters are away from initialisation (nonzero biases)."""
    base = _base(_key(case))
    name = case.get("workload", "")
    if not name:
        prob = _boxes(case, seed)
    elif name == "c2_xpinn_poisson":   # its widths and counts come from its seed
        prob = W.custom_box_problem(base.method, base.pde, 4, 4, [s.widths for s in base.subdomains],
                                    [len(s.res_xy) for s in base.subdomains], max(1, int(round(50 * case["scale"]))),
                                    len(base.interfaces[0].xy), seed=seed)
    elif name.startswith("c5_"):       # so do its cells: the points move inside them
        prob = _moved(base, seed)
    else:
        prob = W.make_problem(name, seed=seed, scale=case["scale"])
    for q, s in enumerate(prob.subdomains):
        s.params = W.perturb_params(s.params, [seed, q], 0.1)
    return prob


def _moved(base, seed):
    """The inverse problem with other points, noise and parameters, at the
    learning rate at which it identifies the conductivity."""
    rng = np.random.default_rng(seed)
    jitter = lambda xy: (xy + 1e-3 * rng.standard_normal(xy.shape)).astype(np.float32)  # noqa: E731
    subs = []
    for s in base.subdomains:
        res, bnd, aux = (rng.permutation(jitter(v)) for v in (s.res_xy, s.bnd_xy, s.aux_xy))
        f = W.diffusion_fields(res[:, 0].astype(float), res[:, 1].astype(float))[2]
        u = W.diffusion_fields(bnd[:, 0].astype(float), bnd[:, 1].astype(float))[0]
        k = W.diffusion_fields(aux[:, 0].astype(float), aux[:, 1].astype(float))[1]
        u = u + 0.005 * rng.standard_normal(u.shape)
        params = np.concatenate([W.glorot_params(rng, w, s.adaptive) for w in (s.widths, s.aux_widths)])
        subs.append(W.Subdomain(widths=list(s.widths), loss_w=s.loss_w, lr=1e-3, res_xy=res,
                                res_f=f.astype(np.float32)[:, None], bnd_xy=bnd, bnd_g=u.astype(np.float32)[:, None],
                                params=params, aux_widths=list(s.aux_widths), aux_xy=aux,
                                aux_g=k.astype(np.float32)[:, None], act=s.act, adaptive=s.adaptive))
    return W.Problem(name=base.name, method=base.method, pde=base.pde, coef=base.coef, subdomains=subs,
                     interfaces=[W.Interface(e.a, e.b, jitter(e.xy), e.normal) for e in base.interfaces],
                     meta=base.meta)


def _eval_points(case, prob, seed):
    """(xy, owner): a grid over the domain in row order (few points: scattered),
    with the subdomains whose closure holds each point."""
    n = case["points"]
    rng = np.random.default_rng([seed, 7])
    if prob.pde == W.PDE_DIFFUSION2D_INV:
        pick = rng.integers(0, len(_base(_key(case)).eval_xy), n)
        if n >= 1000:
            pick = np.sort(pick)
        b = _base(_key(case))
        return b.eval_xy[pick] + np.float32(1e-4) * rng.standard_normal((n, 2)).astype(np.float32), b.eval_owner[pick]
    every = np.concatenate([e.xy for e in prob.interfaces] + [s.res_xy for s in prob.subdomains])
    lo, hi = every.min(0), every.max(0)
    if n >= 1000:
        side = int(math.isqrt(n))
        i = np.arange(n)
        xy = np.stack([(i // side) / max(1, (n - 1) // side), (i % side) / (side - 1)], 1)
        xy = xy + 0.2 / side * (rng.random(2) - 0.5)
    else:
        xy = rng.random((n, 2))
    xy = (lo + np.clip(xy, 0, 1) * (hi - lo)).astype(np.float32)
    # closed boxes around each subdomain's residual points, from the grid lines
    owner = -np.ones((n, 4), np.int32)
    used = np.zeros(n, np.int64)
    for q, (x0, x1, y0, y1) in enumerate(_rectangles(case, prob, lo, hi)):
        at = np.nonzero((xy[:, 0] >= x0) & (xy[:, 0] <= x1) & (xy[:, 1] >= y0) & (xy[:, 1] <= y1))[0]
        at = at[used[at] < 4]
        owner[at, used[at]] = q
        used[at] += 1
    return xy, owner


def _rectangles(case, prob, lo, hi):
    name = case.get("workload", "")
    if not name:
        nx, ny = case["nx"], case["ny"]
    elif name.startswith("burgers_st"):
        nx, ny = prob.meta["nx"], prob.meta["nt"]
    elif name == "c3_cpinn_burgers":
        nx, ny = prob.n_sd, 1
    else:
        nx = ny = math.isqrt(prob.n_sd)
    xs, ys = np.linspace(lo[0], hi[0], nx + 1), np.linspace(lo[1], hi[1], ny + 1)
    return [(xs[i], xs[i + 1], ys[j], ys[j + 1]) for j in range(ny) for i in range(nx)]


# ---------------------------------------------------------------------------
# preparation and one pass


def _adam_state(prob, seed):
    """The state of a run that has been training for a while."""
    rng = np.random.default_rng([seed, 3])
    n = sum(s.params.size for s in prob.subdomains)
    v = (0.1 * (0.5 + rng.random(n))) ** 2
    m = 0.3 * np.sqrt(v) * rng.standard_normal(n)
    return {"params": [s.params for s in prob.subdomains], "m": m.astype(np.float32), "v": v.astype(np.float32),
            "t": 1000}


def prepare(case, seed):
    prob = _problem(case, seed)
    pb = ddpinn.Problem(prob, fused=not case.get("per_subdomain", False), device=DEVICE)
    state = {"do": case["do"], "pb": pb}
    if case["do"] == "train":
        pb.set_state(_adam_state(prob, seed))
        state["steps"] = case["steps"]
    elif case["do"] == "autograd":
        flat = np.concatenate([s.params for s in prob.subdomains])
        state["theta"] = torch.tensor(flat, device=DEVICE, requires_grad=True)
    elif case["do"] == "eval":
        state["xy"], state["owner"] = _eval_points(case, prob, seed)
    return state


def run(state):
    pb, do = state["pb"], state["do"]
    if do == "train":
        terms = pb.step(state["steps"])
        st = pb.get_state()   # the checkpoint
        return {"terms": terms, "params": np.concatenate(st["params"]), "m": st["m"], "v": st["v"]}
    if do == "autograd":
        theta = state["theta"]
        theta.grad = None
        J = ddpinn.DDPLoss.apply(theta, pb)
        J.sum().backward()
        return {"J": J, "grad": theta.grad}
    if do == "eval":
        return {"u": pb.eval(state["xy"], state["owner"])}
    terms, grad = pb.loss_and_grad_static() if do == "static" else pb.loss_and_grad()
    return {"terms": terms, "grad": grad}


# ---------------------------------------------------------------------------
# what a pass cannot do without


def _net_shapes(s):
    return [s.widths] + ([s.aux_widths] if s.aux_widths is not None else [])


def _madds(widths):
    return sum(a * b for a, b in zip(widths[:-1], widths[1:]))


def work(case):
    """Multiply-adds of the layers (all of them, unpadded) over the streams
    each point needs: value, gradient and second order at residual points and
    XPINN interfaces, value and normal derivative at cPINN interfaces, value at
    data; forward once, the two reverse products once.  Interface values of
    the neighbour are its own forward.  Bytes: points, parameters, gradients,
    Adam state, outputs."""
    prob = _base(_key(case))
    n_par = sum(s.params.size for s in prob.subdomains)
    cols = prob.d_out + (1 if prob.pde == W.PDE_DIFFUSION2D_INV else 0)
    if case["do"] == "eval":
        per = sum(2.0 * _madds(w) for s in prob.subdomains for w in _net_shapes(s)) / prob.n_sd
        return {"flops": case["points"] * per, "bytes": case["points"] * (8.0 + 16.0 + 4.0 * cols) + 4.0 * n_par}
    n_if = [0] * prob.n_sd
    for e in prob.interfaces:
        s_if = 4 if (e.method or prob.method) == W.METHOD_XPINN else 2
        n_if[e.a] += s_if * len(e.xy)
        n_if[e.b] += s_if * len(e.xy)
    flops, nbytes = 0.0, 0.0
    for q, s in enumerate(prob.subdomains):
        columns = [4 * len(s.res_xy) + len(s.bnd_xy) + n_if[q]]
        if s.aux_widths is not None:
            columns.append(3 * len(s.res_xy) + len(s.aux_xy) + 3 * n_if[q] // 4)
        flops += sum(6.0 * c * _madds(w) for c, w in zip(columns, _net_shapes(s)))
        nbytes += 4.0 * (len(s.res_xy) * (2 + prob.n_eq) + len(s.bnd_xy) * (2 + prob.d_out))
        nbytes += 12.0 * len(s.aux_xy) if s.aux_widths is not None else 0.0
    nbytes += 8.0 * sum(len(e.xy) for e in prob.interfaces)
    steps = case.get("steps", 1)
    nbytes += 4.0 * n_par * (6.0 if case["do"] == "train" else 2.0)
    return {"flops": flops * steps, "bytes": nbytes * steps}


# ---------------------------------------------------------------------------
# the same in 64 bits


def _t(a):
    return torch.as_tensor(np.asarray(a, np.float64), device=DEVICE)


def _phi(act, y):
    """The activation and its first two derivatives."""
    if act == "tanh":
        t = torch.tanh(y)
        d = 1 - t * t
        return t, d, -2 * t * d
    s, c = torch.sin(y), torch.cos(y)
    return (s, c, -s) if act == "sin" else (c, -s, -c)


def _network(theta, widths, s, z, pde, derivatives=True):
    """Outputs (N, d_out) and, with derivatives, those of the two inputs and
    the second-order sum the operator needs, carried through the layers."""
    h, off, layers = z, 0, []
    for a, b in zip(widths[:-1], widths[1:]):
        layers.append((theta[off:off + a * b].reshape(b, a), theta[off + a * b:off + a * b + b]))
        off += a * b + b
    d1, d2, sec = torch.zeros_like(z), torch.zeros_like(z), torch.zeros_like(z)
    d1[:, 0] = 1
    d2[:, 1] = 1
    for k, (w, b) in enumerate(layers):
        h = h @ w.T + b
        if derivatives:
            d1, d2, sec = d1 @ w.T, d2 @ w.T, sec @ w.T
        if k == len(layers) - 1:
            break
        c = s.slope_n * theta[off + k] if s.adaptive else 1.0
        p0, p1, p2 = _phi(s.act, c * h)
        if derivatives:
            d1, d2, sec = c * d1, c * d2, c * sec
            square = d1 * d1 if pde == W.PDE_BURGERS1D else d1 * d1 + d2 * d2
            d1, d2, sec = p1 * d1, p1 * d2, p1 * sec + p2 * square
        h = p0
    return h, d1, d2, sec


def _size(s, widths):
    return sum(a * b + b for a, b in zip(widths[:-1], widths[1:])) + (len(widths) - 2 if s.adaptive else 0)


def _halves(s, theta):
    n = _size(s, s.widths)
    return theta[:n], theta[n:]


def _operator(prob, s, theta, z):
    """(values, L(u)) at the points z; the inverse problem's values are (u, K)."""
    thu, thk = _halves(s, theta)
    u, ux, uy, ul = _network(thu, s.widths, s, z, prob.pde)
    if prob.pde == W.PDE_POISSON2D:
        return u, -ul, (ux, uy)
    if prob.pde == W.PDE_BURGERS1D:
        return u, uy + u * ux - prob.coef[0] * ul, (ux, uy)
    if prob.pde == W.PDE_NS2D:
        re, U, V = prob.coef[0], u[:, 0], u[:, 1]
        L = torch.stack([U * ux[:, 0] + V * uy[:, 0] + ux[:, 2] - ul[:, 0] / re,
                         U * ux[:, 1] + V * uy[:, 1] + uy[:, 2] - ul[:, 1] / re, ux[:, 0] + uy[:, 1]], 1)
        return u, L, (ux, uy)
    k, kx, ky, _ = _network(thk, s.aux_widths, s, z, prob.pde)
    return torch.cat([u, k], 1), k * ul + kx * ux + ky * uy, (ux, uy)


def _interface(prob, e, s, theta):
    u, L, (ux, uy) = _operator(prob, s, theta, _t(e.xy))
    if (e.method or prob.method) == W.METHOD_XPINN:
        return u, L
    nx, ny = (float(v) for v in e.normal)
    if prob.pde == W.PDE_POISSON2D:
        return u, -(nx * ux + ny * uy)
    if prob.pde == W.PDE_BURGERS1D:
        return u, nx * (0.5 * u * u - prob.coef[0] * ux) + ny * u
    re, U, V, P = prob.coef[0], u[:, 0], u[:, 1], u[:, 2]
    normal = nx * ux + ny * uy
    return u, torch.stack([nx * (U * U + P) + ny * U * V - normal[:, 0] / re,
                           nx * U * V + ny * (V * V + P) - normal[:, 1] / re, nx * U + ny * V], 1)


def _mean(x):
    return (x * x).sum() / max(1, x.shape[0])


def _terms_and_grads(prob, thetas):
    sides = {}   # each side's interface values, as the neighbour receives them
    with torch.no_grad():
        for i, e in enumerate(prob.interfaces):
            for q in (e.a, e.b):
                sides[i, q] = _interface(prob, e, prob.subdomains[q], thetas[q])
    terms, grads = [], []
    for q, s in enumerate(prob.subdomains):
        theta = thetas[q].detach().requires_grad_(True)
        thu, thk = _halves(s, theta)
        t = [torch.zeros((), dtype=torch.float64, device=DEVICE) for _ in range(4)]
        t[0] = t[0] + _mean(_network(thu, s.widths, s, _t(s.bnd_xy), prob.pde, False)[0] - _t(s.bnd_g))
        if s.aux_widths is not None:
            t[0] = t[0] + _mean(_network(thk, s.aux_widths, s, _t(s.aux_xy), prob.pde, False)[0] - _t(s.aux_g))
        t[1] = t[1] + _mean(_operator(prob, s, theta, _t(s.res_xy))[1] - _t(s.res_f))
        for i, e in enumerate(prob.interfaces):
            if q in (e.a, e.b):
                u, o = _interface(prob, e, s, theta)
                un, on = sides[i, e.b if q == e.a else e.a]
                t[2] = t[2] + 0.25 * _mean(u - un)
                t[3] = t[3] + _mean(o - on)
        J = sum(float(np.float32(w)) * v for w, v in zip(s.loss_w, t))
        grads.append(torch.autograd.grad(J, theta)[0])
        terms.append(torch.stack([J] + t).detach())
    return torch.stack(terms), grads


def exact(case, seed):
    prob = _problem(case, seed)
    thetas = [_t(s.params) for s in prob.subdomains]
    if case["do"] == "eval":
        xy, owner = _eval_points(case, prob, seed)
        own = torch.as_tensor(owner, device=DEVICE)
        cols = prob.d_out + (1 if prob.pde == W.PDE_DIFFUSION2D_INV else 0)
        out = torch.zeros(len(xy), cols, dtype=torch.float64, device=DEVICE)
        z = _t(xy)
        for q, s in enumerate(prob.subdomains):
            at = (own == q).any(1).nonzero()[:, 0]
            if len(at):
                thu, thk = _halves(s, thetas[q])
                u = _network(thu, s.widths, s, z[at], prob.pde, False)[0]
                if s.aux_widths is not None:
                    u = torch.cat([u, _network(thk, s.aux_widths, s, z[at], prob.pde, False)[0]], 1)
                out[at] += u
        return {"u": out / (own >= 0).sum(1).clamp(min=1)[:, None]}
    if case["do"] == "train":
        st = _adam_state(prob, seed)
        sizes = [s.params.size for s in prob.subdomains]
        m, v = (list(torch.split(_t(st[k]), sizes)) for k in ("m", "v"))
        b1, b2, eps = (float(np.float32(c)) for c in (0.9, 0.999, 1e-8))
        for t in range(st["t"] + 1, st["t"] + 1 + case["steps"]):
            terms, grads = _terms_and_grads(prob, thetas)
            for q, s in enumerate(prob.subdomains):
                m[q] = b1 * m[q] + (1 - b1) * grads[q]
                v[q] = b2 * v[q] + (1 - b2) * grads[q] ** 2
                step = (m[q] / (1 - b1 ** t)) / ((v[q] / (1 - b2 ** t)).sqrt() + eps)
                thetas[q] = thetas[q] - float(np.float32(s.lr)) * step
        return {"terms": terms, "params": torch.cat(thetas), "m": torch.cat(m), "v": torch.cat(v)}
    terms, grads = _terms_and_grads(prob, thetas)
    if case["do"] == "autograd":
        return {"J": terms[:, 0], "grad": torch.cat(grads)}
    return {"terms": terms, "grad": torch.cat(grads)}
