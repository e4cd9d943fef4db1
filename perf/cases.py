"""The workloads that the library's speed is measured on.

Every case is one pass through the package's public entry points, at the
sizes that programs use them: from a single outline's curves, where the call
itself is the cost, to a whole frame of a large scene.  ``listed()`` names the
fixed ones; ``draw()`` gives further ones of the same kinds and ranges, odd
and ragged sizes among them.

Kinds
  curves  curves (rational ones too) sampled at parameters
  train   curve evaluation and its gradients through autograd
  fit     Adam steps of the least-squares curve fit, in place
  batch   a mixed batch behind a kept plan
  encode  a C0 chain turned into its texel grid and its cache-line tiles
  chain   random-access evaluation of an encoded chain
  grid    tessellation of surface patches on a uniform grid
  points  surfaces and volumes at scattered parameters
"""
import math

import torch

import paper_2603_15447_amd as bz

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZES = {"f32": 4, "f16": 2, "bf16": 2}


def listed():
    return [
        # one glyph's or icon's outline: a handful of 2D cubics, where the cost is the call
        {"name": "outline", "kind": "curves", "n": 64, "n_t": 32, "degree": 3, "dim": 2, "dtype": "f32",
         "method": "decasteljau", "shared": True, "rational": False},
        # a frame's hair or fibre set: 4096 cubic space curves, 256 shared parameters each
        {"name": "frame_cubics", "kind": "curves", "n": 4096, "n_t": 256, "degree": 3, "dim": 3, "dtype": "f32",
         "method": "decasteljau", "shared": True, "rational": False},
        # CAD edges: many rational quintics, each sampled at its own 50 parameters
        {"name": "rational_edges", "kind": "curves", "n": 100003, "n_t": 50, "degree": 5, "dim": 3, "dtype": "f32",
         "method": "bernstein", "shared": False, "rational": True},
        # high-degree motion curves in 16-bit storage, a hundred common time stamps
        {"name": "motion_deg9_bf16", "kind": "curves", "n": 40009, "n_t": 100, "degree": 9, "dim": 4, "dtype": "bf16",
         "method": "auto", "shared": True, "rational": False},
        # one step of a program that trains rational curves with its own optimiser: forward and backward
        {"name": "train_rational", "kind": "train", "n": 16384, "n_t": 100, "degree": 3, "dim": 3, "dtype": "f32",
         "rational": True},
        # fitting scanned strokes of a few hundred samples each, 40 Adam steps between reports
        {"name": "fit_strokes", "kind": "fit", "n": 16384, "n_t": 200, "degree": 3, "dim": 3, "steps": 40},
        # a whole scene's objects in one plan: curves of every degree, rational ones and NURBS
        {"name": "batch_scene", "kind": "batch", "n_bezier": 1 << 20, "n_nurbs": 1 << 16, "n_patches": 0, "n_t": 16,
         "dim": 3, "dtype": "f32", "method": "bernstein"},
        # one drawing's objects in one plan, patches among them, an odd parameter count, 16-bit storage
        {"name": "batch_drawing_f16", "kind": "batch", "n_bezier": 3000, "n_nurbs": 200, "n_patches": 100, "n_t": 10,
         "dim": 3, "dtype": "f16", "method": "bernstein"},
        # a chain that changed since the last frame: encode it and lay out its tiles
        {"name": "encode_chain", "kind": "encode", "n_seg": 1 << 20, "dim": 3, "cubic": False},
        # random access into a long chain
        {"name": "chain_random", "kind": "chain", "n_seg": 1 << 20, "n_q": 1 << 24, "dim": 3, "layout": "tiles"},
        # tessellation into 32 x 32 quads, which have 33 x 33 corners
        {"name": "patches_33x33", "kind": "grid", "n": 16384, "du": 3, "dv": 3, "nu": 33, "nv": 33, "dim": 3,
         "dtype": "f32"},
        # free-form deformation: tricubic volumes, 256 scattered points in each
        {"name": "volume_points", "kind": "points", "n": 1 << 16, "n_per": 256, "du": 3, "dv": 3, "dw": 3, "dim": 3,
         "dtype": "f32"},
    ]


# ------------------------------------------------------------------ draws
def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _count(rng, total_lo, total_hi, per):
    """Objects of `per` queries each, for a total spread over its logarithm."""
    return max(1, _log_int(rng, total_lo, total_hi) // per)


def draw(rng):
    kind = rng.choice(["curves", "curves", "train", "fit", "batch", "encode", "chain", "grid", "points"])
    c = {"kind": kind}
    if kind == "curves":
        n_t = rng.choice([_log_int(rng, 8, 300), 64 * rng.randint(1, 6)])
        c.update(n=_count(rng, 1 << 11, 1 << 22, n_t), n_t=n_t, degree=rng.choice([2, 3, 3, 3, 4, 5, 7, 9, 11]),
                 dim=rng.choice([2, 3, 3, 4]), dtype=rng.choice(["f32", "f32", "f16", "bf16"]),
                 method=rng.choice(["decasteljau", "bernstein", "seiler", "auto"]), shared=rng.random() < 0.5,
                 rational=rng.random() < 0.3)
    elif kind == "train":
        n_t = _log_int(rng, 16, 256)
        c.update(n=_count(rng, 1 << 12, 3 << 19, n_t), n_t=n_t, degree=rng.choice([2, 3, 3, 4, 5, 7]),
                 dim=rng.choice([2, 3, 3]), dtype=rng.choice(["f32", "f32", "f32", "bf16"]),
                 rational=rng.random() < 0.5)
    elif kind == "fit":
        n_t = _log_int(rng, 40, 800)
        c.update(n=_count(rng, 1 << 14, 3 << 20, n_t), n_t=n_t, degree=rng.choice([2, 3, 3, 4, 5]),
                 dim=rng.choice([2, 3]), steps=rng.randint(10, 40))
    elif kind == "batch":
        n_t = rng.choice([8, 10, 16, 16, 25, 32])
        n = _count(rng, 1 << 14, 1 << 23, n_t)
        c.update(n_bezier=n, n_nurbs=n // 16, n_patches=rng.choice([0, n // 16]), n_t=n_t, dim=rng.choice([2, 3, 3]),
                 dtype=rng.choice(["f32", "f32", "f16", "bf16"]), method=rng.choice(["bernstein", "decasteljau"]))
    elif kind == "encode":
        c.update(n_seg=_log_int(rng, 500, 1 << 20), dim=rng.choice([2, 3, 3]), cubic=rng.random() < 0.3)
    elif kind == "chain":
        c.update(n_seg=_log_int(rng, 500, 1 << 20), n_q=_log_int(rng, 1 << 14, 1 << 24), dim=rng.choice([2, 3, 3]),
                 layout=rng.choice(["grid", "tiles", "tiles", "tiles_f16", "cubic_tiles"]))
    elif kind == "grid":
        nu = rng.choice([8, 9, 10, 16, 17, 20, 24, 32, 32, 33, 33, 50, 64, 65])
        nv = rng.choice([nu, nu, rng.randint(5, 70)])
        du = rng.choice([2, 3, 3, 3])
        c.update(n=_count(rng, 1 << 12, 1 << 24, nu * nv), du=du, dv=rng.choice([du, 2]), nu=nu, nv=nv,
                 dim=rng.choice([2, 3, 3]), dtype=rng.choice(["f32", "f32", "f16"]))
    else:
        dw = rng.choice([0, 2, 3, 3])
        n_per = _log_int(rng, 32, 1500)
        d = rng.choice([2, 3, 3])
        c.update(n=_count(rng, 1 << 13, 1 << 23, n_per), n_per=n_per, du=d, dv=d, dw=dw, dim=3,
                 dtype=rng.choice(["f32", "f32", "f16"]))
    return c


# ------------------------------------------------------------------ inputs
def _inputs(c, seed):
    """The arrays of a case, on the GPU, from the seed alone."""
    dev = "cuda"
    g = torch.Generator(device=dev)
    g.manual_seed(seed)

    def uniform(*shape, lo=0.0, hi=1.0):
        return torch.rand(shape, generator=g, device=dev) * (hi - lo) + lo

    def weights(*shape):  # log-uniform in [1/4, 4]
        return torch.exp2(uniform(*shape, lo=-2.0, hi=2.0))

    kind = c["kind"]
    if kind in ("curves", "train"):
        dt = DTYPES[c["dtype"]]
        x = {"ctrl": uniform(c["n"], c["dim"], c["degree"] + 1, lo=-1.0, hi=1.0).to(dt)}
        x["w"] = weights(c["n"], c["degree"] + 1).to(dt) if c["rational"] else None
        if kind == "curves" and c["shared"]:  # a common uniform grid, moved a little by the seed
            x["t"] = ((torch.arange(c["n_t"], device=dev, dtype=torch.float32) + uniform(1)) / c["n_t"]).contiguous()
        else:
            x["t"] = uniform(c["n"], c["n_t"])
        if kind == "train":
            x["g"] = torch.randn((c["dim"], c["n"] * c["n_t"]), generator=g, device=dev)
        return x
    if kind == "fit":  # noisy samples of a curve; the fit starts from the chord and uniform parameters
        n, n_t, dim, d = c["n"], c["n_t"], c["dim"], c["degree"]
        truth = uniform(n, dim, d + 1, lo=-1.0, hi=1.0).double()
        tau = torch.sort(uniform(n, n_t), dim=1)[0].double()
        y = _curve(truth, tau).float() + 0.01 * torch.randn((dim, n * n_t), generator=g, device=dev)
        y3 = y.view(dim, n, n_t)
        f = torch.arange(d + 1, device=dev, dtype=torch.float32) / d
        ctrl = (y3[:, :, 0].T[:, :, None] * (1 - f) + y3[:, :, -1].T[:, :, None] * f).contiguous()
        t = (torch.arange(n_t, device=dev, dtype=torch.float32) / (n_t - 1)).repeat(n, 1).contiguous()
        return {"ctrl": ctrl, "t": t, "y": y.contiguous()}
    if kind == "batch":
        nb, nn, npa, dim = c["n_bezier"], c["n_nurbs"], c["n_patches"], c["dim"]
        n = nb + nn + npa
        # kinds 0 integral, 1 rational, 2 NURBS, 3 bicubic patch, shuffled
        rational = (uniform(nb) < 0.5).long()
        deg = torch.randint(2, 16, (nb,), generator=g, device=dev)
        n_knots = torch.randint(8, 65, (nn,), generator=g, device=dev)
        code = torch.cat([rational << 8 | deg, torch.full((nn,), 2 << 8 | 3, device=dev),
                          torch.full((npa,), 3 << 8 | 3 << 4 | 3, device=dev)])
        ncp = torch.cat([deg + 1, n_knots - 4, torch.full((npa,), 16, device=dev)])
        nk = torch.cat([torch.zeros(nb, dtype=torch.long, device=dev), n_knots,
                        torch.zeros(npa, dtype=torch.long, device=dev)])
        order = torch.randperm(n, generator=g, device=dev)
        code, ncp, nk = code[order], ncp[order], nk[order]
        cp_off = torch.zeros(n + 1, dtype=torch.long, device=dev)
        cp_off[1:] = torch.cumsum(ncp, 0)
        k_off = torch.zeros(n + 1, dtype=torch.long, device=dev)
        k_off[1:] = torch.cumsum(nk, 0)
        total = int(cp_off[-1])
        # clamped knot vectors: four zeros, sorted interior knots, four ones
        counts = nk[nk > 0]
        at = torch.arange(64, device=dev)[None, :]
        inner = (at >= 4) & (at < counts[:, None] - 4)
        v = uniform(nn, 64).clamp(1e-6, 1 - 1e-6) if nn else torch.zeros((0, 64), device=dev)
        v = torch.where(inner, v, (at >= 4).float() * 2.0)
        v = torch.sort(v, dim=1)[0]
        v = torch.where(v > 1.0, torch.ones_like(v), v)
        knots = v[at < counts[:, None]].contiguous()
        dt = DTYPES[c["dtype"]]
        x = {"code": code, "kind_degree": code.to(torch.int16).view(torch.uint16), "cp_offset": cp_off,
             "ctrl": uniform(total * dim, lo=-1.0, hi=1.0).to(dt), "w": weights(total).to(dt), "knot_offset": k_off,
             "knots": knots, "t": uniform(n, c["n_t"])}
        x["v"] = uniform(n, c["n_t"]) if npa else None
        return x
    if kind in ("encode", "chain"):
        cubic = c["cubic"] if kind == "encode" else c["layout"] == "cubic_tiles"
        m = (3 if cubic else 2) * c["n_seg"] + 1
        step = uniform(m, c["dim"], lo=-0.1, hi=0.1).double()
        x = {"chain": torch.cumsum(step, 0).float().contiguous()}
        if kind == "chain":
            x["T"] = (torch.rand(c["n_q"], generator=g, device=dev, dtype=torch.float64) * c["n_seg"]).float()
        return x
    dt = DTYPES[c["dtype"]]
    if kind == "grid":
        return {"ctrl": uniform(c["n"], c["dim"], (c["du"] + 1) * (c["dv"] + 1), lo=-1.0, hi=1.0).to(dt)}
    ncp = (c["du"] + 1) * (c["dv"] + 1) * (c["dw"] + 1)
    return {"ctrl": uniform(c["n"], c["dim"], ncp, lo=-1.0, hi=1.0).to(dt),
            "uvw": uniform(c["n"], c["n_per"], 3 if c["dw"] else 2)}


def prepare(case, seed):
    x = _inputs(case, seed)
    x["case"] = case
    kind = case["kind"]
    if kind == "train":
        for k in ("ctrl", "w", "t"):
            if x[k] is not None:
                x[k].requires_grad_(True)
    elif kind == "fit":
        for k in ("ctrl", "t"):
            x["m_" + k], x["v_" + k] = torch.zeros_like(x[k]), torch.zeros_like(x[k])
        x["loss"] = torch.zeros(case["n"], device="cuda")
        x["step"] = 1
    elif kind == "batch":
        # the plan keeps its own copies of the control points: the arrays it was made from go
        x["plan"] = bz.BatchPlan(x.pop("kind_degree"), x.pop("cp_offset"), x.pop("ctrl"), x.pop("w"), case["dim"],
                                 x.pop("knot_offset"), x.pop("knots"), case["n_t"], method=case["method"])
        x.pop("code")
    elif kind == "chain":
        chain = x.pop("chain")
        if case["layout"] == "cubic_tiles":
            x["tex"] = bz.tile_piecewise_cubic(bz.encode_piecewise_cubic(chain))
        else:
            grid = bz.encode_piecewise(chain)
            x["tex"] = (grid if case["layout"] == "grid" else bz.tile_piecewise(grid) if case["layout"] == "tiles"
                        else bz.tile_piecewise16(grid, torch.float16))
    return x


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "curves":
        if c["rational"]:
            return bz.eval_rational(state["ctrl"], state["w"], state["t"], c["method"])
        return bz.eval_bezier(state["ctrl"], state["t"], c["method"])
    if kind == "train":
        ins = [state[k] for k in ("ctrl", "t", "w") if state[k] is not None]
        out = bz.bezier_curve(state["ctrl"], state["t"], state["w"])
        return [out] + list(torch.autograd.grad(out, ins, state["g"]))
    if kind == "fit":
        bz.fit_adam_run(state["ctrl"], state["t"], state["y"], state["m_ctrl"], state["v_ctrl"], state["m_t"],
                        state["v_t"], state["step"], c["steps"], loss_part=state["loss"])
        state["step"] += c["steps"]
        return [state["ctrl"], state["t"], state["loss"]]
    if kind == "batch":
        return state["plan"](state["t"], v=state["v"])
    if kind == "encode":
        if c["cubic"]:
            grid = bz.encode_piecewise_cubic(state["chain"])
            return [grid, bz.tile_piecewise_cubic(grid)]
        grid = bz.encode_piecewise(state["chain"])
        return [grid, bz.tile_piecewise(grid)]
    if kind == "chain":
        if c["layout"] == "grid":
            return bz.eval_piecewise(state["tex"], state["T"])
        if c["layout"] == "tiles":
            return bz.eval_piecewise_tiled(state["tex"], c["n_seg"], c["dim"], state["T"])
        if c["layout"] == "tiles_f16":
            return bz.eval_piecewise_tiled16(state["tex"], c["n_seg"], c["dim"], state["T"])
        return bz.eval_piecewise_cubic_tiled(state["tex"], c["n_seg"], c["dim"], state["T"])
    if kind == "grid":
        return bz.eval_tensor_patch(state["ctrl"], c["du"], c["dv"], nu=c["nu"], nv=c["nv"])
    return bz.eval_tensor_patch(state["ctrl"], c["du"], c["dv"], c["dw"], uvw=state["uvw"])


# ------------------------------------------------------------------ work
def _degree_work(d, ch):
    """(Bernstein) flops of one curve point with ch channels: basis and contraction."""
    return 4 * d + 2 * (d + 1) * ch


def work(case):
    c = case
    kind = c["kind"]
    if kind in ("curves", "train"):
        d, dim, e = c["degree"], c["dim"], SIZES[c["dtype"]]
        ch = dim + (1 if c["rational"] else 0)
        nq = c["n"] * c["n_t"]
        params = c["n"] * (d + 1) * ch * e
        if kind == "curves":
            return {"bytes": params + 4 * (c["n_t"] if c["shared"] else nq) + 4 * dim * nq,
                    "flops": nq * _degree_work(d, ch)}
        # forward: parameters, t, points; backward: the same inputs, dL/dC and the gradients
        return {"bytes": 3 * params + nq * (4 + 4 * dim + 4 + 4 * dim + 4), "flops": 4 * nq * _degree_work(d, ch)}
    if kind == "fit":
        d, dim = c["degree"], c["dim"]
        nq, npar = c["n"] * c["n_t"], c["n"] * (d + 1) * dim
        flops = nq * c["steps"] * (4 * d + dim * (2 * (d + 1) + 3 * d + 7 + 2 * (d + 1)) + 16)
        return {"bytes": nq * (4 * dim + 6 * 4) + npar * 6 * 4 + 4 * c["n"], "flops": flops}
    if kind == "batch":
        n = c["n_bezier"] + c["n_nurbs"] + c["n_patches"]
        e, dim, nq = SIZES[c["dtype"]], c["dim"], n * c["n_t"]
        pts = c["n_bezier"] * 9.5 * (dim + 0.5) + c["n_nurbs"] * 32 * (dim + 1) + c["n_patches"] * 16 * dim
        return {"bytes": pts * e + c["n_nurbs"] * 36 * 4 + n * 8 + nq * (4 + 4 * dim)
                + c["n_patches"] * c["n_t"] * 4,
                "flops": nq * _degree_work(8.5, dim + 0.5)}
    if kind == "encode":
        ns, dim = c["n_seg"], c["dim"]
        chain = ((3 if c["cubic"] else 2) * ns + 1) * dim * 4
        grid = (ns + 1) * (4 if c["cubic"] else 2) * dim * 4
        w = (3 if c["cubic"] else 2) * dim
        tiles = -(-ns // (32 // w - 1)) * 128
        return {"bytes": chain + grid + tiles, "flops": 4 * ns * dim}
    if kind == "chain":
        per = {"grid": 8, "tiles": 8, "tiles_f16": 4, "cubic_tiles": 12}[c["layout"]]
        return {"bytes": c["n_q"] * (4 + 4 * c["dim"]) + min(c["n_seg"], 2 * c["n_q"]) * per * c["dim"],
                "flops": c["n_q"] * 12 * c["dim"]}
    e, dim = SIZES[c["dtype"]], c["dim"]
    if kind == "grid":
        nq, ncp = c["n"] * c["nu"] * c["nv"], (c["du"] + 1) * (c["dv"] + 1)
        return {"bytes": c["n"] * ncp * dim * e + nq * dim * 4, "flops": nq * 2 * (c["du"] + 1) * dim}
    nu, nv, nw = c["du"] + 1, c["dv"] + 1, c["dw"] + 1
    nq = c["n"] * c["n_per"]
    return {"bytes": c["n"] * nu * nv * nw * dim * e + nq * (4 * (3 if c["dw"] else 2) + 4 * dim),
            "flops": nq * (2 * dim * (nu * nv * nw * (nw > 1) + nu * nv + nu) + 4 * (nu + nv + nw))}


# ------------------------------------------------------------------ 64-bit values
def _basis(t, d):
    """Bernstein basis values of degree d, a list of arrays shaped like t."""
    s = 1.0 - t
    return [math.comb(d, i) * t ** i * s ** (d - i) for i in range(d + 1)]


def _curve(ctrl, t, w=None):
    """Points [dim, n*n_t] of curves ctrl[n, dim, d+1] at t[n, n_t], in 64 bits."""
    B = _basis(t, ctrl.shape[2] - 1)
    if w is not None:
        B = [b * w[:, i, None] for i, b in enumerate(B)]
        total = sum(B)
    out = []
    for k in range(ctrl.shape[1]):
        v = sum(b * ctrl[:, k, i, None] for i, b in enumerate(B))
        out.append((v if w is None else v / total).reshape(-1))
    return torch.stack(out)


def _chain_columns(chain, n_seg, cubic):
    """End points [n_seg+1, dim] and free texels, a list of [n_seg+1, dim], in 64 bits."""
    p = chain.double()
    ends = p[:: 3 if cubic else 2]
    if cubic:
        twice = [3 * p[1::3] - p[:-1:3], 3 * p[2::3] - p[3::3]]
    else:
        twice = [2 * p[1::2]]
    k = torch.arange(n_seg + 1, device=p.device)
    sign = (1 - 2 * (k % 2)).double()[:, None]
    free = []
    for m2 in twice:  # x_0 = M_0, x_(k+1) = 2 M_k - x_k
        y = torch.cat([0.5 * m2[:1], -sign[:-1] * m2])
        free.append(sign * torch.cumsum(y, 0))
    return ends, free


def _exact_fit(c, x):
    ctrl, t, y = x["ctrl"].double(), x["t"].double(), x["y"].double()
    n, n_t, dim, d = c["n"], c["n_t"], c["dim"], c["degree"]
    y3 = y.view(dim, n, n_t)
    mc, vc, mt, vt = (torch.zeros_like(v) for v in (ctrl, ctrl, t, t))
    for step in range(1, c["steps"] + 1):
        B, Bm = _basis(t, d), _basis(t, d - 1)
        gc, gt, loss = torch.zeros_like(ctrl), torch.zeros_like(t), torch.zeros(n, dtype=torch.float64, device=t.device)
        for k in range(dim):
            r = sum(b * ctrl[:, k, i, None] for i, b in enumerate(B)) - y3[k]
            loss += (r * r).sum(1)
            g = 2.0 * r / (n * n_t)
            gt += g * d * sum(b * (ctrl[:, k, i + 1] - ctrl[:, k, i])[:, None] for i, b in enumerate(Bm))
            for i in range(d + 1):
                gc[:, k, i] = (g * B[i]).sum(1)
        for p, g, m, v in ((ctrl, gc, mc, vc), (t, gt, mt, vt)):
            m.mul_(0.9).add_(g, alpha=0.1)
            v.mul_(0.999).addcmul_(g, g, value=0.001)
            p -= 1e-2 * (m / (1 - 0.9 ** step)) / ((v / (1 - 0.999 ** step)).sqrt() + 1e-8)
        t.clamp_(0.0, 1.0)
    return [ctrl, t, loss / (n * n_t)]


def _exact_nurbs(P, w, knots, n_knots, u):
    """Cubic NURBS points [n, n_t, dim]: P[n, 60, dim], w[n, 60], knots[n, 64] (padded), u[n, n_t]."""
    n_t = u.shape[1]
    at = torch.arange(64, device=u.device)[None, None, :]
    below = ((knots[:, None, :] <= u[:, :, None]) & (at < n_knots[:, None, None])).sum(2) - 1
    span = torch.minimum(below.clamp(min=3), n_knots[:, None] - 5)
    knot = lambda off: torch.gather(knots, 1, span + off)  # noqa: E731
    left = [None] + [u - knot(1 - j) for j in (1, 2, 3)]
    right = [None] + [knot(j) - u for j in (1, 2, 3)]
    N = [torch.ones_like(u)]
    for j in (1, 2, 3):  # Cox and de Boor's recursion on the four functions of the span
        new, saved = [], torch.zeros_like(u)
        for r in range(j):
            q = N[r] / (right[r + 1] + left[j - r])
            new.append(saved + right[r + 1] * q)
            saved = left[j - r] * q
        N = new + [saved]
    den = torch.zeros_like(u)
    num = torch.zeros(u.shape[0], n_t, P.shape[2], dtype=u.dtype, device=u.device)
    for j in range(4):
        i = span - 3 + j
        b = N[j] * torch.gather(w, 1, i)
        den += b
        num += b[:, :, None] * torch.gather(P, 1, i[:, :, None].expand(-1, -1, P.shape[2]))
    return num / den[:, :, None]


def _exact_batch(c, x):
    dim, n_t = c["dim"], c["n_t"]
    n = x["code"].shape[0]
    out = torch.empty((dim, n, n_t), dtype=torch.float64, device="cuda")
    cpo, ko, t = x["cp_offset"], x["knot_offset"], x["t"].double()
    for code in torch.unique(x["code"]).tolist():
        kind, deg = code >> 8, code & 255
        objs = torch.nonzero(x["code"] == code)[:, 0]
        if kind == 2:
            ncp = cpo[objs + 1] - cpo[objs]
            i = torch.minimum(torch.arange(60, device="cuda")[None, :], ncp[:, None] - 1)
            w = x["w"][cpo[objs, None] + i].double()
            P = torch.stack([x["ctrl"][cpo[objs, None] * dim + k * ncp[:, None] + i].double() for k in range(dim)], 2)
            nk = ko[objs + 1] - ko[objs]
            j = torch.minimum(torch.arange(64, device="cuda")[None, :], nk[:, None] - 1)
            r = _exact_nurbs(P, w, x["knots"][ko[objs, None] + j].double(), nk, t[objs])
            out[:, objs] = r.permute(2, 0, 1)
            continue
        ncp = 16 if kind == 3 else deg + 1
        i = torch.arange(ncp * dim, device="cuda")[None, :]
        P = x["ctrl"][cpo[objs, None] * dim + i].double().view(-1, dim, ncp)
        if kind == 3:
            Bu, Bv = _basis(t[objs], 3), _basis(x["v"][objs].double(), 3)
            for k in range(dim):
                out[k, objs] = sum(Bu[a] * Bv[b] * P[:, k, 4 * a + b, None] for a in range(4) for b in range(4))
            continue
        w = x["w"][cpo[objs, None] + torch.arange(ncp, device="cuda")[None, :]].double() if kind == 1 else None
        out[:, objs] = _curve(P, t[objs], w).view(dim, -1, n_t)
    return out.reshape(dim, n * n_t)


def exact(case, seed):
    c, x = case, _inputs(case, seed)
    kind = c["kind"]
    if kind == "curves":
        t = x["t"].double()
        t = t[None, :].expand(c["n"], -1) if c["shared"] else t
        return _curve(x["ctrl"].double(), t, None if x["w"] is None else x["w"].double())
    if kind == "train":
        p = [x[k].double().requires_grad_(True) for k in ("ctrl", "t", "w") if x[k] is not None]
        out = _curve(p[0], p[1], p[2] if len(p) > 2 else None)
        return [out.detach()] + list(torch.autograd.grad(out, p, x["g"].double()))
    if kind == "fit":
        return _exact_fit(c, x)
    if kind == "batch":
        return _exact_batch(c, x)
    if kind in ("encode", "chain"):
        ns, dim = c["n_seg"], c["dim"]
        cubic = c["cubic"] if kind == "encode" else c["layout"] == "cubic_tiles"
        ends, free = _chain_columns(x["chain"], ns, cubic)
        if kind == "encode":
            even = (torch.arange(ns + 1, device="cuda") % 2 == 0)[:, None, None]
            rows = [torch.where(even, torch.stack([ends, f], 1), torch.stack([f, ends], 1)) for f in free]
            grid = torch.stack(rows, 1) if cubic else rows[0]
            cols = torch.cat([ends] + free, 1) if cubic else grid.reshape(ns + 1, -1)
            width = cols.shape[1]
            per = 32 // width - 1
            n_tiles = -(-ns // per)
            pad = torch.zeros(n_tiles * per + 1, width, dtype=torch.float64, device="cuda")
            pad[: ns + 1] = cols
            at = torch.arange(n_tiles, device="cuda")[:, None] * per + torch.arange(per + 1, device="cuda")[None, :]
            tiles = torch.zeros(n_tiles, 32, dtype=torch.float64, device="cuda")
            tiles[:, : (per + 1) * width] = pad[at].reshape(n_tiles, -1)
            return [grid, tiles.reshape(-1)]
        store = torch.float16 if c["layout"] == "tiles_f16" else torch.float32
        ends, free = ends.float().to(store).double(), [f.float().to(store).double() for f in free]
        T = x["T"].double().clamp(0, ns)
        k = T.floor().long().clamp(max=ns - 1)
        t = (T - k)[:, None]
        layer = [ends[k] * (1 - t) ** 2 + (f[k] + f[k + 1]) * t * (1 - t) + ends[k + 1] * t * t for f in free]
        v = layer[0] if len(layer) == 1 else (1 - t) * layer[0] + t * layer[1]
        return v.T.contiguous()
    P = x["ctrl"].double()
    if kind == "grid":
        axis = lambda m: torch.arange(m, device="cuda", dtype=torch.float64) / max(m - 1, 1)  # noqa: E731
        Bu, Bv = _basis(axis(c["nu"]), c["du"]), _basis(axis(c["nv"]), c["dv"])
        out = torch.zeros(c["dim"], c["n"], c["nu"], c["nv"], dtype=torch.float64, device="cuda")
        for i, a in enumerate(Bu):
            for j, b in enumerate(Bv):
                ab = a[:, None] * b[None, :]
                for k in range(c["dim"]):
                    out[k] += P[:, k, i * (c["dv"] + 1) + j, None, None] * ab
        return out.reshape(c["dim"], -1)
    uvw = x["uvw"].double()
    Bu, Bv = _basis(uvw[:, :, 0], c["du"]), _basis(uvw[:, :, 1], c["dv"])
    Bw = _basis(uvw[:, :, 2], c["dw"]) if c["dw"] else [torch.ones_like(uvw[:, :, 0])]
    out = torch.zeros(c["dim"], c["n"], c["n_per"], dtype=torch.float64, device="cuda")
    at = 0
    for a in Bu:
        for b in Bv:
            for w in Bw:
                abw = a * b * w
                for k in range(c["dim"]):
                    out[k] += P[:, k, at, None] * abw
                at += 1
    return out.reshape(c["dim"], -1)
