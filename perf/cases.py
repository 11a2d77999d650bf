"""Timing cases: the calls that programs built on this package make.

Each case is a dict of plain values; `path` names the public entry points it
goes through, the other keys are sizes and options:

  step      crom.Stepper.step: the latent step q_n -> q_{n+1} (heat or the
            neo-Hookean bar), Gauss-Newton or linearised, one instance or a
            ragged batch
  decode    crom.Decoder.decode: the value decode of a whole field
  jets      crom.Decoder.decode_jac: values with spatial derivatives and the
            latent Jacobian
  grads     crom.Trainer.grads: loss and gradients of one training batch
  train     crom.Trainer.step: one Adam step of encoder and decoder
  vjp       autograd.decode forward and backward (the decoder inside a
            PyTorch program)
  fd        heat2d.fd_snapshots: the FP64 finite-difference snapshots of a
            training set
  residual  crom.sampling_residual: the residual vectors of candidate sample
            sets (robust sample selection)

Decoder shapes: "1d" (1, 3, 1, 32), "2d" (2, 8, 1, 128), "3d"
(3, 16, 3, 256) as (m, r, d, width), with 5, 5 and 6 hidden layers.
"""
import math

import numpy as np
import torch

from paper_2206_02607_amd import autograd, crom, heat2d

SHAPES = {"1d": (1, 3, 1, 32, 5), "2d": (2, 8, 1, 128, 5), "3d": (3, 16, 3, 256, 6)}
F64 = torch.float64


def listed():
    return [
        # the smallest call: the 1D heat rollout's step (20 samples), one instance
        dict(name="step 1d heat", path="step", shape="1d", precision="fp32", linearized=False, instances=1,
             s_min=20, s_max=20, iters=5),
        # an interactive rollout: one instance of 2D heat at 2,000 samples
        dict(name="step 2d heat", path="step", shape="2d", precision="bf16", linearized=False, instances=1,
             s_min=2000, s_max=2000, iters=5),
        # the bar of 64 x 16 x 16 material points at 500 samples
        dict(name="step bar", path="step", shape="3d", precision="bf16", linearized=False, instances=1, s_min=500,
             s_max=500, iters=5),
        # many-query use: 512 diffusivities at once, ragged sample counts
        dict(name="batch linearised", path="step", shape="2d", precision="bf16", linearized=True, instances=512,
             s_min=200, s_max=2000, iters=1),
        # the same use at full precision with the nonlinear inversion
        dict(name="batch gauss-newton", path="step", shape="2d", precision="fp32", linearized=False, instances=64,
             s_min=200, s_max=2000, iters=5),
        # a frame of the rollout: the field at every node of a 256 x 256 grid
        dict(name="decode field", path="decode", shape="2d", precision="bf16", act="elu", points=65536),
        # derivatives for a user's own PDE terms, an odd number of points
        dict(name="jets fp32", path="jets", shape="2d", precision="fp32", act="elu", points=20011),
        # a training batch: 16 snapshots of 128 x 128 nodes, dense encoder
        dict(name="grads bf16", path="grads", shape="2d", precision="bf16", act="elu", batch=16, nx=128, ny=128,
             hidden=256, encoder="dense"),
        # training at full precision with the convolutional encoder, a ragged grid
        dict(name="train fp32", path="train", shape="2d", precision="fp32", act="elu", batch=5, nx=101, ny=97,
             hidden=32, encoder="conv"),
        # the decoder inside a PyTorch program, a few latents at scattered points
        dict(name="autograd bf16", path="vjp", shape="2d", precision="bf16", act="elu", batch=3, points=4999),
        # a training set's snapshots: 40 diffusivities, 128 x 128 nodes, 5 times
        dict(name="fd snapshots", path="fd", fields=40, nx=128, ny=128, times=5, substeps=1250),
        # one round of sample selection: 10 candidate sets x 40 parameters on 128 x 128 nodes
        dict(name="sample residual", path="residual", shape="2d", precision="bf16", sets=10, params=40, points=16384),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["step", "batch", "bar", "decode", "jets", "grads", "train", "vjp", "fd", "residual"])
    prec = rng.choice(["bf16", "bf16", "fp32"])
    if path == "step":
        if rng.random() < 0.4:
            s = _log(rng, 8, 400)
            return dict(path="step", shape="1d", precision="fp32", linearized=rng.random() < 0.5, instances=1,
                        s_min=s, s_max=s, iters=rng.randint(1, 5))
        s = _log(rng, 40, 4000)
        return dict(path="step", shape="2d", precision=prec, linearized=rng.random() < 0.5, instances=1, s_min=s,
                    s_max=s, iters=rng.randint(1, 5))
    if path == "batch":
        s = _log(rng, 20, 400)
        return dict(path="step", shape="2d", precision=prec, linearized=rng.random() < 0.7,
                    instances=_log(rng, 4, 256), s_min=s, s_max=_log(rng, s, 2000), iters=rng.randint(1, 4))
    if path == "bar":
        s = _log(rng, 40, 800)
        return dict(path="step", shape="3d", precision=prec, linearized=rng.random() < 0.5,
                    instances=rng.randint(1, 2), s_min=s, s_max=s, iters=rng.randint(1, 4))
    if path in ("decode", "jets"):
        shape = rng.choice(["1d", "2d", "2d", "3d"])
        act = "sine" if shape != "3d" and rng.random() < 0.25 else "elu"
        return dict(path=path, shape=shape, precision=prec, act=act,
                    points=_log(rng, 17, 200000 if path == "decode" else 60000))
    if path in ("grads", "train"):
        act = "sine" if prec == "bf16" and rng.random() < 0.2 else "elu"
        enc = rng.choice(["dense", "conv"]) if path == "grads" else "conv"
        return dict(path=path, shape="2d", precision=prec, act=act, batch=rng.randint(1, 16), nx=_log(rng, 24, 128),
                    ny=_log(rng, 24, 128), hidden=rng.choice([32, 64, 256]) if enc == "dense" else 32, encoder=enc)
    if path == "vjp":
        return dict(path="vjp", shape="2d", precision=prec, act="elu", batch=rng.randint(1, 8),
                    points=_log(rng, 17, 30000))
    if path == "fd":
        return dict(path="fd", fields=_log(rng, 1, 40), nx=_log(rng, 17, 256), ny=_log(rng, 17, 256),
                    times=rng.randint(2, 5), substeps=_log(rng, 10, 500))
    return dict(path="residual", shape="2d", precision=prec, sets=rng.randint(1, 10), params=rng.randint(1, 40),
                points=_log(rng, 300, 16384))


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _layers(gen, shape, act):
    """Seeded decoder layers: Xavier-uniform weights with small biases (the
    bar's displacement field: zero biases, small outputs), or the SIREN
    initialisation with its frequency 30 in the weights."""
    m, r, d, width, depth = SHAPES[shape]
    sizes = [m + r] + [width] * depth + [d]
    out = []
    for l, (n_in, n_out) in enumerate(zip(sizes[:-1], sizes[1:])):
        a, b = math.sqrt(6.0 / (n_in + n_out)), 0.0 if shape == "3d" else 0.1
        if act == "sine":
            a = 30.0 / n_in if l == 0 else math.sqrt(6.0 / n_in) / (30.0 if l == depth else 1.0)
            b = (30.0 if l < depth else 1.0) / math.sqrt(n_in)
        scale = 1e-2 if shape == "3d" and l == depth else 1.0  # displacements: small strains
        out.append((gen.uniform(-a, a, (n_out, n_in)).astype(np.float32) * np.float32(scale),
                    gen.uniform(-b, b, n_out).astype(np.float32) * np.float32(scale)))
    return out


def _points(gen, n, m, act="elu"):
    lo = -1.0 if act == "sine" else 0.0
    return torch.from_numpy(gen.uniform(lo, 1.0, (n, m)).astype(np.float32)).cuda()


def _nodes(nx, ny):
    x, y = np.meshgrid(np.linspace(0.0, 1.0, nx), np.linspace(0.0, 1.0, ny), indexing="ij")
    return np.stack([x.ravel(), y.ravel()], axis=1).astype(np.float32)


def _heat_fields(gen, n, nodes):
    """n decayed heat fields [n, P] on the unit square (sine modes)."""
    x = torch.from_numpy(nodes).cuda().to(F64)
    k = torch.arange(1, 5, device="cuda", dtype=F64) * math.pi
    sx, sy = torch.sin(x[:, :1] * k), torch.sin(x[:, 1:] * k)
    amp = torch.from_numpy(gen.uniform(-1.0, 1.0, (4, 4))).cuda()
    t = torch.from_numpy(gen.uniform(0.0, 0.05, n) * gen.uniform(0.1, 1.0, n)).cuda()
    decay = torch.exp(-(k[:, None] ** 2 + k[None, :] ** 2) * t[:, None, None])
    return torch.stack([((sx @ (amp * decay[i])) * sy).sum(1) for i in range(n)])


def _conv_sizes(n):
    """(kernel 6, stride 4) lengths while at least 32 values are left."""
    out = []
    while n >= 6 and (n - 6) // 4 + 1 >= 32:
        n = (n - 6) // 4 + 1
        out.append(n)
    return out


def _encoder(gen, case, n_in, r):
    """Seeded encoder parameter arrays in the order of the flat vector."""
    h, parts = case["hidden"], []
    if case["encoder"] == "conv":
        for n_in in _conv_sizes(n_in):
            parts += [gen.uniform(-0.4, 0.4, (1, 1, 6)), gen.uniform(-0.4, 0.4, 1)]
    for o, i in ((h, n_in), (r, h)):
        a = math.sqrt(6.0 / (i + o))
        parts += [gen.uniform(-a, a, (o, i)), np.zeros(o)]
    return [p.astype(np.float32) for p in parts]


def _inputs(case, seed):
    """Everything a case's inputs are made of, from the seed alone."""
    gen = np.random.Generator(np.random.PCG64(seed))
    path = case["path"]
    if path == "fd":
        nx, ny = case["nx"], case["ny"]
        x, y = np.linspace(0.0, 1.0, nx)[:, None], np.linspace(0.0, 1.0, ny)[None, :]
        u = np.zeros((nx, ny))
        for _ in range(4):
            cx, cy, w, a = gen.uniform(0.25, 0.75), gen.uniform(0.25, 0.75), gen.uniform(0.06, 0.12), gen.uniform(-1, 1)
            u += a * np.exp(-((x - cx) ** 2 + (y - cy) ** 2) / (2 * w * w))
        u *= np.sin(math.pi * x) * np.sin(math.pi * y)
        u[0, :] = u[-1, :] = u[:, 0] = u[:, -1] = 0.0
        dx = 1.0 / (max(nx, ny) - 1)
        dt = 0.16 * dx * dx
        return dict(u=u, mus=gen.uniform(0.1, 1.0, case["fields"]), dx=dx, dt=dt,
                    times=[i * case["substeps"] * dt for i in range(case["times"])])
    m, r, d, width, depth = SHAPES[case["shape"]]
    act = case.get("act", "elu")
    z = dict(m=m, r=r, d=d, act=act, layers=_layers(gen, case["shape"], act))
    if path == "step":
        n = case["instances"]
        counts = gen.integers(case["s_min"], case["s_max"] + 1, n)
        counts = np.maximum(counts, -(-r // d))
        z["offsets"] = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
        z["max_iter"] = case["iters"]
        if case["shape"] == "3d":
            g = np.stack(np.meshgrid(np.arange(64), np.arange(16), np.arange(16), indexing="ij"), -1).reshape(-1, 3)
            idx = np.concatenate([np.sort(gen.choice(len(g), c, replace=False)) for c in counts])
            z["y"] = torch.from_numpy((g[idx] / 15.0).astype(np.float32)).cuda()
            z["clamp"] = torch.from_numpy((g[idx][:, 0] == 0).astype(np.uint8)).cuda()
            z["coef"] = torch.tensor([1e4, 4e3, 1000.0, 0.0, 0.0, -9.81], dtype=F64, device="cuda").repeat(n, 1)
            z["dt"], z["q"] = 1e-3, gen.uniform(-0.1, 0.1, (n, r))
        else:
            z["y"] = _points(gen, int(counts.sum()), m)
            z["clamp"], z["coef"] = None, torch.from_numpy(gen.uniform(0.1, 1.0, n)).cuda()
            z["dt"], z["q"] = 1e-4 if m == 2 else 1e-5, gen.uniform(-1.0, 1.0, (n, r))
        z["q"] = torch.from_numpy(z["q"]).cuda()
    elif path in ("decode", "jets"):
        z["x"] = _points(gen, case["points"], m, act)
        z["q"] = torch.from_numpy(gen.uniform(-1.0, 1.0, r) * (0.1 if m == 3 else 1.0)).cuda()
    elif path in ("grads", "train"):
        nodes = _nodes(case["nx"], case["ny"])
        u = _heat_fields(gen, case["batch"], nodes)
        z["u"] = ((u - u.mean()) / u.std()).to(torch.float32)
        nodes = nodes * 2.0 - 1.0 if act == "sine" else (nodes - 0.5) * 3.4  # standardized coordinates
        z["x"] = torch.from_numpy(nodes.astype(np.float32)).cuda()
        z["enc"] = _encoder(gen, case, len(nodes), r)
    elif path == "vjp":
        z["x"] = _points(gen, case["points"], m, act)
        z["q"] = torch.from_numpy(gen.uniform(-1.0, 1.0, (case["batch"], r)).astype(np.float32)).cuda()
        z["dg"] = torch.from_numpy(gen.normal(0.0, 1.0, (case["batch"], case["points"], d)).astype(np.float32)).cuda()
    else:
        nodes = _points(gen, case["points"], m).cpu().numpy()
        z["x"] = torch.from_numpy(nodes).cuda()
        z["q"] = torch.from_numpy(gen.uniform(-1.0, 1.0, (case["sets"], case["params"], r))).cuda()
        z["ref"] = _heat_fields(gen, case["params"], nodes).unsqueeze(-1).contiguous()
    return z


def _decoder(case, z):
    return crom.Decoder.from_layers(z["layers"], z["m"], precision=case["precision"], act=z["act"])


def prepare(case, seed):
    z = _inputs(case, seed)
    s = dict(path=case["path"], z=z)
    if case["path"] == "fd":
        return s
    s["dec"] = _decoder(case, z)
    if case["path"] == "step":
        s["stepper"] = crom.Stepper(s["dec"], z["offsets"], z["y"], z["clamp"],
                                    pde="neohookean" if z["m"] == 3 else "heat")
        s["opts"] = crom.GNOptions(max_iter=z["max_iter"], linearized=case["linearized"])
        s["q_next"] = torch.empty_like(z["q"])
    elif case["path"] in ("grads", "train"):
        flat = np.concatenate([p.ravel() for p in z["enc"]])
        s["trainer"] = crom.Trainer(s["dec"], flat, case["hidden"], z["x"], case["batch"], case["encoder"])
    elif case["path"] == "vjp":
        s["dec"].params.requires_grad_(True)
        z["q"].requires_grad_(True)
    return s


def run(state):
    z, path = state["z"], state["path"]
    if path == "step":
        return state["stepper"].step(z["q"], z["coef"], z["dt"], state["opts"], state["q_next"])
    if path == "decode":
        return state["dec"].decode(z["x"], z["q"])
    if path == "jets":
        return state["dec"].decode_jac(z["x"], z["q"], dx=True, d2=crom.D2_LAPLACIAN, dq=True)
    if path == "grads":
        loss, gd, ge, q = state["trainer"].grads(z["u"])
        return {"loss": loss, "grad_dec": gd, "grad_enc": ge, "q": q}
    if path == "train":
        t = state["trainer"]
        loss = t.step(z["u"], 1e-3)
        return {"loss": loss, "grad_dec": t.grad_dec, "grad_enc": t.grad_enc, "dec": t.dec.params,
                "enc": t.enc_params}
    if path == "vjp":
        params = state["dec"].params
        g = autograd.decode(state["dec"], z["q"], z["x"])
        gp, gq = torch.autograd.grad(g, (params, z["q"]), z["dg"])
        return {"g": g.detach(), "grad_params": gp, "grad_q": gq}
    if path == "fd":
        return heat2d.fd_snapshots(z["u"], z["mus"], z["times"], z["dx"], z["dt"])
    res, metric = crom.sampling_residual(state["dec"], z["x"], z["q"], z["ref"])
    return {"res": res, "metric": metric}


def work(case):
    """Operations of the algorithm (two per multiply-add; a column through the
    hidden layers is width^2 multiply-adds a layer), inputs read once and
    outputs written once."""
    path = case["path"]
    if path == "fd":
        n = case["fields"] * case["nx"] * case["ny"]
        return {"bytes": 8 * (case["nx"] * case["ny"] + n * case["times"]),
                "flops": 8 * n * (case["times"] - 1) * case["substeps"]}
    m, r, d, w, depth = SHAPES[case["shape"]]
    col = 2 * w * w * (depth - 1) + 2 * w * d  # one column per point
    weights = 4 * (w * (m + r + 1) + (depth - 1) * w * (w + 1) + d * (w + 1))
    if path == "step":
        pts = case["instances"] * (case["s_min"] + case["s_max"]) / 2
        second = 6 if m == 3 else 1
        first = 1 + m + second + d  # value, x tangents, second derivatives, one adjoint per output
        more = 0 if case["linearized"] else case["iters"] * (1 + d)  # trial value and adjoints
        return {"bytes": weights + pts * 4 * m + case["instances"] * 8 * (2 * r + 1), "flops": pts * (first + more) * col}
    if path in ("decode", "jets"):
        p = case["points"]
        cols = 1 if path == "decode" else 1 + m + 1 + d
        outs = d if path == "decode" else d * (1 + m + 1 + r)
        return {"bytes": weights + 4 * p * (m + outs), "flops": p * cols * col}
    if path == "residual":
        p, n = case["points"], case["sets"] * case["params"]
        return {"bytes": weights + p * (4 * m + 8 * d * case["params"] + 8 * case["sets"]) + 8 * n * r,
                "flops": p * n * col}
    if path == "vjp":
        rows = case["batch"] * case["points"]
        return {"bytes": 2 * weights + 4 * case["points"] * m + 8 * rows * d, "flops": 3 * rows * col}
    p = case["nx"] * case["ny"]
    rows = case["batch"] * p
    enc = 4 * case["hidden"] * (p if case["encoder"] == "dense" else 32)
    passes = 2 if path == "grads" else 8  # with Adam: parameters and both moments, read and written, too
    return {"bytes": passes * (weights + enc) + 4 * p * m + 4 * rows,
            "flops": 3 * rows * col + case["batch"] * enc}


# --------------------------------------------------------------------------
# the same results in 64 bits
# --------------------------------------------------------------------------
def _wide(z):
    return [(torch.from_numpy(W).cuda().to(F64), torch.from_numpy(b).cuda().to(F64)) for W, b in z["layers"]]


def _act(z, act):
    return torch.sin(z) if act == "sine" else torch.where(z > 0, z, torch.expm1(z))


def _value(layers, x, q, act="elu"):
    """g [P, d] at x [P, m] for one latent q [r]."""
    a = torch.cat([x, q.expand(len(x), -1)], 1)
    for W, b in layers[:-1]:
        a = _act(a @ W.T + b, act)
    return a @ layers[-1][0].T + layers[-1][1]


def _jets(layers, x, q, act="elu", second="lap"):
    """(g [P, d], dg/dx [P, d, m], second derivatives, dg/dq [P, d, r]) by the
    chain rule; second: "lap" [P, d], "hess" [P, d, m, m] or None."""
    P, m = x.shape
    a = torch.cat([x, q.expand(P, -1)], 1)
    t = torch.eye(a.shape[1], dtype=F64, device=a.device).expand(P, -1, -1)  # [P, m + r, n]
    h = None
    for W, b in layers[:-1]:
        z, dz = a @ W.T + b, t @ W.T
        a = _act(z, act)
        e = torch.exp(z.clamp(max=0.0))
        s1, s2 = (torch.cos(z), -a) if act == "sine" else (torch.where(z > 0, 1.0, e), torch.where(z > 0, 0.0, e))
        dx = dz[:, :m]
        if second == "lap":
            pair = (dx * dx).sum(1)
            h = s2 * pair if h is None else s1 * (h @ W.T) + s2 * pair
        elif second == "hess":
            pair = dx[:, :, None] * dx[:, None]
            s1h, s2h = s1[:, None, None], s2[:, None, None]
            h = s2h * pair if h is None else s1h * (h @ W.T) + s2h * pair
        t = s1[:, None] * dz
    W, b = layers[-1]
    t = (t @ W.T).transpose(1, 2)
    if h is not None:
        h = h @ W.T if second == "lap" else (h @ W.T).permute(0, 3, 1, 2)
    return a @ W.T + b, t[:, :, :m], h, t[:, :, m:]


def _step64(case, z):
    """One latent step per instance: explicit update at the samples, then
    Gauss-Newton with backtracking (or one linearised solve)."""
    layers, m, dt = _wide(z), z["m"], z["dt"]
    out = []
    for i in range(case["instances"]):
        lo, hi = int(z["offsets"][i]), int(z["offsets"][i + 1])
        x, q, c = z["y"][lo:hi].to(F64), z["q"][i], z["coef"][i]
        g, gx, h, J = _jets(layers, x, q, second="hess" if m == 3 else "lap")
        if m == 3:
            lam, mu, rho0, B = c[0], c[1], c[2], c[3:]
            F = torch.eye(3, dtype=F64, device="cuda") + gx
            Fi = torch.linalg.inv(F)
            FiT, lnJ = Fi.transpose(1, 2), torch.log(torch.linalg.det(F))[:, None, None]
            div = torch.zeros_like(g)
            for j in range(3):
                dF = h[:, :, :, j]
                dP = mu * dF + (mu - lam * lnJ) * (FiT @ dF.transpose(1, 2) @ FiT)
                dP = dP + lam * (Fi.transpose(1, 2) * dF).sum((1, 2))[:, None, None] * FiT
                div += dP[:, :, j]
            f = g + dt * dt * (div / rho0 + B)
            f = torch.where(z["clamp"][lo:hi, None] == 1, torch.zeros_like(f), f)
        else:
            f = g + dt * c * h
        for _ in range(1 if case["linearized"] else case["iters"]):
            Jf, res = J.reshape(-1, J.shape[-1]), (f - g).reshape(-1)
            b, phi = Jf.T @ res, 0.5 * (res @ res)
            delta = torch.cholesky_solve(b[:, None], torch.linalg.cholesky(Jf.T @ Jf))[:, 0]
            if case["linearized"]:
                q = q + delta
                break
            small = 1e-6 * (1.0 + q.norm())
            if delta.norm() <= small:
                break
            alpha = 1.0
            for _ in range(11):
                r = f - _value(layers, x, q + alpha * delta)
                if 0.5 * (r * r).sum() <= phi - 1e-4 * alpha * (b @ delta):
                    break
                alpha *= 0.5
            else:
                break
            q = q + alpha * delta
            if alpha * delta.norm() <= small:
                break
            g, _, _, J = _jets(layers, x, q, second=None)
        out.append(q)
    return torch.stack(out)


def _train64(case, z):
    """Loss, gradients and latents of one batch in 64 bits, by autograd."""
    dec = [t.requires_grad_(True) for wb in _wide(z) for t in wb]
    enc = [torch.from_numpy(p).cuda().to(F64).requires_grad_(True) for p in z["enc"]]
    u, x = z["u"].to(F64), z["x"].to(F64)
    a = u
    for k in range(0, len(enc) - 4, 2):
        a = torch.stack([a[:, j:j + 4 * ((a.shape[1] - 6) // 4) + 1:4] for j in range(6)], 2) @ enc[k][0, 0] + enc[k + 1]
        a = _act(a, "elu")
    E1, c1, E2, c2 = enc[-4:]
    q = _act(a @ E1.T + c1, "elu") @ E2.T + c2
    loss = torch.zeros((), dtype=F64, device="cuda")
    layers = list(zip(dec[::2], dec[1::2]))
    for b in range(case["batch"]):
        loss = loss + ((_value(layers, x, q[b], z["act"])[:, 0] - u[b]) ** 2).sum() / u.numel()
    grads = torch.autograd.grad(loss, dec + enc)
    flat = lambda ts: torch.cat([t.reshape(-1) for t in ts]).detach()  # noqa: E731
    gd, ge = flat(grads[:len(dec)]), flat(grads[len(dec):])
    out = {"loss": loss.detach().reshape(1), "grad_dec": gd, "grad_enc": ge}
    if case["path"] == "grads":
        return dict(out, q=q.detach())
    first = lambda p, g: p - 1e-3 * g / (g.abs() + 1e-8)  # noqa: E731  Adam's first step
    return dict(out, dec=first(flat(dec), gd), enc=first(flat(enc), ge))


def exact(case, seed):
    z, path = _inputs(case, seed), case["path"]
    if path == "fd":
        nu = torch.from_numpy(z["mus"]).cuda()[:, None, None]
        u = torch.from_numpy(z["u"]).cuda().repeat(case["fields"], 1, 1)
        out = [u.clone()]
        for _ in range(case["times"] - 1):
            for _ in range(case["substeps"]):
                lap = u[:, 2:, 1:-1] + u[:, :-2, 1:-1] + u[:, 1:-1, 2:] + u[:, 1:-1, :-2] - 4.0 * u[:, 1:-1, 1:-1]
                u[:, 1:-1, 1:-1] += (z["dt"] / z["dx"] ** 2) * nu * lap
            out.append(u.clone())
        return torch.stack(out, 1)
    if path == "step":
        return _step64(case, z)
    if path in ("grads", "train"):
        return _train64(case, z)
    layers = _wide(z)
    if path == "decode":
        return _value(layers, z["x"].to(F64), z["q"], z["act"])
    if path == "jets":
        return _jets(layers, z["x"].to(F64), z["q"], z["act"])
    if path == "vjp":
        ps = [t.requires_grad_(True) for wb in layers for t in wb]
        q = z["q"].detach().to(F64).requires_grad_(True)
        g = torch.stack([_value(layers, z["x"].to(F64), q[b], z["act"]) for b in range(len(q))])
        grads = torch.autograd.grad(g, ps + [q], z["dg"].to(F64))
        return {"g": g.detach(), "grad_params": torch.cat([t.reshape(-1) for t in grads[:-1]]), "grad_q": grads[-1]}
    res = torch.stack([sum((_value(layers, z["x"].to(F64), q) - z["ref"][k]).norm(dim=1) for k, q in enumerate(qs))
                       for qs in z["q"]])
    return {"res": res, "metric": res.mean(1) + res.max(1).values}
