"""Performance cases: the work that a user of the Wilson-Dirac solver has it do.

Five kinds of call, each through the package's public entry points:

* ``apply``   one application of the Wilson operator (:func:`dslash`): native
  fields in FP16, BF16 and FP32, as an outside solver would call it, or canonical
  complex128 fields in FP64, as a check of a solution does; one or several fields;
* ``solve``   the FP64 refinement around a low-precision BiCGStab
  (:func:`solve_mixed_ir`), on the even-odd system or the full matrix, for one or
  several sources, with or without the network as preconditioner;
* ``bicgstab`` one BiCGStab in FP64 (the reference solver of the paper's Table 2);
* ``pairs``   FP32 BiCGStab solutions of a batch of Gaussian sources to 1e-6, stored
  in complex64: the training pairs of the network;
* ``gradient`` the network's residual loss and its weight gradient over a batch of
  Gaussian sources: forward and backward pass of a training step.

Lattices are those of the tests and the benchmark (8^4, 16^4, 24^3 x 48, 32^3 x 64,
48^3 x 96) and others of the same range, with extents that divide no block among them.
All inputs are seeded and made on the GPU.
"""
import math

import numpy as np
import torch

import paper_2602_14450_amd as q

PRECS = {"fp64": q.FP64, "fp32": q.FP32, "fp16": q.FP16, "bf16": q.BF16}
OPS = {"D": q.OP_D, "H": q.OP_H, "Ddag": q.OP_DDAG}
DTYPES = {"fp64": torch.float64, "fp32": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}
REAL_BYTES = {"fp64": 8, "fp32": 4, "fp16": 2, "bf16": 2}
CHANNELS = (1, 2, 2, 1)
FLOP_PER_SITE = 1368  # one application of D: 8 hops of 168, and 1 - kappa H


def _case(name, kind, dims, **more):
    x, y, z, t = dims
    case = {"kind": kind, "x": x, "y": y, "z": z, "t": t, "nrhs": 1}
    case.update(more)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest call: one application on a test lattice, where the launch is all there is
        _case("apply_fp16_8x8x8x8", "apply", (8, 8, 8, 8), prec="fp16", op="D"),
        # the operator of the roofline: 32^3 x 64 in FP16, native fields
        _case("apply_fp16_32x32x32x64", "apply", (32, 32, 32, 64), prec="fp16", op="D"),
        # a check of solutions held in complex128, on a lattice whose x rows divide no block
        _case("apply_fp64_24x24x24x48", "apply", (24, 24, 24, 48), prec="fp64", op="D"),
        # the 12 spin-colour fields of a propagator in one application
        _case("apply_fp16_24x24x24x48_12", "apply", (24, 24, 24, 48), prec="fp16", op="D", nrhs=12),
        # the smallest solve: latency of launches and polls
        _case("solve_fp16_8x8x8x8", "solve", (8, 8, 8, 8), prec="fp16", even_odd=True, inner_tol=1e-3, net=False,
              source="gauss"),
        # the headline solve
        _case("solve_fp16_32x32x32x64", "solve", (32, 32, 32, 64), prec="fp16", even_odd=True, inner_tol=1e-3,
              net=False, source="gauss"),
        # a whole propagator: 12 point sources in one call
        _case("solve_fp16_32x32x32x64_12", "solve", (32, 32, 32, 64), prec="fp16", even_odd=True, inner_tol=1e-3,
              net=False, source="point", nrhs=12),
        # the largest lattice that the benchmark solves on one GPU
        _case("solve_fp16_48x48x48x96", "solve", (48, 48, 48, 96), prec="fp16", even_odd=True, inner_tol=1e-2,
              net=False, source="gauss"),
        # the reference solver in full precision, on a lattice between the tuned ones
        _case("bicgstab_fp64_20x20x20x40", "bicgstab", (20, 20, 20, 40), prec="fp64", even_odd=True),
        # one batch of training pairs
        _case("pairs_fp32_16x16x16x16_16", "pairs", (16, 16, 16, 16), prec="fp32", nrhs=16),
        # the learned form: the network as right preconditioner on a held-out field
        _case("solve_net_16x16x16x16", "solve", (16, 16, 16, 16), prec="fp16", even_odd=False, inner_tol=1e-3,
              net=True, source="gauss"),
        # one training step's gradient at the training batch
        _case("gradient_16x16x16x16_16", "gradient", (16, 16, 16, 16), nrhs=16),
    ]


EXTENTS = (4, 6, 8, 10, 12, 14, 16, 18, 20, 24, 28, 32, 36, 40, 48)


def _draw_dims(rng, sites):
    """Four even extents of a volume up to `sites`, spread over its logarithm from 4^4."""
    want = math.exp(rng.uniform(math.log(256), math.log(sites)))
    while True:
        dims = [rng.choice(EXTENTS) for _ in range(4)]
        if rng.random() < 0.5:
            dims = [dims[0]] * 3 + [dims[3]]
        v = math.prod(dims)
        if v <= sites and want / 2 <= v <= want * 2:
            return dims


def draw(rng):
    kind = rng.choice(("apply", "apply", "solve", "solve", "solve", "bicgstab", "pairs", "gradient"))
    if kind == "apply":
        nrhs = rng.choice((1, 1, 1, 2, 3, 4, 5, 12))
        return _case(None, kind, _draw_dims(rng, 4_000_000 // nrhs), nrhs=nrhs, op=rng.choice(("D", "D", "H", "Ddag")),
                     prec=rng.choice(("fp16", "fp16", "bf16", "fp32", "fp64")))
    if kind == "solve":
        prec = rng.choice(("fp16", "fp16", "fp16", "bf16", "fp32"))
        net = prec == "fp16" and rng.random() < 0.25
        even_odd = rng.random() < 0.7
        nrhs = rng.choice((1, 1, 1, 2, 4)) if net else rng.choice((1, 1, 1, 2, 4, 12))
        return _case(None, kind, _draw_dims(rng, (400_000 if net else 4_000_000) // nrhs), nrhs=nrhs, prec=prec, net=net,
                     even_odd=even_odd, inner_tol=1e-3 if prec == "fp16" else 1e-2, source="gauss")
    if kind == "bicgstab":
        return _case(None, kind, _draw_dims(rng, 2_000_000), prec="fp64", even_odd=rng.random() < 0.7)
    nrhs = rng.choice((4, 8, 15, 16))
    dims = _draw_dims(rng, 1_200_000 // nrhs)
    return _case(None, kind, dims, nrhs=nrhs, prec="fp32") if kind == "pairs" else _case(None, kind, dims, nrhs=nrhs)


# ---------------------------------------------------------------------------
# Inputs, from the seed alone
def _dims(case):
    return (case["x"], case["y"], case["z"], case["t"])


def _volume(case):
    return math.prod(_dims(case))


def _eps_kappa(case):
    """Roughness of the links and hopping parameter of the benchmark's lattices."""
    if _volume(case) > 8_000_000:
        return 0.2, 0.1245
    return 0.3, 0.12 if _volume(case) < 16**4 else 0.124


def _generator(seed, what):
    return torch.Generator(device="cuda").manual_seed(1000 * int(seed) + what)


def _mul3(a, b):
    return (a.unsqueeze(-1) * b.unsqueeze(-3)).sum(-2)


def _links(case, seed):
    """SU(3) links exp(i eps sum_a c_a lambda_a), c_a normal, re-unitarised: complex128 (V, 4, 3, 3)."""
    eps, _ = _eps_kappa(case)
    n = _volume(case) * 4
    gen = _generator(seed, 1)
    u = torch.empty((n, 3, 3), dtype=torch.complex128, device="cuda")
    step = 1 << 21
    for at in range(0, n, step):
        m = min(step, n - at)
        c = torch.randn((8, m), dtype=torch.float64, device="cuda", generator=gen) * eps
        h = torch.zeros((m, 3, 3), dtype=torch.complex128, device="cuda")
        for a, (i, j) in enumerate(((0, 1), (0, 2), (1, 2))):
            h[:, i, j] = torch.complex(c[2 * a], -c[2 * a + 1])
            h[:, j, i] = torch.complex(c[2 * a], c[2 * a + 1])
        d = c[7] / math.sqrt(3.0)
        h[:, 0, 0], h[:, 1, 1], h[:, 2, 2] = (d + c[6]).to(h.dtype), (d - c[6]).to(h.dtype), (-2 * d).to(h.dtype)
        h = h * (1j / 8)
        e = torch.eye(3, dtype=h.dtype, device="cuda") + h / 8
        for k in range(7, 0, -1):  # Taylor series of exp(h), three times squared
            e = torch.eye(3, dtype=h.dtype, device="cuda") + _mul3(h, e) / k
        for _ in range(3):
            e = _mul3(e, e)
        r0 = e[:, 0] / torch.linalg.vector_norm(e[:, 0], dim=1, keepdim=True)
        r1 = e[:, 1] - (r0.conj() * e[:, 1]).sum(1, keepdim=True) * r0
        r1 = r1 / torch.linalg.vector_norm(r1, dim=1, keepdim=True)
        u[at:at + m, 0], u[at:at + m, 1] = r0, r1
        for k in range(3):
            i, j = (k + 1) % 3, (k + 2) % 3
            u[at:at + m, 2, k] = (r0[:, i] * r1[:, j] - r0[:, j] * r1[:, i]).conj()
    return u.view(-1, 4, 3, 3)


def _sources(case, seed):
    """(nrhs, V, 4, 3) complex128: Gaussian with E|z|^2 = 1, or the spin-colour unit point sources at the origin."""
    shape = (case["nrhs"], _volume(case), 4, 3)
    if case.get("source") == "point":
        b = torch.zeros(shape, dtype=torch.complex128, device="cuda")
        for k in range(case["nrhs"]):
            b[k, 0, k // 3, k % 3] = 1
        return b
    return torch.randn(shape, dtype=torch.complex128, device="cuda", generator=_generator(seed, 2))


#: gamma_mu psi = phase[s] psi[perm[s]] in the basis of the library's header
GAMMAS = (((3, 2, 1, 0), (-1j, -1j, 1j, 1j)), ((3, 2, 1, 0), (-1, 1, 1, -1)), ((2, 3, 0, 1), (-1j, 1j, 1j, -1j)),
          ((0, 1, 2, 3), (1, 1, -1, -1)))


def _weights(case, seed):
    """The network's weights in the course of training: the third-order Neumann series, and 1% of noise."""
    _, kappa = _eps_kappa(case)
    rng = np.random.default_rng(int(seed))
    one, hop = np.zeros((9, 4, 4), dtype=np.complex128), np.zeros((9, 4, 4), dtype=np.complex128)
    one[0] = np.eye(4)
    for mu, (perm, phase) in enumerate(GAMMAS):
        gamma = np.zeros((4, 4), dtype=np.complex128)
        gamma[np.arange(4), perm] = phase
        hop[1 + 2 * mu], hop[2 + 2 * mu] = kappa * (np.eye(4) - gamma), kappa * (np.eye(4) + gamma)
    rows = ([[one], [hop]], [[one, one], [hop, hop]], [[one, hop]])
    out = []
    for r in rows:
        w = np.stack([np.stack(c, axis=1) for c in r], axis=1)  # (9, C_out, C_in, 4, 4)
        out.append(w + 0.01 * kappa * (rng.standard_normal(w.shape) + 1j * rng.standard_normal(w.shape)))
    return out


def prepare(case, seed):
    dims, kind = _dims(case), case["kind"]
    _, kappa = _eps_kappa(case)
    g = q.gauge_upload(_links(case, seed), dims)
    s = {"case": case, "g": g, "kappa": kappa}
    b = _sources(case, seed)
    if kind == "apply" and case["prec"] != "fp64":
        prec, n = PRECS[case["prec"]], case["nrhs"]
        s["in"] = torch.zeros(g.spinor_bytes(prec) * n, dtype=torch.uint8, device="cuda")
        s["out"] = torch.zeros_like(s["in"])
        q.convert(g, prec, s["in"], b, want_norm=False)
    elif kind == "gradient":
        s["b"] = b
    else:
        s["b"], s["x"] = b, torch.zeros_like(b)
    if kind == "gradient" or case.get("net"):
        s["net"] = q.PTC(g, CHANNELS, max_batch=case["nrhs"])
        s["net"].set_weights(_weights(case, seed))
    return s


def run(state):
    case, g, kappa, kind = state["case"], state["g"], state["kappa"], state["case"]["kind"]
    if kind == "apply":
        prec = PRECS[case["prec"]]
        if case["prec"] == "fp64":
            return q.dslash(g, kappa, state["x"], state["b"], op=OPS[case["op"]], prec=prec)
        q.dslash(g, kappa, state["out"], state["in"], op=OPS[case["op"]], prec=prec, layout=q.NATIVE, nrhs=case["nrhs"])
        return state["out"].view(DTYPES[case["prec"]])
    if kind == "solve":
        q.solve_mixed_ir(g, kappa, state["x"], state["b"], inner_prec=PRECS[case["prec"]], s=128.0, sigma=64.0,
                         tol=1e-12, inner_tol=case["inner_tol"], even_odd=case["even_odd"], precond=state.get("net"))
        return state["x"]
    if kind == "bicgstab":
        q.bicgstab(g, kappa, state["x"], state["b"], prec=q.FP64, tol=1e-12, even_odd=case["even_odd"], history=False)
        return state["x"]
    if kind == "pairs":
        q.bicgstab(g, kappa, state["x"], state["b"], prec=q.FP32, tol=1e-6, max_iter=5000, history=False)
        return state["x"].to(torch.complex64)
    loss, grad = state["net"].loss_grad_residual(kappa, state["b"])
    # the network's weights and gradients are FP32 numbers in a complex128 array
    return loss, [w.astype(np.complex64) for w in grad]


# ---------------------------------------------------------------------------
# What a pass cannot do without
def work(case):
    v, n = _volume(case), case["nrhs"]
    link, spinor = 48, 24  # reals of a site's four links (two rows each) and of its spinor

    def apply(prec, sites, share=1.0):
        """One application: links once, n fields in and out."""
        return REAL_BYTES[prec] * sites * (share * link + 2 * n * spinor)

    if case["kind"] == "apply":
        return {"bytes": apply(case["prec"], v), "flops": FLOP_PER_SITE * v * n}
    ends = 2 * n * v * spinor * 8  # b and x in complex128
    if case["kind"] == "gradient":
        mix = 8 * sum(9 * 16 * a * b * 3 for a, b in zip(CHANNELS[:-1], CHANNELS[1:]))
        # b once, the links once; products of the forward pass, of the weights' and of the fields' gradients
        return {"bytes": ends / 2 + 4 * v * link, "flops": n * v * (3 * mix + 2 * FLOP_PER_SITE)}
    if case.get("net"):
        # 16 inner iterations: two applications of D and two of the network (three layers, ten fields) each,
        # then about 5 FP64 residuals
        layers = REAL_BYTES["fp16"] * v * (3 * link + 10 * n * spinor)
        mix = 8 * sum(9 * 16 * a * b * 3 for a, b in zip(CHANNELS[:-1], CHANNELS[1:]))
        return {"bytes": ends + 32 * (apply("fp16", v) + layers) + 5 * apply("fp64", v),
                "flops": n * v * (32 * (mix + FLOP_PER_SITE) + 5 * FLOP_PER_SITE)}
    if case["kind"] in ("bicgstab", "pairs"):
        products, exact, prec = (36 if case["prec"] == "fp64" else 34), 1, case["prec"]
    else:
        products, exact, prec = 40, 5, case["prec"]
    # an even-odd application passes over the links twice and over half-size fields, and does one application's work;
    # the full matrix takes twice the applications
    if case.get("even_odd"):
        one, one64 = (2 * REAL_BYTES[p] * v * (link + n * spinor) for p in (prec, "fp64"))
    else:
        products *= 2 if case["kind"] != "pairs" else 1
        one, one64 = apply(prec, v), apply("fp64", v)
    return {"bytes": ends + products * one + exact * one64, "flops": FLOP_PER_SITE * v * n * (products + exact)}


# ---------------------------------------------------------------------------
# The same in 64 bits, in plain torch
def _gamma(mu, f):
    perm, phase = GAMMAS[mu]
    ph = torch.tensor(phase, dtype=f.dtype, device=f.device)
    return f[..., list(perm), :] * ph[:, None]


def _times(u, f):
    """u[..., a, b] f[..., spin, b]"""
    return sum(u[..., None, :, b] * f[..., b, None] for b in range(3))


def _transport(u, mu, sign, f):
    """U_mu(x) f(x + mu), or U_mu(x - mu)^dag f(x - mu); f: (n, t, z, y, x, spin, colour)."""
    axis = 4 - mu
    if sign > 0:
        return _times(u[..., mu, :, :], torch.roll(f, -1, axis))
    return torch.roll(_times(u[..., mu, :, :].transpose(-1, -2).conj(), f), 1, axis)


def _hop(u, f, dag=False):
    out = torch.zeros_like(f)
    for mu in range(4):
        for sign in (1, -1):
            w = _transport(u, mu, sign, f)
            out = out + w + (sign if dag else -sign) * _gamma(mu, w)
    return out


def _solve(apply, b, tol):
    """BiCGStab in 64 bits, one field at a time, restarted until the true residual is below tol |b|."""
    x = torch.zeros_like(b)
    dot = lambda a, c: torch.vdot(a.reshape(-1), c.reshape(-1))  # noqa: E731
    norm_b = torch.linalg.vector_norm(b)
    for _ in range(4):
        r = b - apply(x)
        if torch.linalg.vector_norm(r) <= tol * norm_b:
            break
        shadow, p, rho = r.clone(), r.clone(), dot(r, r)
        for _ in range(400):
            v = apply(p)
            alpha = rho / dot(shadow, v)
            s = r - alpha * v
            t = apply(s)
            omega = dot(t, s) / dot(t, t)
            x = x + alpha * p + omega * s
            r = s - omega * t
            if torch.linalg.vector_norm(r) <= tol / 2 * norm_b:
                break
            new = dot(shadow, r)
            p = r + (new / rho) * (alpha / omega) * (p - omega * v)
            rho = new
    return x


def _native(case, f):
    """Canonical fields (n, V, 4, 3) in the order of the library's native layout, as reals."""
    x, y, z, t = _dims(case)
    n, per = f.shape[0], 16 // (2 * REAL_BYTES[case["prec"]])
    f = f.reshape(n, t, z, y, x, 12)
    at = torch.stack(torch.meshgrid(*(torch.arange(k, device=f.device) for k in (t, z, y, x)), indexing="ij")).sum(0) % 2
    half = _volume(case) // 2
    blocks = -(-half // 64)
    out = torch.zeros((n, 2, blocks * 64, 12), dtype=f.dtype, device=f.device)
    for parity in (0, 1):
        out[:, parity, :half] = f[:, at == parity]
    out = out.reshape(n, 2, blocks, 64, 12 // per, per).transpose(3, 4)
    return torch.view_as_real(out.contiguous()).reshape(-1)


def _network(u, ws, f):
    fields = [f]
    for w in ws:
        paths = [[c] + [_transport(u, mu, sign, c) for mu in range(4) for sign in (1, -1)] for c in fields]
        out = []
        for j in range(w.shape[1]):
            acc = 0
            for i in range(len(fields)):
                for p in range(9):
                    m = w[p, j, i]
                    acc = acc + torch.stack([sum(m[s, k] * paths[i][p][..., k, :] for k in range(4)) for s in range(4)], -2)
            out.append(acc)
        fields = out
    return fields[0]


def exact(case, seed):
    x, y, z, t = _dims(case)
    _, kappa = _eps_kappa(case)
    kind, n = case["kind"], case["nrhs"]
    if kind in ("solve", "pairs", "bicgstab") and (_volume(case) * n > 12_000_000 or case.get("source") == "point"):
        return None
    u = _links(case, seed).view(t, z, y, x, 4, 3, 3)
    b = _sources(case, seed).view(n, t, z, y, x, 4, 3)
    if kind == "apply":
        out = []
        for f in b.split(1):
            h = _hop(u, f, dag=case["op"] == "Ddag")
            out.append(h if case["op"] == "H" else f - kappa * h)
        out = torch.cat(out).view(n, -1, 4, 3)
        return out if case["prec"] == "fp64" else _native(case, out)
    if kind != "gradient":
        out = torch.cat([_solve(lambda f: f - kappa * _hop(u, f), f, 1e-14) for f in b.split(1)])
        return out.view(n, -1, 4, 3)
    ws = [torch.from_numpy(w).cuda().requires_grad_() for w in _weights(case, seed)]
    loss = 0.0
    for f in b.split(1):
        m = _network(u, ws, f)
        r = m - kappa * _hop(u, m) - f
        one = r.abs().square().sum() / f.abs().square().sum() / n
        one.backward()
        loss += one.item()
    return loss, [w.grad for w in ws]
