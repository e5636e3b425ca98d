"""Performance cases of the Wilson-Dirac library.

Each case is one call that a program built on this package makes: a hop of one
checkerboard, the full operator, a hop of many right-hand sides, a solve, or a
training gradient of the learned preconditioner.  Handles are made by
``wd_gauge_create`` and used as they come (no tuner run), on lattices between
8^4, which a test or a first attempt uses, and 32^3 x 64.

``prepare`` draws links and fields on the GPU from the seed alone: links
exp(i eps H) with Gaussian traceless Hermitian H, eps 0.2 to 0.4, and sources
with N(0,1) components.  ``exact`` repeats the call in complex128 from Eq. 3,
with dense gamma matrices and uncompressed links, and lays the result out as
the device field that ``run`` returns.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_0710_2442_amd as wd
from paper_0710_2442_amd import learn

KAPPA = 0.124
T_BC = -1
TOL = 1e-11  # of the solves: a digit past the 1e-10 that the results are quoted to
BATCH8 = "8x8x8x8+12x12x12x12+16x16x16x32+16x16x16x16+20x20x20x40+12x12x12x24+16x16x16x24+8x8x8x16"
BATCH_EPS = (0.2, 0.3, 0.4)
REAL_BYTES = {"f64": 8.0, "f32": 4.0, "f16": 52 / 24, "bf16": 2.0}


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest call: one hop on the 8^4 lattice of the first tests
        {"name": "hop_f64_8x8x8x8", "kind": "hop", "dims": "8x8x8x8", "prec": "f64", "parity": 0, "dagger": False},
        # an uneven lattice (odd half extents, slots that no tile divides), the adjoint hop
        {"name": "hop_f32_dag_12x20x6x28", "kind": "hop", "dims": "12x20x6x28", "prec": "f32", "parity": 1,
         "dagger": True},
        # the headline workload's lattice
        {"name": "hop_f64_32x32x32x64", "kind": "hop", "dims": "32x32x32x64", "prec": "f64", "parity": 0,
         "dagger": False},
        # the operator itself, as a solver outside the library applies it
        {"name": "dirac_f64_16x16x16x32", "kind": "dirac", "dims": "16x16x16x32", "prec": "f64", "one_pass": False},
        # the same in one launch, on the lattice of the propagator runs
        {"name": "dirac_one_f32_24x24x24x48", "kind": "dirac", "dims": "24x24x24x48", "prec": "f32",
         "one_pass": True},
        # the 12 spin-colour components of a propagator, in the storage of the inner solver
        {"name": "mrhs12_bf16_24x24x24x48", "kind": "mrhs", "dims": "24x24x24x48", "prec": "bf16", "nrhs": 12,
         "parity": 0},
        # one source, a small lattice: latency of an iteration
        {"name": "cg_f64_8x8x8x16", "kind": "solve", "solver": "cg", "dims": "8x8x8x16", "prec": "f64"},
        # one source, reduced-precision inner solver
        {"name": "defect_bf16_24x24x24x48", "kind": "solve", "solver": "defect", "dims": "24x24x24x48",
         "prec": "bf16"},
        # one source, flexible GCR with the network as preconditioner
        {"name": "fgcr_net_bf16_16x16x16x32", "kind": "solve", "solver": "fgcr", "dims": "16x16x16x32",
         "prec": "bf16"},
        # 12 sources together on the training lattice
        {"name": "mrhs12_solve_bf16_16x16x16x16", "kind": "solve_mrhs", "dims": "16x16x16x16", "prec": "bf16",
         "nrhs": 12},
        # the eight uneven lattices solved in one call
        {"name": "batch8_solve_bf16", "kind": "batch", "dims": BATCH8, "prec": "bf16"},
        # one gradient of the training loop (forward and backward of 8 pairs)
        {"name": "train_grad_bf16_16x16x16x16", "kind": "train", "dims": "16x16x16x16", "prec": "bf16", "pairs": 8},
    ]


def _draw_dims(rng, lo, hi):
    """Four even extents (multiples of 4 half of the time) with lo <= volume <= hi, the volume spread over its
    logarithm."""
    m = rng.choice([2, 4])
    while True:
        v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        side = v ** 0.25
        d = [max(4, m * round(side * math.exp(rng.uniform(-0.35, 0.35)) / m)) for _ in range(3)]
        d.append(max(4, m * round(v / (d[0] * d[1] * d[2]) / m)))
        if d[3] <= 96 and lo <= d[0] * d[1] * d[2] * d[3] <= hi:
            return d


def _text(d):
    return "x".join(str(x) for x in d)


def draw(rng):
    kind = rng.choice(["hop", "hop", "dirac", "mrhs", "solve", "solve", "solve_mrhs", "batch", "train"])
    c = {"kind": kind}
    if kind == "hop":
        c["dims"] = _text(_draw_dims(rng, 4096, 2097152))
        c["prec"] = rng.choice(["f64", "f64", "f32", "f16", "bf16"])
        c["parity"] = rng.randrange(2)
        c["dagger"] = rng.random() < 0.5
    elif kind == "dirac":
        c["dims"] = _text(_draw_dims(rng, 16384, 1048576))
        c["prec"] = rng.choice(["f64", "f32"])
        c["one_pass"] = rng.random() < 0.5
    elif kind == "mrhs":
        c["dims"] = _text(_draw_dims(rng, 16384, 663552))
        c["prec"] = rng.choice(["f64", "f32", "bf16"])
        c["nrhs"] = rng.choice([3, 4, 7, 12, 12, 16, 24]) if math.prod(_dims(c)) < 262144 else 12
        c["parity"] = rng.randrange(2)
    elif kind == "solve":
        c["solver"] = rng.choice(["cg", "defect", "fgcr"])
        c["dims"] = _text(_draw_dims(rng, 4096, 262144))
        c["prec"] = {"cg": "f64", "defect": rng.choice(["f32", "f16", "bf16"]),
                     "fgcr": rng.choice(["f32", "bf16"])}[c["solver"]]
    elif kind == "solve_mrhs":
        c["dims"] = _text(_draw_dims(rng, 8192, 65536))
        c["prec"] = rng.choice(["f32", "bf16"])
        c["nrhs"] = rng.choice([4, 6, 12])
    elif kind == "batch":
        c["dims"] = "+".join(_text(_draw_dims(rng, 4096, 65536)) for _ in range(rng.randrange(3, 8)))
        c["prec"] = rng.choice(["f32", "bf16"])
    else:
        c["dims"] = _text(_draw_dims(rng, 4096, 65536))
        c["prec"] = rng.choice(["f32", "bf16"])
        c["pairs"] = rng.choice([2, 4, 8])
    return c


def _dims(case):
    return [int(x) for x in case["dims"].split("x")]


def _lattices(case):
    return [[int(x) for x in t.split("x")] for t in case["dims"].split("+")]


# ------------------------------------------------------------------ inputs
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(gen, *shape):
    return torch.complex(*(torch.randn(*shape, generator=gen, device="cuda", dtype=torch.float64) for _ in range(2)))


def _matmul3(a, b):
    return sum(a[..., :, k, None] * b[..., None, k, :] for k in range(3))


def _links(gen, dims, eps):
    """SU(3) links near the unit matrix, (L4, L3, L2, L1, 4, 3, 3) complex128 on the GPU."""
    L1, L2, L3, L4 = dims
    h = _normal(gen, L4, L3, L2, L1, 4, 3, 3)
    h = 0.5 * (h + h.conj().transpose(-1, -2))
    trace = h.diagonal(dim1=-2, dim2=-1).sum(-1) / 3
    one = torch.eye(3, dtype=h.dtype, device=h.device)
    x = 1j * eps * (h - trace[..., None, None] * one)
    del h
    u = one + x + _matmul3(x, x) / 2 + _matmul3(x, _matmul3(x, x)) / 6
    del x
    r0 = u[..., 0, :]
    r0 = r0 / torch.linalg.vector_norm(r0, dim=-1, keepdim=True)
    r1 = u[..., 1, :]
    r1 = r1 - (r0.conj() * r1).sum(-1, keepdim=True) * r0
    r1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
    return torch.stack([r0, r1, torch.linalg.cross(r0, r1).conj()], dim=-2)


def _sources(gen, dims, n=None):
    L1, L2, L3, L4 = dims
    shape = (L4, L3, L2, L1, 4, 3)
    return _normal(gen, *(shape if n is None else (n,) + shape))


def _pairs(gen, dims, u, n):
    """Training pairs: normalised Gaussian r, and e = a truncated Neumann series of D^-1 r."""
    r = _sources(gen, dims, n)
    r = r / torch.linalg.vector_norm(r.reshape(n, -1), dim=1).reshape(n, 1, 1, 1, 1, 1, 1)
    e, t = r.clone(), r
    for _ in range(4):
        t = KAPPA * _hop(u, t)
        e = e + t
    return r, e


def _weights(seed):
    """Near-identity network weights, as training starts from."""
    return learn.init_weights(seed)


# ------------------------------------------------------------------ Eq. 3 in complex128
_GAMMA = (((3, 1j), (2, 1j), (1, -1j), (0, -1j)), ((3, -1), (2, 1), (1, 1), (0, -1)),
          ((2, 1j), (3, -1j), (0, -1j), (1, 1j)), ((2, 1), (3, 1), (0, 1), (1, 1)))


def _gamma(mu, psi):
    return torch.stack([f * psi[..., s, :] for s, f in _GAMMA[mu]], dim=-2)


def _shift(psi, mu, step):
    """psi(x + step mu), with the time-boundary factor."""
    out = torch.roll(psi, -step, dims=-3 - mu)
    if mu == 3:
        edge = out.select(-6, out.shape[-6] - 1 if step > 0 else 0)
        edge.mul_(T_BC)
    return out


def _colour(u, psi, dagger=False):
    if dagger:
        return sum(u[..., b, :].conj().unsqueeze(-2) * psi[..., b:b + 1] for b in range(3))
    return sum(u[..., :, b].unsqueeze(-2) * psi[..., b:b + 1] for b in range(3))


def _transport(u, psi, mu, step):
    """U_{x,mu} psi(x + mu) or U^dag_{x-mu,mu} psi(x - mu)."""
    if step > 0:
        return _colour(u[..., mu, :, :], _shift(psi, mu, 1))
    return _colour(torch.roll(u[..., mu, :, :], 1, dims=-3 - mu), _shift(psi, mu, -1), dagger=True)


def _hop(u, psi, dagger=False):
    s = -1 if dagger else 1
    out = torch.zeros_like(psi)
    for mu in range(4):
        g = _gamma(mu, psi)
        out += _transport(u, psi + s * g, mu, 1)
        out += _transport(u, psi - s * g, mu, -1)
    return out


def _dirac(u, psi, kappa, dagger=False):
    return psi - kappa * _hop(u, psi, dagger)


def _solution(u, b, kappa):
    """D_W x = b by CG on the normal equations, to rounding."""
    x = torch.zeros_like(b)
    s = b.clone()
    r = _dirac(u, s, kappa, True)
    p, rr = r.clone(), torch.linalg.vector_norm(r) ** 2
    stop = 1e-14 * torch.linalg.vector_norm(b)
    for k in range(1500):
        q = _dirac(u, p, kappa)
        alpha = rr / torch.linalg.vector_norm(q) ** 2
        x += alpha * p
        s -= alpha * q
        if k % 16 == 15 and bool(torch.linalg.vector_norm(s) < stop):
            break
        r = _dirac(u, s, kappa, True)
        rr, old = torch.linalg.vector_norm(r) ** 2, rr
        p = r + (rr / old) * p
    return x


def _layer(u, psi, w):
    """One network layer: psi a list of channels, w (9, out, in, 4, 4)."""
    out = [0] * w.shape[1]
    for c, p in enumerate(psi):
        for h in range(9):
            t = p if h == 0 else _transport(u, p, (h - 1) % 4, 1 if h < 5 else -1)
            m = t.movedim(-2, 0)
            for o in range(w.shape[1]):
                out[o] = out[o] + (w[h, o, c] @ m.reshape(4, -1)).reshape(m.shape).movedim(0, -2)
    return out


# ------------------------------------------------------------------ field layout
def _basis(psi):
    """Chiral basis <-> the stored one, where gamma_4 is diagonal."""
    a, b = psi[..., :2, :], psi[..., 2:, :]
    return torch.cat([a + b, a - b], dim=-2) / math.sqrt(2.0)


def _half_sites(dims, parity):
    L1, L2, L3, L4 = dims
    x = [torch.arange(n, device="cuda") for n in (L4, L3, L2, L1)]
    odd = (x[0][:, None, None, None] + x[1][:, None, None] + x[2][:, None] + x[3]) % 2
    return torch.nonzero(odd.reshape(-1) == parity).reshape(-1)


def _stored(psi, prec):
    """The chiral field that a field of precision prec holds for psi (rounded in the stored basis)."""
    v = torch.view_as_real(_basis(psi))
    if prec == "f16":
        m = v.abs().amax(dim=(-1, -2, -3), keepdim=True).float()
        v = m.double() * (v / m).half().double()
    elif prec != "f64":
        v = v.to(torch.float32 if prec == "f32" else torch.bfloat16).double()
    return _basis(torch.view_as_complex(v.contiguous()))


def _layout(psi, dims, prec, parities):
    """The device layout of psi's parities, in float64: chunks of 64 sites, 16-byte packets."""
    per = {"f64": 1, "f32": 2, "f16": 4, "bf16": 4}[prec]
    v, scales, fields = _basis(psi).reshape(-1, 12), [], []
    for p in parities:
        h = v[_half_sites(dims, p)]
        h = torch.cat([h, h.new_zeros(-len(h) % 256, 12)])
        if prec == "f16":
            m = torch.view_as_real(h).abs().amax(dim=(-1, -2))
            scales.append(m.reshape(-1, 64))
            h = h / torch.where(m > 0, m, torch.ones_like(m))[:, None]
        fields.append(torch.view_as_real(h.reshape(-1, 64, 12 // per, per).permute(0, 2, 1, 3).contiguous()).reshape(-1))
    out = torch.cat(fields)
    if prec == "f16":
        return {"values": out.reshape(-1, 3 * 64 * 8), "scales": torch.cat(scales)}
    return out


def _view(field, prec):
    """A device field's numbers."""
    if prec == "f16":
        c = field.view(-1, 208 * 16)
        return {"values": c[:, :192 * 16].view(torch.float16), "scales": c[:, 192 * 16:].view(torch.float32)}
    return field.view({"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}[prec])


def _field(g, psi, prec, parity=wd.WD_FULL):
    f = wd.wd_new_field(g.dims, prec, 1, parity)
    wd.wd_spinor_pack(g, psi.reshape(-1), f, parity, prec)
    return f


# ------------------------------------------------------------------ one call
def _inputs(case, seed):
    """Links and sources of a case, as complex128 arrays on the GPU."""
    gen = _generator(seed)
    kind, n = case["kind"], case.get("nrhs")
    if kind == "batch":
        lat = _lattices(case)
        return [(d, _links(gen, d, BATCH_EPS[i % 3]), _sources(gen, d)) for i, d in enumerate(lat)]
    dims = _dims(case)
    u = _links(gen, dims, 0.3)
    if kind == "train":
        return dims, u, _pairs(gen, dims, u, case["pairs"])
    return dims, u, _sources(gen, dims, n)


def _params(case, net=None):
    prec = case["prec"]
    if case["kind"] == "solve" and case["solver"] == "cg":
        return wd.wd_solve_params_default(solver=wd.WD_SOLVER_CG)
    if case["kind"] == "solve" and case["solver"] == "fgcr":
        return wd.wd_solve_params_default(solver=wd.WD_SOLVER_DEFECT_FGCR, inner_prec=prec, inner_tol=1e-2, fgcr_m=4,
                                          precond=net)
    return wd.wd_solve_params_default(solver=wd.WD_SOLVER_DEFECT_CG, inner_prec=prec,
                                      inner_tol=1e-3 if prec == "f32" else 1e-2)


def prepare(case, seed):
    kind, prec = case["kind"], case["prec"]
    s = {"case": case}
    if kind == "batch":
        s["g"], s["b"], s["x"] = [], [], []
        for d, u, b in _inputs(case, seed):
            g = wd.Gauge(u.cpu().numpy(), d, T_BC, "f64")
            s["g"].append(g)
            s["b"].append(_field(g, b, "f64"))
            s["x"].append(wd.wd_new_field(d, "f64"))
        s["params"] = _params(case)
        s["out"] = [_view(x, "f64") for x in s["x"]]
        return s
    dims, u, psi = _inputs(case, seed)
    g = s["g"] = wd.Gauge(u.cpu().numpy(), dims, T_BC, prec if kind == "hop" else "f64")
    if kind == "hop":
        s["in"] = _field(g, psi, prec, 1 - case["parity"])
        out = s["res"] = wd.wd_new_field(dims, prec, 1, case["parity"])
    elif kind == "dirac":
        s["in"] = _field(g, psi, prec)
        out = s["res"] = wd.wd_new_field(dims, prec)
    elif kind == "mrhs":
        s["in"] = torch.cat([_field(g, p, prec, 1 - case["parity"]) for p in psi])
        out = s["res"] = wd.wd_new_field(dims, prec, case["nrhs"], case["parity"])
    elif kind == "solve":
        if case["solver"] == "fgcr":
            s["net"] = wd.Ptc(g, _weights(seed), "bf16")
        s["b"], s["params"] = _field(g, psi, "f64"), _params(case, s.get("net"))
        out = s["x"] = wd.wd_new_field(dims, "f64")
        prec = "f64"
    elif kind == "solve_mrhs":
        s["b"], s["params"] = torch.cat([_field(g, p, "f64") for p in psi]), _params(case)
        out = s["x"] = wd.wd_new_field(dims, "f64", case["nrhs"])
        prec = "f64"
    else:
        s["net"] = wd.Ptc(g, _weights(seed), prec)
        s["r"], s["e"] = (torch.cat([_field(g, p, "f32") for p in q]) for q in psi)
        return s
    s["out"] = _view(out, prec)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "hop":
        wd.wd_dslash_ex(s["g"], s["in"], s["res"], 1.0, case["parity"], case["prec"],
                        wd.WD_DAGGER if case["dagger"] else 0)
    elif kind == "dirac":
        wd.wd_dslash_ex(s["g"], s["in"], s["res"], KAPPA, wd.WD_FULL, case["prec"],
                        wd.WD_ONE_PASS if case["one_pass"] else 0)
    elif kind == "mrhs":
        wd.wd_dslash_mrhs(s["g"], s["in"], s["res"], KAPPA, case["parity"], case["prec"], case["nrhs"])
    elif kind == "solve":
        wd.wd_solve(s["g"], s["b"], s["x"], KAPPA, TOL, s["params"])
    elif kind == "solve_mrhs":
        wd.wd_solve_mrhs(s["g"], s["b"], s["x"], case["nrhs"], KAPPA, TOL, s["params"])
    elif kind == "batch":
        wd.wd_solve_batch(s["g"], s["b"], s["x"], [KAPPA] * len(s["g"]), TOL, s["params"])
    else:
        # the loss is a mean over FP32 activations
        loss, grad = wd.wd_ptc_loss_grad(s["net"], s["r"], s["e"], case["pairs"])
        return {"loss": np.float32(loss), "grad": grad}
    return s["out"]


# ------------------------------------------------------------------ 64-bit results and work
def exact(case, seed):
    kind, prec = case["kind"], case["prec"]
    if kind == "batch":
        return [_layout(_solution(u, b, KAPPA), d, "f64", (0, 1)) for d, u, b in _inputs(case, seed)]
    dims, u, psi = _inputs(case, seed)
    if kind == "hop":
        return _layout(_hop(u, _masked(_stored(psi, prec), dims, 1 - case["parity"]), case["dagger"]), dims, prec,
                       (case["parity"],))
    if kind == "dirac":
        return _layout(_dirac(u, _stored(psi, prec), KAPPA), dims, prec, (0, 1))
    if kind == "mrhs":
        q = case["parity"]
        return torch.cat([_layout(KAPPA * _hop(u, _masked(_stored(p, prec), dims, 1 - q)), dims, prec, (q,))
                          for p in psi])
    if kind == "solve":
        return _layout(_solution(u, psi, KAPPA), dims, "f64", (0, 1))
    if kind == "solve_mrhs":
        return torch.cat([_layout(_solution(u, b, KAPPA), dims, "f64", (0, 1)) for b in psi])
    flat = torch.from_numpy(_weights(seed)).cuda().view(torch.complex64).to(torch.complex128).requires_grad_()
    w1, w2 = flat[:288].reshape(9, 2, 1, 4, 4), flat[288:].reshape(9, 1, 2, 4, 4)
    loss = 0.0
    for r, e in zip(*psi):
        y = _layer(u, _layer(u, [_stored(r, "f32")], w1), w2)[0]
        one = (y - _stored(e, "f32")).abs().square().sum() / case["pairs"]
        one.backward()
        loss += float(one)
    return {"loss": loss, "grad": torch.view_as_real(flat.grad).reshape(-1)}


def _masked(psi, dims, parity):
    out = torch.zeros_like(psi).reshape(-1, 12)
    at = _half_sites(dims, parity)
    out[at] = psi.reshape(-1, 12)[at]
    return out.reshape(psi.shape)


def _hop_work(dims, prec, nrhs=1, parities=1):
    """Links (12 reals each, FP64 or FP32) and spinors once; 1320 flop a site (Sec. 5)."""
    v = math.prod(dims)
    link = 8.0 if prec == "f64" else 4.0
    sites = v / 2 * parities
    return {"bytes": v * 48 * link + sites * nrhs * 48 * REAL_BYTES[prec], "flops": 1320.0 * sites * nrhs}


def work(case):
    """For a solve: the hops of a typical number of iterations at this kappa, on vectors of the inner precision."""
    kind, prec = case["kind"], case["prec"]
    if kind == "batch":
        each = [_scaled(_hop_work(d, prec), 280) for d in _lattices(case)]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    dims = _dims(case)
    if kind == "hop":
        return _hop_work(dims, prec)
    if kind == "dirac":
        return _hop_work(dims, prec, parities=2)
    if kind == "mrhs":
        return _hop_work(dims, prec, case["nrhs"])
    if kind == "solve":
        return _scaled(_hop_work(dims, prec), {"cg": 260, "defect": 290, "fgcr": 120}[case["solver"]])
    if kind == "solve_mrhs":
        return _scaled(_hop_work(dims, prec, case["nrhs"]), 280)
    # five layer-sized contractions a pair: two forward, one input gradient, two weight gradients
    v = math.prod(dims)
    return {"bytes": v * (192.0 + 192.0 * case["pairs"]), "flops": 5 * 9 * 132 * 8.0 * v * case["pairs"]}


def _scaled(w, n):
    return {k: n * x for k, x in w.items()}
