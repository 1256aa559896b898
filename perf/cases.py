"""Workloads of the library, as a flow solver issues them, for timing and for
comparing results between builds.

A case is a dict of plain values.  ``listed()`` gives the fixed ones,
``draw(rng)`` one more of the same ranges; ``prepare(case, seed)`` makes what
the solver holds before the call (states, mesh, network, mechanism handle) on
the GPU, ``run(state)`` is one pass through the public entry points and
returns its outputs, ``work(case)`` the bytes and operations the pass cannot
do without, and ``exact(case, seed)`` the same outputs in plain 64-bit torch
where they have a closed form.

What the kinds stand for:

* ``plain``    the chemistry of one flow step by the stiff integrator
               (chem_integrate).  A flow solver calls it on every cell of its
               subdomain each step; the state is restored from a kept copy
               first, as bench.py does, so that every pass does the same work.
* ``served``   the same step by the trained network with checks and fallback
               (chem_surrogate_infer), one network or one per species.
* ``train``    a training run on labelled states (chem_surrogate_train), its
               result read back as a program that saves it does.
* ``props``    temperature from enthalpy, then mixture viscosity, conductivity
               and diffusion coefficients of a field (the Thermo calls).
* ``laplace``  the implicit Laplacian of one equation: straight into CSR, or
               Algorithm 1 in ldu form and its conversion.

A trained network is not available to a case (training takes seconds and its
result would depend on the build), so the served networks are seeded: random
weights whose output layer is projected onto the element-conserving
subspace, with an output scale that keeps every prediction acceptable, as
a trained network's are.  The cells that fall back are chosen by the input:
burnt hot spots above the training box's 2500 K.
"""
from __future__ import annotations

import functools
import math
import os
import tempfile

import numpy as np
import torch

from chemgen.fields import P_ATM, end_states
from chemgen.mechanism import R_U, standard_mechanism
from chemgen.mesh import box_mesh
from chemgen.surrogate_data import epoch_orders, init_params, init_species_params, network_dims
from chemgen.transport import transport_fits
from paper_2312_13513_amd import chem

F64 = torch.float64
MIX_SEED = 7        # the mixture of bench.py's trained network and served fields
TRANSPORT_SEED = 11


def listed():
    return [
        # a subdomain of a few hundred cells: one launch's latency
        {"name": "plain_few", "kind": "plain", "mech": "M9", "field": "random", "n": 257, "dt": 1e-6},
        # the benchmark's default step: 64^3 flame, mechanism compiled in
        {"name": "plain_flame64", "kind": "plain", "mech": "M9", "field": "flame", "n": 262144, "dt": 1e-6},
        # a user's mechanism of the CH4 case's size (20 species, 85 reactions, fall-off): table-driven kernels
        {"name": "plain_ch4", "kind": "plain", "mech": "CH4R", "field": "flame", "n": 20011, "dt": 1e-6},
        # 35 species / 200 reactions: labelling of training states, and the step without a network
        {"name": "plain_m35", "kind": "plain", "mech": "M35", "field": "flame", "n": 65536, "dt": 1e-6},
        # the same with FP32 Jacobian and LU (the mixed mode of the three-zone workload)
        {"name": "plain_m35_mixed", "kind": "plain", "mech": "M35", "field": "flame", "n": 16383, "dt": 1e-6,
         "precision": 1},
        # served step of a small subdomain, nothing rejected
        {"name": "served_few", "kind": "served", "mech": "M35", "n": 1000, "dt": 1e-5, "hot": 0.0},
        # the benchmark's served field: 256 x 128 x 128 cells, one in 10^5 integrated
        {"name": "served_field", "kind": "served", "mech": "M35", "n": 4194304, "dt": 1e-5, "hot": 1e-5},
        # the paper's per-species networks (1600-800-400 each)
        {"name": "served_species", "kind": "served", "mech": "M9", "n": 65536, "dt": 1e-6, "hot": 0.0,
         "per_species": True},
        # training, the benchmark's batch
        {"name": "train", "kind": "train", "mech": "M35", "n": 65536, "batch": 4096, "epochs": 2},
        # one GPU's share of the 256^3 TGV mesh
        {"name": "props_tgv", "kind": "props", "mech": "M9", "n": 4194304},
        # the same of the larger mechanism, ragged
        {"name": "props_m35", "kind": "props", "mech": "M35", "n": 500003},
        # the benchmark's mesh, assembled straight into CSR
        {"name": "laplace_128", "kind": "laplace", "nx": 128, "ny": 128, "nz": 128, "direct": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plain", "plain", "plain", "served", "served", "train", "props", "props", "laplace", "laplace"])
    if kind == "plain":
        c = rng.choice([
            # (mechanism, field, largest, precision, schedule): schedule -1 is the library's choice, 2 the
            # 16-lane tiles that serve small mechanisms which are not compiled in
            ("M9", "random", 32768, 0, -1), ("M9", "flame", 262144, 0, -1), ("H2R", "random", 32768, 0, -1),
            ("H2R", "flame", 262144, 0, -1), ("M9", "flame", 65536, 0, 2), ("CH4R", "flame", 20000, 0, -1),
            ("M35", "flame", 16384, 0, -1), ("M35", "flame", 16384, 1, -1)])
        return {"kind": "plain", "mech": c[0], "field": c[1], "n": _log_int(rng, 100, c[2]), "dt": 1e-6,
                "precision": c[3], "schedule": c[4]}
    if kind == "served":
        if rng.random() < 0.3:
            return {"kind": "served", "mech": "M9", "n": _log_int(rng, 200, 65536), "dt": 1e-6, "hot": 0.0,
                    "per_species": True}
        return {"kind": "served", "mech": rng.choice(["M9", "M35", "M35"]), "n": _log_int(rng, 200, 4194304),
                "dt": 1e-5, "hot": rng.choice([0.0, 1e-6, 1e-5, 1e-4])}
    if kind == "train":
        return {"kind": "train", "mech": rng.choice(["M9", "M35"]), "n": _log_int(rng, 8192, 65536),
                "batch": rng.choice([1024, 2048, 4096, 8192]), "epochs": 2}
    if kind == "props":
        m = rng.choice(["M9", "H2R", "CH4R", "M35"])
        return {"kind": "props", "mech": m, "n": _log_int(rng, 500, 4000000 if m in ("M9", "H2R") else 500000)}
    return {"kind": "laplace", "nx": _log_int(rng, 5, 128), "ny": _log_int(rng, 5, 128), "nz": _log_int(rng, 5, 128),
            "direct": rng.random() < 0.5}


# --------------------------------------------------------------------------- inputs


@functools.lru_cache(maxsize=None)
def _mechanism(name):
    return standard_mechanism(name)


@functools.lru_cache(maxsize=None)
def _end_states(name):
    return end_states(_mechanism(name), np.random.default_rng(MIX_SEED))


@functools.lru_cache(maxsize=None)
def _transport(name):
    return transport_fits(_mechanism(name), TRANSPORT_SEED)


@functools.lru_cache(maxsize=4)
def _mesh(nx, ny, nz):
    return box_mesh(nx, ny, nz, grading=(2.0, 1.0, 0.5))


def _handle(name):
    with tempfile.TemporaryDirectory() as d:
        path = os.path.join(d, name + ".mech")
        _mechanism(name).write(path)
        return chem.Mechanism(path, 0)


def _gpu(a):
    return torch.tensor(np.asarray(a), dtype=F64, device="cuda")


def _flame(mech, n, seed):
    """(T, p, Y) of n cells of a smooth flame field: 300 + 1900 c K and the
    mixture of the end states at c, c a normalised sum of Fourier modes."""
    rng = np.random.default_rng(seed)
    side = max(1, round(n ** (1.0 / 3.0)))
    i = torch.arange(n, device="cuda")
    x = torch.stack([(i % side).to(F64), ((i // side) % side).to(F64), (i // (side * side)).to(F64)]) / side
    s = torch.zeros(n, dtype=F64, device="cuda")
    for _ in range(8):
        k = rng.integers(-3, 4, 3)
        k[rng.integers(3)] += 0 if k.any() else 1
        s += rng.uniform(0.5, 1.0) * torch.cos(2.0 * math.pi * (k[0] * x[0] + k[1] * x[1] + k[2] * x[2])
                                               + rng.uniform(0.0, 2.0 * math.pi))
    c = (s - s.min()) / (s.max() - s.min())
    Yu, Yb = _end_states(mech)
    Y = (1.0 - c)[None, :] * _gpu(Yu)[:, None] + c[None, :] * _gpu(Yb)[:, None]
    return 300.0 + 1900.0 * c, torch.full((n,), P_ATM, dtype=F64, device="cuda"), Y.contiguous()


def _random(mech, n, seed):
    """(T, p, Y): T uniform in 900 .. 2200 K, Y from Dirichlet(1)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    T = 900.0 + 1300.0 * torch.rand(n, generator=g, dtype=F64, device="cuda")
    Y = -torch.log1p(-torch.rand(_mechanism(mech).K, n, generator=g, dtype=F64, device="cuda")) + 1e-12
    return T, torch.full((n,), P_ATM, dtype=F64, device="cuda"), (Y / Y.sum(0)).contiguous()


def _served_states(case, seed):
    T, p, Y = _flame(case["mech"], case["n"], seed)
    hot = int(round(case["hot"] * case["n"]))
    if hot:
        rng = np.random.default_rng(seed + 1)
        at = torch.tensor(rng.choice(case["n"], hot, replace=False), device="cuda")
        T[at] = _gpu(rng.uniform(2510.0, 2590.0, hot))
        Y[:, at] = _gpu(_end_states(case["mech"])[1])[:, None].expand(-1, hot)
    return T, p, Y


def _norm(mech, dt, scale):
    """Normalisation: feature means and deviations over a flame line, output scale ``scale``, mean 0."""
    Yu, Yb = _end_states(mech)
    c = np.linspace(0.0, 1.0, 1025)
    Y = (1.0 - c) * Yu[:, None] + c * Yb[:, None]
    raw = np.concatenate([(300.0 + 1900.0 * c)[None], np.full((1, c.size), P_ATM), (Y ** 0.1 - 1.0) / 0.1])
    sig = raw.std(axis=1)
    sig[1] = 0.0   # constant pressure
    return np.concatenate([raw.mean(axis=1), sig, np.zeros_like(scale), scale, [dt]])


def _network(case, seed):
    """(flat FP32 parameters, normalisation) of the served network (see the module's first lines)."""
    m = _mechanism(case["mech"])
    Yu, Yb = _end_states(case["mech"])
    if case.get("per_species"):
        # one output per network: nothing to project; a scale small enough for the element check
        scale = np.maximum(1e-5 * np.minimum(Yu, Yb), 1e-7)
        return init_species_params(m.K, (1600, 800, 400), seed), _norm(case["mech"], case["dt"], scale)
    flat = init_params(network_dims(m.K), seed)
    scale = np.maximum(2e-3 * np.minimum(Yu, Yb), 1e-8)
    A = (m.counts.T / m.molar_masses()) * scale
    P = np.eye(m.K) - np.linalg.pinv(A) @ A
    o = flat.size - m.K - m.K * 128
    flat[o:o + m.K * 128] = (P @ flat[o:o + m.K * 128].reshape(m.K, 128).astype(np.float64)).ravel()
    return flat, _norm(case["mech"], case["dt"], scale)


def _train_data(case, seed):
    T, p, Y = _flame(case["mech"], case["n"], seed)
    g = torch.Generator(device="cuda").manual_seed(seed)
    f = 1.0 + 0.02 * torch.randn(Y.shape, generator=g, dtype=F64, device="cuda")
    Yn = Y * f
    Yn = (Yn / Yn.sum(0)).contiguous()
    order = epoch_orders(case["n"], case["epochs"], seed)
    return T, p, Y, Yn, order


def _train_norm(case):
    """Scale of the targets: the deviation of 2 % changes along the flame line."""
    Yu, Yb = _end_states(case["mech"])
    return _norm(case["mech"], 1e-5, 0.02 * np.maximum(np.maximum(Yu, Yb), 1e-6))


def _laplace_fields(mesh, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda n: torch.rand(n, generator=g, dtype=F64, device="cuda")  # noqa: E731
    x = _gpu(mesh.centres)
    gc = 1.0 + 0.5 * torch.sin(6.0 * x[:, 0] + 6.3 * r(1)) * torch.cos(5.0 * x[:, 1]) + 0.2 * r(mesh.ncells)
    return gc, 0.5 + r(mesh.nbfaces), 2.0 * r(mesh.nbfaces) - 1.0


# --------------------------------------------------------------------------- prepare and run


def prepare(case, seed):
    return {"plain": _prepare_plain, "served": _prepare_served, "train": _prepare_train, "props": _prepare_props,
            "laplace": _prepare_laplace}[case["kind"]](case, seed)


def run(state):
    return state["run"](state)


def _states(case, seed):
    return {"random": _random, "flame": _flame}[case["field"]](case["mech"], case["n"], seed)


def _prepare_plain(case, seed):
    T, p, Y = _states(case, seed)
    opts = chem.chem_default_opts()
    opts.precision = case.get("precision", 0)
    opts.schedule = case.get("schedule", -1)
    return {"run": _run_plain, "mech": _handle(case["mech"]), "opts": opts, "dt": case["dt"], "T0": T, "p": p, "Y0": Y,
            "T": T.clone(), "Y": Y.clone(), "status": torch.zeros(case["n"], dtype=torch.int32, device="cuda")}


def _run_plain(s):
    s["T"].copy_(s["T0"])
    s["Y"].copy_(s["Y0"])
    s["mech"].integrate(s["T"], s["p"], s["Y"], s["dt"], s["opts"], status=s["status"])
    return {"T": s["T"], "Y": s["Y"], "status": s["status"]}


def _prepare_served(case, seed):
    T, p, Y = _served_states(case, seed)
    mech = _handle(case["mech"])
    hidden = (1600, 800, 400) if case.get("per_species") else (512, 256, 128)
    net = chem.Surrogate(mech, *hidden, per_species=bool(case.get("per_species")))
    params, norm = _network(case, seed)
    net.set_params(params)
    net.set_norm(norm)
    net.reserve(case["n"])
    return {"run": _run_served, "mech": mech, "net": net, "dt": case["dt"], "T0": T, "p": p, "Y0": Y, "T": T.clone(),
            "Y": Y.clone(), "mask": torch.zeros(case["n"], dtype=torch.int32, device="cuda"),
            "count": torch.zeros(1, dtype=torch.int64, device="cuda")}


def _run_served(s):
    s["T"].copy_(s["T0"])
    s["Y"].copy_(s["Y0"])
    s["net"].infer(s["T"], s["p"], s["Y"], s["dt"], mask=s["mask"], fallback_count=s["count"])
    return {"T": s["T"], "Y": s["Y"], "mask": s["mask"], "count": s["count"]}


def _prepare_train(case, seed):
    T, p, Y, Yn, order = _train_data(case, seed)
    mech = _handle(case["mech"])
    net = chem.Surrogate(mech, 512, 256, 128)
    net.set_params(init_params(network_dims(mech.K), seed))
    net.set_norm(_train_norm(case))
    return {"run": _run_train, "mech": mech, "net": net, "T": T, "p": p, "Y": Y, "Yn": Yn,
            "order": torch.tensor(order, device="cuda"), "epochs": case["epochs"], "batch": case["batch"]}


def _run_train(s):
    losses = s["net"].train(s["T"], s["p"], s["Y"], s["Yn"], s["epochs"], s["batch"], order=s["order"])
    return {"losses": losses, "params": s["net"].get_params()}


def _prepare_props(case, seed):
    T, p, Y = _flame(case["mech"], case["n"], seed)
    g = torch.Generator(device="cuda").manual_seed(seed)
    guess = T + 40.0 * torch.rand(case["n"], generator=g, dtype=F64, device="cuda") - 20.0
    mech = _handle(case["mech"])
    mech.set_transport(*_transport(case["mech"]))
    e = lambda: torch.empty(case["n"], dtype=F64, device="cuda")  # noqa: E731
    return {"run": _run_props, "mech": mech, "h": _h_cp(case["mech"], T, Y)[0], "guess": guess, "p": p, "Y": Y, "T": e(),
            "cp": e(), "mu": e(), "lam": e(), "D": torch.empty_like(Y)}


def _run_props(s):
    s["T"].copy_(s["guess"])
    s["mech"].T_from_h(s["h"], s["Y"], s["T"], cp=s["cp"])
    s["mech"].transport(s["T"], s["p"], s["Y"], mu=s["mu"], lam=s["lam"], D=s["D"])
    return {k: s[k] for k in ("T", "cp", "mu", "lam", "D")}


def _prepare_laplace(case, seed):
    mesh = _mesh(case["nx"], case["ny"], case["nz"])
    gc, gb, pb = _laplace_fields(mesh, seed)
    m = chem.LduMesh(mesh, 0)
    e = lambda n: torch.empty(n, dtype=F64, device="cuda")  # noqa: E731
    s = {"run": _run_laplace, "mesh": m, "gc": gc, "gb": gb, "pb": pb, "csr": e(m.nnz), "rhs": e(m.ncells)}
    if not case["direct"]:
        s["ldu"] = [e(m.nfaces), e(m.nfaces), e(m.ncells), e(m.nbfaces), e(m.nbfaces)]
    return s


def _run_laplace(s):
    if "ldu" not in s:
        s["mesh"].laplacian_csr(s["gc"], s["gb"], s["pb"], s["csr"], s["rhs"])
        return {"csr": s["csr"], "rhs": s["rhs"]}
    s["mesh"].laplacian(s["gc"], s["gb"], s["pb"], *s["ldu"])
    s["mesh"].to_csr(*s["ldu"], s["csr"], s["rhs"])
    return {"csr": s["csr"], "rhs": s["rhs"], **dict(zip(("lower", "upper", "diag", "internal", "boundary"), s["ldu"]))}


# --------------------------------------------------------------------------- work


#: Mean right-hand sides, Jacobians, Newton iterations and steps per cell of the integrator's method on each field.
_COUNTS = {("M9", "flame"): (12.0, 3.0, 9.3, 7.1), ("M9", "random"): (60.0, 9.5, 57.0, 49.6),
           ("H2R", "flame"): (6.2, 1.6, 4.2, 3.3), ("H2R", "random"): (46.4, 9.0, 43.4, 36.3),
           ("CH4R", "flame"): (45.1, 8.5, 42.1, 35.3), ("M35", "flame"): (399.4, 44.4, 396.4, 334.8)}


def work(case):
    if case["kind"] == "laplace":
        nx, ny, nz = case["nx"], case["ny"], case["nz"]
        c = nx * ny * nz
        f = 3 * c - nx * ny - ny * nz - nx * nz
        b = 2 * (nx * ny + ny * nz + nx * nz)
        # gamma, geometry of every face, boundary values in; matrix and right-hand side out
        out = 8 * ((c + 2 * f) + c) + (0 if case["direct"] else 8 * (2 * f + c + 2 * b))
        return {"bytes": 8 * c + 24 * f + 40 * b + out, "flops": 8 * f + 4 * b}
    m, n = _mechanism(case["mech"]), case["n"]
    K, R, N = m.K, m.R, m.K + 1
    state = 8 * (2 * K + 3) * n
    if case["kind"] == "plain":
        rhs, jac, newton, steps = _COUNTS[case["mech"], case["field"]]
        f = rhs * (40 * K + 60 * R + 28) + newton * (2 * N * N + 9 * N + 20) + steps * (21 * N + 60)
        f += jac * (77 * K + 115 * R + 10 * K * K + N * (N - 1) // 2 + (N - 1) * N * (2 * N - 1) // 3 + 2 * N * N)
        return {"bytes": state + 4 * n, "flops": f * n}
    if case["kind"] == "served":
        per = K * 2 * ((K + 2) * 1600 + 1600 * 800 + 800 * 400 + 400) if case.get("per_species") \
            else 2 * ((K + 2) * 512 + 512 * 256 + 256 * 128 + 128 * K)
        return {"bytes": state + 4 * n, "flops": per * n}
    if case["kind"] == "train":
        per = 2 * ((K + 2) * 512 + 512 * 256 + 256 * 128 + 128 * K)
        return {"bytes": 8 * (2 * K + 2) * n, "flops": 3 * per * n * case["epochs"]}
    return {"bytes": 8 * (2 * K + 8) * n, "flops": (7 * K * K + 13 * K * (K - 1) // 2 + 38 * K + 62 + 4 * (22 * K + 10)) * n}


# --------------------------------------------------------------------------- exact


def exact(case, seed):
    # the stiff integration has no closed form, and one in plain torch to 64-bit accuracy takes minutes
    if case["kind"] == "plain" or case.get("hot"):
        return None
    return {"served": _exact_served, "train": _exact_train, "props": _exact_props,
            "laplace": _exact_laplace}[case["kind"]](case, seed)


def _h_cp(mech, T, Y):
    """Mixture enthalpy (J/kg) and cp (J/(kg K)) from the NASA-7 polynomials."""
    m = _mechanism(mech)
    W = m.molar_masses()
    nasa = _gpu(m.nasa)
    h, cp = torch.zeros_like(T), torch.zeros_like(T)
    for k in range(m.K):
        a = [torch.where(T < nasa[k, 1], nasa[k, 3 + j], nasa[k, 10 + j]) for j in range(6)]
        cp += Y[k] * (R_U / W[k]) * (a[0] + T * (a[1] + T * (a[2] + T * (a[3] + T * a[4]))))
        h += Y[k] * (R_U / W[k]) * (T * (a[0] + T * (a[1] / 2 + T * (a[2] / 3 + T * (a[3] / 4 + T * a[4] / 5)))) + a[5])
    return h, cp


def _T_from_h(mech, h, Y, T):
    for _ in range(12):
        hm, cp = _h_cp(mech, T, Y)
        T = torch.clamp(T - (hm - h) / cp, 200.0, 3500.0)
    return T


def _features(norm, K, T, p, Y):
    raw = torch.cat([T[:, None], p[:, None], ((Y.clamp_min(0.0) ** 0.1 - 1.0) / 0.1).T], dim=1)
    mu, sig = _gpu(norm[:K + 2]), _gpu(norm[K + 2:2 * K + 4])
    return torch.where(sig < 1e-12, torch.zeros_like(raw), (raw - mu) / sig.clamp_min(1e-12))


def _layers(flat, dims):
    out, o = [], 0
    for i, j in dims:
        out.append((_gpu(flat[o:o + i * j].reshape(j, i)), _gpu(flat[o + i * j:o + i * j + j])))
        o += i * j + j
    return out


def _forward(layers, x):
    for k, (W, b) in enumerate(layers):
        x = x @ W.T + b
        if k + 1 < len(layers):
            x = torch.nn.functional.gelu(x)
    return x


def _exact_served(case, seed):
    K = _mechanism(case["mech"]).K
    T, p, Y = _served_states(case, seed)
    params, norm = _network(case, seed)
    if case.get("per_species"):
        dims = [(K + 2, 1600), (1600, 800), (800, 400), (400, 1)]
        each = params.size // K
        nets = [_layers(params[g * each:(g + 1) * each], dims) for g in range(K)]
    else:
        nets = [_layers(params, network_dims(K))]
    scale = _gpu(norm[3 * K + 4:4 * K + 4])
    Tn, Yn = torch.empty_like(T), torch.empty_like(Y)
    for a in range(0, case["n"], 262144):
        s = slice(a, a + 262144)
        x = _features(norm, K, T[s], p[s], Y[:, s])
        y = Y[:, s] + (torch.cat([_forward(net, x) for net in nets], dim=1) * scale).T
        y = y.clamp_min(0.0)
        Yn[:, s] = y / y.sum(0)
        Tn[s] = _T_from_h(case["mech"], _h_cp(case["mech"], T[s], Y[:, s])[0], Yn[:, s], T[s])
    return {"T": Tn, "Y": Yn, "mask": None, "count": None}


def _exact_train(case, seed):
    K, n, batch = _mechanism(case["mech"]).K, case["n"], case["batch"]
    T, p, Y, Yn, order = _train_data(case, seed)
    norm = _train_norm(case)
    x = _features(norm, K, T, p, Y)
    y = ((Yn - Y) / _gpu(norm[3 * K + 4:4 * K + 4])[:, None]).T
    w = [t.requires_grad_() for wb in _layers(init_params(network_dims(K), seed), network_dims(K)) for t in wb]
    m, v = [torch.zeros_like(t) for t in w], [torch.zeros_like(t) for t in w]
    per = -(-n // batch)
    losses, t = [], 0
    for ep in range(case["epochs"]):
        idx = torch.tensor(order[ep * n:(ep + 1) * n].astype(np.int64), device="cuda")
        total = 0.0
        for b in range(per):
            rows = idx[b * batch:(b + 1) * batch]
            d = _forward(list(zip(w[::2], w[1::2])), x[rows]) - y[rows]
            total = total + (d.detach() ** 2).sum()
            g = torch.autograd.grad((d ** 2).mean(), w)
            lr = 1e-5 + 0.5 * (1e-3 - 1e-5) * (1.0 + math.cos(math.pi * t / (per * case["epochs"])))
            t += 1
            with torch.no_grad():
                for i, gi in enumerate(g):
                    m[i].mul_(0.9).add_(gi, alpha=0.1)
                    v[i].mul_(0.999).addcmul_(gi, gi, value=0.001)
                    w[i] -= lr * (m[i] / (1 - 0.9 ** t)) / ((v[i] / (1 - 0.999 ** t)).sqrt() + 1e-8)
        losses.append(float(total) / (n * K))
    return {"losses": np.array(losses), "params": torch.cat([t.detach().reshape(-1) for t in w])}


def _poly(c, x):
    r = torch.zeros_like(x)
    for i in range(4, -1, -1):
        r = r * x + float(c[i])
    return r


def _exact_props(case, seed):
    m = _mechanism(case["mech"])
    visc, cond, diff = _transport(case["mech"])
    W = m.molar_masses()
    T, p, Y = _flame(case["mech"], case["n"], seed)
    cp = _h_cp(case["mech"], T, Y)[1]
    L = torch.log(T)
    y = Y.clamp_min(0.0)
    y = y / y.sum(0)
    X = y / _gpu(W)[:, None]
    X = X / X.sum(0)
    muk = [(T ** 0.25 * _poly(visc[k], L)) ** 2 for k in range(m.K)]
    lamk = [T.sqrt() * _poly(cond[k], L) for k in range(m.K)]
    mu, D = torch.zeros_like(T), torch.empty_like(Y)
    for k in range(m.K):
        den, s = torch.zeros_like(T), torch.zeros_like(T)
        for j in range(m.K):
            den += X[j] * (1.0 + (muk[k] / muk[j]).sqrt() * (W[j] / W[k]) ** 0.25) ** 2 / math.sqrt(8.0 * (1.0 + W[k] / W[j]))
            if j != k:
                s += X[j] * p / (T ** 1.5 * _poly(diff[j, k], L))
        mu += X[k] * muk[k] / den
        D[k] = (1.0 - y[k]) / s
    lam = 0.5 * (sum(X[k] * lamk[k] for k in range(m.K)) + 1.0 / sum(X[k] / lamk[k] for k in range(m.K)))
    return {"T": T, "cp": cp, "mu": mu, "lam": lam, "D": D}


def _exact_laplace(case, seed):
    mesh = _mesh(case["nx"], case["ny"], case["nz"])
    gc, gb, pb = _laplace_fields(mesh, seed)
    own, nei, fc = (torch.tensor(a.astype(np.int64), device="cuda") for a in (mesh.owner, mesh.neighbour, mesh.face_cells))
    w = _gpu(mesh.weight)
    up = (w * gc[own] + (1.0 - w) * gc[nei]) * _gpu(mesh.delta) * _gpu(mesh.mag_sf)
    n = mesh.ncells
    diag = torch.zeros(n, dtype=F64, device="cuda").index_add_(0, own, -up).index_add_(0, nei, -up)
    fixed = _gpu(np.repeat(mesh.patch_type == 0, np.diff(mesh.patch_start)).astype(np.float64))
    coef = gb * _gpu(mesh.bmag_sf) * _gpu(mesh.bdelta) * fixed
    rhs = torch.zeros(n, dtype=F64, device="cuda").index_add_(0, fc, coef * pb)
    full = diag.clone().index_add_(0, fc, -coef)
    i = torch.arange(n, device="cuda")
    key = torch.cat([own * n + nei, nei * n + own, i * n + i])
    out = {"csr": torch.cat([up, up, full])[torch.argsort(key)], "rhs": rhs}
    if not case["direct"]:
        out |= {"lower": up, "upper": up, "diag": diag, "internal": -coef, "boundary": coef * pb}
    return out
