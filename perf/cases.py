"""The work that a user of this framework has it do, as cases that can be timed.

Every case is one pass through the public entry points of ``paper_2312_07008_amd`` on
inputs that are already on the GPU, with the outputs and workspaces a program keeps
between calls allocated beforehand.  The kinds of case:

  call      density build, natural-orbital truncation and energy correction in one
            call sequence: what a user runs for one small molecule
  label     one labelling pass of the pair screen: the plain pass with per-pair norms,
            the pair features and the training targets
  build     the density pass alone (FP64, BF16 slices or INT8 digits; with or without
            active holes and a pair mask)
  truncate  natural orbitals of a virtual density and the cumulative-occupation cut
  correct   the kept-space energy and the additive correction
  train     a stretch of full-batch training steps of the screen's network
  a9        the terms of the density with active particles, singles and cumulant
  naf       compression to natural auxiliary functions
  ladder    the particle-particle ladder in the kept space

Inputs follow the recipes of the repository's generator: uniform energies, integrals
B^Q_ia = 0.06 / (1 + eps_a) N(0, 1), active densities with eigenvalue pairs (x, 2 - x).
"""
from __future__ import annotations

import math

import torch

import paper_2312_07008_amd as dp
from paper_2312_07008_amd import api

S_FLOW = 0.5
P_O = 0.985
PRECISION = {"f64": dp.FP64, "bf16": dp.BF16_SLICED, "int8": dp.INT8_SLICED}


# --------------------------------------------------------------------------- cases

def listed():
    return [
        # the smallest workload of the repository, as its smoke test runs it: latency
        # and launches count
        {"name": "call-c1-f64", "kind": "call", "prec": "f64", "n_core": 10, "n_act": 0, "n_vir": 60, "n_aux": 200},
        # one of the 200 small input sets whose pairs train the screen
        {"name": "label-c1", "kind": "label", "prec": "f64", "n_core": 10, "n_act": 0, "n_vir": 60, "n_aux": 200},
        # a molecule with an active space in plain FP64 (the c2 workload's sizes)
        {"name": "build-c2-f64", "kind": "build", "prec": "f64", "n_core": 40, "n_act": 8, "n_vir": 400,
         "n_aux": 1600, "masked": 0.0},
        # odd sizes: the virtual count of Ni(CO)4, an odd auxiliary count, a quarter of
        # the pairs screened away
        {"name": "build-539-bf16", "kind": "build", "prec": "bf16", "n_core": 31, "n_act": 0, "n_vir": 539,
         "n_aux": 1867, "masked": 0.25},
        # the benchmark's own workload: ~1300 basis functions on split BF16
        {"name": "build-c3-bf16", "kind": "build", "prec": "bf16", "n_core": 80, "n_act": 0, "n_vir": 1200,
         "n_aux": 4000, "masked": 0.0},
        # INT8 digits with active holes, between the two
        {"name": "build-800-int8", "kind": "build", "prec": "int8", "n_core": 36, "n_act": 4, "n_vir": 800,
         "n_aux": 2800, "masked": 0.0},
        # the eigenproblem of the benchmark's workload
        {"name": "truncate-1200", "kind": "truncate", "n_vir": 1200},
        # the correction of the benchmark's workload (INT8 digits hold its error)
        {"name": "correct-c3-int8", "kind": "correct", "prec": "int8", "n_core": 80, "n_act": 0, "n_vir": 1200,
         "n_aux": 4000, "n_kept": 894},
        # training on the pairs of 200 small input sets
        {"name": "train-11000", "kind": "train", "samples": 11000, "steps": 12},
        # the rest of the density's terms at the c2 workload's sizes
        {"name": "a9-c2", "kind": "a9", "n_core": 40, "n_act": 8, "n_vir": 400, "n_aux": 1600},
        # a redundant auxiliary set, half of which is kept
        {"name": "naf-1200", "kind": "naf", "n_core": 16, "n_act": 0, "n_vir": 300, "n_aux": 1200, "rank": 600},
        # the ladder in a truncated space, half the linear size of the c2 workload
        {"name": "ladder-200", "kind": "ladder", "n_vir": 200, "n_aux": 800, "n_amp": 400, "n_kept": 133},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["call", "label", "build", "build", "build", "build", "build", "truncate", "correct", "train",
                       "a9", "naf", "ladder"])
    while True:
        if kind in ("call", "label"):
            n_vir = _log_int(rng, 24, 200)
            c = {"kind": kind, "prec": rng.choice(["f64", "bf16", "int8"]) if kind == "call" else "f64",
                 "n_core": _log_int(rng, 3, 16), "n_act": rng.choice([0, 0, 2, 4]) if kind == "call" else 0,
                 "n_vir": n_vir, "n_aux": int(n_vir * rng.uniform(2.6, 4.2)) + 1}
        elif kind == "build":
            n_vir = _log_int(rng, 48, 1200)
            c = {"kind": kind, "prec": rng.choice(["f64", "bf16", "bf16", "int8"]), "n_core": _log_int(rng, 4, 80),
                 "n_act": rng.choice([0, 0, 2, 4, 8]), "n_vir": n_vir, "n_aux": int(n_vir * rng.uniform(2.6, 4.2)) + 1,
                 "masked": rng.choice([0.0, 0.0, rng.uniform(0.05, 0.4)])}
        elif kind == "truncate":
            c = {"kind": kind, "n_vir": _log_int(rng, 24, 1200)}
        elif kind == "correct":
            n_vir = _log_int(rng, 48, 1200)
            c = {"kind": kind, "prec": rng.choice(["f64", "bf16", "int8", "int8"]), "n_core": _log_int(rng, 4, 80),
                 "n_act": rng.choice([0, 0, 2, 4]), "n_vir": n_vir, "n_aux": int(n_vir * rng.uniform(2.6, 4.2)) + 1,
                 "n_kept": max(2, int(n_vir * rng.uniform(0.5, 0.85)))}
        elif kind == "train":
            c = {"kind": kind, "samples": _log_int(rng, 600, 30000), "steps": rng.randint(4, 12)}
        elif kind == "a9":
            n_vir = _log_int(rng, 60, 700)
            c = {"kind": kind, "n_core": _log_int(rng, 6, 60), "n_act": rng.choice([2, 4, 6, 8]), "n_vir": n_vir,
                 "n_aux": int(n_vir * rng.uniform(2.6, 4.2)) + 1}
        elif kind == "naf":
            n_aux = _log_int(rng, 120, 1200)
            c = {"kind": kind, "n_core": _log_int(rng, 4, 24), "n_act": rng.choice([0, 2]),
                 "n_vir": max(40, int(n_aux * rng.uniform(0.25, 0.4))), "n_aux": n_aux,
                 "rank": int(n_aux * rng.uniform(0.4, 0.8))}
            if (c["n_core"] + c["n_act"]) * c["n_vir"] < 2 * n_aux:
                continue
        else:
            n_vir = _log_int(rng, 40, 200)
            c = {"kind": kind, "n_vir": n_vir, "n_aux": int(n_vir * rng.uniform(2.6, 4.2)) + 1,
                 "n_amp": _log_int(rng, 16, 400), "n_kept": max(8, int(n_vir * rng.uniform(0.5, 0.85)))}
        # FP64 work goes at a fraction of the rate of the sliced paths
        if work(c)["flops"] * (1.0 if c.get("prec") in ("bf16", "int8") else 3.0) <= 6.0e13:
            return c


# ------------------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _uniform(g, lo, hi, n):
    return torch.sort(torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * (hi - lo) + lo).values


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float64)


def _decay(eps):
    return 0.06 / (1.0 + eps)


def _gamma(g, n_act):
    if not n_act:
        return None
    x = torch.rand(n_act // 2, generator=g, device="cuda", dtype=torch.float64).cpu() * 2.0
    q = torch.linalg.qr(_normal(g, n_act, n_act).cpu()).Q
    lam = torch.cat([x, 2.0 - x])
    m = (q * lam) @ q.T
    return (0.5 * (m + m.T)).cuda().contiguous()


def _molecule(c, g):
    n_core, n_act, n_vir, n_aux = c["n_core"], c["n_act"], c["n_vir"], c["n_aux"]
    d = {"eps_vir": _uniform(g, 0.1, 5.0, n_vir), "gamma": _gamma(g, n_act)}
    d["eps_hole"] = torch.cat([_uniform(g, -1.5, -0.3, n_core), _uniform(g, -0.3, 0.0, n_act)])
    n_h = n_core + n_act
    if c.get("rank"):
        r = c["rank"]
        B = (_normal(g, n_h * n_vir, r) @ _normal(g, r, n_aux)).view(n_h, n_vir, n_aux) / math.sqrt(r)
        B += 1e-7 * _normal(g, n_h, n_vir, n_aux)
    else:
        B = _normal(g, n_h, n_vir, n_aux)
    d["B"] = B.mul_(_decay(d["eps_vir"])[None, :, None]).contiguous()
    return d


def _opts(c, prec=None):
    return dp.make_opts(c["n_core"], c["n_act"], c["n_vir"], c["n_aux"], S_FLOW,
                        precision=PRECISION[prec or c.get("prec", "f64")])


def _bytes(n):
    return torch.empty(max(int(n), 1), dtype=torch.uint8, device="cuda")


def _out(*shape, dtype=torch.float64):
    return torch.empty(shape, dtype=dtype, device="cuda")


def _density(c, g):
    """A virtual density: dominated by its diagonal, decaying over two orders of magnitude."""
    n = c["n_vir"]
    d = _decay(_uniform(g, 0.1, 5.0, n)) ** 1.5
    z = _normal(g, n, 16 * n)
    D = (z @ z.T) * (1e6 / (16 * n)) * d[:, None] * d[None, :]
    return (0.5 * (D + D.T)).contiguous()


def _orbitals(g, n):
    """Natural orbitals close to the virtuals they come from, as columns."""
    a = torch.eye(n, dtype=torch.float64) + _normal(g, n, n).cpu() * (0.3 / math.sqrt(n))
    return torch.linalg.qr(a).Q.cuda().contiguous()


def _mlp(g):
    return torch.cat([_normal(g, 320) / math.sqrt(5.0), _normal(g, 64) * 0.0, _normal(g, 4096) / 8.0,
                      _normal(g, 64) * 0.0, _normal(g, 64) / 8.0, _normal(g, 1) * 0.0]).float().contiguous()


def _cumulant(g, n):
    a = _normal(g, n, n, n, n)
    lam = 0.05 * (a + a.permute(1, 0, 3, 2))
    return (0.5 * (lam + lam.permute(2, 3, 0, 1))).contiguous()


def prepare(case, seed):
    c, g, kind = case, _gen(seed), case["kind"]
    if kind == "truncate":
        n = c["n_vir"]
        return {"case": c, "D": _density(c, g), "occ": _out(n), "no_vecs": _out(n, n),
                "ws": _bytes(dp.fno_truncate_workspace_size(n))}
    if kind == "train":
        n = c["samples"]
        e = torch.rand(n, 2, generator=g, device="cuda", dtype=torch.float64) * 1.2 - 1.5
        lw, x3 = 2.6 + 0.05 * _normal(g, n), -0.02 * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
        x4 = -0.1 + 0.05 * e.sum(1) + 0.01 * _normal(g, n)
        feats = torch.stack([e[:, 0], e[:, 1], lw, x3, x4], 1).float().contiguous()
        y = (-0.8 - 0.15 * e.sum(1) + 0.1 * e[:, 0] * e[:, 1] + 0.03 * _normal(g, n)).float().contiguous()
        return {"case": c, "feats": feats, "y": y, "W0": _mlp(g)}
    if kind == "ladder":
        n, na, npair = c["n_vir"], c["n_aux"], c["n_amp"]
        eps = _uniform(g, 0.1, 5.0, n)
        z = _normal(g, n, n, na)
        z = (z + z.transpose(0, 1)) * math.sqrt(0.5)
        d = _decay(eps)
        B = (z * torch.sqrt(d[:, None] * d[None, :])[:, :, None]).contiguous()
        T = (0.05 * _normal(g, npair, n, n) / (1.0 + eps[None, :, None] + eps[None, None, :])).contiguous()
        k = c["n_kept"]
        return {"case": c, "B": B, "T": T, "X": _orbitals(g, n), "R": _out(npair, k, k),
                "ws": _bytes(dp.pp_ladder_workspace_size(n, na, npair, k))}

    d = _molecule(c, g)
    n_h, n = c["n_core"] + c["n_act"], c["n_vir"]
    d.update(case=c, opts=_opts(c))
    if kind in ("call", "label", "build"):
        d.update(D=_out(n, n), e=_out(2), ws=_bytes(dp.workspace_size(d["opts"])))
    if kind in ("label", "build"):
        d.update(pe=_out(n_h, n_h), tn=_out(n_h, n_h, dtype=torch.float32))
    if kind == "build" and c["masked"]:
        m = torch.rand(n_h, n_h, generator=g, device="cuda") < c["masked"]
        m = m.triu()
        m = m | m.T
        m[c["n_core"]:] = False
        m[:, c["n_core"]:] = False
        d["mask"] = (~m).to(torch.uint8).contiguous()
    if kind == "call":
        d.update(occ=_out(n), no_vecs=_out(n, n), ws_t=_bytes(dp.fno_truncate_workspace_size(n)),
                 ws_c=_bytes(dp.pt2_correction_workspace_size(d["opts"], n)))
    if kind == "correct":
        # the full-space energy as the pass returned it
        e = -1.6e-7 * n_h * n_h * n * n * c["n_aux"]
        d.update(no_vecs=_orbitals(g, n), e_full=torch.tensor([e, 0.0], dtype=torch.float64, device="cuda"),
                 ws=_bytes(dp.pt2_correction_workspace_size(d["opts"], c["n_kept"])))
    if kind == "a9":
        n_a, n_aux = c["n_act"], c["n_aux"]
        ba = _normal(g, n_h, n_a, n_aux) * _decay(d["eps_hole"][c["n_core"]:])[None, :, None]
        blk = ba[c["n_core"]:].clone()
        ba[c["n_core"]:] = (blk + blk.transpose(0, 1)) * math.sqrt(0.5)
        d.update(B_act=ba.contiguous(), lam=_cumulant(g, n_a), D0=_density(c, g), t1=_out(n_h, n))
    return d


# ---------------------------------------------------------------------------- run

def _build(s, **kw):
    return dp.build_vv_density(s["opts"], s["eps_hole"], s["eps_vir"], s["gamma"], s["B"], s.get("mask"),
                               D_vv=s["D"], e_pt2=s["e"], workspace=s["ws"], **kw)


def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind == "build":
        _build(s, pair_energy=s["pe"], pair_tnorm=s["tn"])
        return {"D_vv": s["D"], "e_pt2": s["e"], "pair_energy": s["pe"], "pair_tnorm": s["tn"]}
    if kind == "label":
        _build(s, pair_tnorm=s["tn"])
        f, ls = dp.pairscreen_features(s["opts"], s["eps_hole"], s["eps_vir"], s["B"])
        y = dp.pairscreen_targets(s["tn"], ls, c["n_core"], c["n_core"])
        return {"feats": f, "log_scale": ls, "targets": y, "pair_tnorm": s["tn"]}
    if kind == "call":
        _build(s)
        t = dp.fno_truncate(s["D"], P_O, occ=s["occ"], no_vecs=s["no_vecs"], workspace=s["ws_t"])
        r = dp.pt2_energy_correction(s["opts"], s["eps_hole"], s["eps_vir"], s["gamma"], s["B"], s["no_vecs"],
                                     t["n_kept"], s["e"], workspace=s["ws_c"])
        return {"D_vv": s["D"], "e_pt2": s["e"], "occ": s["occ"], "n_kept": t["n_kept"], "e_kept": r["e_kept"],
                "correction": r["correction"]}
    if kind == "truncate":
        t = dp.fno_truncate(s["D"], P_O, occ=s["occ"], no_vecs=s["no_vecs"], workspace=s["ws"])
        return {"occ": s["occ"], "no_vecs": s["no_vecs"], "n_kept": t["n_kept"]}
    if kind == "correct":
        r = dp.pt2_energy_correction(s["opts"], s["eps_hole"], s["eps_vir"], s["gamma"], s["B"], s["no_vecs"],
                                     c["n_kept"], s["e_full"], workspace=s["ws"])
        return {"e_kept": r["e_kept"], "correction": r["correction"]}
    if kind == "train":
        W = s["W0"].clone()
        m, v = torch.zeros_like(W), torch.zeros_like(W)
        losses = dp.pairscreen_train(W, m, v, s["feats"], s["y"], c["steps"], 3e-3)
        return {"W": W, "m": m, "v": v, "losses": losses}
    if kind == "a9":
        D = s["D0"].clone()
        args = (s["opts"], s["eps_hole"], s["eps_vir"], s["gamma"])
        dp.add_active_particle_density(*args, s["B"], s["B_act"], D)
        api.add_cumulant_singles_density(*args, s["lam"], s["B"], s["B_act"], D, t1=s["t1"])
        return {"D_vv": D, "t1": s["t1"]}
    if kind == "naf":
        r = dp.naf_compress(s["opts"], s["B"], 1e-10)
        return {"B_naf": r["B_naf"], "sigma": r["sigma"], "n_naf": r["n_naf"]}
    dp.pp_ladder(s["B"], s["T"], s["X"], c["n_kept"], R=s["R"], workspace=s["ws"])
    return {"R": s["R"]}


# --------------------------------------------------------------------------- work

def _build_work(c, n_vir=None, density=True):
    n_h, n, q = c["n_core"] + c["n_act"], n_vir or c["n_vir"], c["n_aux"]
    pairs = n_h * (n_h + 1) / 2
    if c.get("masked"):
        pairs -= c["masked"] * c["n_core"] * (c["n_core"] + 1) / 2
    flops = 2.0 * pairs * n * n * q + (4.0 * pairs * n ** 3 / 2 * 2 if density else 0.0)
    return {"bytes": 8.0 * (n_h * n * q + (n * n if density else 0)), "flops": flops}


def _eigh_work(n):
    return {"bytes": 16.0 * n * n, "flops": (4.0 / 3.0 + 2.0) * n ** 3}


def work(case):
    c, kind = case, case["kind"]
    if kind == "build":
        return _build_work(c)
    if kind == "label":
        w = _build_work(c)
        return {"bytes": w["bytes"], "flops": w["flops"] + 3.0 * c["n_core"] * c["n_vir"] * c["n_aux"]}
    if kind in ("call", "correct"):
        n_h, n, q = c["n_core"] + c["n_act"], c["n_vir"], c["n_aux"]
        k = c.get("n_kept", int(0.7 * n))
        parts = [_build_work(c, k, density=False), _eigh_work(k), {"bytes": 0.0, "flops": 2.0 * n_h * n * k * q}]
        if kind == "call":
            parts += [_build_work(c), _eigh_work(n)]
        b = 8.0 * n_h * n * q + 8.0 * n * n * (2 if kind == "call" else 1)
        return {"bytes": b, "flops": sum(p["flops"] for p in parts)}
    if kind == "truncate":
        return _eigh_work(c["n_vir"])
    if kind == "train":
        n = c["samples"]
        return {"bytes": 24.0 * n + 6 * 4.0 * 4609, "flops": c["steps"] * n * 6.0 * (5 * 64 + 64 * 64 + 64)}
    if kind == "a9":
        n_h, a, n, q = c["n_core"] + c["n_act"], c["n_act"], c["n_vir"], c["n_aux"]
        ints = 2.0 * n * n_h * n_h * a * q  # the amplitudes, common to all terms
        gemm = 2.0 * n * n * n_h * n_h * a
        cum = 2.0 * n * n * (2 * n_h * a * a + a ** 3 + n_h + 2 * a) + 2.0 * a * a * n * n * (q / 2 + a * a + n)
        return {"bytes": 8.0 * (n_h * n * q + n_h * a * q + 2 * n * n + a ** 4), "flops": ints + gemm + cum}
    if kind == "naf":
        rows, q, r = (c["n_core"] + c["n_act"]) * c["n_vir"], c["n_aux"], c["rank"]
        return {"bytes": 8.0 * rows * (q + r), "flops": 1.0 * rows * q * q + 2.0 * rows * q * r + (4.0 / 3) * q ** 3 +
                2.0 * q * q * r}
    n, k, q, p = c["n_vir"], c["n_kept"], c["n_aux"], c["n_amp"]
    flops = 2.0 * q * (n * n * k + n * k * k) + 2.0 * p * (n * n * k + n * k * k) + 2.0 * k ** 4 * (q / 2 + p)
    return {"bytes": 8.0 * (n * n * q + p * n * n + p * k * k), "flops": flops}


# -------------------------------------------------------------------------- exact

def _regularized(V, eps_pair, eps_v):
    """(t, renormalized V) for V[..., a, b] with denominators eps_pair - eps_a - eps_b."""
    dl = eps_pair - (eps_v[:, None] + eps_v[None, :])
    x = torch.exp(-S_FLOW * dl * dl)
    return V * ((1.0 - x) / dl), V * (1.0 + x)


def _exact_pass(c, eps_h, eps_v, gamma, B, mask=None, density=True):
    """Energy, density, pair energies and norms, summed over hole pairs with plain products."""
    n_c, n_a = c["n_core"], c["n_act"]
    n_h, n = n_c + n_a, B.shape[1]
    D = torch.zeros(n, n, dtype=torch.float64, device="cuda") if density else None
    E = torch.zeros((), dtype=torch.float64, device="cuda")
    pe = torch.zeros(n_h, n_h, dtype=torch.float64, device="cuda")
    tn = torch.zeros(n_h, n_h, dtype=torch.float64, device="cuda")

    def dot(a, b):
        return (a * b).sum((-2, -1))

    def add(T, Vr, Tt, w):
        """w/4 <Vr, 2 Tt - Tt^T> and w/2 T (2 Tt - Tt^T)^T over a stack of pairs and their transposes."""
        nonlocal E, D
        Y = 2.0 * Tt - Tt.transpose(1, 2)
        E = E + (w * dot(Vr, Y)).sum() / 4.0
        if density:
            Yw = Y * w[:, None, None]
            D += 0.5 * (T.transpose(0, 1).reshape(n, -1) @ Yw.transpose(0, 1).reshape(n, -1).T)

    def stack(i, js):
        V = (B[i] @ B[js].reshape(-1, B.shape[2]).T).view(n, len(js), n).transpose(0, 1)
        return _regularized(V, (eps_h[i] + eps_h[js])[:, None, None], eps_v)

    chunk = max(1, int(4e8 // (n * n)))
    act = torch.arange(n_c, n_h, device="cuda")
    for i in range(n_c):
        js = [j for j in range(i, n_c) if mask is None or bool(mask[i, j])]
        for j0 in range(0, len(js), chunk):
            j = torch.tensor(js[j0:j0 + chunk], device="cuda")
            T, Vr = stack(i, j)
            pair = dot(Vr, 2.0 * T - T.transpose(1, 2))
            pe[i, j] = pair
            pe[j, i] = pair
            tn[i, j] = torch.sqrt(dot(T, T))
            tn[j, i] = tn[i, j]
            one = torch.ones_like(pair)
            add(T, Vr, 4.0 * T, one)
            off = (j != i).double()
            Tt = T.transpose(1, 2).contiguous()
            add(Tt, Vr.transpose(1, 2), 4.0 * Tt, off)
        if n_a:
            T, Vr = stack(i, act)
            tn[i, act] = torch.sqrt(dot(T, T))
            tn[act, i] = tn[i, act]
            Tt = 2.0 * (gamma @ T.reshape(n_a, -1)).view_as(T)
            one = torch.ones(n_a, dtype=torch.float64, device="cuda")
            add(T, Vr, Tt, one)
            add(T.transpose(1, 2).contiguous(), Vr.transpose(1, 2), Tt.transpose(1, 2).contiguous(), one)
    if n_a:
        T, Vr = (torch.cat(x) for x in zip(*[stack(u, act) for u in range(n_c, n_h)]))
        tn[n_c:, n_c:] = torch.sqrt(dot(T, T)).view(n_a, n_a)
        gg = torch.kron(gamma, gamma)
        add(T, Vr, (gg @ T.reshape(n_a * n_a, -1)).view_as(T),
            torch.ones(n_a * n_a, dtype=torch.float64, device="cuda"))
        pe[n_c:] = math.nan
        pe[:, n_c:] = math.nan
    if density:
        D = 0.5 * (D + D.T)
    return D, torch.stack([E, torch.zeros_like(E)]), pe, tn


def _exact_orbitals(D):
    w, v = torch.linalg.eigh(D.cpu())
    w, v = w.flip(0), v.flip(1)
    big = v.gather(0, v.abs().argmax(0, keepdim=True))
    return w, v * torch.where(big < 0, -1.0, 1.0)


def _exact_correct(c, d, vecs, n_kept, e_full):
    Vk = vecs[:, :n_kept].cuda()
    F = Vk.T @ (d["eps_vir"][:, None] * Vk)
    et, W = torch.linalg.eigh((0.5 * (F + F.T)).cpu())
    U = Vk @ W.cuda()
    Bt = torch.matmul(U.T.contiguous(), d["B"])
    _, e, _, _ = _exact_pass(c, d["eps_hole"], et.cuda(), d["gamma"], Bt, density=False)
    return e, e_full - e


def _exact_features(c, d, tn):
    n_c, e, ev = c["n_core"], d["eps_hole"], d["eps_vir"]
    q2 = (d["B"][:n_c] ** 2).sum(1)
    q = torch.sqrt(q2)
    U, W = q @ q.T, torch.sqrt(q2 @ q2.T)
    i, j = torch.triu_indices(n_c, n_c, device="cuda")
    lo, hi = 0.5, 2.0
    for _ in range(200):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if 2 * mid * mid * math.exp(-mid * mid) > -math.expm1(-mid * mid) else (lo, mid)
    peak = torch.tensor(lo / math.sqrt(S_FLOW), dtype=torch.float64, device="cuda")

    def f(x):
        return -torch.expm1(-S_FLOW * x * x) / x

    a, b = (e[i] + e[j] - 2 * ev[0]).abs(), (e[i] + e[j] - 2 * ev[-1]).abs()
    a, b = torch.minimum(a, b), torch.maximum(a, b)
    g = torch.where((a <= peak) & (peak <= b), f(peak), torch.maximum(f(a), f(b)))
    lw, lu, dg = torch.log(W[i, j]), torch.log(U[i, j]), torch.log(torch.diagonal(W))
    feats = torch.stack([e[i], e[j], lu - lw, 0.1 * (lw - 0.5 * (dg[i] + dg[j])), 0.1 * (torch.log(g) + lw)], 1)
    scale = torch.stack([torch.log(g) + lw, torch.log(g) + lu], 1)
    return {"feats": feats, "log_scale": scale, "targets": torch.log(tn[i, j]) - scale[:, 0], "pair_tnorm": tn}


def _exact_train(c, d):
    X, y, w = d["feats"].double(), d["y"].double(), d["W0"].double()
    m, v, losses, n = torch.zeros_like(w), torch.zeros_like(w), [], d["y"].numel()
    for t in range(1, c["steps"] + 1):
        W1, b1, W2, b2, w3, b3 = torch.split(w, [320, 64, 4096, 64, 64, 1])
        W1, W2 = W1.view(64, 5), W2.view(64, 64)
        h1 = torch.tanh(X @ W1.T + b1)
        h2 = torch.tanh(h1 @ W2.T + b2)
        r = h2 @ w3 + b3 - y
        losses.append((r * r).mean())
        do = 2.0 * r / n
        z2 = do[:, None] * w3[None, :] * (1.0 - h2 * h2)
        z1 = (z2 @ W2) * (1.0 - h1 * h1)
        g = torch.cat([(z1.T @ X).reshape(-1), z1.sum(0), (z2.T @ h1).reshape(-1), z2.sum(0), h2.T @ do,
                       do.sum()[None]])
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        w = w - 3e-3 * (m / (1 - 0.9 ** t)) / (torch.sqrt(v / (1 - 0.999 ** t)) + 1e-8)
    return {"W": w, "m": m, "v": v, "losses": torch.stack(losses)}


def _exact_a9(c, d):
    n_c, n_a, eps, ev, G, lam = c["n_core"], c["n_act"], d["eps_hole"], d["eps_vir"], d["gamma"], d["lam"]
    n_h, n = n_c + n_a, c["n_vir"]
    ea = eps[n_c:]
    eta = 2.0 * torch.eye(n_a, dtype=torch.float64, device="cuda") - G
    V = (d["B"].reshape(n_h * n, -1) @ d["B_act"].reshape(n_h * n_a, -1).T).view(n_h, n, n_h, n_a)
    dl = (eps[:, None, None, None] + eps[None, None, :, None] - ev[None, :, None, None] - ea[None, None, None, :])
    X = (V * (1.0 - torch.exp(-S_FLOW * dl * dl)) / dl).permute(0, 2, 1, 3).contiguous()  # [i, j, e, x]
    w = torch.eye(n_h, dtype=torch.float64, device="cuda")
    w[n_c:, n_c:] = 0.5 * G
    tc = 2.0 * X - X.transpose(0, 1)
    Z = (w @ tc.reshape(n_h, -1)).view_as(X).transpose(0, 1).contiguous()
    Z = (w @ Z.view(n_h, -1)).view(n_h, n_h, n, n_a).transpose(0, 1)
    L, R = torch.matmul(X, eta).permute(2, 0, 1, 3).reshape(n, -1), Z.permute(2, 0, 1, 3).reshape(n, -1)
    E = L @ R.T
    D = d["D0"] + 0.5 * (E + E.T)
    # singles
    ux = (ea[None, :] - ea[:, None]) * G.T
    tcu = 2.0 * X[:, n_c:] - X[n_c:].transpose(0, 1)  # [i, u, e, x]
    src = 0.5 * torch.einsum("ux,iuex->ie", ux, tcu)
    ds = eps[:, None] - ev[None, :]
    t1 = src * (1.0 - torch.exp(-S_FLOW * ds * ds)) / ds
    tm, tu = t1[:n_c], t1[n_c:]
    Xaa, Xca, Xac = X[n_c:, n_c:], X[:n_c, n_c:], X[n_c:, :n_c].transpose(0, 1)
    C = 2.0 * tm.T @ tm + tu.T @ G @ tu
    C = C + tu.T @ torch.einsum("xyfv,uvxy->uf", Xaa, lam) + torch.einsum("uvey,uvxy->ex", Xaa, lam) @ tu
    Ba = d["B"][n_c:]
    Vv = (Ba.reshape(n_a * n, -1) @ Ba.reshape(n_a * n, -1).T).view(n_a, n, n_a, n).permute(0, 2, 1, 3)
    T, _ = _regularized(Vv, (ea[:, None] + ea[None, :])[:, :, None, None], ev)
    T = T.reshape(n_a * n_a, n, n)
    Tl = (lam.reshape(n_a * n_a, n_a * n_a) @ T.reshape(n_a * n_a, -1)).view_as(T)
    C = C + T.permute(1, 0, 2).reshape(n, -1) @ Tl.permute(1, 0, 2).reshape(n, -1).T

    def both(a, b):  # sum over [m, p, q]: a[m, e, p, q] b[m, f, p, q]
        return a.permute(1, 0, 2, 3).reshape(n, -1) @ b.permute(1, 0, 2, 3).reshape(n, -1).T

    def left(a):  # sum_vy a[m, v, e, y] lam[u, v, x, y] -> [m, e, x, u]
        return torch.einsum("mvey,uvxy->mexu", a, lam)

    def p_terms(a, av, b, bx):
        r = [x.permute(0, 2, 1, 3) for x in (b, bx)]  # [m, f, x, u]
        s1, s2 = left(a), left(av)
        s3 = torch.einsum("mvex,uvxy->meyu", av, lam)
        return 2.0 * both(s1, r[0]) - both(s1, r[1]) - both(s2, r[0]) - both(s3, r[1])

    C = C + p_terms(Xca, Xac, Xca, Xac)
    XE = torch.matmul(Xaa, eta)
    XL = (lam.reshape(n_a * n_a, n_a * n_a) @ Xaa.reshape(n_a * n_a, -1)).view_as(Xaa)
    C = C + 0.5 * XE.permute(2, 0, 1, 3).reshape(n, -1) @ XL.permute(2, 0, 1, 3).reshape(n, -1).T
    aw, av = Xaa, Xaa.transpose(0, 1)  # t_ey^wv and t_ey^vw, both [w, v, e, y]
    bz, bx = (torch.einsum("wz,zxfu->wxfu", G, q) for q in (aw, av))
    C = C + 0.5 * p_terms(aw, av, bz, bx)
    return {"D_vv": D + 0.5 * (C + C.T), "t1": t1}


def exact(case, seed):
    c, kind = case, case["kind"]
    d = prepare(c, seed)
    if kind in ("build", "label", "call"):
        D, e, pe, tn = _exact_pass(c, d["eps_hole"], d["eps_vir"], d["gamma"], d["B"], d.get("mask"),
                                   density=kind != "label")
        if kind == "build":
            return {"D_vv": D, "e_pt2": e, "pair_energy": pe, "pair_tnorm": tn}
        if kind == "label":
            return _exact_features(c, d, tn)
        occ, vecs = _exact_orbitals(D)
        total, cum = occ.sum(), occ.cumsum(0)
        n_kept = min(int((cum < P_O * total).sum()) + 1, c["n_vir"])
        e_kept, corr = _exact_correct(c, d, vecs, n_kept, e)
        return {"D_vv": D, "e_pt2": e, "occ": occ, "n_kept": n_kept, "e_kept": e_kept, "correction": corr}
    if kind == "truncate":
        occ, vecs = _exact_orbitals(d["D"])
        n_kept = min(int((occ.cumsum(0) < P_O * occ.sum()).sum()) + 1, c["n_vir"])
        return {"occ": occ, "no_vecs": vecs, "n_kept": n_kept}
    if kind == "correct":
        e_kept, corr = _exact_correct(c, d, d["no_vecs"], c["n_kept"], d["e_full"])
        return {"e_kept": e_kept, "correction": corr}
    if kind == "train":
        return _exact_train(c, d)
    if kind == "a9":
        return _exact_a9(c, d)
    if kind == "naf":
        J = d["B"].reshape(-1, c["n_aux"])
        sigma, U = _exact_orbitals(J.T @ J)
        keep = int((sigma > 1e-10 * sigma[0]).sum())
        n_h = c["n_core"] + c["n_act"]
        return {"B_naf": (J @ U[:, :keep].cuda()).view(n_h, c["n_vir"], keep), "sigma": sigma, "n_naf": keep}
    X = d["X"][:, :c["n_kept"]].contiguous()
    k, q = c["n_kept"], c["n_aux"]
    B = torch.matmul(X.T.contiguous(), d["B"].permute(2, 0, 1).contiguous()) @ X  # [Q, a, c]
    rows = B.permute(1, 0, 2).contiguous()                                         # [a, Q, c]
    R = torch.empty(c["n_amp"], k, k, dtype=torch.float64, device="cuda")
    for p in range(c["n_amp"]):
        t = X.T @ d["T"][p] @ X
        R[p] = (rows.reshape(k * q, k) @ t).view(k, -1) @ rows.view(k, -1).T
    return {"R": R}
