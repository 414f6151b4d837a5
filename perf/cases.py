"""Workloads that the library's speed is measured on: what a user's program calls, over the sizes it calls it with.

The range.  A residual is one evaluation of the T1/T2 equations at given amplitudes; an iteration of every solver
here is one residual and one update.  Sizes run from the o5 v20 Q60 system to o30 v270 Q900; between them lie the
request stream's shapes (o 4 to 24, v = 9 o, Q = 3 (o + v)) and the smaller v/o of plain double-zeta sets.  Larger
sets (o40 v360 Q1200) hold more than 100 GB each.  Precisions, both vvvv storages, several states on one integral
set, the 1-CSF transformed Hamiltonian with the partial linearisation, the build of an integral set, whole solves
and a served batch of requests are all among them.

Inputs.  Density-fitting factors are Gaussian with the width at which the iteration converges (naux nv sigma^2 = 3),
orbital energies lie below and above the gap, doubles are the first-order amplitudes of those integrals plus a small
random part and singles are small and random, as in the middle of a solve.
"""
import math

import numpy as np
import torch

import paper_2501_10515_amd as A

PREC = {"fp64": A.ASCC_PREC_FP64, "fp32": A.ASCC_PREC_FP32, "bf16x3": A.ASCC_PREC_BF16X3}
VVVV = {"full": A.ASCC_VVVV_FULL, "packed": A.ASCC_VVVV_PACKED}
STEPS = 12  # iterations of a ground-state solve from T = 0 to the tolerances below, about


def listed():
    return [
        # the smallest system, one evaluation: launches and latency only
        dict(name="residual o5 v20 fp64", kind="residual", o=5, v=20, q=60, prec="fp64", vvvv="full"),
        # ... and its whole solve, a student's or a test's first call
        dict(name="solve o5 v20 fp64", kind="solve", o=5, v=20, q=60, prec="fp64", vvvv="full", tol=1e-8),
        # a small request of the stream in the precision of the bulk iterations
        dict(name="residual o8 v72 bf16x3", kind="residual", o=8, v=72, q=240, prec="bf16x3", vvvv="packed"),
        # the stream's middle, odd everywhere
        dict(name="residual o13 v117 fp64", kind="residual", o=13, v=117, q=390, prec="fp64", vvvv="packed"),
        # single-precision contractions on sizes that fit no tile
        dict(name="residual o17 v131 fp32", kind="residual", o=17, v=131, q=443, prec="fp32", vvvv="packed"),
        # the o20 v180 Q600 workload: FP64 with the full vvvv block, and the low-precision bulk iteration
        dict(name="residual o20 v180 fp64", kind="residual", o=20, v=180, q=600, prec="fp64", vvvv="full"),
        dict(name="residual o20 v180 bf16x3", kind="residual", o=20, v=180, q=600, prec="bf16x3", vvvv="packed"),
        # the largest: one state of the o30 v270 Q900 system
        dict(name="residual o30 v270 fp64", kind="residual", o=30, v=270, q=900, prec="fp64", vvvv="packed"),
        # several states of one Hamiltonian, four to a pass
        dict(name="batch o12 v108 fp64", kind="batch", o=12, v=108, q=360, prec="fp64", vvvv="packed", states=8, group=4),
        # an excited state's equations: transformed Hamiltonian, partial linearisation
        dict(name="plascc o15 v135 fp64", kind="plascc", o=15, v=135, q=450, prec="fp64", vvvv="packed"),
        # a new geometry: the integral set in a kept workspace and its first evaluation
        dict(name="build o18 v162 bf16x3", kind="build", o=18, v=162, q=540, prec="bf16x3", vvvv="packed"),
        # a handful of requests from host arrays to energies through the request server
        dict(name="serve o4-o8 bf16x3", kind="serve", o=8, v=72, q=240, prec="bf16x3", vvvv="packed", requests=8, tol=1e-7),
    ]


def draw(rng):
    kind = rng.choice(["residual"] * 6 + ["solve", "batch", "plascc", "build", "serve"])
    most = {"residual": 24, "solve": 14, "batch": 14, "plascc": 18, "build": 20, "serve": 8}[kind]
    o = int(round(math.exp(rng.uniform(math.log(4), math.log(most)))))
    v = max(o + 1, int(round(o * rng.uniform(4.0, 9.0))))
    q = int(round((o + v) * rng.uniform(2.6, 3.2)))
    c = dict(kind=kind, o=o, v=v, q=q, prec=rng.choice(["fp64", "fp64", "bf16x3", "fp32"]),
             vvvv=rng.choice(["packed", "packed", "full"]))
    if kind == "solve":
        c.update(tol=1e-8, prec="fp64")
    if kind == "batch":
        c["states"] = rng.randint(2, 8)
        c["group"] = rng.randint(1, min(4, c["states"]))
    if kind == "serve":
        c.update(requests=rng.randint(4, 8), tol=1e-7, vvvv="packed", prec=rng.choice(["fp64", "bf16x3"]))
    return c


# --- inputs -----------------------------------------------------------------------------------------------------

def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _gen(seed):
    return torch.Generator(device=_device()).manual_seed(seed)


def _system(o, v, q, g):
    """(B, eps) on the device: B[Q] symmetric, orbital energies sorted, occupied ones first."""
    n, dev = o + v, _device()
    sigma = 0.05 * math.sqrt(1200.0 / (q * v))
    B = torch.randn((q, n, n), dtype=torch.float64, device=dev, generator=g).mul_(sigma)
    up = torch.triu(B)
    B = up + torch.triu(B, 1).transpose(1, 2)
    eo = torch.rand(o, dtype=torch.float64, device=dev, generator=g).mul_(1.7).sub_(2.0).sort().values
    ev = torch.rand(v, dtype=torch.float64, device=dev, generator=g).mul_(4.9).add_(0.1).sort().values
    return B.contiguous(), torch.cat([eo, ev])


def _amplitudes(B, eps, o, g):
    """t1 small and random; t2 = (ia|jb) / D plus a small random pair-symmetric part."""
    v = eps.numel() - o
    t1 = torch.randn((o, v), dtype=torch.float64, device=B.device, generator=g).mul_(0.02)
    Bov = B[:, :o, o:].reshape(B.shape[0], o * v)
    t2 = (Bov.T @ Bov).reshape(o, v, o, v).permute(0, 2, 1, 3).contiguous()
    d = eps[:o, None] - eps[None, o:]
    t2 /= d[:, None, :, None] + d[None, :, None, :]
    x = torch.randn((o, o, v, v), dtype=torch.float64, device=B.device, generator=g).mul_(0.001)
    t2 += x + x.permute(1, 0, 3, 2)
    return t1, t2


def _states(case, seed):
    """The system and its amplitude sets (one, or one per state)."""
    g, o, v = _gen(seed), case["o"], case["v"]
    B, eps = _system(o, v, case["q"], g)
    t1, t2 = zip(*[_amplitudes(B, eps, o, g) for _ in range(case.get("states", 1))])
    t1, t2 = torch.stack(t1), torch.stack(t2)
    if case["kind"] == "plascc":  # on the guess of the highest occupied to lowest virtual state
        t1[0, o - 1, 0] += 1.0 / math.sqrt(2.0)
        t2[0, o - 1, o - 1, 0, 0] -= 0.5
    return B, eps, t1, t2


def _requests(case, seed):
    """Shapes (v = 9 o, Q = 3 (o + v), o up to the case's) and inputs of the served systems."""
    g = _gen(seed)
    low = min(4, case["o"])
    for k in range(case["requests"]):
        o = low + k % (case["o"] - low + 1)
        v = max(o + 1, round(o * case["v"] / case["o"]))
        yield o, *_system(o, v, 3 * (o + v), g)


# --- what a program keeps, and one pass -------------------------------------------------------------------------

def prepare(case, seed):
    kind, o, v, q = case["kind"], case["o"], case["v"], case["q"]
    prec, mode = PREC[case["prec"]], VVVV[case["vvvv"]]
    if kind == "serve":
        reqs = [(o, B.cpu().numpy(), e.cpu().numpy()) for o, B, e in _requests(case, seed)]
        server = A.Server(hbm_budget=6 << 30, max_active=16, precision=prec, vvvv_mode=mode, tol_rnorm=case["tol"])
        return dict(kind=kind, server=server, reqs=reqs)
    if kind == "solve":
        B, eps = _system(o, v, q, _gen(seed))
        ints = A.ascc_build_ints(B, eps, o, precision=prec, vvvv_mode=mode)
        t1 = torch.zeros((o, v), dtype=torch.float64, device=B.device)
        t2 = torch.zeros((o, o, v, v), dtype=torch.float64, device=B.device)
        return dict(kind=kind, ints=ints, t1=t1, t2=t2, tol=case["tol"])
    B, eps, t1, t2 = _states(case, seed)
    s = dict(kind=kind, t1=t1, t2=t2, r1=torch.empty_like(t1), r2=torch.empty_like(t2),
             e=torch.empty(t1.shape[0], dtype=torch.float64, device=B.device))
    if kind == "build":
        need = A.ascc_workspace_bytes(o, v, q, prec, mode)[0]
        s.update(B=B, eps=eps, o=o, prec=prec, mode=mode,
                 ws=torch.empty(need, dtype=torch.uint8, device=B.device))
    elif kind == "plascc":
        s["ints"] = A.ascc_build_ints_hbar(B, eps, o, o - 1, o, precision=prec, vvvv_mode=mode)
        A.ascc_set_plascc(s["ints"], o - 1, o)
    else:
        s["ints"] = A.ascc_build_ints(B, eps, o, precision=prec, vvvv_mode=mode)
        if kind == "batch":
            need = A.ascc_batch_workspace_bytes(o, v, q, case["states"], case["group"], prec, mode)
            s["ws"] = torch.empty(need // 8, dtype=torch.float64, device=B.device)
            A.ascc_batch_reserve_ws(s["ints"], case["states"], case["group"], s["ws"])
    return s


def run(s):
    kind = s["kind"]
    if kind == "serve":
        srv = s["server"]
        ids = [srv.submit(B, eps, o, 0.0) for o, B, eps in s["reqs"]]
        queued = running = 1
        while queued or running:
            queued, running, _ = srv.step(0.0)
        infos = [srv.info(i) for i in ids]
        return np.array([[x["e_ref"], x["e_corr"]] for x in infos])
    if kind == "solve":
        s["t1"].zero_()
        s["t2"].zero_()
        res = A.ascc_solve(s["ints"], s["t1"], s["t2"], tol_rnorm=s["tol"], maxiter=60)
        return s["t1"], s["t2"], np.float64(res["e_corr"])
    if kind == "batch":
        A.ascc_residual_batch(s["ints"], list(s["t1"]), list(s["t2"]), list(s["r1"]), list(s["r2"]), s["e"])
    elif kind == "build":
        ints = A.ascc_build_ints_ws(s["B"], s["eps"], s["o"], s["ws"], precision=s["prec"], vvvv_mode=s["mode"])
        A.ascc_residual(ints, s["t1"][0], s["t2"][0], s["r1"][0], s["r2"][0], s["e"])
        ints.close()
    else:
        A.ascc_residual(s["ints"], s["t1"][0], s["t2"][0], s["r1"][0], s["r2"][0], s["e"])
    return s["r1"], s["r2"], s["e"]


# --- what a pass cannot do without ------------------------------------------------------------------------------

def _residual_work(o, v, q, prec, vvvv):
    """Operations of the N^6 terms (ladder over the pair halves, W/Z, hole-hole ladder, rings); bytes of the integral
    blocks, the fitting factors and the doubles, once each (4 bytes a value of the large blocks in low precision)."""
    to, tv, so, sv = o * (o + 1) // 2, v * (v + 1) // 2, o * (o - 1) // 2, v * (v - 1) // 2
    flops = 2.0 * (to * tv**2 + so * sv**2) + 4.0 * o**4 * v**2 + 10.0 * o**3 * v**3
    word = 8 if prec == "fp64" else 4
    large = (v**4 if vvvv == "full" and prec == "fp64" else 2 * tv**2) + v * v * (o * v + o * o) + 2 * (o * v) ** 2
    return word * large + 8.0 * (q * (o + v) ** 2 + (o * v) ** 2 * 3), flops


def work(case):
    o, v, q = case["o"], case["v"], case["q"]
    b, f = _residual_work(o, v, q, case["prec"], case["vvvv"])
    if case["kind"] == "solve":
        b, f = STEPS * b, STEPS * f
    elif case["kind"] == "batch":  # the integrals are read once for all states
        per = 8.0 * (o * v) ** 2 * 3
        b, f = b + (case["states"] - 1) * per, f * case["states"]
    elif case["kind"] == "build":  # the (ac|bd) slabs with b >= a, (kc|bd) and (ia|jb)
        f += 2.0 * q * (v * v * v * (v + 1) / 2 + o * v**3 + (o * v) ** 2)
        b *= 2
    elif case["kind"] == "serve":
        b = f = 0.0
        low = min(4, o)
        for k in range(case["requests"]):
            x = low + k % (o - low + 1)
            y = max(x + 1, round(x * v / o))
            db, df = _residual_work(x, y, 3 * (x + y), case["prec"], "packed")
            b, f = b + STEPS * db, f + STEPS * df
    return {"bytes": float(b), "flops": float(f)}


# --- the same results in 64 bits, plainly -----------------------------------------------------------------------

def _two_electron(B, o):
    """sum_k 2 (pq|kk) - (pk|kq)."""
    dk = B[:, range(o), range(o)].sum(1)
    K = torch.zeros(B.shape[1:], dtype=B.dtype, device=B.device)
    for Bq in B.split(64):
        K += torch.matmul(Bq[:, :, :o], Bq[:, :o, :]).sum(0)
    return 2.0 * torch.tensordot(dk, B, 1) - K


def _residual(B, h, fov, t1, t2):
    """Closed-shell singles and doubles residual and energy, T1-dressed, every term as it is written."""
    o, v = t1.shape
    n, dev = o + v, B.device
    X, Y = torch.eye(n, dtype=B.dtype, device=dev), torch.eye(n, dtype=B.dtype, device=dev)
    X[o:, :o] = -t1.T
    Y[:o, o:] = t1
    Bh = torch.matmul(torch.matmul(X, B), Y.T)
    F = X @ h @ Y.T + _two_electron(Bh, o)
    oo, ov, vo, vv = (Bh[:, p, q].contiguous() for p in (slice(0, o), slice(o, n)) for q in (slice(0, o), slice(o, n)))
    q = B.shape[0]

    def block(L, R):
        return (L.reshape(q, -1).T @ R.reshape(q, -1)).reshape(*L.shape[1:], *R.shape[1:])

    u = 2.0 * t2 - t2.transpose(2, 3)
    kcld, kiac, aikc = block(ov, ov), block(oo, vv), block(vo, ov)
    flat = lambda x, *p: x.permute(*p).reshape(x.shape[p[0]] * x.shape[p[1]], -1)  # noqa: E731
    # sum_ld B_Q,ld u_kl^cd
    N = (ov.reshape(q, -1) @ flat(u, 1, 3, 0, 2)).reshape(q, o, v)
    r1 = torch.einsum("qkd,qad->ka", N, vv) - torch.einsum("qli,qla->ia", oo, N)
    r1 = r1 + torch.einsum("ikac,kc->ia", u, F[:o, o:]) + F[o:, :o].T
    r2 = block(vo, vo).permute(1, 3, 0, 2).contiguous()
    step = max(1, min(v, int(2e9 / v**3)))
    for a in range(0, v, step):  # sum_cd t_ij^cd (ac|bd)^
        na = min(step, v - a)
        g = block(vv[:, a:a + na].contiguous(), vv).permute(1, 3, 0, 2).reshape(v * v, -1)
        r2[:, :, a:a + na] += (t2.reshape(o * o, -1) @ g).reshape(o, o, na, v)
        del g
    chi = block(oo, oo).permute(1, 3, 0, 2).reshape(o * o, -1) + t2.reshape(o * o, -1) @ flat(kcld, 1, 3, 0, 2)
    r2 += (chi @ t2.reshape(o * o, -1)).reshape(r2.shape)
    # rings, as [ia][kc] matrices
    tx, um = flat(t2, 0, 3, 1, 2), flat(u, 0, 2, 1, 3)                # t_ik^ca at [i a][k c], u_ik^ac
    K = flat(kcld, 0, 3, 2, 1)                                          # (kd|lc) at [k c][l d]
    L = 2.0 * flat(kcld, 0, 1, 2, 3) - K
    kiac_m = flat(kiac, 1, 2, 0, 3)                                     # (ki|ac) at [i a][k c]
    Xc = kiac_m - 0.5 * (tx @ K)
    Zd = 2.0 * flat(aikc, 1, 0, 2, 3) - kiac_m + 0.5 * (um @ L)
    p1 = (tx @ Xc.T).reshape(o, v, o, v)                                # [j b][i a] for t_kj^bc, Xc[i a][k c]
    p2 = (um @ Zd.T).reshape(o, v, o, v)
    del tx, um, K, L, Xc, Zd, kiac_m
    x = 0.5 * (p2 - p1).permute(2, 0, 3, 1) - p1.permute(0, 2, 3, 1)
    Fv = F[o:, o:] - torch.einsum("qkb,qkc->bc", N, ov)
    Fo = F[:o, :o] + torch.einsum("qkd,qjd->kj", ov, N)
    x = x + torch.matmul(t2, Fv.T) - torch.einsum("ikab,kj->ijab", t2, Fo)
    r2 += x + x.permute(1, 0, 3, 2)
    g = kcld.permute(0, 2, 1, 3)
    tau = t2 + t1[:, None, :, None] * t1[None, :, None, :]
    e = (tau * (2.0 * g - g.transpose(2, 3))).sum() + 2.0 * (fov * t1).sum()
    return r1, r2, e.reshape(1)


def _hamiltonian(B, eps, o):
    return torch.diag(eps) - _two_electron(B, o)


def _solved(B, eps, o, tol=1e-12):
    """The converged amplitudes and energy from T = 0 (Jacobi steps with an 8-vector extrapolation)."""
    v = eps.numel() - o
    h, fov = _hamiltonian(B, eps, o), torch.zeros((o, v), dtype=B.dtype, device=B.device)
    d1 = eps[:o, None] - eps[None, o:]
    d2 = d1[:, None, :, None] + d1[None, :, None, :]
    x = torch.zeros(o * v + (o * v) ** 2, dtype=B.dtype, device=B.device)
    ts, es = [], []
    for _ in range(60):
        t1, t2 = x[:o * v].reshape(o, v), x[o * v:].reshape(o, o, v, v)
        r1, r2, e = _residual(B, h, fov, t1, t2)
        if math.sqrt(float(r1.square().sum() + r2.square().sum())) < tol:
            break
        s = torch.cat([(r1 / d1).reshape(-1), (r2 / d2).reshape(-1)])
        ts, es = (ts + [x + s])[-8:], (es + [s])[-8:]
        m = len(es)
        M = torch.zeros((m + 1, m + 1), dtype=torch.float64)
        E = torch.stack(es)
        M[:m, :m] = (E @ E.T).cpu()
        M[:m, :m] /= M[:m, :m].diagonal().max()
        M[m, :m] = M[:m, m] = -1.0
        c = torch.linalg.lstsq(M, -torch.eye(m + 1, dtype=torch.float64)[:, m:], driver="gelsd").solution[:m, 0]
        x = c.to(x.device) @ torch.stack(ts)
    return t1.clone(), t2.clone(), e


def exact(case, seed):
    kind, o = case["kind"], case["o"]
    if kind == "serve":
        rows = []
        for o, B, eps in _requests(case, seed):
            h = _hamiltonian(B, eps, o)
            e0 = (h.diagonal()[:o] + eps[:o]).sum()
            rows.append([float(e0), float(_solved(B, eps, o)[2])])
        return np.array(rows)
    if kind == "solve":
        B, eps = _system(o, case["v"], case["q"], _gen(seed))
        t1, t2, e = _solved(B, eps, o)
        return t1, t2, np.float64(float(e))
    B, eps, t1, t2 = _states(case, seed)
    h, fov = _hamiltonian(B, eps, o), torch.zeros_like(t1[0])
    if kind == "plascc":
        # x -> (1 + K) x (1 - K) with K = E_hp / sqrt 2
        K = torch.zeros_like(h)
        K[o - 1, o] = 1.0 / math.sqrt(2.0)
        one = torch.eye(h.shape[0], dtype=h.dtype, device=h.device)
        B = torch.matmul(torch.matmul(one + K, B), one - K)
        h = (one + K) @ h @ (one - K)
        fov = (h + _two_electron(B, o))[:o, o:]
    outs = [_residual(B, h, fov, a, b) for a, b in zip(t1, t2)]
    r1, r2, e = (torch.stack([x[k] for x in outs]) for k in range(3))
    if kind == "plascc":
        # without the part quadratic in the mixed doubles (index sets that touch the hole or the particle, the
        # all-primary one left out): half the sum at +tM and -tM, less the value at 0
        tm = torch.zeros_like(t2[0])
        tm[o - 1], tm[:, o - 1] = t2[0][o - 1], t2[0][:, o - 1]
        tm[:, :, 0], tm[:, :, :, 0] = t2[0][:, :, 0], t2[0][:, :, :, 0]
        tm[o - 1, o - 1, 0, 0] = 0.0
        plus, minus, zero = (_residual(B, h, fov, t1[0], s * tm)[1] for s in (1.0, -1.0, 0.0))
        r2 = r2 - (0.5 * (plus + minus) - zero)
    return r1, r2, e.reshape(-1)
