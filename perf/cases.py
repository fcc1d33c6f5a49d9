"""Performance cases of the Alternating Metropolis-Hastings sampler.

What a program built on this package has the GPU do, through the package's public entry
points: alternation cycles of a sampler that is resumed from a checkpoint, whole short
jobs, batched and served proteins, float64 energies, conformations and gradients, and
L-BFGS minimisation.  Everything a pass reads is made here from a seed, with torch and
numpy alone: reference torsions from a Ramachandran-like mixture, a distogram table of
37 bins around the reference C-beta distances mixed with Dirichlet(0.5) noise, and
conformations of a given spread around the reference ("noise", radians), as a run that
starts from a predicted structure has them, or the extended chain.

    listed()           the cases
    draw(rng)          one more case of the same ranges
    prepare(case, s)   inputs and handles a program has before the call
    run(state)         one pass
    work(case)         bytes and operations a pass cannot do without
    exact(case, s)     the pass in 64 bits by plain torch, where that is possible
"""
import math

import numpy as np
import torch

from paper_2211_03193_amd import amh

N_BINS, D_MIN, BIN_W = 37, 2.0, 0.5

# Kinds of case and what they stand for:
#   cycle     resume from a checkpoint, advance the chains, take the next checkpoint: the
#             inner loop of every run of the sampler
#   job       a whole short run from the extended chain: context, sweeps, best states
#   batch     one cycle of several proteins of different lengths in shared launches
#   serve     jobs from host tables through the continuous-batching server
#   energy    float64 energies and C-beta coordinates of given conformations
#   conformation   atom coordinates of given torsions
#   grad      float64 energies and torsion gradients of given conformations
#   minimize  L-BFGS from given conformations


def _cycle(name, L, C, d=12, sweeps=10, noise=0.3, t=2500, S=5000, every=10, n_global=1, anchor=10,
           cascade=0, sigma_end=0.0):
    return {"name": name, "kind": "cycle", "L": L, "C": C, "d": d, "sweeps": sweeps, "noise": noise, "t": t,
            "S": S, "every": every, "n_global": n_global, "anchor": anchor, "cascade": cascade,
            "sigma_end": sigma_end}


def listed():
    return [
        # the smallest: one chain of a small protein (64 residues, window 8)
        _cycle("cycle_L64_C1", 64, 1, d=8, t=10000, S=20000),
        # odd sizes and the schedule's options: cascaded radii, a narrowing proposal, two
        # global sweeps in a cycle of seven, anchors that fall between them
        _cycle("cycle_L97_C37_options", 97, 37, d=9, sweeps=14, every=7, n_global=2, anchor=3, cascade=5,
               sigma_end=4.0, t=2506),
        # one GPU's share when 1024 chains are split over eight
        _cycle("cycle_L300_C128", 300, 128),
        # the benchmark's size: 300 residues, 1024 chains, near the predicted structure
        _cycle("cycle_L300_C1024", 300, 1024),
        # the longest protein that is served
        _cycle("cycle_L800_C64", 800, 64, noise=0.1),
        # a whole run of 20 sweeps from the extended chain, a chain count that is no power of two
        {"name": "job_L250_C1500", "kind": "job", "L": 250, "C": 1500, "d": 12, "sweeps": 20},
        # a ragged batch: eight proteins of 50 to 600 residues, 64 chains each
        {"name": "batch_8_L50-600", "kind": "batch", "n": 8, "lo": 50, "hi": 600, "C": 64, "sweeps": 10,
         "noise": 0.3},
        # a handful of queued jobs of 50 to 200 residues, from submission to the last result
        {"name": "serve_6_L50-200", "kind": "serve", "n": 6, "lo": 50, "hi": 200, "C": 64, "sweeps": 20},
        # scoring every chain of the benchmark's run
        {"name": "energy_L300_B1024", "kind": "energy", "L": 300, "B": 1024, "noise": 0.3},
        # writing out a few structures
        {"name": "conformation_L150_B64", "kind": "conformation", "L": 150, "B": 64, "noise": 0.3},
        # gradients at the size of the hybrid run (400 residues, 512 conformations)
        {"name": "grad_L400_B512", "kind": "grad", "L": 400, "B": 512, "noise": 0.3},
        # refining sampled conformations
        {"name": "minimize_L200_B128", "kind": "minimize", "L": 200, "B": 128, "noise": 0.1, "iters": 20},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["cycle", "cycle", "cycle", "job", "batch", "serve", "energy", "conformation", "grad",
                       "minimize"])
    if kind == "cycle":
        L = _log_int(rng, 24, 800)
        # no more chains than the largest listed cycle's work allows
        C = _log_int(rng, 1, max(2, min(1280, 300 * 300 * 1024 // (L * L * (2 if L > 300 else 1)))))
        c = _cycle("", L, C, d=rng.choice([4, 8, 9, 12, 15]), noise=rng.choice([0.05, 0.1, 0.3, 0.5]),
                   t=rng.choice([0, 990, 2500, 4500]))
        if rng.random() < 0.3:
            c.update(every=7, n_global=rng.choice([1, 2]), anchor=rng.choice([2, 7]), sweeps=7,
                     cascade=rng.choice([0, 4, 7]), sigma_end=rng.choice([0.0, 4.0]), t=rng.choice([0, 2506, 4501]),
                     C=max(1, C // 2))
        del c["name"]
        return c
    if kind == "job":
        L = _log_int(rng, 40, 300)
        C = _log_int(rng, 16, min(1500, 1500 * 250 * 250 // (L * L)))
        return {"kind": kind, "L": L, "C": C, "d": rng.choice([8, 12]), "sweeps": 20}
    if kind == "batch":
        return {"kind": kind, "n": rng.randint(2, 8), "lo": rng.randint(40, 90), "hi": rng.randint(150, 600),
                "C": _log_int(rng, 8, 64), "sweeps": 10, "noise": 0.3}
    if kind == "serve":
        return {"kind": kind, "n": rng.randint(2, 6), "lo": rng.randint(40, 80), "hi": rng.randint(100, 200),
                "C": _log_int(rng, 8, 64), "sweeps": 20}
    L = _log_int(rng, 24, 500)
    most = max(1, 1024 * 300 * 300 // (L * L))
    B = _log_int(rng, 1, min(1024 if kind in ("energy", "conformation") else 512, most))
    if kind == "minimize":
        L = min(L, 300)
        return {"kind": kind, "L": L, "B": min(B, 256), "noise": rng.choice([0.05, 0.1]), "iters": rng.choice([5, 20])}
    return {"kind": kind, "L": L, "B": B, "noise": rng.choice([0.05, 0.1, 0.3, 1.0])}


# --- inputs ---------------------------------------------------------------------------

# ideal backbone: bonds (A) and angles (degrees)
_NCA, _CAC, _CN, _CB = 1.458, 1.525, 1.329, 1.53
_A_NCAC, _A_CACN, _A_CNCA, _A_NCACB = (math.radians(a) for a in (111.2, 116.2, 121.7, 110.5))
_OMEGA, _T_CB = math.radians(180.0), math.radians(-122.5)


def _place(A, B, C, l, angle, tor):
    """The atom at bond l, angle and torsion tor (tensor or number) after A, B, C [..., 3]."""
    b = C - B
    b = b / b.norm(dim=-1, keepdim=True)
    n = torch.linalg.cross(B - A, b, dim=-1)
    n = n / n.norm(dim=-1, keepdim=True)
    m = torch.linalg.cross(n, b, dim=-1)
    tor = torch.as_tensor(tor, dtype=C.dtype, device=C.device)
    return (C - l * math.cos(angle) * b + l * math.sin(angle) * (torch.cos(tor)[..., None] * m
                                                                 + torch.sin(tor)[..., None] * n))


def _atoms(s):
    """N, CA, C, C-beta [B][L][4][3] of torsions s [B][2L], in s's type and on its device."""
    Bn, L = s.shape[0], s.shape[1] // 2
    v = lambda x, y: torch.tensor([x, y, 0.0], dtype=s.dtype, device=s.device).expand(Bn, 3)  # noqa: E731
    N, CA = v(0.0, 0.0), v(_NCA, 0.0)
    C = v(_NCA - _CAC * math.cos(_A_NCAC), _CAC * math.sin(_A_NCAC))
    rows = [(N, CA, C)]
    for c in range(1, L):
        N2 = _place(N, CA, C, _CN, _A_CACN, s[:, 2 * c - 1])
        CA2 = _place(CA, C, N2, _NCA, _A_CNCA, _OMEGA)
        C2 = _place(C, N2, CA2, _CAC, _A_NCAC, s[:, 2 * c])
        N, CA, C = N2, CA2, C2
        rows.append((N, CA, C))
    N, CA, C = (torch.stack([r[i] for r in rows], 1) for i in range(3))
    return torch.stack([N, CA, C, _place(C, N, CA, _CB, _A_NCACB, _T_CB)], 2)


def _wrap(a):
    w = np.mod(a + np.pi, 2.0 * np.pi) - np.pi
    return np.where(w <= -np.pi, w + 2.0 * np.pi, w)


def _protein(L, seed):
    """(reference torsions [2L] numpy, table [L(L-1)/2][37] float32 CPU tensor) of a seed."""
    rng = np.random.Generator(np.random.PCG64(seed))
    mu = np.radians(np.array([[-63.0, -43.0], [-120.0, 130.0], [57.0, 47.0]]))
    s = mu[rng.choice(3, size=L, p=[0.55, 0.40, 0.05])] + np.radians(15.0) * rng.standard_normal((L, 2))
    s = _wrap(s.reshape(-1))
    cb = _atoms(torch.from_numpy(s[None]))[0, :, 3]
    i, j = torch.triu_indices(L, L, 1)
    d = (cb[i] - cb[j]).norm(dim=1)
    knots = D_MIN + BIN_W * (torch.arange(N_BINS, dtype=torch.float64) + 0.5)
    log_g = torch.log_softmax(-0.5 * (knots[None] - d[:, None]) ** 2, 1)
    # Dirichlet(0.5): normalised squares of normal variates
    z = torch.from_numpy(rng.standard_normal((len(d), N_BINS), dtype=np.float32)).double().square_().clamp_(min=1e-30)
    log_q = torch.log(z / z.sum(1, keepdim=True))
    return s, -torch.logaddexp(math.log(0.9) + log_g, math.log(0.1) + log_q).float()


def _around(s, n, noise, seed):
    """n conformations [n][2L] float64 numpy around s."""
    rng = np.random.Generator(np.random.PCG64(seed))
    return np.ascontiguousarray(_wrap(s[None] + noise * rng.standard_normal((n, len(s)))))


def _config(L, C, key, d, S, every=10, n_global=1, anchor=10, cascade=0, sigma_end=0.0):
    cfg = amh.AmhConfig(L=L, n_chains=C, n_bins=N_BINS, window_d=d, d_min=D_MIN, bin_w=BIN_W, global_every=every,
                        anchor_every=anchor, sigma=math.radians(10.0), T0=1.0, T1=0.01, total_sweeps=S, seed=key,
                        n_global=n_global, sigma_end=math.radians(sigma_end))
    if cascade:
        cfg.n_cascade = 1
        cfg.cascade_d[0] = cascade
    return cfg


def _cycle_config(case, seed):
    return _config(case["L"], case["C"], 0x414D4800 + seed, case["d"], case["S"], case["every"], case["n_global"],
                   case["anchor"], case["cascade"], case["sigma_end"])


def _lengths(case):
    """The lengths of a batch or of served jobs, spread evenly with both ends."""
    n = case["n"]
    return [case["lo"] + (case["hi"] - case["lo"]) * q // (n - 1) for q in range(n)]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "cycle":
        s, y = _protein(case["L"], seed)
        s0 = torch.from_numpy(_around(s, case["C"], case["noise"], seed + 1)).cuda()
        ctx = amh.Context(_cycle_config(case, seed), y.cuda(), s0)
        ck = ctx.get_state()
        ck["t"] = case["t"]
        return {"case": case, "ctx": ctx, "checkpoint": ck}
    if kind == "job":
        _, y = _protein(case["L"], seed)
        return {"case": case, "y": y.cuda(), "cfg": _config(case["L"], case["C"], 0x414D4800 + seed, case["d"], 5000)}
    if kind == "batch":
        ctxs, cks = [], []
        for q, L in enumerate(_lengths(case)):
            s, y = _protein(L, seed + 100 * q)
            s0 = torch.from_numpy(_around(s, case["C"], case["noise"], seed + 100 * q + 1)).cuda()
            ctxs.append(amh.Context(_config(L, case["C"], 0x414D4800 + seed + q, 12, 5000), y.cuda(), s0))
            cks.append(dict(ctxs[-1].get_state(), t=2500))
        return {"case": case, "ctxs": ctxs, "batch": amh.Batch(ctxs), "checkpoints": cks}
    if kind == "serve":
        return {"case": case, "jobs": [(_config(L, case["C"], 0x414D4800 + seed + q, 12, case["sweeps"]),
                                        _protein(L, seed + 100 * q)[1].numpy())
                                       for q, L in enumerate(_lengths(case))]}
    s, y = _protein(case["L"], seed)
    conf = torch.from_numpy(_around(s, case["B"], case["noise"], seed + 1)).cuda()
    if kind == "conformation":
        return {"case": case, "s": conf}
    return {"case": case, "s": conf, "ctx": amh.Context(_config(case["L"], 1, seed, 12, 10), y.cuda())}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "cycle":
        ctx = state["ctx"]
        ctx.set_state(state["checkpoint"])
        ctx.sweep(case["sweeps"])
        return ctx.get_state()
    if kind == "job":
        ctx = amh.Context(state["cfg"], state["y"])
        ctx.sweep(case["sweeps"])
        V, s, cb = ctx.energy(which=1, want_s=True, want_cb=True)
        ctx.poll()
        ctx.close()
        return {"V": V, "s": s, "cb": cb}
    if kind == "batch":
        for ctx, ck in zip(state["ctxs"], state["checkpoints"]):
            ctx.set_state(ck)
        state["batch"].sweep(case["sweeps"])
        out = []
        for ctx in state["ctxs"]:
            V, s, cb = ctx.energy(which=0, want_s=True, want_cb=True)
            out.append({"V": V, "s": s, "cb": cb})
        return out
    if kind == "serve":
        server = amh.Server(hbm_budget_bytes=8 << 30, sweeps_per_round=10)
        ids = [server.submit(cfg, y, -1e30) for cfg, y in state["jobs"]]
        while sum(server.step()) > 0:
            pass
        out = [{k: j[k] for k in ("best_V", "s_best", "v")} for j in (server.job(i, want_state=True) for i in ids)]
        server.close()
        return out
    if kind == "energy":
        V, s, cb = state["ctx"].energy(state["s"], want_cb=True)
        return {"V": V, "cb": cb}
    if kind == "conformation":
        return amh.conformation(state["s"])
    if kind == "grad":
        V, g = state["ctx"].grad(state["s"])
        return {"V": V, "g": g}
    s = state["s"].clone()
    out = state["ctx"].minimize(s, amh.lbfgs_opts(n_iter=case["iters"]))
    return {"V": out["V"], "s": s}


# --- the work a pass cannot do without -----------------------------------------------
# Operations: a squared distance and its test 9, a spline 20, the rotation of a point 18;
# its derivative and the two force updates of a gradient pair 30 more.

_TEST, _SPLINE, _ROTATE, _FORCE = 9, 20, 18, 30
_PLACE = 60   # one atom placed from three others


def _near_pairs(L):
    """Pairs inside the last knot of a folded protein, about (measured: 60 partners each)."""
    return min(L * (L - 1) // 2, 30 * L)


def _sweep_work(L, C, d, n_local, n_global, anchors):
    h = d // 2
    window = 0
    for k in range(1, 2 * L - 1):
        c, p = k >> 1, (k >> 1) + (k & 1)
        lo, hi = max(0, c - h), min(L - 1, c + h)
        window += max(0, p - lo) * max(0, hi - p + 1)
    local = window * (2 * (_TEST + _SPLINE) + _ROTATE) + 2 * L * d * _ROTATE
    # every downstream C-beta turned, every near pair across the pivot scored: one in three
    # of them on average, and those of the pivot's own row and column
    glob = L * L * _ROTATE + 2 * L * (_near_pairs(L) / 3 + 30) * (_TEST + _SPLINE)
    anchor = 4 * L * _PLACE + _near_pairs(L) * (_TEST + _SPLINE)
    state = C * (2 * L * 8 * 3 + 12 * L * 8 * 2 + 64)   # torsions in and out, best torsions, atoms in and out
    return {"bytes": state + L * (L - 1) // 2 * N_BINS * 4,
            "flops": C * (n_local * local + n_global * glob + anchors * anchor)}


def work(case):
    kind = case["kind"]
    if kind == "cycle":
        t = range(case["t"], case["t"] + case["sweeps"])
        g = sum(q % case["every"] >= case["every"] - case["n_global"] for q in t)
        a = sum((q + 1) % case["anchor"] == 0 for q in t)
        return _sweep_work(case["L"], case["C"], case["d"], len(t) - g, g, a)
    if kind == "job":
        n = case["sweeps"]
        return _sweep_work(case["L"], case["C"], case["d"], n - n // 10, n // 10, n // 10)
    if kind in ("batch", "serve"):
        n = case["sweeps"]
        parts = [_sweep_work(L, case["C"], 12, n - n // 10, n // 10, n // 10) for L in _lengths(case)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    L, B = case["L"], case["B"]
    table = L * (L - 1) // 2 * N_BINS * 4
    if kind == "conformation":
        return {"bytes": B * (16 * L + 48 * L), "flops": B * 4 * L * _PLACE}
    if kind == "energy":
        return {"bytes": table + B * (16 * L + 12 * L + 8),
                "flops": B * (4 * L * _PLACE + _near_pairs(L) * (_TEST + _SPLINE))}
    grad = 4 * L * _PLACE + _near_pairs(L) * (_TEST + _SPLINE + _FORCE) + 2 * L * 30
    if kind == "grad":
        return {"bytes": table + B * (32 * L + 8), "flops": B * grad}
    # a minimisation evaluates the gradient at least once per iteration, and reads and
    # writes its torsions once
    return {"bytes": table + B * (32 * L + 8), "flops": B * (case["iters"] + 1) * grad}


# --- the same in 64 bits ---------------------------------------------------------------


def _pair_energy(rows, d):
    """Catmull-Rom value of table rows [..., 37] (float64) at distances d: the knots are the
    bin centres, mirrored ghosts at both ends, constant outside."""
    t = ((d - (D_MIN + 0.5 * BIN_W)) / BIN_W).clamp(0.0, N_BINS - 1.0)
    b = t.floor().clamp(max=N_BINS - 2.0)
    f, b = t - b, b.long()
    take = lambda k: rows.gather(-1, k[..., None])[..., 0]  # noqa: E731
    y0, y1, y2 = take((b - 1).abs()), take(b), take(b + 1)
    y3 = take(torch.where(b + 2 > N_BINS - 1, b, b + 2))
    return y1 + 0.5 * f * ((y2 - y0) + f * ((2 * y0 - 5 * y1 + 4 * y2 - y3) + f * (3 * (y1 - y2) + y3 - y0)))


def _energies(cb, y):
    """V [B] of C-beta coordinates cb [B][L][3] for the table y [P][37] (float64)."""
    L = cb.shape[1]
    i, j = torch.triu_indices(L, L, 1, device=cb.device)
    return torch.stack([_pair_energy(y, (x[i] - x[j]).norm(dim=1)).sum() for x in cb])


def _philox(k, t, chain, key):
    """Philox4x32-10 (Salmon et al., SC'11) of counters (k, t, chain, 0) as unsigned 32-bit words."""
    m = 0xFFFFFFFF
    x = [np.asarray(v, dtype=np.uint64) for v in np.broadcast_arrays(k, t, chain, 0)]
    k0, k1 = key & m, key >> 32
    for _ in range(10):
        a, b = x[0] * np.uint64(0xD2511F53), x[2] * np.uint64(0xCD9E8D57)
        x = [(b >> np.uint64(32)) ^ x[1] ^ np.uint64(k0), b & np.uint64(m),
             (a >> np.uint64(32)) ^ x[3] ^ np.uint64(k1), a & np.uint64(m)]
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return x


def _exact_cycle(case, seed):
    """The sampler's definition, all chains side by side: systematic scan of single-torsion
    proposals, the changed pairs of the window or of the whole protein, Metropolis rule."""
    L, C, n = case["L"], case["C"], 2 * case["L"]
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    s_ref, y32 = _protein(L, seed)
    y = y32.double().to(dev)
    s = torch.from_numpy(_around(s_ref, C, case["noise"], seed + 1)).to(dev)
    x = _atoms(s)
    V = _energies(x[:, :, 3], y)
    best, s_best = V.clone(), s.clone()
    counters = torch.zeros(C, 4, dtype=torch.int64, device=dev)
    counters[:, 2] = -1
    key, chain = 0x414D4800 + seed, np.arange(C)
    for t in range(case["t"], case["t"] + case["sweeps"]):
        glob = t % case["every"] >= case["every"] - case["n_global"]
        frac = t / (case["S"] - 1)
        beta = 1.0 / (1.0 * 0.01 ** frac)
        sigma = math.radians(10.0)
        if case["sigma_end"] > 0:
            sigma *= (math.radians(case["sigma_end"]) / sigma) ** frac
        h = (case["cascade"] if case["cascade"] and t % 2 else case["d"]) // 2
        for k in range(n):
            w = _philox(k, t, chain, key)
            u = [(v.astype(np.float64) + 0.5) / 2.0 ** 32 for v in w[:3]]
            delta = torch.from_numpy(sigma * np.sqrt(-2 * np.log(u[0])) * np.cos(2 * np.pi * u[1])).to(dev)
            log_u = torch.from_numpy(np.log(u[2])).to(dev)
            c, odd = k >> 1, k & 1
            p = c + odd
            a, e = x[:, c, odd], x[:, c, odd + 1]
            lo, hi = (0, L - 1) if glob else (max(0, c - h), min(L - 1, c + h))
            dE = torch.zeros(C, dtype=torch.float64, device=dev)
            new = None
            if k not in (0, n - 1):
                axis = (e - a) / (e - a).norm(dim=1, keepdim=True)
                r = x[:, p:] - a[:, None, None]
                ax = axis[:, None, None].expand_as(r)
                cd, sd = torch.cos(delta)[:, None, None, None], torch.sin(delta)[:, None, None, None]
                new = a[:, None, None] + cd * r + sd * torch.linalg.cross(ax, r, dim=-1) \
                    + (1 - cd) * (ax * r).sum(-1, keepdim=True) * ax
                if not odd:
                    new[:, 0, :2] = x[:, p, :2]
                if p > lo and hi >= p:
                    i, j = torch.arange(lo, p, device=dev), torch.arange(p, hi + 1, device=dev)
                    rows = y[(i * L - i * (i + 1) // 2 - i - 1)[:, None] + j[None]][None].expand(C, -1, -1, -1)
                    far = x[:, lo:p, None, 3]
                    d0 = (x[:, None, p:hi + 1, 3] - far).norm(dim=-1)
                    d1 = (new[:, None, :hi + 1 - p, 3] - far).norm(dim=-1)
                    dE = (_pair_energy(rows, d1) - _pair_energy(rows, d0)).sum((1, 2))
            acc = (dE <= 0) | (log_u < -beta * dE)
            m = torch.where(acc, s[:, k] + delta, s[:, k])
            s[:, k] = torch.where(m > math.pi, m - 2 * math.pi, torch.where(m <= -math.pi, m + 2 * math.pi, m))
            if new is not None:
                x[:, p:] = torch.where(acc[:, None, None, None], new, x[:, p:])
            counters[:, 1 if glob else 0] += acc
        if (t + 1) % case["anchor"] == 0:
            x = _atoms(s)
            V = _energies(x[:, :, 3], y)
            better = V < best
            best, s_best = torch.where(better, V, best), torch.where(better[:, None], s, s_best)
            counters[:, 3] += 1
    return {"s": s, "s_best": s_best, "v": torch.stack([V, best], 1), "counters": counters, "atoms": x,
            "t": case["t"] + case["sweeps"]}


def exact(case, seed):
    kind = case["kind"]
    if kind == "cycle":
        # a proposal costs some milliseconds here, whatever its size; a larger run also takes
        # a near-tie the other way in some chain, as any change of rounding does
        if 2 * case["L"] * case["sweeps"] > 3000 or case["C"] > 64:
            return None
        return _exact_cycle(case, seed)
    if kind in ("job", "batch", "serve", "minimize"):
        # runs of many chains take near-ties, and line searches near-equal trial values, by
        # the last bits of an energy: no value in 64 bits is theirs
        return None
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    s_ref, y = _protein(case["L"], seed)
    s = torch.from_numpy(_around(s_ref, case["B"], case["noise"], seed + 1)).to(dev)
    if kind == "conformation":
        return _atoms(s)
    y = y.double().to(dev)
    if kind == "energy":
        cb = _atoms(s)[:, :, 3]
        return {"V": _energies(cb, y), "cb": cb}
    V, g = [], []
    for part in s.split(128):
        part = part.clone().requires_grad_(True)
        cb = _atoms(part)[:, :, 3]
        # the energy's gradient at the C-beta positions, one conformation at a time, then back
        # through the geometry for all at once
        leaf = cb.detach().requires_grad_(True)
        for b in range(len(part)):
            v = _energies(leaf[b:b + 1], y)
            V.append(v.detach())
            v.backward(torch.ones_like(v))
        cb.backward(leaf.grad)
        g.append(part.grad)
    return {"V": torch.cat(V), "g": torch.cat(g)}
