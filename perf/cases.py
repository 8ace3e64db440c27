"""Performance cases of the library: what is timed, on which inputs, and the
values the timed calls should return.

Each case names one kind of call a program makes (a rank-2 run, a grouped
run, an adjoint, a receiver run, a full-order run) and its sizes.  `listed`
gives the fixed cases, `draw` one more of the same ranges, `prepare` the
inputs and the objects a program keeps between calls (context, plan),
`run` one call, `work` the bytes and operations the call cannot do without,
and `exact` the call's results in 64-bit arithmetic with plain torch.

Reduced operators are random as in the paper's performance study (Sec. 4.2):
Avs ~ N(0, 1/Ks) entrywise, Asv = -Avs^T (skew) or -diag(w) Avs^T with
w ~ U[0.5, 1.5] (a positive material weight times the negative transpose,
what staggered finite differences give); dt is half the stability limit.
"""
import math
import random

import numpy as np
import torch

from paper_2009_11742_amd.rom import Fom, GroupPlan, Rom

DEV = "cuda"


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # a small projected model (POD of a few snapshots: Kv = 30, Ks = 28)
        # stepped a little way for one sample: launch and call latency
        rank2("small_f32", "f32", 30, 28, 1, 20, skew=False),
        # the paper's plain method: FP64, a handful of samples, long horizon,
        # quantity of interest and probe trace kept
        rank2("plain_f64", "f64", 64, 64, 8, 2000, probe="Jy"),
        # the benchmark workload: 256 samples of a K = 256 model, 10^4 steps
        rank2("bench_f32", "f32", 256, 256, 256, 10000, probe="J"),
        # a projected model of odd sizes with material weights, an odd
        # ensemble, the second source signal, the whole probe trace
        rank2("ragged_f32", "f32", 150, 130, 300, 1000, skew=False, probe="Jy", source="gauss1"),
        # FP64 production of a mid-size projected model
        rank2("mid_f64", "f64", 300, 280, 128, 200, skew=False, probe="J"),
        # the precision study's size in FP32 and with BF16 operators
        rank2("large_f32", "f32", 1024, 1024, 1024, 500, probe="J"),
        rank2("large_bf16", "bf16", 1024, 1024, 1024, 500, probe="J"),
        # the top of the paper's scaling study (K = 4096)
        rank2("scaling_f32", "f32", 4096, 4096, 1024, 8),
        # many models of uneven size advanced together
        {"name": "grouped_f32", "kind": "grouped", "G": 64, "sizes": 0, "nsteps": 200},
        # gradients of the quantity of interest at the differentiation size
        {"name": "adjoint_f32", "kind": "adjoint", "kv": 512, "ks": 512, "M": 256, "nsteps": 1000, "skew": True},
        # seismograms and ensemble statistics at 16 receivers
        {"name": "receivers_f32", "kind": "receivers", "kv": 256, "ks": 256, "M": 256, "R": 16, "nsteps": 1000,
         "skew": True},
        # the full-order model the reduced ones come from (785,152 unknowns)
        {"name": "fom_f64", "kind": "fom", "nr": 256, "nth": 1024, "M": 16, "nsteps": 100},
    ]


def rank2(name, dtype, kv, ks, M, nsteps, skew=True, probe="none", source="ricker", operand="pair"):
    return {"name": name, "kind": "rank2", "dtype": dtype, "kv": kv, "ks": ks, "M": M, "nsteps": nsteps,
            "skew": skew, "probe": probe, "source": source, "operand": operand}


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _steps(rng, flops_per_step, lo, hi, budget):
    return max(4, min(_log(rng, lo, hi), int(budget / flops_per_step)))


def _sizes(rng, lo, hi):
    """Square about half the time (rounded to 64 in half of those), else any
    Kv and Ks within a factor of two."""
    kv = _log(rng, lo, hi)
    r = rng.random()
    if r < 0.3 and kv >= 64:
        kv = kv // 64 * 64
        return kv, kv
    if r < 0.55:
        return kv, kv
    return kv, max(lo, int(kv * rng.uniform(0.5, 1.0)))


def draw(rng):
    """One more case.  Ranges: FP32 rank-2 runs K 16..1600, M 1..1024; FP64
    K 16..640, M 1..512; BF16 / FP8 operators K 64..1024, M 1..1024; grouped
    runs of 2..48 models of the listed case's sizes; adjoints K 32..640,
    M 4..256; receivers K 32..512, M 1..512, R 1..16; full-order grids up to
    the listed one, M 1..32."""
    kind = rng.choice(["f32", "f32", "f32", "f32", "f64", "f64", "lowp", "grouped", "adjoint", "receivers", "fom"])
    probe = rng.choice(["none", "J", "Jy"])
    source = rng.choice(["ricker", "gauss1"])
    if kind in ("f32", "f64"):
        kv, ks = _sizes(rng, 16, 1600 if kind == "f32" else 640)
        M = _log(rng, 1, 1024 if kind == "f32" else 512)
        n = _steps(rng, 4.0 * kv * ks * M, 20, 600 if kind == "f32" or kv <= 128 else 200, 1.5e11)
        c = rank2("", kind, kv, ks, M, n, rng.random() < 0.5, probe, source)
        del c["name"]
        return c
    if kind == "lowp":
        kv, ks = _sizes(rng, 64, 1024)
        M = _log(rng, 1, 1024)
        c = rank2("", rng.choice(["bf16", "fp8"]), kv, ks, M, _steps(rng, 4.0 * kv * ks * M, 20, 400, 1.5e11),
                  rng.random() < 0.5, probe, source)
        del c["name"]
        return c
    if kind == "grouped":
        return {"kind": "grouped", "G": _log(rng, 2, 48), "sizes": rng.randrange(1, 1000), "nsteps": _log(rng, 20, 200)}
    if kind == "adjoint":
        kv, ks = _sizes(rng, 32, 640)
        M = _log(rng, 4, 256)
        return {"kind": "adjoint", "kv": kv, "ks": ks, "M": M, "skew": rng.random() < 0.5,
                "nsteps": _steps(rng, 12.0 * kv * ks * M, 30, 500, 1e11)}
    if kind == "receivers":
        kv, ks = _sizes(rng, 32, 512)
        M = _log(rng, 1, 512)
        return {"kind": "receivers", "kv": kv, "ks": ks, "M": M, "R": _log(rng, 1, 16), "skew": rng.random() < 0.5,
                "nsteps": _steps(rng, 4.0 * kv * ks * M, 30, 1000, 5e10)}
    return {"kind": "fom", "nr": _log(rng, 32, 256), "nth": _log(rng, 64, 1024), "M": _log(rng, 1, 16),
            "nsteps": _log(rng, 10, 100)}


# ------------------------------------------------------------------- inputs

def _gen(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + salt)
    return g


def _f32(x):
    return x.to(torch.float32).to(torch.float64)


def _model(kv, ks, M, skew, seed, salt=0, rounded=True):
    """Operators, source, samples, probe and dt on the GPU in FP64; rounded
    to FP32 values for runs with FP32 inputs."""
    g = _gen(seed, salt)
    A = torch.randn((kv, ks), generator=g, device=DEV, dtype=torch.float64) / math.sqrt(ks)
    b = torch.randn(kv, generator=g, device=DEV, dtype=torch.float64)
    c = torch.randn(kv, generator=g, device=DEV, dtype=torch.float64)
    mu = 0.5 + 0.5 * torch.rand(M, generator=g, device=DEV, dtype=torch.float64)
    w = 0.5 + torch.rand(ks, generator=g, device=DEV, dtype=torch.float64)
    dt = 0.5 / (1.0 + math.sqrt(kv / ks))
    if rounded:
        A, b, c, dt = _f32(A), _f32(b), _f32(c), float(np.float32(dt))
    B = -A.t().contiguous()
    if not skew:
        B = w[:, None] * B
        B = _f32(B) if rounded else B
    return {"A": A, "B": B, "b": b, "c": c, "mu": mu, "dt": dt}


def _host(X):
    """Column-major host copy."""
    return X.t().contiguous().cpu().numpy().T


def _rom(m, **kw):
    return Rom(_host(m["A"]), _host(m["B"]), m["b"].cpu().numpy(), m["dt"], **kw)


def _group_sizes(case):
    """(K, M) of each model: K uniform over 128, 192, ..., 768, M log-uniform
    in 16 .. 512 (the grouped workload's distribution)."""
    rng = random.Random(case["sizes"])
    return [(64 * rng.randint(2, 12), _log(rng, 16, 512)) for _ in range(case["G"])]


def _grid(case, seed):
    """Heterogeneous medium on a staggered grid (unit spacing): inverse
    density at the velocity points, stiffness at the two stress families,
    point source, time step inside the CFL limit, centre frequencies."""
    nr, nth, M = case["nr"], case["nth"], case["M"]
    g = _gen(seed)

    def field(*shape):
        return 0.8 + 0.4 * torch.rand(shape, generator=g, device=DEV, dtype=torch.float64)

    m = {"ir": field(nr, nth), "k1": field(nr - 1, nth), "k2": field(nr, nth - 1), "dt": 0.4}
    f = torch.zeros((nr, nth), dtype=torch.float64, device=DEV)
    f[nr // 3, nth // 5] = 1.0
    m["f"] = f
    m["mu"] = 0.1 + 0.1 * torch.rand(M, generator=g, device=DEV, dtype=torch.float64)
    return m


def _grid_csr(m):
    """Av (divergence over density) and As (stiffness times gradient)."""
    ir, k1, k2 = (m[k].cpu().numpy() for k in ("ir", "k1", "k2"))
    nr, nth = ir.shape
    n1 = (nr - 1) * nth
    i, j = np.meshgrid(np.arange(nr), np.arange(nth), indexing="ij")
    cols = np.stack([(i - 1) * nth + j, i * nth + j, n1 + i * (nth - 1) + j - 1, n1 + i * (nth - 1) + j], -1)
    vals = np.stack([-ir, ir, -ir, ir], -1)
    keep = np.stack([i > 0, i < nr - 1, j > 0, j < nth - 1], -1)
    ptr = np.concatenate([[0], np.cumsum(keep.sum(-1).ravel())])
    Av = (ptr.astype(np.int32), cols[keep].astype(np.int32), vals[keep])
    r1 = np.arange(n1)
    i2, j2 = np.meshgrid(np.arange(nr), np.arange(nth - 1), indexing="ij")
    r2 = (i2 * nth + j2).ravel()
    cols = np.concatenate([np.stack([r1, r1 + nth], -1), np.stack([r2, r2 + 1], -1)])
    k = np.concatenate([k1.ravel(), k2.ravel()])
    vals = np.stack([-k, k], -1)
    As = (np.arange(0, 2 * k.size + 1, 2, dtype=np.int32), cols.ravel().astype(np.int32), vals.ravel())
    return Av, As


def prepare(case, seed):
    kind = case["kind"]
    if kind == "rank2":
        f64 = case["dtype"] == "f64"
        m = _model(case["kv"], case["ks"], case["M"], case["skew"], seed, rounded=not f64)
        rom = _rom(m, state="f64" if f64 else "f32", ops=case["dtype"], source=case["source"],
                   state_operand=case["operand"])
        st = {"case": case, "rom": rom, "mu": m["mu"]}
        if case["probe"] != "none":
            st["c"] = m["c"].to(rom.torch_dtype).contiguous()
        return st
    if kind == "grouped":
        roms, mus, sizes = [], [], _group_sizes(case)
        for i, (K, M) in enumerate(sizes):
            m = _model(K, K, M, True, seed, salt=1 + i)
            roms.append(_rom(m, state="f32"))
            mus.append(m["mu"])
        # all states in one buffer, so that a program clears them at once
        flat = torch.zeros(sum(2 * K * M for K, M in sizes), dtype=torch.float32, device=DEV)
        Vs, Ss, o = [], [], 0
        for K, M in sizes:
            Vs.append(flat[o:o + K * M].view(M, K))
            Ss.append(flat[o + K * M:o + 2 * K * M].view(M, K))
            o += 2 * K * M
        return {"case": case, "plan": GroupPlan(roms, mus, Vs, Ss), "flat": flat}
    if kind == "adjoint":
        m = _model(case["kv"], case["ks"], case["M"], case["skew"], seed)
        return {"case": case, "rom": _rom(m, state="f32"), "mu": m["mu"], "c": m["c"].to(torch.float32)}
    if kind == "receivers":
        m = _model(case["kv"], case["ks"], case["M"], case["skew"], seed)
        C = _receiver_rows(case, seed)
        return {"case": case, "rom": _rom(m, state="f32"), "mu": m["mu"], "C": C}
    m = _grid(case, seed)
    Av, As = _grid_csr(m)
    fom = Fom(Av, As, m["f"].cpu().numpy().ravel(), m["dt"])
    return {"case": case, "fom": fom, "mu": m["mu"]}


def _receiver_rows(case, seed):
    return torch.randn((case["R"], case["kv"]), generator=_gen(seed, 77), device=DEV, dtype=torch.float32)


# ----------------------------------------------------------------- one call

def run(st):
    case = st["case"]
    kind, n = case["kind"], case["nsteps"]
    if kind == "grouped":
        st["flat"].zero_()
        st["plan"].run(n)
        return {"states": st["flat"]}
    if kind == "fom":
        V, S = st["fom"].zeros(case["M"])
        st["fom"].run(st["mu"], V, S, n)
        return {"V": V, "S": S}
    rom, mu = st["rom"], st["mu"]
    if kind == "adjoint":
        return rom.adjoint(mu, n, st["c"])
    V, S = rom.zeros(case["M"])
    if kind == "receivers":
        out = rom.run_receivers(mu, V, S, n, st["C"])
        return {"V": V, "S": S, "Y": out["Y"], "stats": out["stats"]}
    out = {"V": V, "S": S}
    J = y = None
    if case["probe"] != "none":
        J = out["J"] = torch.zeros(case["M"], dtype=torch.float64, device=DEV)
        if case["probe"] == "Jy":
            y = out["y"] = torch.empty((n, case["M"]), dtype=torch.float64, device=DEV)
    rom.run_rank2(mu, V, S, n, c=st.get("c"), J=J, y=y)
    return out


def work(case):
    kind, n = case["kind"], case["nsteps"]
    if kind == "grouped":
        sizes = _group_sizes(case)
        return {"bytes": sum(8.0 * K * K + 16.0 * K * M for K, M in sizes),
                "flops": sum(4.0 * K * K * M * n for K, M in sizes)}
    if kind == "fom":
        nr, nth, M = case["nr"], case["nth"], case["M"]
        n1 = (nr - 1) * nth + nr * (nth - 1)
        return {"bytes": 16.0 * M * (nr * nth + n1) + 12.0 * 4 * n1, "flops": 2.0 * 4 * n1 * M * n}
    kv, ks, M = case["kv"], case["ks"], case["M"]
    f = 4.0 * kv * ks * M * n
    if kind == "adjoint":
        return {"bytes": 16.0 * kv * ks + 24.0 * M, "flops": 3 * f}
    if kind == "receivers":
        R = case["R"]
        return {"bytes": 8.0 * kv * ks + 8.0 * (kv + ks) * M + 8.0 * n * R * (M + 5),
                "flops": f + 2.0 * kv * R * M * n}
    sb = 8.0 if case["dtype"] == "f64" else 4.0
    ob = {"f64": 8.0, "f32": 4.0, "bf16": 2.0, "fp8": 1.0}[case["dtype"]]
    y = 8.0 * n * M if case["probe"] == "Jy" else 0.0
    return {"bytes": 2 * ob * kv * ks + 2 * sb * (kv + ks) * M + y, "flops": f}


# ------------------------------------------------------------ 64-bit results

def _forcing(source, t, mu):
    if source == "gauss1":
        x = math.pi * (mu * t - 3.0)
        return -math.sqrt(2.0 * math.e) * x * torch.exp(-x * x)
    a = (math.pi * (mu * t - 1.5)) ** 2
    return (1.0 - 2.0 * a) * torch.exp(-a)


def _forcing_dmu(t, mu):
    x = math.pi * (mu * t - 1.5)
    return (4.0 * x ** 3 - 6.0 * x) * torch.exp(-x * x) * (math.pi * t)


def _operators(case, m):
    """The operators as a run of the case's type holds them."""
    A, B = m["A"], m["B"]
    if case["dtype"] == "bf16":
        return (X.to(torch.float32).to(torch.bfloat16).to(torch.float64) for X in (A, B))
    if case["dtype"] == "fp8":
        scale = torch.maximum(A.abs().max(), B.abs().max()).to(torch.float32) / 448.0
        return ((X.to(torch.float32) / scale).to(torch.float8_e4m3fn).to(torch.float32).to(torch.float64)
                * scale.to(torch.float64) for X in (A, B))
    return A, B


def _step(A, B, b, dt, V, S, u):
    V.addmm_(A, S, alpha=dt)
    V.addr_(b, u, alpha=dt)
    S.addmm_(B, V, alpha=dt)


def exact(case, seed):
    kind, n = case["kind"], case["nsteps"]
    if kind == "fom":
        return _exact_fom(case, seed)
    if kind == "grouped":
        parts = []
        for i, (K, M) in enumerate(_group_sizes(case)):
            m = _model(K, K, M, True, seed, salt=1 + i)
            V, S = (torch.zeros((K, M), dtype=torch.float64, device=DEV) for _ in range(2))
            for k in range(n):
                _step(m["A"], m["B"], m["b"], m["dt"], V, S, _forcing("ricker", k * m["dt"], m["mu"]))
            parts += [V.t().reshape(-1), S.t().reshape(-1)]
        return {"states": torch.cat(parts)}
    kv, ks, M = case["kv"], case["ks"], case["M"]
    m = _model(kv, ks, M, case["skew"], seed, rounded=case.get("dtype") != "f64")
    b, c, mu, dt = m["b"], m["c"], m["mu"], m["dt"]
    V = torch.zeros((kv, M), dtype=torch.float64, device=DEV)
    S = torch.zeros((ks, M), dtype=torch.float64, device=DEV)
    if kind == "adjoint":
        return _exact_adjoint(m, V, S, n)
    if kind == "receivers":
        C = _receiver_rows(case, seed).to(torch.float64)
        Y = torch.empty((n, case["R"], M), dtype=torch.float64, device=DEV)
        for k in range(n):
            _step(m["A"], m["B"], b, dt, V, S, _forcing("ricker", k * dt, mu))
            Y[k] = C @ V
        srt = Y.sort(dim=2).values
        rank = [srt[:, :, max(1, -(-p * M // 100)) - 1] for p in (5, 50, 95)]
        mean = Y.mean(dim=2)
        var = ((Y - mean[:, :, None]) ** 2).mean(dim=2)
        # one sample has no spread: nothing to compare a zero variance with
        return {"V": V.t().contiguous(), "S": S.t().contiguous(), "Y": Y, "stats": torch.stack([mean, var] + rank, 2)}
    A, B = _operators(case, m)
    J = torch.zeros(M, dtype=torch.float64, device=DEV)
    y = torch.empty((n, M), dtype=torch.float64, device=DEV) if case["probe"] == "Jy" else None
    for k in range(n):
        _step(A, B, b, dt, V, S, _forcing(case["source"], k * dt, mu))
        if case["probe"] != "none":
            r = c @ V
            J.addcmul_(r, r, value=dt)
            if y is not None:
                y[k] = r
    out = {"V": V.t().contiguous(), "S": S.t().contiguous()}
    if case["probe"] != "none":
        out["J"] = J
    if y is not None:
        out["y"] = y
    return out


def _exact_adjoint(m, V, S, n):
    A, B, b, c, mu, dt = (m[k] for k in ("A", "B", "b", "c", "mu", "dt"))
    M = mu.numel()
    Vt = torch.empty((n + 1,) + tuple(V.shape), dtype=torch.float64, device=DEV)
    St = torch.empty((n + 1,) + tuple(S.shape), dtype=torch.float64, device=DEV)
    J = torch.zeros(M, dtype=torch.float64, device=DEV)
    Vt[0], St[0] = V, S
    for k in range(n):
        _step(A, B, b, dt, V, S, _forcing("ricker", k * dt, mu))
        Vt[k + 1], St[k + 1] = V, S
        r = c @ V
        J.addcmul_(r, r, value=dt)
    dA, dB, dmu = torch.zeros_like(A), torch.zeros_like(B), torch.zeros_like(J)
    p, q = torch.zeros_like(V), torch.zeros_like(S)
    At, Bt = A.t().contiguous(), B.t().contiguous()
    for k in range(n - 1, -1, -1):
        p.addmm_(Bt, q, alpha=dt)
        p.addr_(c, c @ Vt[k + 1], alpha=2.0 * dt)
        dB.addmm_(q, Vt[k + 1].t(), alpha=dt)
        dA.addmm_(p, St[k].t(), alpha=dt)
        dmu.addcmul_(b @ p, _forcing_dmu(k * dt, mu), value=dt)
        q.addmm_(At, p, alpha=dt)
    return {"J": J, "dAvs": dA, "dAsv": dB, "dmu": dmu}


def _exact_fom(case, seed):
    m = _grid(case, seed)
    nr, nth, M = case["nr"], case["nth"], case["M"]
    dt, ir, k1, k2, f = m["dt"], m["ir"][..., None], m["k1"][..., None], m["k2"][..., None], m["f"][..., None]
    V, s1, s2 = (torch.zeros(s + (M,), dtype=torch.float64, device=DEV)
                 for s in ((nr, nth), (nr - 1, nth), (nr, nth - 1)))
    for k in range(case["nsteps"]):
        d = torch.zeros_like(V)
        d[:-1] += s1
        d[1:] -= s1
        d[:, :-1] += s2
        d[:, 1:] -= s2
        V += dt * (ir * d + f * _forcing("ricker", k * dt, m["mu"]))
        s1 += dt * (k1 * (V[1:] - V[:-1]))
        s2 += dt * (k2 * (V[:, 1:] - V[:, :-1]))
    return {"V": V.reshape(nr * nth, M), "S": torch.cat([s1.reshape(-1, M), s2.reshape(-1, M)])}
