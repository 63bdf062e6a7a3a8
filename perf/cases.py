"""The workloads whose speed this framework is judged by, through its public entry points.

Six kinds of work cover what a program does with the library:
  heff     one application of the two-site effective Hamiltonian (FP64, or the FP32-operator form) on
           the caller's environments: the inner step of an external eigensolver;
  svd      truncated SVDs of two-site matrices, single or a uniform batch, FP64 or FP32 in and out;
  visit    a bond visited back and forth at fixed chi with a fixed number of matvecs: the step whose
           rate the benchmark quotes;
  sweep    a full sweep of one chain under the PID controller, Lanczos to its tolerance;
  batch    a sweep of many chains in lockstep;
  circuit  one ansatz layer (two gate layers) of a circuit at its bond-dimension cap, and the state
           read back.
listed() names one or more sizes of each, draw() takes sizes from the same ranges."""
import math

import numpy as np
import torch

import paper_2604_03960_amd as tna
import synth

PID_GAINS = (2.0, 0.1, 0.5)  # the Heisenberg gains
MODELS = {"heisenberg": (tna.MODEL_XXZ, [1.0, 1.0, 0.0], 5), "j1j2": (tna.MODEL_J1J2, [1.0, 0.241], 8),
          "tfim": (tna.MODEL_TFIM, [1.0, 1.0], 3)}
EXACT_SVD_ROWS = 1100  # above this a 64-bit library SVD on the host takes too long to wait for


def listed():
    return [
        # a short bond (chi held at its lower bound): launches and latency
        {"name": "heff_chi16", "kind": "heff", "chi_l": 16, "chi_r": 16, "model": "heisenberg", "prec": "f64"},
        # a bond of an adaptive run: odd and unequal dimensions, the J1-J2 chain's wider MPO
        {"name": "heff_ragged_j1j2", "kind": "heff", "chi_l": 203, "chi_r": 331, "model": "j1j2", "prec": "f64"},
        # the FP32-operator form at a middle size
        {"name": "heff_chi512_f32", "kind": "heff", "chi_l": 512, "chi_r": 512, "model": "heisenberg", "prec": "f32"},
        # the largest bond: the headline's own product
        {"name": "heff_chi2048", "kind": "heff", "chi_l": 2048, "chi_r": 2048, "model": "heisenberg", "prec": "f64"},
        # two-site matrices of many chains at chi = 16, one batched call
        {"name": "svd_32_batch64", "kind": "svd", "m": 32, "n": 32, "batch": 64, "keep": 16, "tau": 8.0,
         "dtype": "f64"},
        # a bond between two of unequal dimension, odd sizes
        {"name": "svd_517x331", "kind": "svd", "m": 517, "n": 331, "batch": 1, "keep": 166, "tau": 64.0,
         "dtype": "f64"},
        # chi = 256, the grid's batch of 16, FP32 in and out
        {"name": "svd_512_batch16_f32", "kind": "svd", "m": 512, "n": 512, "batch": 16, "keep": 256, "tau": 64.0,
         "dtype": "f32"},
        # chi = 2048, the largest matrix the library takes
        {"name": "svd_4096", "kind": "svd", "m": 4096, "n": 4096, "batch": 1, "keep": 2048, "tau": 512.0,
         "dtype": "f64"},
        # fixed-chi throughput mode at a centre bond, 20 matvecs a visit
        {"name": "visit_chi512", "kind": "visit", "N": 20, "chi": 512, "matvecs": 20, "model": "heisenberg"},
        # the adaptive run at its lower bound: short bonds all along the chain
        {"name": "sweep_n32_pid", "kind": "sweep", "N": 32, "chi_min": 16, "chi_max": 64, "model": "heisenberg"},
        # many chains in lockstep
        {"name": "batch_16_chains", "kind": "batch", "chains": 16, "n_min": 16, "n_max": 32, "chi_min": 8,
         "chi_max": 64},
        # a hardware-efficient ansatz at its cap: one group of SVDs per gate layer
        {"name": "circuit_n32_chi64", "kind": "circuit", "N": 32, "chi": 64},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["heff", "heff", "heff", "svd", "svd", "svd", "visit", "sweep", "batch", "circuit"])
    if kind == "heff":
        model = rng.choice(["heisenberg", "heisenberg", "j1j2", "tfim"])
        top = 2048 if model == "heisenberg" else 1100
        chi_l = _log_int(rng, 3, top)
        chi_r = max(1, min(top, int(chi_l * math.exp(rng.uniform(-0.7, 0.7)))))
        return {"kind": kind, "chi_l": chi_l, "chi_r": chi_r, "model": model,
                "prec": rng.choice(["f64", "f64", "f64", "f32"])}
    if kind == "svd":
        m = _log_int(rng, 7, 1400)
        n = max(4, min(1400, int(m * math.exp(rng.uniform(-0.5, 0.5)))))
        r = min(m, n)
        batch = rng.choice([1, 1, 1 + rng.randrange(24)])
        if batch * m * n > 16 * 512 * 512:
            batch = 1
        return {"kind": kind, "m": m, "n": n, "batch": batch, "keep": max(1, r // 2),
                "tau": round(rng.uniform(0.12, 0.3) * r + 1.0, 3), "dtype": rng.choice(["f64", "f64", "f32"])}
    if kind == "visit":
        return {"kind": kind, "N": 2 * rng.randrange(8, 11), "chi": _log_int(rng, 48, 512),
                "matvecs": rng.randrange(8, 21), "model": rng.choice(["heisenberg", "tfim"])}
    if kind == "sweep":
        chi_min = rng.randrange(4, 17)
        return {"kind": kind, "N": _log_int(rng, 12, 64), "chi_min": chi_min, "chi_max": 64,
                "model": rng.choice(["heisenberg", "heisenberg", "tfim"])}
    if kind == "batch":
        return {"kind": kind, "chains": _log_int(rng, 3, 48), "n_min": 12, "n_max": rng.randrange(16, 33),
                "chi_min": rng.randrange(6, 13), "chi_max": 64}
    return {"kind": kind, "N": _log_int(rng, 10, 40), "chi": _log_int(rng, 8, 64)}


# ------------------------------------------------------------------ inputs
def _generator(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + stream)
    return g


def _randn(seed, stream, *shape):
    return torch.randn(*shape, dtype=torch.float64, device="cuda", generator=_generator(seed, stream))


def _mpo_pair(case):
    model, params, D = MODELS[case["model"]]
    W = torch.from_numpy(tna.mpo_build(model, 2, params)).cuda()
    return W[0].contiguous(), W[1].contiguous(), D


def _heff_inputs(case, seed):
    cl, cr = case["chi_l"], case["chi_r"]
    W1, W2, D = _mpo_pair(case)
    # environments are symmetric under the exchange of bra and ket; a two-site tensor has unit norm
    L = _randn(seed, 1, cl, D, cl)
    R = _randn(seed, 2, cr, D, cr)
    L = (0.5 * (L + L.permute(2, 1, 0))).contiguous()
    R = (0.5 * (R + R.permute(2, 1, 0))).contiguous()
    theta = _randn(seed, 3, cl, 2, 2, cr)
    return L, W1, W2, R, (theta / theta.norm()).contiguous()


def _svd_input(case, seed):
    """Two-site matrices with the spectrum exp(-k / tau) and Haar-distributed factors."""
    b, m, n = case["batch"], case["m"], case["n"]
    r = min(m, n)
    q = []
    for stream, rows in ((4, m), (5, n)):
        u, t = torch.linalg.qr(_randn(seed, stream, b, rows, r))
        q.append(u * torch.sign(torch.diagonal(t, dim1=-2, dim2=-1))[:, None, :])
    s = torch.exp(-torch.arange(r, dtype=torch.float64, device="cuda") / case["tau"])
    A = torch.stack([(q[0][i] * s) @ q[1][i].T.contiguous() for i in range(b)])
    return (A if case["dtype"] == "f64" else A.float()).contiguous()


def _chain_lengths(case):
    c, lo, hi = case["chains"], case["n_min"], case["n_max"]
    return [lo + (i * (hi - lo)) // max(1, c - 1) for i in range(c)]


def prepare(case, seed):
    kind = case["kind"]
    ctx = tna.Context(0)
    st = {"case": case, "ctx": ctx}
    if kind == "heff":
        st["L"], st["W1"], st["W2"], st["R"], st["theta"] = _heff_inputs(case, seed)
        st["out"] = torch.empty_like(st["theta"])
        st["prec"] = tna.HEFF_F64 if case["prec"] == "f64" else tna.HEFF_F32
    elif kind == "svd":
        A = _svd_input(case, seed)
        st["A"] = A[0].contiguous() if case["batch"] == 1 else A
    elif kind == "visit":
        model, params, _ = MODELS[case["model"]]
        W = tna.mpo_build(model, case["N"], params)
        A, chi, _ = synth.random_mps(case["N"], 2, case["chi"], seed)
        dm = tna.Dmrg(ctx, W, A, chi, tna.pid_params(*PID_GAINS, 1.0, 0.3, 16, case["chi"]),
                      fixed_iters=case["matvecs"], fixed_chi=case["chi"])
        st["bond"] = case["N"] // 2 - 1
        for b in range(st["bond"]):
            dm.visit(b, 0)
        for h in (0, 1, 0, 1):  # settled, as the benchmark's own warm-up leaves it
            dm.visit(st["bond"], h)
        st["dm"] = dm
    elif kind == "sweep":
        model, params, _ = MODELS[case["model"]]
        W = tna.mpo_build(model, case["N"], params)
        A, chi, _ = synth.random_mps(case["N"], 2, case["chi_min"], seed)
        st["dm"] = tna.Dmrg(ctx, W, A, chi, tna.pid_params(*PID_GAINS, 1.0, 0.3, case["chi_min"], case["chi_max"]))
    elif kind == "batch":
        lens = _chain_lengths(case)
        fields = 1.0 + synth.uniform53(seed, 0, len(lens))  # transverse fields of the disordered-phase chains
        Ws = [tna.mpo_build(tna.MODEL_TFIM, n, [1.0, float(h)]) for n, h in zip(lens, fields)]
        mps = [synth.random_mps(n, 2, case["chi_min"], seed * 1000 + i) for i, n in enumerate(lens)]
        st["bt"] = tna.DmrgBatch(ctx, Ws, [a for a, _, _ in mps], [c for _, c, _ in mps],
                                 tna.pid_params(*PID_GAINS, 1.0, 0.3, case["chi_min"], case["chi_max"]))
    else:
        N, chi = case["N"], case["chi"]
        layers = int(math.ceil(math.log2(chi))) + 2
        par, gates, _ = synth.hea_circuit(N, layers + 1, seed)
        gates = np.ascontiguousarray(gates, dtype=np.float64).reshape(-1, 16)
        c = tna.Circuit(ctx, N, tna.pid_params(*PID_GAINS, 1.0, 0.3, 4, chi), fixed_chi=chi)
        per = [len(range(p, N - 1, 2)) for p in par]
        cut = sum(per[:-2])
        c.run(par[:-2], gates[:cut])  # the cap is reached before the layer that is timed
        st["circuit"], st["par"], st["gates"] = c, par[-2:], gates[cut:].copy()
    return st


# ------------------------------------------------------------------ one pass
VISIT_INTS = ("m", "n", "k", "chi_ctrl")
VISIT_FLOATS = ("E", "S", "S_ema", "eps", "wdisc", "sigma0", "P", "I", "D", "u")
GATE_FLOATS = ("S", "S_ema", "eps", "wdisc", "sigma0", "u")


def _records(recs, floats, ints):
    return {"values": np.array([[r[f] for f in floats] for r in recs]),
            "ranks": np.array([[r[f] for f in ints] for r in recs], dtype=np.int64)}


def run(state):
    kind, ctx = state["case"]["kind"], state["ctx"]
    if kind == "heff":
        return ctx.heff_apply(state["L"], state["W1"], state["W2"], state["R"], state["theta"], state["prec"],
                              out=state["out"])
    if kind == "svd":
        keep = state["case"]["keep"]
        if state["case"]["batch"] == 1:
            S, U, Vt, spec, k, _, status = ctx.svd_truncate(state["A"], keep)
        else:
            S, U, Vt, spec, _, status = ctx.svd_truncate_batched(state["A"], keep)
        return {"S": S, "U": U, "Vt": Vt, "spec": spec, "status": status}
    if kind == "visit":
        dm, b = state["dm"], state["bond"]
        E0, r0, s0 = dm.visit(b, 0)
        E1, r1, s1 = dm.visit(b, 1)
        return {"E": np.array([E0, E1]), "status": [s0, s1], **_records([r0, r1], VISIT_FLOATS, VISIT_INTS)}
    if kind == "sweep":
        E, recs, status = state["dm"].sweep()
        chi, _ = state["dm"].state()
        return {"E": E, "status": status, "chi": chi, **_records(recs, VISIT_FLOATS, VISIT_INTS)}
    if kind == "batch":
        E, per, _, status = state["bt"].sweep()
        return {"E": E, "status": status,
                **_records([r for recs in per for r in recs], VISIT_FLOATS, VISIT_INTS)}
    chi_map, recs = state["circuit"].run(state["par"], state["gates"])
    sites, chi = state["circuit"].mps()
    return {"map": chi_map, "sites": sites, "chi": chi, **_records(recs, GATE_FLOATS, VISIT_INTS)}


# ------------------------------------------------------------------ work and exact values
def _heff_work(cl, cr, D):
    flops = 2.0 * D * 4 * cl * cr * (cl + cr) + 2.0 * (4 * D) ** 2 * cl * cr
    return 8.0 * (D * cl * cl + D * cr * cr + 8 * cl * cr + 8 * D * D), flops


def _svd_work(m, n, k):
    r, c = min(m, n), max(m, n)
    # bidiagonalisation and k vectors of each side
    return 8.0 * (m * n + r + m * k + k * n), 4.0 * r * r * (c - r / 3.0) + 4.0 * r * k * (m + n) / 2.0


def _visit_work(cl, cm, cr, D, matvecs, k):
    by, fl = _heff_work(cl, cr, D)
    sb, sf = _svd_work(2 * cl, 2 * cr, k)
    basis = 8.0 * 4 * cl * cr * matvecs  # every Krylov vector written once
    env = 2.0 * 2 * D * cl * k * (cl + k)
    return by + sb + basis, 8.0 * cl * cm * cr + matvecs * fl + sf + env


def work(case):
    kind = case["kind"]
    if kind == "heff":
        by, fl = _heff_work(case["chi_l"], case["chi_r"], MODELS[case["model"]][2])
    elif kind == "svd":
        by, fl = _svd_work(case["m"], case["n"], case["keep"])
        by *= case["batch"] * (1.0 if case["dtype"] == "f64" else 0.5)
        fl *= case["batch"]
    elif kind == "visit":
        c = [min(case["chi"], 2 ** j) for j in (case["N"] // 2 - 1, case["N"] // 2)]
        by, fl = _visit_work(c[0], c[1], c[0], MODELS[case["model"]][2], case["matvecs"], c[1])
        by, fl = 2 * by, 2 * fl
    elif kind in ("sweep", "batch"):
        by = fl = 0.0
        lens = [case["N"]] if kind == "sweep" else _chain_lengths(case)
        D = MODELS[case["model"]][2] if kind == "sweep" else MODELS["tfim"][2]
        for n in lens:
            dims = [1] + synth.initial_bond_dims(n, 2, case["chi_min"]) + [1]
            for b in range(n - 1):
                x, y = _visit_work(dims[b], dims[b + 1], dims[b + 2], D, 8, dims[b + 1])
                by, fl = by + 2 * x, fl + 2 * y
    else:
        dims = [1] + synth.initial_bond_dims(case["N"], 2, case["chi"]) + [1]
        by = fl = 0.0
        for b in range(case["N"] - 1):
            cl, cm, cr = dims[b], dims[b + 1], dims[b + 2]
            x, y = _svd_work(2 * cl, 2 * cr, cm)
            by, fl = by + x, fl + y + 8.0 * cl * cm * cr * 2
    return {"bytes": by, "flops": fl}


def _gauge(U, Vt):
    """The largest-magnitude entry of every column of U positive."""
    i = np.abs(U).argmax(axis=0)
    sg = np.where(U[i, np.arange(U.shape[1])] < 0, -1.0, 1.0)
    return U * sg, Vt * sg[:, None]


def exact(case, seed):
    if case["kind"] == "heff":
        L, W1, W2, R, theta = _heff_inputs(case, seed)
        cl, cr = case["chi_l"], case["chi_r"]
        D = L.shape[1]
        M = torch.tensordot(W1, W2, dims=([1], [0]))  # [w][s][s'][w''][t][t']
        M = M.permute(1, 4, 3, 0, 2, 5).reshape(4 * D, 4 * D)  # [(s,t,w'')][(w,s',t')]
        X = (L.reshape(cl * D, cl) @ theta.reshape(cl, 4 * cr)).reshape(cl, 4 * D, cr)
        Z = (M @ X.permute(1, 0, 2).reshape(4 * D, cl * cr)).reshape(4 * D, cl, cr)
        Z = Z.permute(1, 0, 2).reshape(cl * 4, D * cr).contiguous()
        return (Z @ R.reshape(cr, D * cr).T.contiguous()).reshape(cl, 2, 2, cr)
    if case["kind"] == "svd" and min(case["m"], case["n"]) <= EXACT_SVD_ROWS:
        A = _svd_input(case, seed).double().cpu().numpy()
        k = min(case["keep"], case["m"], case["n"])
        S, U, V, P = [], [], [], []
        for a in A:
            u, s, v = np.linalg.svd(a, full_matrices=False)
            u, v = _gauge(u[:, :k], v[:k])
            z, tail = np.sum(s * s), np.sum(s[k:] ** 2)
            p = s * s / z
            gap = (s[k - 1] - s[k]) / s[0] if k < len(s) else 1.0
            S.append(s), U.append(u), V.append(v)
            P.append([z, -np.sum(p * np.log(p)), math.sqrt(tail), tail / z, math.sqrt(np.sum(s[:k] ** 2)), gap])
        got = {"S": np.stack(S), "U": np.stack(U), "Vt": np.stack(V), "spec": np.array(P)}
        if case["batch"] == 1:
            got = {n: v[0] for n, v in got.items()}
        return {**got, "status": None}
    return None
