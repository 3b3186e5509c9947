"""Performance cases of the IC-D2S hot path: what a solver run asks of the library.

A run of the method alternates Tabu search, control-parameter selection, the
batched annealer on the extracted sub-QUBOs and the write-back with its field
update; the learned selector adds feature scoring and a training step.  Each
case calls one of these stages (or a whole short run) through the package's
public calls on synthetic instances, with the state that the stage meets in a
run: solutions after a Tabu pass, sub-QUBOs of the best-ranked variables.

``listed()`` names the cases, ``draw(rng)`` gives another one of the same
ranges, ``prepare(case, seed)`` builds inputs and handles on the GPU,
``run(state)`` is one pass, ``work(case)`` what the pass cannot do without
and ``exact(case, seed)`` the values in 64 bits where the outputs have a
closed form.  The searches (Tabu, annealer, whole runs) return whole numbers
that only the sequential search itself defines, so they have none.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2502_13947_amd import inputs, qb
from paper_2502_13947_amd.solver import Solver, default_thresholds, feature_scales

THR_BITS = 10   # bits of the acceptance table's index, as the benchmark uses
NSW_PREP = 64   # sweeps of the acceptance table of the initial pass in whole runs


def listed():
    return [
        # a whole short run at the paper's own solution count (Table 1: z = 4): the initial pass block after block,
        # then two outer iterations; small launches and one search's latency, the chip nearly empty
        dict(name="run_n2500_z4", kind="run", n=2500, density=0.1, lim=100, z=4, k=4, m_lo=128, m_hi=128, R=1, nsw=200,
             init_m=128, iters=2),
        # Alg. 1 on the fully dense n = 7000 workload, a solution for every compute unit
        dict(name="tabu_n7000_z256", kind="tabu", n=7000, density=1.0, lim=100, z=256),
        # Alg. 1 on the large sparse workload, alpha = 5 n = 100,000 steps
        dict(name="tabu_sparse_n20000_z16", kind="tabu", n=20000, sparse=True, z=16),
        # the smallest annealer call: 16 sub-QUBOs of 128 (the n = 2500 workload)
        dict(name="anneal_n2500_m128", kind="anneal", n=2500, density=0.1, lim=100, z=4, k=4, m_lo=128, m_hi=128,
             R=1, nsw=200),
        # one sub-QUBO of 512 per solution, the n = 5000 workload's annealer call
        dict(name="anneal_n5000_m512", kind="anneal", n=5000, density=0.5, lim=100, z=256, k=1, m_lo=512, m_hi=512,
             R=1, nsw=1000),
        # uneven batch: four sub-QUBOs of 128 to 1024 per solution, the n = 7000 workload's annealer call
        dict(name="anneal_n7000_mixed", kind="anneal", n=7000, density=1.0, lim=100, z=256, k=4, m_lo=128, m_hi=1024,
             R=1, nsw=1000),
        # couplings beyond int8, ragged sizes, several replicas a job
        dict(name="anneal_n1003_int16_r4", kind="anneal", n=1003, density=0.5, lim=1000, z=16, k=3, m_lo=100, m_hi=300,
             R=4, nsw=300),
        # sparse sub-QUBOs of 1024 with 16 replicas, the n = 20000 workload's annealer call
        dict(name="anneal_ell_n20000_r16", kind="anneal", n=20000, sparse=True, z=16, k=8, m_lo=1024, m_hi=1024, R=16,
             nsw=1000),
        # Alg. 4 keys, ranking, selection and extraction on the large sparse workload
        dict(name="select_sparse_n20000", kind="select", n=20000, sparse=True, z=16, k=8, m_lo=1024, m_hi=1024),
        # write-back, field update, energy and best of the n = 7000 workload
        dict(name="apply_n7000_z256", kind="apply", n=7000, density=1.0, lim=100, z=256, k=4, m_lo=128, m_hi=1024),
        # the learned selector's forward path: features, MLP scores and their order
        dict(name="learned_n7000_z256", kind="learned", n=7000, density=1.0, lim=100, z=256),
        # the learned selector's training step (gradient and Adam) at the trainer's batch size
        dict(name="train_b4096", kind="train", batch=4096),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_instance(rng, n_hi=7000, sparse_hi=20000):
    if rng.random() < 0.35:
        return dict(n=_log_int(rng, 400, sparse_hi), sparse=True)
    return dict(n=_log_int(rng, 100, n_hi), density=rng.choice([0.1, 0.5, 1.0]), lim=rng.choice([100, 100, 1000]))


def _draw_jobs(rng, c, k_hi=4):
    k = rng.randint(1, k_hi)
    m_hi = _log_int(rng, 16, min(1024, c["n"] // k))
    return dict(k=k, m_lo=rng.randint(max(1, m_hi // 8), m_hi), m_hi=m_hi)


def draw(rng):
    """One more case of the listed ones' ranges."""
    kind = rng.choice(["tabu", "tabu", "anneal", "anneal", "anneal", "select", "apply", "learned", "train", "run"])
    if kind == "train":
        return dict(kind=kind, batch=_log_int(rng, 64, 8000))
    if kind == "learned":
        return dict(kind=kind, n=_log_int(rng, 500, 7000), density=rng.choice([0.1, 0.5, 1.0]), lim=100,
                    z=_log_int(rng, 4, 256))
    if kind == "run":
        n = _log_int(rng, 200, 2500)
        return dict(kind=kind, n=n, density=rng.choice([0.1, 0.5]), lim=100, z=_log_int(rng, 1, 16), k=2, m_lo=n // 20,
                    m_hi=n // 10, R=rng.choice([1, 2]), nsw=rng.randint(20, 200), init_m=min(n // 2, 128),
                    iters=rng.randint(1, 3))
    c = dict(kind=kind, **_draw_instance(rng))
    c["z"] = _log_int(rng, 1, 16 if c.get("sparse") else 256)
    if kind == "tabu":
        return c
    c.update(_draw_jobs(rng, c))
    if kind == "anneal":
        c["R"] = rng.choice([1, 1, 2, 3, 4, 8, 16])
        # at most the sparse workload's replicas in flight, and the dense one's attempts
        jobs = max(1, min(c["z"], (2048 if c.get("sparse") else 1024) // (c["k"] * c["R"])))
        c["z"] = jobs
        c["nsw"] = _log_int(rng, 50, 1000 if c["R"] == 1 or c.get("sparse") else 300)
    return c


# ------------------------------------------------------------------ inputs
def _instance(case, seed, dev):
    """The problem handle and, for a dense one, Q."""
    if case.get("sparse"):
        cols = max(4, int(round(math.sqrt(2.0 * case["n"]))))
        rows = max(4, case["n"] // cols)
        return qb.Problem.from_csr(*inputs.torus_graph_qubo(rows, cols, 4.0, seed), device=dev), None
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    n, lim = case["n"], case["lim"]
    Q = torch.randint(-lim, lim + 1, (n, n), generator=g, device=dev, dtype=torch.int16)
    if case["density"] < 1.0:
        Q *= torch.rand((n, n), generator=g, device=dev) < case["density"]
    Q = torch.triu(Q)
    Q = (Q + torch.triu(Q, 1).T).contiguous()
    return qb.Problem(Q), Q


def _solutions(P, z, seed, dev, alpha):
    """Random solutions with their fields and energies, after `alpha` Tabu
    steps (0: as drawn), with the flip statistics."""
    n = P.n
    X = torch.zeros((z, n), dtype=torch.uint8, device=dev)
    H = torch.zeros((z, n), dtype=torch.int32, device=dev)
    E = torch.zeros(z, dtype=torch.int64, device=dev)
    T, LF = torch.zeros_like(H), torch.zeros_like(H)
    qb.init_solutions(n, z, seed, X)
    qb.field(P, X, H)
    qb.energy(X, H, E)
    if alpha:
        qb.tabu(P, X, H, E, alpha, _tenure(n), True, T, LF)
    return X, H, E, T, LF


def _tenure(n):
    return max(1, n // 150)


def _sizes(case):
    """[z, k] job sizes: part of the case, the same for every seed."""
    seed = case["z"]
    rng = np.random.Generator(np.random.PCG64(seed))
    lo, hi = case["m_lo"], case["m_hi"]
    if lo == 128 and hi == 1024:   # the n = 7000 workload's sizes
        return inputs.job_sizes(case["z"], case["k"], (128, 256, 512, 1024), seed)
    return rng.integers(lo, hi + 1, size=(case["z"], case["k"])).astype(np.int32)


def _selected(case, seed, dev):
    """A solution set after a short Tabu pass and the batch of its
    best-ranked sub-QUBOs."""
    P, Q = _instance(case, seed, dev)
    z, n = case["z"], P.n
    st = dict(P=P, Q=Q, n=n, alpha=n)
    st["X"], st["H"], st["E"], st["T"], st["LF"] = _solutions(P, z, seed + 1, dev, st["alpha"])
    job_m = _sizes(case)
    b = st["b"] = qb.Batch(n, z, np.repeat(np.arange(z, dtype=np.int32), case["k"]), job_m.reshape(-1))
    st["K"] = torch.zeros((z, n), dtype=torch.int64, device=dev)
    st["order"] = torch.zeros((z, n), dtype=torch.int32, device=dev)
    words = qb.ell_tile_words(b, P.ell_width) if P.sparse else max(b.tile_elems, 16)
    st["tiles"] = torch.zeros(words, dtype=torch.int32 if P.sparse else qb.tile_dtype(P), device=dev)
    st["F0"] = torch.zeros(b.total, dtype=torch.int32, device=dev)
    st["y0"] = torch.zeros(b.total, dtype=torch.uint8, device=dev)
    return st


def _select(st):
    P, b = st["P"], st["b"]
    qb.keys(P, st["X"], st["T"], st["K"], t_bound=st["alpha"])
    qb.rank(st["K"], st["order"])
    qb.select(b, st["order"])
    (qb.extract_ell if P.sparse else qb.extract)(P, b, st["X"], st["H"], st["tiles"], st["F0"], st["y0"])


def _anneal(st):
    b = st["b"]
    if st["P"].sparse:
        qb.anneal_ell(b, st["P"].ell_width, st["tiles"], st["F0"], st["y0"], st["thr"], st["R"], st["seed"], 0,
                      st["Y"], st["e"], THR_BITS)
    else:
        qb.anneal(b, st["tiles"], st["F0"], st["y0"], st["thr"], st["R"], st["seed"], 0, st["Y"], st["e"], THR_BITS)


def _annealer(st, case, seed, dev):
    b, R = st["b"], case.get("R", 1)
    st.update(R=R, seed=seed + 3, Y=torch.zeros(b.total * R, dtype=torch.uint8, device=dev),
              e=torch.zeros(b.J * R, dtype=torch.int64, device=dev),
              thr=torch.as_tensor(default_thresholds(st["P"], case.get("nsw", 20), THR_BITS), device=dev))


def prepare(case, seed):
    dev = torch.device("cuda")
    kind = case["kind"]
    if kind == "train":
        g = torch.Generator(device=dev)
        g.manual_seed(seed)
        n = case["batch"]
        f = torch.randn((n, 8), generator=g, device=dev)
        f[:, 5:] = torch.rand((n, 3), generator=g, device=dev)   # eta, gamma and Delta lie in [0, 1]
        st = dict(feat=f.to(torch.bfloat16).view(torch.int16),
                  label=(torch.rand(n, generator=g, device=dev) < 0.05).to(torch.uint8), t=0,
                  master=torch.zeros(qb.NPARAM, device=dev), W=torch.zeros(qb.NPARAM, dtype=torch.int16, device=dev),
                  loss=torch.zeros(1, device=dev),
                  work=torch.zeros(qb.mlp_train_workspace(n), dtype=torch.uint8, device=dev))
        qb.mlp_init(seed, st["master"], st["W"])
        st.update({k: torch.zeros_like(st["master"]) for k in ("grad", "m", "v")})
    elif kind == "run":
        P, Q = _instance(case, seed, dev)
        thr = default_thresholds(P, case["nsw"], THR_BITS)
        n = case["n"]
        st = dict(solver=Solver(Q, z=case["z"], seed=seed + 1, job_m=_sizes(case), init_m=case["init_m"],
                                thr_init=default_thresholds(P, NSW_PREP, THR_BITS), thr=thr, B=THR_BITS, R=case["R"],
                                alpha=5 * n, tenure=_tenure(n)), iters=case["iters"])
    elif kind == "tabu":
        P, Q = _instance(case, seed, dev)
        X, H, E, T, LF = _solutions(P, case["z"], seed + 1, dev, 0)
        st = dict(P=P, Q=Q, n=P.n, start=(X.clone(), H.clone(), E.clone()), X=X, H=H, E=E, T=T, LF=LF)
    elif kind == "learned":
        P, Q = _instance(case, seed, dev)
        z, n = case["z"], P.n
        X, H, E, T, LF = _solutions(P, z, seed + 1, dev, n)
        master, W = torch.zeros(qb.NPARAM, device=dev), torch.zeros(qb.NPARAM, dtype=torch.int16, device=dev)
        qb.mlp_init(seed, master, W)
        g = torch.Generator(device=dev)
        g.manual_seed(seed)
        G = torch.randint(0, max(2, int(P.sigma)), (z, n), generator=g, device=dev, dtype=torch.int32)
        G *= torch.rand((z, n), generator=g, device=dev) < 0.1
        st = dict(P=P, Q=Q, X=X, H=H, T=T, LF=LF, G=G, W=W, alpha=n, scales=feature_scales(P, n, z),
                  F=torch.zeros((z, n, 8), dtype=torch.int16, device=dev),
                  score=torch.zeros((z, n), device=dev), K=torch.zeros((z, n), dtype=torch.int64, device=dev),
                  order=torch.zeros((z, n), dtype=torch.int32, device=dev))
    else:
        st = _selected(case, seed, dev)
        if kind != "select":
            _select(st)
            _annealer(st, case, seed, dev)
        if kind == "apply":
            _anneal(st)
            z, n = case["z"], st["n"]
            st.update(start=(st["X"].clone(), st["H"].clone()), dX=torch.zeros((z, n), dtype=torch.int8, device=dev),
                      ebest=torch.zeros(1, dtype=torch.int64, device=dev), ej=torch.zeros_like(st["e"][:st["b"].J]),
                      xbest=torch.zeros(n, dtype=torch.uint8, device=dev))
    st["kind"] = kind
    return st


# ------------------------------------------------------------------ one pass
def run(st):
    kind = st["kind"]
    if kind == "tabu":
        # every pass searches from the kept start
        for a, b in zip((st["X"], st["H"], st["E"]), st["start"]):
            a.copy_(b)
        qb.tabu(st["P"], st["X"], st["H"], st["E"], 5 * st["n"], _tenure(st["n"]), True, st["T"], st["LF"])
        return {k: st[k] for k in ("X", "H", "E", "T", "LF")}
    if kind == "anneal":
        _anneal(st)
        return {"Y": st["Y"], "e": st["e"]}
    if kind == "select":
        _select(st)
        return {k: st[k] for k in ("K", "order", "tiles", "F0", "y0")}
    if kind == "apply":
        for a, b in zip((st["X"], st["H"]), st["start"]):
            a.copy_(b)
        st["ebest"].fill_(2**63 - 1)
        qb.zero(st["dX"])
        qb.writeback(st["b"], st["R"], st["Y"], st["e"], st["y0"], st["X"], st["dX"], st["ej"])
        qb.rankk(st["P"], st["dX"], st["H"])
        qb.energy(st["X"], st["H"], st["E"])
        qb.best(st["X"], st["E"], st["ebest"], st["xbest"])
        return {k: st[k] for k in ("X", "dX", "H", "E", "ebest", "xbest", "ej")}
    if kind == "learned":
        qb.features(st["P"], st["X"], st["H"], st["T"], st["LF"], st["G"], st["alpha"], st["scales"], st["F"])
        qb.mlp_score(st["F"], st["W"], st["K"], st["score"])
        qb.rank(st["K"], st["order"])
        return {k: st[k] for k in ("F", "score", "K", "order")}
    if kind == "train":
        st["t"] += 1
        qb.mlp_grad(st["feat"], st["label"], st["W"], st["grad"], st["loss"], st["work"])
        qb.mlp_adam(st["grad"], st["master"], st["m"], st["v"], st["t"], 2e-3, st["W"])
        return {k: st[k] for k in ("loss", "grad", "master", "m", "v", "W")}
    S = st["solver"]
    trace = S.run(st["iters"])
    return {"trace": trace, "X": S.X, "H": S.H, "E": S.E, "ebest": S.ebest, "xbest": S.xbest}


# ------------------------------------------------------------------ what a pass needs
def work(case):
    """Inputs read once and outputs written once; operations: a Tabu step is a
    multiply-add and a comparison on every move value (on the flipped row's
    entries and one comparison for the argmin's tree on a sparse problem), an
    annealer attempt a quarter of a Philox call (80 operations) and 3 more."""
    kind = case["kind"]
    if kind == "train":
        b = case["batch"]
        return {"bytes": b * 17 + qb.NPARAM * 28, "flops": 6 * b * 4672}
    n, z = case["n"], case["z"]
    esz = 2 if case.get("lim", 100) > 127 else 1
    q = n * 20 * 4 if case.get("sparse") else n * n * esz
    per_step = 3 * 8 + 15 if case.get("sparse") else 3 * n
    m = case.get("k", 0) * (case.get("m_lo", 0) + case.get("m_hi", 0)) // 2   # mean variables of a solution's jobs
    tile = 0
    if m:
        tile = z * m * 80 if case.get("sparse") else z * m * esz * (case["m_lo"] + case["m_hi"]) // 2
    if kind == "tabu":
        return {"bytes": q + z * n * 18, "flops": z * 5 * n * per_step}
    if kind == "anneal":
        return {"bytes": tile + z * m * (5 + case["R"]) + case["nsw"] * 4096, "flops": 23 * z * m * case["R"] * case["nsw"]}
    if kind == "select":
        return {"bytes": z * n * 17 + q + 2 * tile, "flops": z * n * (8 + 2 * math.log2(n))}
    if kind == "apply":
        return {"bytes": q + z * n * 12, "flops": 2 * z * n * n}
    if kind == "learned":
        return {"bytes": z * n * (17 + 16 + 12 + 4), "flops": 2 * z * n * 4672}
    it = case["iters"]
    return {"bytes": q + z * n * 18,
            "flops": it * (z * 5 * n * per_step + 23 * z * m * case["R"] * case["nsw"]) + 23 * z * n * NSW_PREP}


# ------------------------------------------------------------------ 64-bit values
def _unpack(W):
    w = W.view(torch.bfloat16).double()
    return (w[:512].view(64, 8), w[512:576], w[576:4672].view(64, 64), w[4672:4736], w[4736:4800], w[4800])


def _bf16(x):
    return x.float().to(torch.bfloat16).double()


def _forward(f, W):
    W1, b1, W2, b2, W3, b3 = _unpack(W)
    h1 = _bf16(torch.relu(f @ W1.T + b1))
    h2 = _bf16(torch.relu(h1 @ W2.T + b2))
    return h1, h2, h2 @ W3 + b3


def exact(case, seed):
    kind = case["kind"]
    if kind not in ("train", "learned", "apply", "select"):
        return None
    st = prepare(case, seed)
    if kind == "train":
        f = st["feat"].view(torch.bfloat16).double()
        y = st["label"].double()
        _, _, W2, _, W3, _ = _unpack(st["W"])
        h1, h2, s = _forward(f, st["W"])
        loss = torch.nn.functional.softplus(s) - y * s
        ds = (torch.sigmoid(s) - y) / len(y)
        d2 = ds[:, None] * W3 * (h2 > 0)
        d1 = (d2 @ W2) * (h1 > 0)
        grad = torch.cat([(d1.T @ f).reshape(-1), d1.sum(0), (d2.T @ h1).reshape(-1), d2.sum(0), ds @ h2,
                          ds.sum()[None]])
        m, v = 0.1 * grad, 0.001 * grad * grad
        master = st["master"].double() - 2e-3 * grad / (grad.abs() + 1e-8)   # Adam's first step
        return {"loss": loss.mean()[None], "grad": grad, "master": master, "m": m, "v": v, "W": None}
    if kind == "learned":
        f = st["F"]
        qb.features(st["P"], st["X"], st["H"], st["T"], st["LF"], st["G"], st["alpha"], st["scales"], f)
        rows = f.view(torch.bfloat16).view(-1, 8)
        score = torch.cat([_forward(r.double(), st["W"])[2] for r in rows.split(1 << 18)])
        return {"F": None, "score": score.view(st["score"].shape), "K": None, "order": None}
    if kind == "select":
        P, X, T, z = st["P"], st["X"], st["T"].long(), case["z"]
        eta = P.eta()
        c = X.long().sum(0)
        tm = T.max(1, keepdim=True).values.clamp(min=1)
        K = 2 * eta * z * tm + 2 * (z - (2 * c - z).abs()) * P.eta_max * tm - (tm - T) * P.eta_max * z
        order = torch.sort(-K, dim=1, stable=True).indices
        return {"K": K, "order": order, "tiles": None, "F0": None, "y0": None}
    # apply: the chosen replica's bits written back, the field and energy of the result
    b, X = st["b"], st["X"].clone()
    idx = b.idx(X.device).long()
    sol = torch.as_tensor(np.repeat(b.sol, b.sizes), device=X.device).long()
    X[sol, idx] = st["Y"]          # one replica a job
    if st["Q"] is not None:
        H = (X.double() @ st["Q"].double()).round()
        E = (X.double() * H).sum(1)
    else:
        H = E = None
    dX = X.to(torch.int8) - st["X"].to(torch.int8)
    return {"X": X, "dX": dX, "H": H, "E": E, "ebest": None if E is None else E.min()[None],
            "xbest": None if E is None else X[E.argmin()], "ej": st["e"]}
