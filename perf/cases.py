"""The work that users of the library have it do, as timed cases.

Every case goes through the public entry points of ``paper_2004_03972_amd.hqa``: whole
anneals (reset, run, window mean, read-out) of dense and sparse instances in each storage
form, the captured pass over an uneven batch, the tabu read-out, exact energies of given
spin vectors, and the learned early stop (its checkpointed run, its training steps and its
inference).  Sizes are those of the repository's benchmark workloads and tests, with
shorter schedules so that one pass stays short; couplings are made on the GPU from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2004_03972_amd import hqa, instances

# on-chip register and LDS capacity (256 CUs); couplings above it are streamed every step
ON_CHIP_BYTES = 160e6


def listed():
    return [
        # a single small glass, tuned: latency of one short anneal (the test suite's size)
        dict(name="sk64", kind="md", family="sk", N=64, R=8, prec="bf16", tune=20, T=200, W=100,
             n_amb=0),
        # the library's defaults (binary32, untuned) on a mid-size glass of odd sizes
        dict(name="sk509_f32", kind="md", family="sk", N=509, R=33, prec="f32", tune=0, T=200,
             W=100, n_amb=0),
        # one MAX-CUT instance with all its replicas: anneal and exact n = 20 read-out
        dict(name="er800", kind="md", family="er", N=800, p=0.06, R=256, prec="fp8", tune=50,
             T=1000, W=100, n_amb=20),
        # a large glass with fields, 16 initial conditions, H_MD at the end (schedule sweeps)
        dict(name="glass10k", kind="md", family="glass", N=10000, R=16, prec="bf16", tune=20,
             T=1000, W=100, n_amb=0, hmd=1),
        # the large dense shape: matrix-core throughput
        dict(name="pm8192", kind="md", family="pm", N=8192, R=512, prec="fp8", tune=10, T=100,
             W=100, n_amb=0),
        # the periodic 3D lattice with many replicas, sparse plan that stays on chip
        dict(name="ea16", kind="md", family="ea3d", L=16, R=1024, prec="f32", tune=20, T=1000,
             W=100, n_amb=20),
        # a serving-style pass over uneven instances (glasses in BF16, graphs in FP8)
        dict(name="pass24", kind="pass", count=24, R=64, T=500, W=100, n_amb=20),
        # sparse MAX-CUT at the early stop's evaluation size: checkpointed run
        dict(name="es_run10k", kind="es_run", N=10000, deg=50.0, R=128, T=1000, W=100, K=500,
             Ks=100, stride=10),
        # training of the early-stop classifier: minibatches in host memory, as train() has them
        dict(name="es_train", kind="es_train", n=8192, steps=8, mem="host"),
        # one checkpoint's inference: N = 10^4 spins x 128 replicas, BF16
        dict(name="es_predict", kind="es_predict", n=1280000, bf16=1),
        # the K2000 read-out that hands 1000 spins to the tabu search
        dict(name="tabu2000", kind="tabu", family="pm", N=2000, R=16, n_amb=1000, iters=20000,
             tenure=50),
        # scoring given spin vectors exactly on a large glass with fields
        dict(name="energy5000", kind="energy", family="glass", N=5000, V=256),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["md", "md", "md", "csr", "pass", "es_run", "es_train", "es_predict", "tabu",
                       "energy"])
    if kind == "md":
        N = _log(rng, 48, 6000)
        R = min(_log(rng, 1, 512), max(1, int(3.0e10 / (2.0 * N * N))))
        fam, prec = rng.choice([("sk", "bf16"), ("glass", "bf16"), ("er", "fp8"), ("pm", "fp8"),
                                ("sk", "f32"), ("glass", "f32")])
        T = rng.randrange(100, 400)
        return dict(kind="md", family=fam, N=N, p=rng.uniform(0.01, 0.1), R=R, prec=prec,
                    tune=rng.choice([0, 20]), T=T, W=min(100, T),
                    n_amb=rng.choice([0, min(N, 12), min(N, 20)]), hmd=int(rng.random() < 0.3))
    if kind == "csr":
        T = rng.randrange(100, 400)
        c = dict(kind="md", R=_log(rng, 4, 512), prec="f32", tune=rng.choice([0, 20]), T=T,
                 W=min(100, T), n_amb=rng.choice([0, 12, 20]))
        if rng.random() < 0.5:
            c.update(family="ea3d", L=rng.randrange(5, 17))
        else:
            c.update(family="er_sparse", N=_log(rng, 300, 10000), deg=rng.uniform(4.0, 50.0))
            c["R"] = min(c["R"], 128)
        return c
    if kind == "pass":
        return dict(kind="pass", count=rng.randrange(3, 13), R=_log(rng, 8, 96),
                    T=rng.randrange(100, 300), W=100, n_amb=rng.choice([8, 16, 20]))
    if kind == "es_run":
        K = rng.randrange(100, 300)
        return dict(kind="es_run", N=_log(rng, 300, 8000), deg=rng.uniform(6.0, 50.0),
                    R=_log(rng, 4, 128), T=2 * K, W=min(100, K), K=K, Ks=rng.randrange(20, 100),
                    stride=rng.choice([1, 5, 10]))
    if kind == "es_train":
        return dict(kind="es_train", n=_log(rng, 200, 65536), steps=rng.randrange(1, 9),
                    mem=rng.choice(["host", "device"]))
    if kind == "es_predict":
        return dict(kind="es_predict", n=_log(rng, 500, 1200000), bf16=rng.choice([0, 1]))
    if kind == "tabu":
        fam = rng.choice(["pm", "glass"])
        N = _log(rng, 200, 3000)
        n = _log(rng, 25, N)
        return dict(kind="tabu", family=fam, N=N, R=rng.randrange(2, 33), n_amb=n,
                    iters=rng.randrange(500, 10000), tenure=max(1, n // 20))
    return dict(kind="energy", family=rng.choice(["glass", "sk", "pm", "er", "er_sparse"]),
                N=_log(rng, 100, 5000), p=rng.uniform(0.01, 0.1), deg=rng.uniform(4.0, 50.0),
                V=_log(rng, 1, 300))


# ------------------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _dense(family, N, seed, p=0.05):
    """(J, h or None) of one dense instance, binary64 on the GPU (the recipes of instances.py)."""
    g = _gen(seed)
    kw = dict(generator=g, device="cuda", dtype=torch.float64)
    h = None
    if family == "sk":
        J = torch.randn((N, N), **kw) / math.sqrt(N)
    elif family == "glass":
        J = torch.rand((N, N), **kw) * 2.0 - 1.0
        h = torch.rand((N,), **kw) * 4.0 - 2.0
    elif family == "pm":
        J = torch.where(torch.rand((N, N), **kw) < 0.5, -1.0, 1.0).to(torch.float64)
    else:
        J = (torch.rand((N, N), **kw) < p).to(torch.float64)
    J = torch.triu(J, 1)
    return (J + J.T).contiguous(), h


def _csr(case, seed):
    if case["family"] == "ea3d":
        return instances.ea3d(case["L"], seed)
    return instances.er_sparse(case["N"], min(case["deg"], case["N"] / 4), seed)


class _DeviceProblem:
    """A dense instance whose couplings are already in device memory."""

    def __init__(self, J, h=None, prec="f32", override=False):
        self.J, self.h, self.n = J, h, J.shape[0]
        storage = hqa.PRECISIONS[prec] if override else 0
        self.c = hqa.hqa_problem(self.n, hqa.HQA_DENSE, hqa.HQA_DEVICE, storage, J.data_ptr(), None,
                                 None, self.n * self.n, None if h is None else h.data_ptr())


def _is_csr(case):
    return case.get("family") in ("ea3d", "er_sparse") or case["kind"] == "es_run"


def _size(case):
    return case["L"] ** 3 if case.get("family") == "ea3d" else case["N"]


def _problem(case, seed):
    if _is_csr(case):
        rp, ci, v = _csr({**case, "family": case.get("family", "er_sparse")}, seed)
        return hqa.Problem(row_ptr=rp, col=ci, val=v)
    J, h = _dense(case["family"], case["N"], seed, case.get("p", 0.05))
    return _DeviceProblem(J, h)


def _pass_specs(case, seed):
    """Half Sherrington-Kirkpatrick (BF16), half Erdos-Renyi graphs (FP8), uneven sizes that
    depend on the case alone."""
    rng = np.random.default_rng(case["count"])
    out = []
    for k in range(case["count"]):
        if k < case["count"] // 2:
            out.append(("sk", int(rng.integers(100, 2001)), 0.0, seed + k))
        else:
            out.append(("er", int(rng.integers(500, 5001)), float(rng.uniform(0.01, 0.1)), seed + k))
    return out


def _es_samples(n, seed):
    """Feature rows with the ranges of the library's own features, and their labels."""
    g = _gen(seed)
    x = torch.randn((n, hqa.HQA_ES_NFEAT), generator=g, device="cuda")
    u = torch.rand((n, hqa.HQA_ES_NFEAT), generator=g, device="cuda")
    for k in (1, 2, 7, 9, 10):
        x[:, k] = x[:, k].abs()
    x[:, 2] = x[:, 0].abs() + 0.1 * u[:, 2]
    x[:, 3] = x[:, 0] + 0.3 * x[:, 3]
    for k in (4, 5):
        x[:, k] = u[:, k]
    x[:, 11] = 0.05 * torch.ceil(20.0 * u[:, 11])
    y = torch.where(x[:, 3] > 0, 0, 1)
    y = torch.where(x[:, 2] + 0.2 * u[:, 0] < 0.4, 2, y).to(torch.int32)
    return x.contiguous(), y.contiguous()


def _es_params(seed):
    """Classifier weights uniform in +-1/sqrt(fan in), zero biases (binary32)."""
    rng = np.random.default_rng(seed)
    P = []
    for fan_in, out in ((12, 64), (64, 64), (64, 3)):
        P += [rng.uniform(-1.0, 1.0, fan_in * out) / math.sqrt(fan_in), np.zeros(out)]
    return np.concatenate(P).astype(np.float32)


_CW = (0.8, 0.9, 1.4)
_LR = 3e-3


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case, "seed": seed}
    if kind in ("md", "es_run"):
        prob = _problem(case, seed)
        sch = hqa.make_schedule(case["T"], W=case["W"])
        st["md"] = hqa.MD(prob, sch, case["R"], case.get("prec", "f32"), seed=seed)
        if not _is_csr(case):
            prob.J = prob.h = None              # the handle holds its own copy
        if case.get("tune"):
            st["md"].tune(case["tune"])
        N = _size(case)
        if kind == "md":
            st["phibar"] = torch.empty((case["R"], N), dtype=torch.float64, device="cuda")
        else:
            st["es"] = hqa.ES()
            st["es"].params = _es_params(seed)
            st["prob"] = torch.empty((case["R"] * N, 3), dtype=torch.float32, device="cuda")
    elif kind == "pass":
        probs = [_DeviceProblem(*_dense(f, N, s, p), prec="bf16" if f == "sk" else "fp8",
                                override=True) for f, N, p, s in _pass_specs(case, seed)]
        sch = hqa.make_schedule(case["T"], W=case["W"])
        st["md"] = hqa.MD(probs, sch, case["R"], "bf16", seed=seed)
        for q in probs:
            q.J = q.h = None
        shape = (case["count"], case["R"])
        st["out"] = [torch.empty(shape, dtype=torch.float64, device="cuda") for _ in range(2)]
    elif kind == "tabu":
        # a finished anneal: the window sums as such a run leaves them
        prob = _problem(case, seed)
        sch = hqa.make_schedule(1000, W=100)
        prec = "fp8" if case["family"] == "pm" else "bf16"
        st["md"] = hqa.MD(prob, sch, case["R"], prec, seed=seed)
        prob.J = prob.h = None
        st["md"].set_state(hqa.HQA_STATE_WSUM, _wsum(case, seed).cpu().numpy())
        hqa.hqa_md_set_step(st["md"].h, 1000)
    elif kind == "es_train":
        xs = [_es_samples(case["n"], seed + 100 * k) for k in range(case["steps"])]
        cw = torch.tensor(_CW, dtype=torch.float32)
        st["es"] = hqa.ES()
        st["params"] = _es_params(seed)
        if case["mem"] == "host":
            st["batches"] = [(x.cpu().numpy(), y.cpu().numpy()) for x, y in xs]
            st["cw"] = cw.numpy()
        else:
            st["batches"], st["cw"] = xs, cw.cuda()
            st["loss"] = torch.empty(case["steps"], dtype=torch.float32, device="cuda")
    elif kind == "es_predict":
        st["es"] = hqa.ES()
        st["es"].params = _es_params(seed)
        st["x"], _ = _es_samples(case["n"], seed)
        st["prob"] = torch.empty((case["n"], 3), dtype=torch.float32, device="cuda")
    else:
        if case["family"] == "er_sparse":
            rp, ci, v = _csr(case, seed)
            st["arrays"] = [torch.from_numpy(a).cuda() for a in (rp, ci, v)]
            rp, ci, v = st["arrays"]
            st["prob"] = hqa.hqa_problem(case["N"], hqa.HQA_CSR, hqa.HQA_DEVICE, 0, v.data_ptr(),
                                         rp.data_ptr(), ci.data_ptr(), v.numel(), None)
        else:
            st["arrays"] = _problem(case, seed)
            st["prob"] = st["arrays"].c
        st["spins"] = _spins(case["V"], case["N"], seed)
        st["out"] = [torch.empty(case["V"], dtype=torch.float64, device="cuda") for _ in range(2)]
    torch.cuda.synchronize()
    return st


def _wsum(case, seed):
    g = _gen(seed + 7)
    x = torch.randn((case["R"], case["N"]), generator=g, device="cuda", dtype=torch.float64)
    return (x.to(torch.float32) * 100.0).to(torch.float64)


def _spins(V, N, seed):
    g = _gen(seed + 13)
    s = torch.randint(0, 2, (V, N), generator=g, device="cuda", dtype=torch.int8)
    return (2 * s - 1).contiguous()


# ---------------------------------------------------------------------------- one pass
def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "md":
        md = st["md"]
        md.reset(st["seed"])
        md.run()
        hqa.hqa_md_state(md.h, 0, hqa.HQA_STATE_PHIBAR, st["phibar"], hqa.HQA_DEVICE)
        out = {"phibar": st["phibar"]}
        if case.get("hmd"):
            out["H"] = md.hamiltonian()
        if case["n_amb"]:
            out.update(md.classify(case["n_amb"], solve=True))
        return out
    if kind == "pass":
        md, (E, C) = st["md"], st["out"]
        md.run_pass(st["seed"], case["n_amb"], solve=True, graph=True, energy=E, cut=C)
        md.sync()
        return [E, C]
    if kind == "es_run":
        md = st["md"]
        md.reset(st["seed"])
        # a threshold no checkpoint reaches: every checkpoint is evaluated
        q, conf = md.run_es(st["es"], case["K"], case["Ks"], case["stride"], 2.0,
                            prob=st["prob"])
        return [st["prob"], q, conf]
    if kind == "tabu":
        return st["md"].classify_tabu(case["n_amb"], case["iters"], case["tenure"])
    if kind == "es_train":
        es = st["es"]
        es.params = st["params"]                 # a fresh training run: Adam starts again
        if case["mem"] == "host":
            loss = np.array([es.train_step(x, y, st["cw"], _LR) for x, y in st["batches"]])
        else:
            loss = st["loss"]
            for k, (x, y) in enumerate(st["batches"]):
                hqa.hqa_es_train_step(es.h, x, y, case["n"], st["cw"], _LR, loss[k:],
                                      hqa.HQA_DEVICE)
        return [loss, es.params]
    if kind == "es_predict":
        return st["es"].predict(st["x"], bf16=bool(case["bf16"]), out=st["prob"])
    E, C = st["out"]
    hqa.hqa_ising_energy(st["prob"], st["spins"], case["V"], E, C, hqa.HQA_DEVICE)
    return [E, C]


# ----------------------------------------------------------------------- work of a pass
def _md_work(N, R, T, jbytes, nnz, window):
    """Bytes and operations of T steps: the couplings once if they can stay on chip, else
    every step; momenta in as one seed, the window mean out."""
    stream = jbytes * (T if jbytes > ON_CHIP_BYTES else 1)
    return {"bytes": stream + 8.0 * N * R, "flops": (2.0 * nnz + 14.0 * N) * R * T}


def work(case):
    kind = case["kind"]
    if kind in ("md", "es_run"):
        N, R, T = _size(case), case["R"], case["T"]
        if _is_csr(case):
            nnz = 6.0 * N if case.get("family") == "ea3d" else case["deg"] * N
            w = _md_work(N, R, T, 8.0 * nnz, nnz, case["W"])
        else:
            esz = {"f32": 4.0, "bf16": 2.0, "fp8": 1.0}[case["prec"]]
            w = _md_work(N, R, T, esz * N * N, float(N) * N, case["W"])
        if case.get("hmd"):
            w["bytes"] += 8.0 * N * N
            w["flops"] += 2.0 * N * N * R
        if case.get("n_amb"):
            w["bytes"] += 1.0 * R * N
            w["flops"] += R * 2.0 ** case["n_amb"] * 2.0
        if kind == "es_run":
            w["bytes"] += 2 * 12.0 * N * R
            w["flops"] += 2 * 2.0 * 5056 * N * R
        return w
    if kind == "pass":
        w = {"bytes": 0.0, "flops": 0.0}
        jb = sum((2.0 if f == "sk" else 0.125) * N * N for f, N, _, _ in _pass_specs(case, 0))
        R, T = case["R"], case["T"]
        for _, N, _, _ in _pass_specs(case, 0):
            w["flops"] += (2.0 * N + 14.0) * N * R * T + R * 2.0 ** case["n_amb"] * 2.0
            w["bytes"] += 16.0 * R
        w["bytes"] += jb * (T if jb > ON_CHIP_BYTES else 1)
        return w
    if kind == "tabu":
        N, R, n, it = case["N"], case["R"], case["n_amb"], case["iters"]
        return {"bytes": 8.0 * N * N + 5.0 * N * R, "flops": R * (3.0 * n * it + 2.0 * N * N)}
    if kind == "es_train":
        n = case["n"] * case["steps"]
        return {"bytes": 52.0 * n, "flops": 6.0 * 5056 * n}
    if kind == "es_predict":
        return {"bytes": 60.0 * case["n"], "flops": 2.0 * 5056 * case["n"]}
    N, V = case["N"], case["V"]
    if case["family"] == "er_sparse":
        return {"bytes": 12.0 * case["deg"] * N + N * V, "flops": 2.0 * case["deg"] * N * V}
    return {"bytes": 8.0 * N * N + N * V, "flops": 2.0 * N * N * V}


# ------------------------------------------------------- the same results, plainly, in 64 bits
def _momenta(seed, R, N):
    """p(0) = +-1 from the SplitMix64 output function at counter seed + (r N + i + 1) gamma."""
    with np.errstate(over="ignore"):
        z = np.uint64(seed) + (np.arange(R * N, dtype=np.uint64) + np.uint64(1)) * \
            np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z = z ^ (z >> np.uint64(31))
    p = np.where(z >> np.uint64(63), -1.0, 1.0).reshape(R, N)
    return torch.from_numpy(p).cuda()


def _schedule(T):
    """alpha and beta at tau_k = k / 2T, the paper's parameters."""
    tau = np.arange(2 * T + 1) / (2.0 * T)
    poly = lambda f, a, b: f * ((tau + a * (1.0 - tau)) + b * (tau * (tau - 1.0)))
    return poly(0.008, 4.0, 3.0), poly(0.12, 0.05, 1.0)


def _exact_md(case, seed):
    """phibar (and H_MD) of the anneal in binary64: x is [N][R]."""
    N, R, T, W = _size(case), case["R"], case["T"], case["W"]
    h = None
    if _is_csr(case):
        rp, ci, v = _csr(case, seed)
        J = torch.sparse_csr_tensor(torch.from_numpy(rp.astype(np.int64)),
                                    torch.from_numpy(ci.astype(np.int64)),
                                    torch.from_numpy(v), size=(N, N)).cuda()
    else:
        J, h = _dense(case["family"], N, seed, case.get("p", 0.05))
    al, be = _schedule(T)
    x = torch.zeros((N, R), dtype=torch.float64, device="cuda")
    p = _momenta(seed, R, N).T.contiguous()
    S = torch.zeros_like(x)

    def force(x, k):
        g = J @ x
        if h is not None:
            g = g + 2.0 * h[:, None] * x.abs()
        return al[k] * 6.0 * x ** 5 + be[k] * g
    for q in range(T):
        p = p - (0.5 if q == 0 else 1.0) * force(x, 2 * q)
        x = x + al[2 * q + 1] * p
        if q + 1 >= T - W + 1:
            S += x
    out = {"phibar": (S / W).T.contiguous()}
    if case.get("hmd"):
        pm = p - 0.5 * force(x, 2 * T)
        H = al[2 * T] * (0.5 * pm * pm + x ** 6).sum(0) + be[2 * T] * 0.5 * (x * (J @ x)).sum(0)
        if h is not None:
            H = H + be[2 * T] * (h[:, None] * x.abs() * x).sum(0)
        out["H"] = H.cpu().numpy()
    # the read-out of a long anneal follows every rounding of the trajectory before it
    if case["n_amb"]:
        out.update({k: None for k in ("spins", "amb_idx", "energy", "cut", "h_eff", "code",
                                      "e_reduced")})
    return out


def _energy_cut(J, h, s):
    """E = 1/2 s J s + h s and the cut sum_{i<j, s_i != s_j} J_ij of the rows of s."""
    s = s.to(torch.float64)
    q = ((s @ J) * s).sum(1)
    E = 0.5 * q if h is None else 0.5 * q + s @ h
    return E, 0.25 * (J.sum() - q)


def _exact_tabu(case, seed):
    N, R, n = case["N"], case["R"], case["n_amb"]
    if case["family"] != "pm":
        return None                              # real couplings: ties follow the roundings
    Jd, _ = _dense("pm", N, seed)
    J = Jd.cpu().numpy()
    phibar = (_wsum(case, seed).cpu().numpy().astype(np.float32) / np.float32(100.0))
    spins = np.where(phibar < 0, -1, 1).astype(np.int64)
    amb = np.sort(np.argsort(np.abs(phibar), axis=1, kind="stable")[:, :n], axis=1)
    rows = np.arange(R)
    Jr = np.stack([J[np.ix_(a, a)] for a in amb])
    x = np.take_along_axis(spins, amb, 1).astype(np.float64)
    full = np.stack([J[a] @ spins[r] for r, a in enumerate(amb)])
    inner = np.einsum("rab,rb->ra", Jr, x)
    heff, f = full - inner, full
    f = f.copy()
    D, Db, xb = np.zeros(R), np.zeros(R), x.copy()
    until = np.zeros((R, n), dtype=np.int64)
    ten = min(case["tenure"], n - 1)
    for t in range(1, case["iters"] + 1):
        d = -2.0 * x * f
        ok = (until < t) | (D[:, None] + d < Db[:, None])
        a = np.argmin(np.where(ok, d, np.inf), axis=1)
        D = D + d[rows, a]
        f -= 2.0 * Jr[rows, a] * x[rows, a][:, None]
        x[rows, a] = -x[rows, a]
        until[rows, a] = t + ten
        b = D < Db
        Db = np.where(b, D, Db)
        xb[b] = x[b]
    np.put_along_axis(spins, amb, xb.astype(np.int64), 1)
    E, C = _energy_cut(Jd, None, torch.from_numpy(spins).cuda())
    return {"spins": None, "amb_idx": None, "energy": E.cpu().numpy(), "cut": C.cpu().numpy(),
            "h_eff": heff, "code": None, "e_reduced": Db}


def _mlp64(P, x, bf):
    r = (lambda t: t.to(torch.bfloat16).to(torch.float64)) if bf else (lambda t: t)
    W1, b1, W2, b2, W3, b3 = (P[a:b] for a, b in ((0, 768), (768, 832), (832, 4928),
                                                  (4928, 4992), (4992, 5184), (5184, 5187)))
    gelu = lambda z: 0.5 * z * (1.0 + torch.erf(z / math.sqrt(2.0)))
    a = r(x)
    a = r(gelu(a @ r(W1).view(64, 12).T + b1))
    a = r(gelu(a @ r(W2).view(64, 64).T + b2))
    return a @ r(W3).view(3, 64).T + b3


def _exact_es_train(case, seed):
    P = torch.from_numpy(_es_params(seed)).cuda().to(torch.float64)
    m, v, losses = torch.zeros_like(P), torch.zeros_like(P), []
    cw = torch.tensor(_CW, dtype=torch.float32).to(torch.float64).cuda()
    lr, b1, b2 = float(np.float32(_LR)), float(np.float32(0.9)), float(np.float32(0.999))
    for t in range(1, case["steps"] + 1):
        x, y = _es_samples(case["n"], seed + 100 * (t - 1))
        Q = P.clone().requires_grad_(True)
        lp = torch.log_softmax(_mlp64(Q, x.to(torch.float64), False), 1)
        w = cw[y.long()]
        loss = -(w * lp.gather(1, y.long()[:, None])[:, 0]).sum() / w.sum()
        loss.backward()
        m = b1 * m + (1 - b1) * Q.grad
        v = b2 * v + (1 - b2) * Q.grad ** 2
        P = P - lr * (m / (1 - b1 ** t)) / ((v / (1 - b2 ** t)).sqrt() + 1e-8)
        losses.append(loss.detach())
    losses = torch.stack(losses)
    return [losses.cpu().numpy() if case["mem"] == "host" else losses, P.cpu().numpy()]


def _exact_es_predict(case, seed):
    P = torch.from_numpy(_es_params(seed)).cuda().to(torch.float64)
    x, _ = _es_samples(case["n"], seed)
    return torch.softmax(_mlp64(P, x.to(torch.float64), bool(case["bf16"])), 1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "md":
        # 16-bit operands leave the binary64 trajectory within a few hundred steps
        if case["prec"] != "f32" and case["T"] > (400 if case["family"] == "sk" else 100):
            return None
        if not _is_csr(case) and 2.0 * _size(case) ** 2 * case["R"] * case["T"] > 2e13:
            return None
        return _exact_md(case, seed)
    if kind == "tabu":
        return _exact_tabu(case, seed)
    if kind == "es_train":
        return _exact_es_train(case, seed)
    if kind == "es_predict":
        return _exact_es_predict(case, seed)
    if kind == "energy":
        s = _spins(case["V"], case["N"], seed)
        if case["family"] == "er_sparse":
            J = torch.from_numpy(instances.csr_to_dense(case["N"], *_csr(case, seed))).cuda()
            return list(_energy_cut(J, None, s))
        J, h = _dense(case["family"], case["N"], seed, case.get("p", 0.05))
        return list(_energy_cut(J, h, s))
    return None                                  # whole chaotic anneals: no such value
