"""The work this library is used for, as measured cases: bandwidth criteria, their gradients, density-derivative
functionals and dataset preparation, from single calls on a thousand points to batches on millions.

Sizes follow the benchmark workloads of this repository (``bench.py``, ``synth/``) and the paper's speed runs
(Sec. 6.3), with odd and uneven ones beside them.  Inputs are normal mixtures; bandwidths are the normal-scale
pilots and the random full matrices that the benchmark uses.  ``exact`` evaluates the same binned sums with plain
torch operations in float64.
"""
import itertools
import math

import numpy as np
import torch

import paper_1511_07482_amd as kf

DEV = "cuda"


def listed():
    return [
        # the smallest call: one univariate candidate on a prepared sample; latency of a call
        dict(name="scv_one_d1", kind="scv", d=1, n=1000, M=64, B=1, nds=1),
        # the benchmark's step: prepare a bivariate sample, psi_4 at its pilot, SCV and gradient of 256
        # bandwidths, captured once and replayed, as a serving loop does
        dict(name="step_d2", kind="step", d=2, n=100000, M=256, B=256, r=4),
        # a batched SCV call with a ragged grid and an odd number of candidates
        dict(name="scv_d2", kind="scv", d=2, n=50001, M=203, B=101, nds=1),
        # training-style use: objective forward, adjoint backward, trivariate
        dict(name="autograd_d3", kind="autograd", d=3, n=200000, M=64, B=16),
        # one batch over unequal datasets in four dimensions, 64 bandwidths each: the largest arithmetic
        dict(name="scv_uneven_d4", kind="scv", d=4, n=400000, M=32, B=256, nds=4),
        # a new four-dimensional sample: preparation and psi_4, the plug-in selector's pilot stage
        dict(name="psi_batch_d4", kind="psi_batch", d=4, n=500000, M=32, r=4),
        # a large sample binned and transformed
        dict(name="prepare_d2", kind="prepare", d=2, n=2000000, M=256),
        # the paper's literal steps on its benchmark shape
        dict(name="psi_plain_d2", kind="psi", d=2, n=100000, M=256, r=4, mode="plain"),
        # a one-off functional in three dimensions, fused
        dict(name="psi_fused_d3", kind="psi", d=3, n=200000, M=64, r=2, mode="fused"),
        # selection of the bandwidth of a second derivative: LSCV_2 over a candidate set, ragged grid
        dict(name="lscv2_d2", kind="crit", d=2, n=30000, M=230, B=200, r=2, crit="lscv"),
        # a whole minimisation from several starts (few evaluations: far from the stopping tests)
        dict(name="minimize_d2", kind="minimize", d=2, n=20000, M=128, B=4, evals=10),
        # the paper's speed-run shape, truncated support (fft-L)
        dict(name="fftl_d2", kind="fftl", d=2, n=4000, M=160, r=0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_M_RANGE = {1: (32, 1000), 2: (32, 300), 3: (12, 64), 4: (8, 32)}


def draw(rng):
    kind = rng.choice(["scv", "scv", "step", "autograd", "psi_batch", "prepare", "psi", "psi", "crit", "minimize",
                       "fftl"])
    d = rng.choice([1, 2, 2, 3, 4])
    if kind in ("psi", "fftl"):
        d = rng.choice([1, 2, 2, 3])
    if kind in ("crit", "minimize", "step"):
        d = rng.choice([1, 2, 2, 3])
    c = dict(kind=kind, d=d, n=_log(rng, 1000, 2000000 if kind == "prepare" else 300000), M=_log(rng, *_M_RANGE[d]),
             aniso=rng.random() < 0.4)
    if kind == "scv":
        c.update(nds=rng.choice([1, 1, 2, 3]))
        c.update(B=c["nds"] * _log(rng, 1, 256 if d < 3 else 48))
    elif kind in ("step", "autograd"):
        c.update(B=_log(rng, 1, 256 if d < 3 else 32))
        if kind == "step":
            c.update(r=4)
    elif kind == "psi_batch":
        c.update(r=rng.choice([0, 2, 4]))
    elif kind == "psi":
        c.update(r=rng.choice([0, 2, 4]), mode=rng.choice(["plain", "fused"]))
    elif kind == "crit":
        c.update(crit=rng.choice(["lscv", "lscv_exact", "qr"]), r=rng.choice([1, 2, 3]),
                 B=_log(rng, 1, 256 if d < 3 else 8))
    elif kind == "minimize":
        c.update(B=rng.choice([1, 3, 4, 8]), evals=8)
    elif kind == "fftl":
        c.update(r=rng.choice([0, 2]), n=_log(rng, 1000, 100000), M=min(c["M"], 256 if d < 3 else 48))
    return c


# ------------------------------------------------------------------ inputs


def _Ms(case):
    d, M = case["d"], case["M"]
    return [max(6, M - (M // 7) * k) if case.get("aniso") else M for k in range(d)]


def _haar(d, rng):
    Q, R = np.linalg.qr(rng.standard_normal((d, d)))
    return Q * np.sign(np.diag(R))[None, :]


def _vech(H):
    L = np.linalg.cholesky(H)
    d = H.shape[-1]
    return np.concatenate([L[..., j:, j] for j in range(d)], axis=-1)


def _sample(n, d, rng, seed):
    """n points of a two- to four-component normal mixture on the GPU, and the mixture's covariance."""
    k = 4 if d == 2 else 2
    mean = rng.standard_normal((k, d))
    mean = 1.5 * mean / np.linalg.norm(mean, axis=1, keepdims=True)
    cov = []
    for _ in range(k):
        Q = _haar(d, rng)
        cov.append(Q @ np.diag(10.0 ** rng.uniform(-1.0, 0.0, size=d)) @ Q.T)
    L = torch.from_numpy(np.stack([np.linalg.cholesky(0.5 * (s + s.T)) for s in cov])).to(DEV)
    g = torch.Generator(device=DEV).manual_seed(seed)
    lab = torch.randint(k, (n,), generator=g, device=DEV)
    z = torch.randn((n, d), generator=g, device=DEV, dtype=torch.float64)
    X = torch.from_numpy(mean).to(DEV)[lab]
    for i in range(d):
        for j in range(i + 1):
            X[:, i] += L[lab, i, j] * z[:, j]
    m = mean.mean(axis=0)
    S = sum(cov) / k + (mean - m).T @ (mean - m) / k
    return X.contiguous(), 0.5 * (S + S.T)


def _inputs(case, seed):
    """Samples, pilots and candidate bandwidths of a case: plain tensors and arrays."""
    rng = np.random.default_rng(seed)
    d, n, nds = case["d"], case["n"], case.get("nds", 1)
    X, S, G = [], [], []
    for j in range(nds):
        nj = max(200, n * (j + 1) // nds - 7 * j)   # unequal sizes in a batch
        x, s = _sample(nj, d, rng, seed * 16 + j)
        X.append(x)
        S.append(s)
        G.append(nj ** (-2.0 / (d + 6)) * s)
    B = case.get("B", 1)
    if case["kind"] == "minimize":
        ns = (4.0 / (d + 2)) ** (2.0 / (d + 4)) * n ** (-2.0 / (d + 4)) * S[0]
        H = np.stack([ns * np.exp(rng.uniform(0.5, 2.0)) for _ in range(B)])
    else:
        H = np.stack([Q @ np.diag(np.exp(rng.uniform(-3.0, 0.0, size=d))) @ Q.T
                      for Q in (_haar(d, rng) for _ in range(B))])
    v = _vech(0.5 * (H + np.swapaxes(H, -1, -2)))
    Gpsi = [x.shape[0] ** (-2.0 / (d + case.get("r", 4) + 4)) * s for x, s in zip(X, S)]
    return dict(X=X, G=G, Gpsi=Gpsi, vech=torch.from_numpy(v).to(DEV),
                w=torch.from_numpy(rng.uniform(0.5, 1.5, size=B)).to(DEV))


def _per(case):
    nds, B = case.get("nds", 1), case.get("B", 1)
    return [B // nds + (1 if j < B % nds else 0) for j in range(nds)]


# ------------------------------------------------------------------ the cases


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    s["M"] = _Ms(case)
    kind = case["kind"]
    if kind in ("scv", "autograd", "crit", "minimize"):
        s["ds"] = [kf.Dataset(x, g, M=s["M"]) for x, g in zip(s["X"], s["G"])]
    if kind == "step":
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _step(s)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            s["out"] = _step(s)
    return s


def _step(s):
    ds = kf.Dataset(s["X"][0], s["G"][0], M=s["M"])
    psi = kf.psi_batch([ds], [s["Gpsi"][0]], s["case"]["r"])
    obj, grad = kf.scv([ds], s["vech"])
    return dict(psi=psi, obj=obj, grad=grad, keep=ds.counts())


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "step":
        s["graph"].replay()
        return s["out"]
    if kind == "scv":
        obj, grad = kf.scv(s["ds"], s["vech"], per_ds=_per(case))
        return dict(obj=obj, grad=grad)
    if kind == "autograd":
        v = s["vech"].detach().requires_grad_()
        obj = kf.SCV.apply(v, s["ds"][0])
        obj.backward(s["w"])
        return dict(obj=obj.detach(), grad=v.grad)
    if kind == "crit":
        return dict(obj=kf.crit(s["ds"], s["vech"], case["crit"], case["r"], grad=False))
    if kind == "minimize":
        x, f, info = kf.minimize(s["vech"], "scv", datasets=s["ds"], evals=case["evals"])
        return dict(x=x, f=f, info=info)
    X = s["X"][0]
    if kind == "prepare":
        ds = kf.Dataset(X, s["G"][0], M=s["M"])
        return dict(counts=ds.counts(), lag=ds.lag_array())
    if kind == "psi_batch":
        ds = kf.Dataset(X, s["G"][0], M=s["M"])
        return dict(psi=kf.psi_batch([ds], [s["Gpsi"][0]], case["r"]), counts=ds.counts())
    if kind == "psi":
        return dict(psi=kf.psi(X, s["Gpsi"][0], case["r"], M=s["M"], mode=case["mode"]))
    psi, L, P = kf.psi_fftl(X, s["Gpsi"][0], case["r"], M=s["M"])
    return dict(psi=psi, L=L, P=P)


def work(case):
    """Samples read once, grid arrays that a call takes or returns read or written once, and for the criteria one
    multiply-add per Gaussian and lag of the half lag set."""
    d, n, nds, B = case["d"], case["n"], case.get("nds", 1), case.get("B", 1)
    kind = case["kind"]
    M = _Ms(case)
    nodes = float(np.prod(M))
    lags = 0.5 * float(np.prod([2.0 * m - 1.0 for m in M]))
    pts = 8.0 * n * d
    fft = 2.5 * 2.0 * lags * math.log2(2.0 * lags)   # one real transform of the padded grid
    q = d * (d + 1) // 2
    nu = math.comb(d + case.get("r", 0) - 1, case.get("r", 0))
    small = 16.0 * B * (1 + q)
    if kind == "scv":
        return dict(bytes=8.0 * nds * lags + small, flops=4.0 * B * lags)
    if kind == "autograd":
        return dict(bytes=16.0 * lags + small, flops=8.0 * B * lags)
    if kind == "crit":
        return dict(bytes=8.0 * lags + small, flops=(2.0 if case["crit"] == "qr" else 4.0) * B * lags)
    if kind == "minimize":
        return dict(bytes=8.0 * lags + small, flops=4.0 * B * case["evals"] * lags)
    if kind == "step":
        return dict(bytes=pts + 16.0 * nodes + small, flops=2.0 * fft + (4.0 * B + 2.0 * nu) * lags)
    if kind == "prepare":
        return dict(bytes=pts + 8.0 * nodes + 16.0 * lags, flops=2.0 * fft)
    if kind == "psi_batch":
        return dict(bytes=pts + 8.0 * nodes + 8.0 * nu, flops=2.0 * fft + 2.0 * nu * lags)
    return dict(bytes=pts + 8.0 * nu, flops=fft + 2.0 * nu * lags)


# ------------------------------------------------------------------ the same values by plain torch, float64


def _bin(X, G, Ms):
    """Counts of linear binning in 2^-40 quanta, grid spacing: bounds padded by four kernel standard deviations."""
    d = X.shape[1]
    lo = X.amin(0).cpu().numpy() - 4.0 * np.sqrt(np.diag(G))
    hi = X.amax(0).cpu().numpy() + 4.0 * np.sqrt(np.diag(G))
    delta = (hi - lo) / (np.array(Ms) - 1)
    j, f = [], []
    for k in range(d):
        # tensors, not host scalars: a true division, one operation each
        t = (X[:, k] - torch.tensor(lo[k], device=X.device)) / torch.full_like(X[:, k], delta[k])
        jk = torch.clamp(torch.floor(t), max=float(Ms[k] - 2))
        j.append(jk.long())
        f.append(t - jk)
    q, idx = [], []
    for b in range(1 << d):
        w, i = None, torch.zeros_like(j[0])
        for k in range(d):
            up = (b >> k) & 1
            wk = f[k] if up else 1.0 - f[k]
            w = wk if w is None else w * wk
            i = i * Ms[k] + j[k] + up
        q.append(torch.round(w * 2.0 ** 40).long())
        idx.append(i)
    q = torch.stack(q)
    best = torch.zeros(X.shape[0], dtype=torch.long, device=X.device)   # the largest corner, lowest on ties
    top = q[0].clone()
    for b in range(1, 1 << d):
        best = torch.where(q[b] > top, torch.full_like(best, b), best)
        top = torch.maximum(top, q[b])
    q.scatter_add_(0, best[None], (2 ** 40 - q.sum(0))[None])
    counts = torch.zeros(int(np.prod(Ms)), dtype=torch.long, device=X.device)
    for b in range(1 << d):
        counts.index_add_(0, idx[b], q[b])
    return counts.view(*Ms), delta


def _lags(counts):
    """Autocorrelation of the counts on lags -(M-1)..(M-1) of every axis."""
    M = counts.shape
    c = counts.double() * 2.0 ** -40
    P = [2 * m for m in M]
    A = torch.fft.irfftn(torch.fft.rfftn(c, s=P).abs().square(), s=P)
    for k, m in enumerate(M):
        A = torch.cat([A.narrow(k, m + 1, m - 1), A.narrow(k, 0, m)], dim=k)
    return A


def _axes(shape, delta):
    d = len(shape)
    out = []
    for k, s in enumerate(shape):
        x = torch.arange(-(s // 2), s // 2 + 1, device=DEV, dtype=torch.float64) * float(delta[k])
        out.append(x.view([-1 if i == k else 1 for i in range(d)]))
    return out


def _phi(x, S):
    d = len(x)
    P = np.linalg.inv(S)
    q = sum(float(P[i, j]) * x[i] * x[j] for i in range(d) for j in range(d))
    return torch.exp(-0.5 * q) / math.sqrt((2 * math.pi) ** d * np.linalg.det(S))


def _hermite(x, S, order):
    """He_alpha(S^-1 x) of every multi-index of at most `order`: D^alpha phi = (-1)^|alpha| He_alpha phi."""
    d = len(x)
    P = np.linalg.inv(S)
    z = [sum(float(P[i, j]) * x[j] for j in range(d)) for i in range(d)]
    he = {(0,) * d: torch.ones((), device=DEV, dtype=torch.float64)}
    for s in range(1, order + 1):
        for t in itertools.combinations_with_replacement(range(d), s):
            a = tuple(t.count(k) for k in range(d))
            k = t[0]
            b = list(a)
            b[k] -= 1
            v = z[k] * he[tuple(b)]
            for j in range(d):
                if b[j]:
                    c = list(b)
                    c[j] -= 1
                    v = v - float(b[j] * P[k, j]) * he[tuple(c)]
            he[a] = v
    return he


def _tuples(d, r):
    return [tuple(t.count(k) for k in range(d)) for t in itertools.combinations_with_replacement(range(d), r)]


def _psi_exact(A, delta, G, n, r):
    x = _axes(A.shape, delta)
    w = _phi(x, G) * A
    he = _hermite(x, G, r)
    return torch.stack([(w * he[a]).sum() for a in _tuples(len(x), r)]) / float(n) ** 2


def _scv_exact(A, delta, G, n, vech):
    d = A.dim()
    x = _axes(A.shape, delta)
    const = (_phi(x, 2 * G) * A).sum() / float(n) ** 2
    obj, grad = [], []
    for v in vech.cpu().numpy():
        L = np.zeros((d, d))
        t = 0
        for j in range(d):
            for i in range(j, d):
                L[i, j] = v[t]
                t += 1
        H = L @ L.T
        first = (4 * math.pi) ** (-d / 2) / (n * abs(np.prod(np.diag(L))))
        val, gH = first, -0.5 * first * np.linalg.inv(H)
        for S, wo, wg in ((2 * H + 2 * G, 1.0, 1.0), (H + 2 * G, -2.0, -1.0)):
            w = _phi(x, S) * A
            m0 = float(w.sum()) / float(n) ** 2
            val = val + wo * m0
            m2 = np.empty((d, d))
            for i in range(d):
                for j in range(i, d):
                    other = [k for k in range(d) if k not in (i, j)]
                    u = w.sum(dim=other, keepdim=True) if other else w
                    m2[i, j] = m2[j, i] = float((u * x[i] * x[j]).sum()) / float(n) ** 2
            P = np.linalg.inv(S)
            gH = gH + wg * (P @ m2 @ P - P * m0)
        g = 2.0 * gH @ L
        obj.append(val + float(const))
        grad.append([g[i, j] for j in range(d) for i in range(j, d)])
    return torch.tensor(obj, dtype=torch.float64), torch.tensor(grad, dtype=torch.float64)


def _eta(x, S, r):
    """(Laplacian)^r phi_S at the points x."""
    d = len(x)
    he = _hermite(x, S, 2 * r)
    t = 0.0
    for a in _tuples(d, r):
        m = math.factorial(r) / math.prod(math.factorial(k) for k in a)
        t = t + m * he[tuple(2 * k for k in a)]
    return t * _phi(x, S)


def _crit_exact(A, delta, n, vech, crit, r):
    d = A.dim()
    x = _axes(A.shape, delta)
    zero = [torch.zeros((), device=DEV, dtype=torch.float64) for _ in range(d)]
    out = []
    for v in vech.cpu().numpy():
        L = np.zeros((d, d))
        L[np.triu_indices(d)[1], np.triu_indices(d)[0]] = v   # columns of the lower triangle
        H = L @ L.T
        if crit == "qr":
            out.append(float((_eta(x, H, r) * A).sum()) / float(n) ** 2)
            continue
        m = n - 1.0 if crit == "lscv_exact" else float(n)
        s = float(((_eta(x, 2 * H, r) - 2.0 * n / m * _eta(x, H, r)) * A).sum()) / float(n) ** 2
        out.append((-1) ** r * (s + 2.0 / m * float(_eta(zero, H, r))))
    return torch.tensor(out, dtype=torch.float64)


def exact(case, seed):
    kind = case["kind"]
    if kind == "minimize":
        return None
    s = _inputs(case, seed)
    Ms = _Ms(case)
    r = case.get("r", 0)
    if kind in ("psi", "fftl"):
        counts, delta = _bin(s["X"][0], s["Gpsi"][0], Ms)
    else:
        counts, delta = _bin(s["X"][0], s["G"][0], Ms)
    n = s["X"][0].shape[0]
    A = _lags(counts)
    if kind == "prepare":
        lag = None
        if all(m & (m - 1) == 0 for m in Ms):
            # the circular layout of the lag array: lag l at index l mod 2M
            P = [2 * m for m in Ms]
            lag = torch.zeros(P, dtype=torch.float64, device=A.device)
            idx = torch.meshgrid(*[torch.arange(-(m - 1), m, device=A.device) % (2 * m) for m in Ms], indexing="ij")
            lag[idx] = A * float(np.prod(P))
        return dict(counts=counts, lag=lag)
    if kind == "psi_batch":
        return dict(psi=_psi_exact(A, delta, s["Gpsi"][0], n, r)[None], counts=counts)
    if kind == "psi":
        return dict(psi=_psi_exact(A, delta, s["Gpsi"][0], n, r))
    if kind == "fftl":
        lam = float(np.linalg.eigvalsh(s["Gpsi"][0])[-1])
        for k, m in enumerate(Ms):
            L = min(m - 1, math.ceil(3.7 * math.sqrt(lam) / delta[k]))
            A = A.narrow(k, m - 1 - L, 2 * L + 1)
        return dict(psi=_psi_exact(A, delta, s["Gpsi"][0], n, r), L=None, P=None)
    if kind == "crit":
        return dict(obj=_crit_exact(A, delta, n, s["vech"], case["crit"], r))
    if kind == "step":
        obj, grad = _scv_exact(A, delta, s["G"][0], n, s["vech"])
        return dict(psi=_psi_exact(A, delta, s["Gpsi"][0], n, r)[None], obj=obj, grad=grad, keep=counts)
    obj, grad, at = [], [], 0
    for j, b in enumerate(_per(case)):
        if j:
            counts, delta = _bin(s["X"][j], s["G"][j], Ms)
            A = _lags(counts)
        o, g = _scv_exact(A, delta, s["G"][j], s["X"][j].shape[0], s["vech"][at:at + b])
        obj.append(o)
        grad.append(g)
        at += b
    obj, grad = torch.cat(obj), torch.cat(grad)
    if kind == "autograd":
        grad = grad * s["w"].cpu()[:, None]
    return dict(obj=obj, grad=grad)
