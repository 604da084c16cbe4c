"""The work that users of this library have it do, as cases that can be timed and compared.

A case is one whole sampling job through the Python binding -- init_chains, every chain
to its last draw with the FSM runtime, free -- or one call of the potential on a job that
the caller keeps, or one batch of unlike jobs.  Sizes are those of the benchmark, the
tests and the serving mix (chains, dimensions, rows and observations), with fewer draws
where a full job would take seconds.

    listed()            the fixed cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) target arrays, starts and output buffers on the GPU
    run(state)          one pass; returns the draws (and loop counts), or U and its gradient
    work(case)          bytes and operations one pass cannot do without
    exact(case, seed)   the outputs in 64 bits, where a chain's path does not hang on rounding
"""
import math

import numpy as np
import torch

from paper_2503_17405_amd import fsmmc as F
from paper_2503_17405_amd import inputs

# Mean loop counts per draw that the workloads show (log-likelihoods, leapfrogs, tries,
# density evaluations); used to price the work only.
LOOPS = dict(ess_gauss=8, ess_logistic=7, nuts_logreg=5, nuts_mixture=7.5, gp_hyper=6, dr=2, drsym=1.6, slice=7.5)

# The benchmark's leapfrog step on logistic regression.  At depth 10 a posterior whose
# period meets a power of two of leapfrogs can take hundreds of them per draw; drawn cases
# cap the depth at 6 so that their length is known.
STEP = 0.05


def listed():
    return [
        # latent GP regression in FP64, the closed-form posterior: few chains, tiny vectors
        dict(name="ess_gauss_d16_f64", kind="ess_gauss", dim=16, chains=64, draws=1000),
        # the benchmark's headline target and chain count (a fifth of its draws)
        dict(name="ess_logistic_d1024", kind="ess_logistic", dim=1024, chains=8192, draws=400),
        # the smallest job of the serving mix: a handful of chains on a small regression
        dict(name="nuts_logreg_c16_d10", kind="nuts_logreg", chains=16, dim=10, rows=1000, depth=10, draws=200),
        # the benchmark's logistic regression at its configured chain count
        dict(name="nuts_logreg_c4096_d100", kind="nuts_logreg", chains=4096, dim=100, rows=10000, depth=10,
             draws=100),
        # U and its gradient for a caller's own loop (step-size search, diagnostics)
        dict(name="potential_p4096_d100", kind="potential", chains=4096, dim=100, rows=10000),
        # the 100-D correlated mixture, the paper's larger chain count
        dict(name="nuts_mixture_c500_d100", kind="nuts_mixture", chains=500, dim=100, draws=200),
        # GP hyperparameters: a Cholesky in every loop, at a middling and at the paper's data size
        dict(name="gp_hyper_n100", kind="gp_hyper", obs=100, chains=1024, draws=60),
        dict(name="gp_hyper_n414", kind="gp_hyper", obs=414, chains=512, draws=16),
        # delayed rejection on the funnel, many chains
        dict(name="dr_funnel_c65536", kind="dr", dim=10, chains=65536, draws=500),
        # symmetric delayed rejection on N(0, 1), the paper's chain count
        dict(name="drsym_c1024", kind="drsym", dim=1, chains=1024, draws=2000),
        # slice sampling on the funnel
        dict(name="slice_funnel_c1024", kind="slice", dim=10, chains=1024, draws=500),
        # unlike jobs stepped together: four GP targets, a regression and a funnel
        dict(name="batch_mixed", kind="batch", dims="1000,417,256,96", chains=512, draws=200, funnel=8192),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["ess_gauss", "ess_logistic", "nuts_logreg", "potential", "nuts_mixture", "gp_hyper", "gp_hyper",
                       "dr", "drsym", "slice", "batch"])
    if kind == "ess_gauss":
        return dict(kind=kind, dim=_log_int(rng, 8, 64), chains=_log_int(rng, 32, 1024), draws=_log_int(rng, 100, 1000))
    if kind == "ess_logistic":
        dim, chains = _log_int(rng, 64, 1024), _log_int(rng, 16, 8192)
        return dict(kind=kind, dim=dim, chains=chains, draws=min(_log_int(rng, 100, 2000), 2 ** 31 // (dim * chains)))
    if kind == "nuts_logreg":
        chains = _log_int(rng, 16, 4096)
        return dict(kind=kind, chains=chains, dim=_log_int(rng, 10, 100), rows=_log_int(rng, 1000, 10000),
                    depth=6, draws=min(_log_int(rng, 20, 200), max(20, 2 ** 17 // chains)))
    if kind == "potential":
        return dict(kind=kind, chains=_log_int(rng, 1, 4096), dim=_log_int(rng, 2, 100), rows=_log_int(rng, 100, 10000))
    if kind == "nuts_mixture":
        return dict(kind=kind, chains=_log_int(rng, 50, 2048), dim=rng.randint(90, 110), draws=_log_int(rng, 20, 200))
    if kind == "gp_hyper":
        obs = _log_int(rng, 16, 414)
        chains = _log_int(rng, 64, 1024)
        most = 1.6e11 / (chains * max(obs, 40) ** 3)
        return dict(kind=kind, obs=obs, chains=chains, draws=max(2, min(200, int(most))))
    if kind == "dr":
        return dict(kind=kind, dim=rng.randint(2, 16), chains=_log_int(rng, 256, 65536), draws=_log_int(rng, 50, 500))
    if kind == "drsym":
        return dict(kind=kind, dim=rng.randint(1, 4), chains=_log_int(rng, 256, 65536), draws=_log_int(rng, 100, 2000))
    if kind == "slice":
        return dict(kind=kind, dim=rng.randint(2, 16), chains=_log_int(rng, 256, 65536), draws=_log_int(rng, 50, 500))
    dims = ",".join(str(_log_int(rng, 64, 1000)) for _ in range(rng.randint(2, 4)))
    return dict(kind="batch", dims=dims, chains=_log_int(rng, 128, 512), draws=_log_int(rng, 50, 200),
                funnel=_log_int(rng, 1024, 8192))


# ------------------------------------------------------------------ inputs
def _dev(a, dtype=torch.float32):
    return torch.tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


class State:
    """What a caller holds: the context, targets, samplers, starts and output buffers."""

    def __init__(self):
        self.ctx = F.Context(0)
        self.jobs = []  # (target, sampler, chains, draws, seed, x0, out)
        self.kept = None  # a job that the caller keeps between calls

    def add(self, target, sampler, chains, draws, seed, dim, x0=None):
        t = torch.float32 if sampler.dtype == F.F32 else torch.float64
        out = torch.zeros((chains, draws, dim), dtype=t, device="cuda")
        self.jobs.append((target, sampler, chains, draws, seed, x0, out))

    def __del__(self):
        if self.kept is not None:
            self.kept.free()
        self.ctx.close()


def _regression(case, seed):
    d = inputs.logreg(n_data=case["rows"], dim=case["dim"], seed=seed)
    lap = inputs.logreg_laplace(d["X"], d["y"], case["chains"], seed=seed + 1)
    return d, lap


def _gp_data(case, seed):
    if case["kind"] == "ess_gauss":
        return inputs.gp_gauss(dim=case["dim"], seed=seed)
    return inputs.gp_logistic(dim=case["dim"], seed=seed)


def prepare(case, seed):
    kind, s = case["kind"], State()
    s.kind = kind
    data, chain = 2 * seed + 1, 1000003 * seed + 17
    if kind == "ess_gauss":
        w = _gp_data(case, data)
        f64 = torch.float64
        s.add(F.gp_target(_dev(w["L"], f64), _dev(w["y"], f64), w["noise_sd"]), F.ess_sampler(F.F64), case["chains"],
              case["draws"], chain, case["dim"])
    elif kind == "ess_logistic":
        w = _gp_data(case, data)
        s.add(F.gp_target(_dev(w["L"]), _dev(w["y"])), F.ess_sampler(F.F32), case["chains"], case["draws"], chain,
              case["dim"])
    elif kind == "nuts_logreg":
        d, lap = _regression(case, data)
        s.add(F.logreg_target(_dev(d["X"]), _dev(d["y"])), F.nuts_sampler(STEP, case["depth"]), case["chains"], case["draws"],
              chain, case["dim"], _dev(lap["x0"]))
    elif kind == "potential":
        d, lap = _regression(case, data)
        s.theta = _dev(lap["x0"])
        s.kept = F.Job(s.ctx, F.logreg_target(_dev(d["X"]), _dev(d["y"])), F.nuts_sampler(STEP, 10), case["chains"], 1,
                       chain)
    elif kind == "nuts_mixture":
        w = inputs.mog(dim=case["dim"], n_chains=case["chains"], seed=data)
        s.add(F.mog_target(_dev(w["means"]), _dev(w["log_weights"]), _dev(w["prec"])), F.nuts_sampler(0.0473, 10),
              case["chains"], case["draws"], chain, case["dim"], _dev(w["x0"]))
    elif kind == "gp_hyper":
        w = inputs.gp_hyper(n=case["obs"], n_chains=case["chains"], seed=data)
        f64 = torch.float64
        s.add(F.gp_hyper_target(_dev(w["X"], f64), _dev(w["y"], f64), w["jitter"]), F.ess_sampler(F.F64),
              case["chains"], case["draws"], chain, 3, _dev(w["x0"], f64))
    elif kind == "dr":
        s.add(F.funnel_target(case["dim"]), F.dr_sampler(), case["chains"], case["draws"], chain, case["dim"])
    elif kind == "drsym":
        s.add(F.gauss_target(torch.ones(case["dim"], device="cuda")), F.drsym_sampler(100, 0.1), case["chains"],
              case["draws"], chain, case["dim"])
    elif kind == "slice":
        s.add(F.funnel_target(case["dim"]), F.slice_sampler(1.0), case["chains"], case["draws"], chain, case["dim"])
    else:
        m, n = case["chains"], case["draws"]
        for i, dim in enumerate(_dims(case)):
            w = inputs.gp_logistic(dim=dim, seed=data + i)
            s.add(F.gp_target(_dev(w["L"]), _dev(w["y"])), F.ess_sampler(F.F32), m, n, chain + i, dim)
        small = _small_regression(case)
        d, lap = _regression(small, data)
        s.add(F.logreg_target(_dev(d["X"]), _dev(d["y"])), F.nuts_sampler(STEP, small["depth"]), small["chains"], small["draws"],
              chain + 50, small["dim"], _dev(lap["x0"]))
        s.add(F.funnel_target(10), F.dr_sampler(), case["funnel"], n, chain + 60, 10)
    return s


def _dims(case):
    return [int(v) for v in case["dims"].split(",")]


def _small_regression(case):
    return dict(chains=case["chains"] // 4, dim=20, rows=2000, depth=6, draws=max(10, case["draws"] // 8))


# ------------------------------------------------------------------ one pass
def run(s):
    if s.kind == "potential":
        U, g = s.kept.potential(s.theta)
        return dict(U=U, grad=g)
    if s.kind == "batch":
        jobs = [F.Job(s.ctx, tg, smp, m, n, seed, x0=x0, out=out) for tg, smp, m, n, seed, x0, out in s.jobs]
        b = F.Batch(s.ctx, jobs)
        b.run(0)
        b.free()
        for j in jobs:
            j.free()
        return [j[-1] for j in s.jobs]
    tg, smp, m, n, seed, x0, out = s.jobs[0]
    job = F.Job(s.ctx, tg, smp, m, n, seed, x0=x0, out=out)
    job.step_fsm(0)
    counts = job.counts() if m * n <= 1 << 18 else None  # small jobs: the loop counts too
    job.free()
    return dict(draws=out) if counts is None else dict(draws=out, counts=counts)


# ------------------------------------------------------------------ the work
def _counts_bytes(case):
    n = case["chains"] * case["draws"]
    return 4 * n if n <= 1 << 18 else 0


def work(case):
    kind = case["kind"]
    if kind == "batch":
        parts = [dict(kind="ess_logistic", dim=d, chains=case["chains"], draws=case["draws"]) for d in _dims(case)]
        parts += [dict(_small_regression(case), kind="nuts_logreg"),
                  dict(kind="dr", dim=10, chains=case["funnel"], draws=case["draws"])]
        w = [work(p) for p in parts]
        return dict(bytes=sum(x["bytes"] for x in w), flops=sum(x["flops"] for x in w))
    m = case["chains"]
    if kind == "potential":
        N, D = case["rows"], case["dim"]
        return dict(bytes=4 * (N * D + N + 2 * m * D + m), flops=4.0 * m * N * D)
    draws, loops = m * case["draws"], LOOPS[kind]
    if kind in ("ess_gauss", "ess_logistic"):  # nu = L z per draw, x' and its log-likelihood per loop
        D, es = case["dim"], 8 if kind == "ess_gauss" else 4
        return dict(bytes=es * (draws * D + D * (D + 1) // 2 + D) + _counts_bytes(case),
                    flops=draws * (D * (D + 1.0) + loops * 8.0 * D))
    if kind == "nuts_logreg":
        N, D = case["rows"], case["dim"]
        return dict(bytes=4 * (draws * D + N * D + N + m * D) + _counts_bytes(case), flops=draws * loops * 4.0 * N * D)
    if kind == "nuts_mixture":
        D = case["dim"]
        return dict(bytes=4 * (draws * D + D * D + 4 * D + m * D) + _counts_bytes(case), flops=draws * loops * 2.0 * D * D)
    if kind == "gp_hyper":
        n = case["obs"]
        return dict(bytes=8 * (3 * draws + 7 * n + 3 * m) + _counts_bytes(case),
                    flops=draws * loops * (n ** 3 / 3.0 + 12.0 * n * n))
    D = case["dim"]  # lane-per-chain samplers: a proposal (normals included) and a density per loop
    return dict(bytes=4 * draws * D + _counts_bytes(case), flops=draws * loops * (150.0 + 25.0 * D))


# ------------------------------------------------------------------ 64-bit values
# Philox4x32-10 streams and the maps to uniforms and normals as include/fsmmc.h's random
# streams define them: block (chain, draw, role << 24 | sub, block) under the 64-bit seed.
ROLE_NU, ROLE_INIT, ROLE_THRESH, ROLE_ANGLE = 1, 2, 3, 4


def _philox(seed, chain, draw_, role, sub, block):
    u = np.uint64
    lo = u(0xFFFFFFFF)
    x, y, z, w = [np.asarray(v, dtype=u) for v in np.broadcast_arrays(chain, draw_, (role << 24) | np.asarray(sub), block)]
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = u(0xD2511F53) * x, u(0xCD9E8D57) * z
        x, y, z, w = (p1 >> u(32)) ^ y ^ u(k0), p1 & lo, (p0 >> u(32)) ^ w ^ u(k1), p0 & lo
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return x, y, z, w


def _u01(w):
    return ((w >> np.uint64(9)).astype(np.float64) + 0.5) * 2.0 ** -23


def _uniform(seed, chain, draw_, role, sub):
    return _u01(_philox(seed, chain, draw_, role, sub, 0)[0])


def _normals(seed, chain, draw_, role, dim):
    """(len(chain), dim) normals of the vector streams of (chain, draw)."""
    nb = (dim + 3) // 4
    b = np.broadcast_to(np.arange(nb), (len(chain), nb))
    w = [_u01(v) for v in _philox(seed, chain[:, None], np.asarray(draw_)[:, None], role, 0, b)]
    z = []
    for u1, u2 in ((w[0], w[1]), (w[2], w[3])):
        r = np.sqrt(-2.0 * np.log(u1))
        z += [r * np.cos(2 * np.pi * u2), r * np.sin(2 * np.pi * u2)]
    return np.stack(z, axis=-1).reshape(len(chain), 4 * nb)[:, :dim]


def _ess_exact(m, n, dim, seed, x, direction, loglik):
    """Elliptical slice sampling in FP64, every chain at its own pace; (draws, loop counts)."""
    ids = np.arange(m)
    out, counts = np.zeros((m, n, dim)), np.zeros((m, n), dtype=np.int32)
    lx = loglik(x)
    t, k = np.zeros(m, dtype=np.int64), np.zeros(m, dtype=np.int64)
    nu = direction(ids, t)
    logu = np.log(_uniform(seed, ids, t, ROLE_THRESH, 0))
    phi = 2 * np.pi * _uniform(seed, ids, t, ROLE_ANGLE, 0)
    lo, hi = phi - 2 * np.pi, phi.copy()
    while True:
        a = np.nonzero(t < n)[0]
        if a.size == 0:
            return out, counts
        xp = x[a] * np.cos(phi[a])[:, None] + nu[a] * np.sin(phi[a])[:, None]
        lp = loglik(xp)
        k[a] += 1
        ok = lp - lx[a] > logu[a]
        d, r = a[ok], a[~ok]
        x[d], lx[d] = xp[ok], lp[ok]
        out[d, t[d]], counts[d, t[d]] = x[d], k[d]
        t[d] += 1
        k[d] = 0
        if d.size:
            nu[d] = direction(d, t[d])
            logu[d] = np.log(_uniform(seed, d, t[d], ROLE_THRESH, 0))
            phi[d] = 2 * np.pi * _uniform(seed, d, t[d], ROLE_ANGLE, 0)
            lo[d], hi[d] = phi[d] - 2 * np.pi, phi[d]
        neg = phi[r] < 0
        lo[r] = np.where(neg, phi[r], lo[r])
        hi[r] = np.where(neg, hi[r], phi[r])
        phi[r] = lo[r] + (hi[r] - lo[r]) * _uniform(seed, r, t[r], ROLE_ANGLE, k[r])


def exact(case, seed):
    """FP32 chains have no 64-bit value to be held to: their accept decisions turn on
    rounding now and then, and a chain's path parts there for good.  The potential and
    the FP64 samplers do."""
    kind, data, chain = case["kind"], 2 * seed + 1, 1000003 * seed + 17
    if kind == "potential":
        d, lap = _regression(case, data)
        X, y = (_dev(d[k]).double() for k in ("X", "y"))
        th = _dev(lap["x0"]).double()
        eta = th @ X.T
        U = 0.5 * (th * th).sum(1) - (eta @ y - torch.nn.functional.softplus(eta, threshold=1e9).sum(1))
        return dict(U=U, grad=th - (y - torch.sigmoid(eta)) @ X)
    if kind not in ("ess_gauss", "gp_hyper") or case["chains"] * case["draws"] > 1 << 18:
        return None
    m, n = case["chains"], case["draws"]
    if kind == "ess_gauss":
        w = _gp_data(case, data)
        D, L, y, iv = case["dim"], w["L"], w["y"], 1.0 / (2.0 * w["noise_sd"] ** 2)
        x = _normals(chain, np.arange(m), np.zeros(m, dtype=np.int64), ROLE_INIT, D) @ L.T
        out, counts = _ess_exact(m, n, D, chain, x, lambda c, t: _normals(chain, c, t, ROLE_NU, D) @ L.T,
                                 lambda f: -((y - f) ** 2).sum(1) * iv)
        return dict(draws=out, counts=None)
    w = inputs.gp_hyper(n=case["obs"], n_chains=m, seed=data)
    X, y = _dev(w["X"], torch.float64), _dev(w["y"], torch.float64)
    r2 = ((X[:, None, :] - X[None, :, :]) ** 2).sum(2)
    eye = torch.eye(case["obs"], dtype=torch.float64, device="cuda")

    def loglik(theta):
        th = torch.tensor(theta, device="cuda")[:, :, None, None] ** 2
        C = th[:, 0] * torch.exp(-th[:, 1] * r2) + (th[:, 2] + w["jitter"]) * eye
        L, info = torch.linalg.cholesky_ex(C)
        z = torch.linalg.solve_triangular(L, y[:, None].expand(len(theta), -1, 1), upper=False)[:, :, 0]
        ll = -0.5 * (z * z).sum(1) - torch.diagonal(L, dim1=1, dim2=2).log().sum(1)
        return torch.where(info == 0, ll, torch.full_like(ll, -math.inf)).cpu().numpy()

    out, _ = _ess_exact(m, n, 3, chain, w["x0"].copy(), lambda c, t: _normals(chain, c, t, ROLE_NU, 3), loglik)
    return dict(draws=out, counts=None)
