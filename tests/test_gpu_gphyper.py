"""GPU parity of elliptical slice sampling on GP-regression hyperparameters
(Sec. 7.2): an O(n^3) Cholesky of the n x n kernel matrix inside every loop
iteration, computed in FP64 by the chain's wavefront (n <= 96) or by a
block with a blocked factorisation (n > 96).  FSM runtime ==
synchronized runtime (vmap and compact) bit for bit; draws match the FP64
oracle per draw (1e-9 relative: both sides FP64, the factorisations add up
in different orders)."""
import numpy as np
import pytest
import torch

import parity
from oracle import oracle as O
from paper_2503_17405_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2503_17405_amd import fsmmc
    return fsmmc


@pytest.fixture(scope="module")
def ctx(F):
    c = F.Context(0)
    yield c
    c.close()


def target(F, w):
    return F.gp_hyper_target(torch.tensor(w["X"], device="cuda"), torch.tensor(w["y"], device="cuda"),
                             w["jitter"])


def run(F, ctx, w, m, n, seed, runtime="fsm", max_steps=0, x0=None):
    x0t = None if x0 is None else torch.tensor(x0, device="cuda")
    job = F.Job(ctx, target(F, w), F.ess_sampler(F.F64), m, n, seed, x0=x0t)
    try:
        if runtime == "fsm":
            for _ in range(100000):
                if job.step_fsm(max_steps):
                    break
        else:
            assert job.step_synchronized(n, F.SYNC_VMAP if runtime == "vmap" else F.SYNC_COMPACT)
        return job.samples(), job.counts(), job.stats()
    finally:
        job.free()


@pytest.mark.parametrize("nobs,m,n", [(40, 96, 30), (300, 24, 6)])
def test_gphyper_runtimes_bit_exact(F, ctx, nobs, m, n):
    w = inputs.gp_hyper(n=nobs, seed=11)
    seed = 12
    S0, C0, st0 = run(F, ctx, w, m, n, seed, runtime="vmap")
    for runtime, steps in [("fsm", 0), ("fsm", 3), ("compact", 0)]:
        S, C, st = run(F, ctx, w, m, n, seed, runtime, steps)
        assert np.array_equal(S, S0) and np.array_equal(C, C0), (runtime, steps)
        assert st["steps"] == C.sum()
    assert st0["steps"] + st0["padded_steps"] == m * C0.max(axis=0).sum()
    assert st0["guard_trips"] == 0 and np.isfinite(S0).all()
    print("GP hyper n=%d: mean evaluations %.2f, mean max over %d chains %.1f, R %.2f"
          % (nobs, C0.mean(), m, C0.max(axis=0).mean(), st0["r_hat"]))


@pytest.mark.parametrize("nobs", [1, 25, 64, 65, 96, 97, 100, 128, 129, 250, 414])
def test_gphyper_oracle_parity(F, ctx, nobs):
    # up to 96: the chain's wave (one row per lane up to 64, two above);
    # 97 .. 414: the block factorisation (a ragged last panel at 97, 100, 129,
    # 250 and 414; 414 is the paper's data size)
    m = 32 if nobs <= 128 else 8
    w = inputs.gp_hyper(n=nobs, n_chains=m, seed=20 + nobs)
    n, seed = (100 if nobs < 96 else 40 if nobs <= 128 else 12), 21 + nobs
    x0 = w["x0"]
    S, C, _ = run(F, ctx, w, m, n, seed, x0=x0)
    tg = O.gp_hyper_target(w["X"], w["y"], w["jitter"])
    sp = O.ess_sampler(np.eye(3))
    R, RC, _ = O.run_chains(tg, sp, seed, range(m), n, x0=x0)
    r = parity.check_chains(S, C, R, RC, tg, sp, seed, range(m), x0, first=n, tol=1e-9)
    print(parity.summary("GP hyper n=%d" % nobs, r))
    assert r["worst"] <= 1e-9 and not r["bad"]
    assert r["flip_frac"] <= 0.05


def test_gphyper_default_start(F, ctx):
    # no x0: theta0 from the prior on the INIT stream, as the oracle's ESS start
    w = inputs.gp_hyper(n=10, seed=3)
    m, n, seed = 16, 50, 4
    S, C, _ = run(F, ctx, w, m, n, seed)
    tg = O.gp_hyper_target(w["X"], w["y"], w["jitter"])
    sp = O.ess_sampler(np.eye(3))
    R, RC, _ = O.run_chains(tg, sp, seed, range(m), n)
    x_init = np.array([O.ess_init(np.eye(3), seed, j) for j in range(m)])
    r = parity.check_chains(S, C, R, RC, tg, sp, seed, range(m), x_init, first=n, tol=1e-9)
    assert r["worst"] <= 1e-9 and not r["bad"]


def test_gphyper_argument_errors(F, ctx):
    w = inputs.gp_hyper(n=513, seed=1)
    with pytest.raises(F.FsmmcError) as e:
        F.Job(ctx, target(F, w), F.ess_sampler(F.F64), 4, 4, 1)
    assert e.value.status == F.ENOTSUP
    w = inputs.gp_hyper(n=10, seed=1)
    with pytest.raises(F.FsmmcError) as e:
        F.Job(ctx, target(F, w), F.ess_sampler(F.F32), 4, 4, 1)
    assert e.value.status == F.ENOTSUP


@pytest.mark.parametrize("nobs", [15, 16, 17, 31, 32, 63, 127, 191, 192, 255, 256, 257, 271, 272, 511, 512])
def test_gphyper_tile_edges(F, ctx, nobs):
    # the factorisation's 16 x 16 tiles: one short of, at and past a tile; the
    # largest of each block class (31, 63, 127, 191, 255) and the smallest of the
    # next; leading columns through memory from 256 on (1 to 17 of them).
    # 1e-9 as above: both sides FP64, sums in different orders
    m, n, seed = 6, 4, 31 + nobs
    w = inputs.gp_hyper(n=nobs, n_chains=m, seed=40 + nobs)
    S, C, _ = run(F, ctx, w, m, n, seed, x0=w["x0"])
    tg = O.gp_hyper_target(w["X"], w["y"], w["jitter"])
    sp = O.ess_sampler(np.eye(3))
    R, RC, _ = O.run_chains(tg, sp, seed, range(m), n, x0=w["x0"])
    r = parity.check_chains(S, C, R, RC, tg, sp, seed, range(m), w["x0"], first=n, tol=1e-9)
    assert r["worst"] <= 1e-9 and not r["bad"]


@pytest.mark.parametrize("nobs", [5, 40, 300])
def test_gphyper_singular_start(F, ctx, nobs):
    # tau = 1, lambda = sigma = 0 and no jitter: C is all ones, its second pivot
    # exactly 0, log L = -inf; the first proposal with a finite value is taken
    m, n, seed = 4, 5, 77
    w = inputs.gp_hyper(n=nobs, n_chains=m, seed=78)
    x0 = np.tile(np.array([1.0, 0.0, 0.0]), (m, 1))
    w["jitter"] = 0.0
    S, C, _ = run(F, ctx, w, m, n, seed, x0=x0)
    tg = O.gp_hyper_target(w["X"], w["y"], 0.0)
    sp = O.ess_sampler(np.eye(3))
    R, RC, _ = O.run_chains(tg, sp, seed, range(m), n, x0=x0)
    assert np.array_equal(C, RC) and np.all(C[:, 0] == 1)
    assert np.abs(S - R).max() <= 1e-9


@pytest.mark.parametrize("nobs,m", [(5, 3), (31, 2), (64, 16), (96, 7), (97, 1), (100, 30), (128, 2), (300, 1), (512, 1), (512, 9)])
def test_gphyper_under_a_budget(F, ctx, nobs, m):
    """A budget of the chain state, the data and (above 96 observations) a work
    matrix per chain is enough at every size: where the squared distances do not
    fit it, the kernels form them, with the same bits."""
    n, seed = 4, 91
    w = inputs.gp_hyper(n=nobs, n_chains=m, seed=92)
    S0, C0, _ = run(F, ctx, w, m, n, seed, x0=w["x0"])
    N, p, ld = nobs, w["X"].shape[1], (nobs + 31) // 32 * 32
    state = m * (3 * 4 + 8 + 8 + 4 * n + n * 24 + 2 * 24 + 5 * 8) + 64 + 4 * n + 64 + N * p * 8 + N * 8
    tight = F.Context(0, hbm_budget_bytes=state + (m * ld * ld * 8 if N > 96 else 0))
    try:
        for runtime, steps in (("fsm", 0), ("vmap", 0)):
            S, C, _ = run(F, tight, w, m, n, seed, runtime, steps, x0=w["x0"])
            assert np.array_equal(S, S0) and np.array_equal(C, C0)
    finally:
        tight.close()
