"""The lane-per-chain FSM kernels compiled for each dimension (delayed rejection and
slice sampling): draws, loop counts and step counts are those of the synchronized
runtime bit for bit, for every dimension, for chain counts around a wave and for runs
cut into pieces by a step budget."""
import numpy as np
import pytest
import torch

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


def run(F, ctx, tg, smp, m, n, seed, runtime, budget=0):
    job = F.Job(ctx, tg, smp, m, n, seed)
    try:
        if runtime == "fsm":
            for _ in range(10000):
                if job.step_fsm(budget):
                    break
        else:
            assert job.step_synchronized(n, F.SYNC_COMPACT)
        return job.samples(), job.counts(), job.stats()
    finally:
        job.free()


@pytest.mark.parametrize("sampler", ["dr", "slice"])
@pytest.mark.parametrize("D", list(range(1, 17)))
def test_every_dimension(F, ctx, sampler, D):
    smp = F.dr_sampler((1.0, 0.3, 0.1)) if sampler == "dr" else F.slice_sampler(0.7)
    targets = [F.gauss_target(torch.linspace(0.5, 3.0, D, device="cuda"))]
    if D >= 2:
        targets.append(F.funnel_target(D))
    for tg in targets:
        m, n, seed = (1, 70, 300)[D % 3], 37, 100 + D
        S0, C0, st0 = run(F, ctx, tg, smp, m, n, seed, "sync")
        for budget in (0, 5):
            S, C, st = run(F, ctx, tg, smp, m, n, seed, "fsm", budget)
            assert np.array_equal(S, S0) and np.array_equal(C, C0), budget
            assert st["steps"] == st0["steps"] and st["draws"] == m * n
            assert st["lane_slots"] >= st["active_lanes"] and st["lane_slots"] % 64 == 0


def test_slice_window_edges(F, ctx):
    # draws around the 256-draw window, and many chains (64 per wave)
    for m, n in ((3, 255), (3, 256), (3, 257), (20000, 3)):
        tg, smp = F.funnel_target(5), F.slice_sampler(1.0)
        S0, C0, _ = run(F, ctx, tg, smp, m, n, 9, "sync")
        S, C, _ = run(F, ctx, tg, smp, m, n, 9, "fsm")
        assert np.array_equal(S, S0) and np.array_equal(C, C0), (m, n)
