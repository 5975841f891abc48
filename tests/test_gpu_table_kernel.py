"""The table-driven step kernel where calls still reach it by themselves: instances
that the wave and team kernels do not take.  Tempering with per-draw estimates
(fields near the int32 range), batches of dense jobs with a common factor past 16
bits, and short schedules whose launch shape is timed first.  Bit-exact against
the oracle."""
import numpy as np
import pytest

import oracle
from paper_1806_08815_amd import instances

pytestmark = pytest.mark.gpu

KEYS = ("best_x", "best_E", "final_x", "final_E", "n_accept")


@pytest.fixture(scope="module")
def api():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_1806_08815_amd import api as a
    a.lib()
    return a


def _field_bound(Q):
    W = Q.astype(np.int64) + Q.T.astype(np.int64)
    np.fill_diagonal(W, 0)
    return int((np.abs(W).sum(axis=1) + np.abs(np.diag(Q).astype(np.int64))).max())


def _large_fields(N, seed):
    """Fields up to about 2^30 - 2^23, couplings around 2^21, no common factor."""
    g = np.random.default_rng(seed)
    q = (2**30 - 2**23) // (N - 1)
    mag = q - g.integers(0, 1000, size=(N, N))
    return np.triu(mag * g.choice([-1, 1], size=(N, N)), 1).astype(np.int32)


@pytest.mark.parametrize("chains", [2, 40])
def test_tempering_estimates(api, chains):
    """Few replicas: estimates from random-number waves; many: from the compute
    lanes under lazy draws."""
    N, M, K, rounds = 700, 16, 300, 6
    Q = _large_fields(N, 4)
    hb = _field_bound(Q)
    temps = np.geomspace(1e4, 2.0**21, M)
    # past the wave kernels' int32 sums, within the estimates' bound
    assert 2 * hb + 11.8 * temps[-1] > 2**31 and hb <= 2**30 - 2**22 - 256
    ctx = api.da_create(Q)
    gpu = api.da_pt(ctx, temps, chains, rounds, K, 2**16, 11)
    st = api.da_last_kernel_stats(ctx)
    assert st["draw_estimates"] == 1 and (st["rng_waves"] > 0) == (chains == 2)
    c = chains - 1
    ref = oracle.pt(Q, temps, chains=1, rounds=rounds, steps_per_round=K, eoff_inc=2**16,
                    seed=11, chain_base=c)
    rows = slice(c * M, (c + 1) * M)
    for k in KEYS + ("slot",):
        assert np.array_equal(gpu[k][rows], ref[k]), k


@pytest.mark.parametrize("trial", ["parallel", "single"])
@pytest.mark.parametrize("beside", [False, True])
def test_dense_batch(api, trial, beside):
    """Dense jobs of a factor of 2^15 in int16, with and without per-draw estimates,
    alone or beside jobs of the wave kernels."""
    import torch
    f = 2**15
    g = np.random.default_rng(3)
    specs = []
    for N, lim, R in ((300, 60, 5), (64, 1, 9), (1100, 1, 2)):
        Q = np.triu(g.integers(-lim, lim + 1, size=(N, N)), 1).astype(np.int32) * f
        specs.append((Q, 2, R, 3e5, 1e4, trial))
    if beside:
        for N, R in ((50, 7), (600, 3)):
            Q = instances.ising_to_qubo(instances.sk_bimodal(N, 2))[0]
            specs.append((Q, 0, R, 30.0, 1.0, "parallel"))
    items = []
    for a, (Q, hint, R, T_hi, T_lo, tr) in enumerate(specs):
        sch = api.schedule(T_hi, T_lo, "geometric", 5, eoff_inc=f if hint else 1, init="random",
                           trial=tr)
        ctx = api.da_create(Q, hint)
        assert (ctx.info()["wscale"] >= f) == (hint == 2)
        items.append(dict(ctx=ctx, schedule=sch, replicas=R, steps=400, seed=20 + a,
                          out_dev=api.device_outputs(R, Q.shape[0])))
    api.da_anneal_batch(items)
    torch.cuda.synchronize()
    st = api.da_last_kernel_stats(items[0]["ctx"])
    assert st["threads"] == 1024 and st["draw_estimates"] == (1 if trial == "parallel" else 0)
    for a, (Q, hint, R, T_hi, T_lo, tr) in enumerate(specs):
        for r in (0, R - 1):
            ref = oracle.anneal(Q, T_hi=T_hi, T_lo=T_lo, n_levels=5, eoff_inc=f if hint else 1,
                                init=1, trial=int(tr == "single"), replica_base=r, replicas=1,
                                steps=400, seed=20 + a)
            for k in KEYS:
                assert np.array_equal(items[a]["out_dev"][k].cpu().numpy()[r], ref[k][0]), (a, r, k)


@pytest.mark.parametrize("N,S,L", [(71, 100, 128), (93, 65, 128), (111, 300, 64), (133, 575, 128)])
@pytest.mark.parametrize("form", ["sparse", "factor"])
def test_timed_short_schedules(api, N, S, L, form):
    """Fewer than 576 steps, on contexts whose launch shape is timed: the window it
    is timed on stays inside the schedule.  Each N is new to the process."""
    Q = instances.random_qubo(N, 31, lo=-3, hi=3)
    f = 1 if form == "sparse" else 2**15
    N += form == "factor"
    Q = np.pad(Q, ((0, N - Q.shape[0]),) * 2).astype(np.int32) * f
    ctx = api.da_create(Q, api.DA_STORE_SPARSE if form == "sparse" else 2)
    sch = api.schedule(20.0 * f, 1.0 * f, "geometric", L, eoff_inc=2 * f)
    gpu = api.da_anneal(ctx, sch, 3, S, 9)
    ref = oracle.anneal(Q, T_hi=20.0 * f, T_lo=1.0 * f, n_levels=L, eoff_inc=2 * f, replicas=3,
                        steps=S, seed=9)
    for k in KEYS:
        assert np.array_equal(gpu[k], ref[k]), k


def test_served_jobs(api):
    """Jobs of both kernels in one server, epochs that cut levels and steps."""
    f = 2**15
    g = np.random.default_rng(8)
    jobs = []
    for N, R, S in ((90, 5, 1000), (300, 3, 700)):
        Q = np.triu(g.integers(-2, 3, size=(N, N)), 1).astype(np.int32) * f
        jobs.append((Q, api.schedule(3e5, 1e4, "geometric", 6, eoff_inc=f), R, S, N, 2))
    Q = instances.ising_to_qubo(instances.sk_bimodal(70, 2))[0]
    jobs.append((Q, api.schedule(30.0, 1.0, "geometric", 6, eoff_inc=1), 9, 900, 1, 0))
    want = [api.da_anneal(api.da_create(Q, hint), sch, R, S, seed)
            for Q, sch, R, S, seed, hint in jobs]
    srv = api.da_server_create(1 << 30, epoch_steps=151)
    tickets = [api.da_submit(srv, Q, sch, R, S, seed, hint) for Q, sch, R, S, seed, hint in jobs]
    got = [api.da_wait(srv, t) for t in tickets]
    srv.close()
    for a, (Q, sch, R, S, seed, hint) in enumerate(jobs):
        ref = oracle.anneal(Q, T_hi=sch.T_hi, T_lo=sch.T_lo, n_levels=6, eoff_inc=sch.eoff_inc,
                            replica_base=R - 1, replicas=1, steps=S, seed=seed)
        for k in KEYS:
            assert np.array_equal(got[a][k], want[a][k]), (a, k)
            assert np.array_equal(got[a][k][R - 1], ref[k][0]), (a, k)
