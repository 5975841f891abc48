"""The step kernels of one wave and of teams of waves (chosen by da_anneal)
against the CPU oracle: every number of flips per lane at its smallest and largest N and at
ragged ones, every coupling type with W in LDS and in global memory, couplings
from +-1 to 10^7 (fixed point with and without fraction bits, brackets from two
units to hundreds), levels that change the fixed point, schedules with more
levels than steps, per-step schedules, single trials, T = 0, large offsets, and
replica counts that share workgroups.  Whole numbers: bit-exact."""
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


def _instance(kind, N, seed=5):
    """Q, hottest and coldest temperature, offset increment."""
    if kind == "sk":
        u = max(1.0, N ** 0.5)
        return instances.ising_to_qubo(instances.sk_bimodal(N, seed))[0], 3.0 * u, 0.05 * u, 1
    if kind == "cold":   # degenerate flips at temperatures far below a coupling
        return instances.ising_to_qubo(instances.sk_bimodal(N, seed))[0], 1.0, 0.01, 1
    if kind == "gauss":
        q = instances.ising_to_qubo(instances.sk_gaussian(N, seed, scale=2**16))[0]
        return q, 3.0 * 2**16, 0.05 * 2**16, 2**16
    lim = int(kind[1:])  # qLIM: dense, coefficients up to LIM
    q = instances.random_qubo(N, seed, lo=-lim, hi=lim)
    u = 0.5 * lim * N ** 0.5
    return q, 3.0 * u, 0.05 * u, lim


def _check(api, Q, dtype, R, S, L, T_hi, T_lo, inc, kind="geometric", init="zeros",
           trial="parallel", seed=11):
    ctx = api.da_create(Q, dtype)
    sch = api.schedule(T_hi, T_lo, kind, L, eoff_inc=inc, init=init, trial=trial)
    gpu = api.da_anneal(ctx, sch, R, S, seed)
    rows = sorted({0, R // 2, R - 1})
    for r in rows:
        ref = oracle.anneal(Q, T_hi=T_hi, T_lo=T_lo, kind=int(kind != "geometric"), n_levels=L,
                            eoff_inc=inc, init=int(init != "zeros"), trial=int(trial != "parallel"),
                            replica_base=r, replicas=1, steps=S, seed=seed)
        for k in KEYS:
            assert np.array_equal(gpu[k][r], ref[k][0]), (k, r)
    return ctx


@pytest.mark.parametrize("kind", ["sk", "cold", "gauss", "q100", "q100000"])
@pytest.mark.parametrize("N", [1, 2, 33, 64, 65, 127, 128, 129, 200, 256, 257, 449, 500, 512])
def test_sizes(api, kind, N):
    Q, T_hi, T_lo, inc = _instance(kind, N)
    ctx = _check(api, Q, 0, 3, 1500, 12, T_hi, T_lo, inc, init="random" if N % 2 else "zeros")
    assert api.da_last_kernel_stats(ctx)["rng_waves"] == 0


@pytest.mark.parametrize("dtype", [1, 2, 4])
@pytest.mark.parametrize("kind,N,R", [("sk", 64, 600), ("sk", 100, 700), ("sk", 180, 520),
                                      ("sk", 250, 300), ("sk", 390, 260), ("sk", 460, 1100)])
def test_types_and_shared_workgroups(api, kind, N, R, dtype):
    Q, T_hi, T_lo, inc = _instance(kind, N)
    _check(api, Q, dtype, R, 400, 6, T_hi, T_lo, inc)


@pytest.mark.parametrize("N", [20, 90, 210, 400])
@pytest.mark.parametrize("kind,L,S,extra", [
    ("sk", 700, 300, {}),                              # levels skipped
    ("gauss", 1, 300, {}),
    ("sk", 0, 700, dict(kind="linear_beta")),          # a new temperature every step
    ("gauss", 0, 300, dict(init="random")),
    ("sk", 5, 900, dict(trial="single")),
    ("q100", 0, 900, dict(trial="single")),
    ("q100", 3, 0, {}), ("sk", 0, 1, {}),
])
def test_schedules(api, N, kind, L, S, extra):
    Q, T_hi, T_lo, inc = _instance(kind, N)
    _check(api, Q, 0, 3, S, L, T_hi, T_lo, inc, **extra)


@pytest.mark.parametrize("N", [40, 130, 300])
@pytest.mark.parametrize("inc", [0, 7, 2**30, 2**31 - 1])
def test_zero_temperature_and_offsets(api, N, inc):
    Q = instances.random_qubo(N, 3, lo=-300, hi=300)
    _check(api, Q, 0, 3, 400, 4, 0.0, 0.0, inc)
    _check(api, Q, 0, 3, 200, 0, 0.0, 0.0, inc)
    _check(api, Q, 0, 3, 400, 4, 200.0, 1e-3, inc)


@pytest.mark.parametrize("scale", [2**10, 2**16, 2**20])
@pytest.mark.parametrize("dtype", [1, 2, 4])
def test_common_factors(api, scale, dtype):
    """Large common factors: few or no fraction bits, or another kernel."""
    Q = instances.ising_to_qubo(instances.sk_bimodal(100, 5))[0] * scale
    _check(api, Q, dtype, 3, 600, 8, 30.0 * scale, 0.1 * scale, scale)
    _check(api, Q, dtype, 3, 300, 8, 30.0, 0.1, 1)    # T far below a coupling


# teams of waves: 8 and 16 flips per lane, random-number waves that draw two
# blocks, one, and none (by replicas per compute unit)
@pytest.mark.parametrize("kind", ["sk", "gauss", "q100000"])
@pytest.mark.parametrize("N,R", [
    (513, 3), (600, 3), (1000, 3), (1024, 3), (999, 600), (1000, 1100), (1000, 1200),
    (1025, 2), (1500, 2), (2048, 300), (1300, 1100), (1300, 1300),
    (2049, 2), (3000, 2), (4096, 2), (2100, 300), (2100, 600),
    (4097, 2), (8192, 2), (5000, 300)])
def test_teams(api, kind, N, R):
    Q, T_hi, T_lo, inc = _instance(kind, N)
    S = 60 if N > 2048 else 200
    if R < 10:
        S *= 2
    _check(api, Q, 0, R, S, 7, T_hi, T_lo, inc, init="random")


@pytest.mark.parametrize("N,R", [(700, 3), (1000, 600), (700, 1100), (1500, 2), (3000, 2), (4200, 2)])
@pytest.mark.parametrize("kind,L,S,extra", [
    ("sk", 150, 100, {}), ("cold", 4, 150, {}), ("sk", 0, 150, dict(kind="linear_beta")),
    ("gauss", 0, 70, {}), ("q100", 3, 150, dict(trial="single")), ("sk", 3, 0, {}), ("sk", 0, 1, {}),
])
def test_team_schedules(api, N, R, kind, L, S, extra):
    Q, T_hi, T_lo, inc = _instance(kind, N)
    _check(api, Q, 0, R, S, L, T_hi, T_lo, inc, **extra)


def test_resume(api):
    """Pieces that cut levels and groups of steps equal the whole run."""
    for N in (50, 100, 220, 480, 800, 1400):
        Q, T_hi, T_lo, inc = _instance("sk", N)
        ctx = api.da_create(Q)
        sch = api.schedule(T_hi, T_lo, "geometric", 9, eoff_inc=inc)
        whole = api.da_anneal(ctx, sch, 5, 1000, 3)
        c2 = api.da_create(Q)
        for a, b in [(0, 1), (1, 67), (67, 555), (555, 998), (998, 1000)]:
            part = api.da_anneal_steps(c2, sch, 0, 5, 1000, a, b, 3)
        for k in KEYS:
            assert np.array_equal(part[k], whole[k]), (N, k)


@pytest.mark.parametrize("fill", [0, 9000])
def test_mixed_batch(api, fill):
    """One launch per coupling type and mode, every shape among them; with `fill`
    more replicas than the chip holds, in the shapes of a full chip."""
    import torch
    specs = [("sk", 40, 1, 9, "geometric", {}), ("gauss", 64, 0, 3, "geometric", {}),
             ("sk", 100, 2, 5, "geometric", {}), ("q100000", 200, 0, 4, "geometric", {}),
             ("gauss", 300, 0, 3, "geometric", {}), ("sk", 512, 0, 6, "linear_beta", {}),
             ("cold", 600, 0, 2, "geometric", {}), ("gauss", 1024, 0, 2, "geometric", {}),
             ("sk", 1500, 1, 2, "geometric", {}), ("gauss", 2049, 0, 2, "geometric", {}),
             ("sk", 4200, 0, 1, "geometric", {}), ("q100", 150, 0, 5, "geometric", dict(trial="single")),
             ("q100000", 1100, 0, 2, "geometric", {})]
    items, alone = [], []
    for i, (kind, N, dtype, R, sk, extra) in enumerate(specs):
        Q, T_hi, T_lo, inc = _instance(kind, N, seed=i + 1)
        R = fill if fill and i == 0 else R
        S, L = 120 + 10 * i, 0 if sk == "linear_beta" else 5
        sch = api.schedule(T_hi, T_lo, sk, L, eoff_inc=inc, init="random", **extra)
        ctx = api.da_create(Q, dtype)
        alone.append(api.da_anneal(ctx, sch, R, S, 50 + i))
        items.append(dict(ctx=api.da_create(Q, dtype), schedule=sch, replicas=R, steps=S,
                          seed=50 + i, out_dev=api.device_outputs(R, N)))
    api.da_anneal_batch(items)
    torch.cuda.synchronize()
    for i, it in enumerate(items):
        for k in KEYS:
            assert np.array_equal(it["out_dev"][k].cpu().numpy(), alone[i][k]), (i, k)


# one replica, both ends of what the step kernel sweeps itself, more than that;
# captured rounds (at least 64) and single launches; one wave and teams
@pytest.mark.parametrize("N,M,chains,rounds,K", [
    (60, 1, 3, 4, 30), (60, 2, 300, 66, 3), (100, 64, 2, 5, 40), (100, 65, 2, 5, 40),
    (300, 17, 3, 70, 9), (700, 16, 2, 5, 40), (700, 5, 1, 0, 40), (60, 4, 2, 5, 0)])
def test_tempering_sweeps(api, N, M, chains, rounds, K):
    Q, T_hi, T_lo, _ = _instance("sk", N)
    temps = T_lo * (T_hi / T_lo) ** (np.arange(M) / max(M - 1, 1))
    gpu = api.da_pt(api.da_create(Q), temps, chains, rounds, K, 1, 5)
    ref = oracle.pt(Q, temps, chains=chains, rounds=rounds, steps_per_round=K, eoff_inc=1, seed=5)
    for k in KEYS + ("slot", "n_swaps", "pair_swaps"):
        assert np.array_equal(np.asarray(gpu[k]).reshape(-1), np.asarray(ref[k]).reshape(-1)[:np.asarray(gpu[k]).size]), k


# one wave of 16 flips per lane with four replicas in a workgroup: four replicas
# per compute unit, and from six on (256 units), ragged N and last workgroups
@pytest.mark.parametrize("kind", ["sk", "gauss", "q100000"])
@pytest.mark.parametrize("N,R", [(1000, 1000), (999, 1500), (513, 1021), (1024, 1793)])
def test_one_wave_of_sixteen(api, kind, N, R):
    Q, T_hi, T_lo, inc = _instance(kind, N)
    ctx = _check(api, Q, 0, R, 150, 7, T_hi, T_lo, inc, init="random")
    st = api.da_last_kernel_stats(ctx)
    assert (st["flips_per_lane"], st["rng_waves"], st["replicas_per_block"]) == (16, 0, 4)


@pytest.mark.parametrize("dtype", [1, 2, 4])
def test_one_wave_of_sixteen_types(api, dtype):
    Q, T_hi, T_lo, inc = _instance("sk", 830)
    ctx = _check(api, Q, dtype, 1022, 200, 6, T_hi, T_lo, inc)
    assert api.da_last_kernel_stats(ctx)["flips_per_lane"] == 16


@pytest.mark.parametrize("N,R", [(700, 1000), (700, 1500)])
@pytest.mark.parametrize("kind,L,S,extra", [
    ("sk", 150, 100, {}), ("cold", 4, 150, {}), ("sk", 0, 150, dict(kind="linear_beta")),
    ("gauss", 0, 70, {}), ("q100", 3, 150, dict(trial="single")), ("sk", 3, 0, {}), ("sk", 0, 1, {}),
])
def test_one_wave_of_sixteen_schedules(api, N, R, kind, L, S, extra):
    Q, T_hi, T_lo, inc = _instance(kind, N)
    ctx = _check(api, Q, 0, R, S, L, T_hi, T_lo, inc, **extra)
    st = api.da_last_kernel_stats(ctx)
    assert (st["flips_per_lane"], st["rng_waves"]) == (16, 0)


# the shapes of teams by replicas per compute unit (256 units)
@pytest.mark.parametrize("N,R,F,NH", [
    (513, 3, 8, 1), (1024, 512, 8, 1), (999, 600, 8, 2), (1000, 1100, 8, 2), (1000, 1280, 8, 2),
    (1025, 2, 8, 2), (2048, 300, 8, 4), (1300, 1024, 8, 3), (1300, 1100, 16, 0),
    (2049, 2, 8, 3), (4096, 256, 8, 4), (2100, 300, 16, 3), (2100, 600, 16, 0),
    (4097, 2, 16, 5), (5000, 300, 16, 0)])
def test_team_shapes(api, N, R, F, NH):
    Q, T_hi, T_lo, inc = _instance("sk", N)
    ctx = _check(api, Q, 0, R, 20, 3, T_hi, T_lo, inc)
    st = api.da_last_kernel_stats(ctx)
    waves = -(-N // (64 * F))
    assert (st["flips_per_lane"], st["rng_waves"]) == (F, NH)
    assert (st["threads"], st["blocks"]) == (64 * (waves + NH), R)
