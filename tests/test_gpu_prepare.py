"""Instances made on the device (N > 224) and on the host against numpy: storage
type and common factor, energies, at the edges of the 64 x 64 tiles, couplings
of the largest size, none at all, and what is refused.  Whole numbers: exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_1806_08815_amd import api as a
    a.lib()
    return a


def _q(kind, N):
    g = np.random.Generator(np.random.PCG64(N))
    if kind == "diag":
        return np.diag(g.integers(-9, 10, size=N)).astype(np.int32)
    if kind == "one":       # one coupling of 2^30 - 1, in the last tile
        Q = np.zeros((N, N), np.int32)
        Q[N - 2, N - 1] = 2**30 - 1
        return Q
    if kind == "cancel":    # Q_ij = -Q_ji up to one pair: large entries, small couplings
        A = np.triu(g.integers(-2**31 + 1, 2**31, size=(N, N), dtype=np.int64), 1)
        Q = (A - A.T).astype(np.int32)
        Q[0, N - 1] -= 3 if Q[0, N - 1] > 0 else -3
        return Q
    f, lim = {"g1": (1, 60), "g6": (6, 100), "g2^20": (2**20, 1), "wide": (1, 30000)}[kind]
    Q = np.triu(g.integers(-lim, lim + 1, size=(N, N)) * f).astype(np.int32)
    Q[np.diag_indices(N)] = g.integers(-50, 51, size=N)
    return Q


@pytest.mark.parametrize("kind", ["g1", "g6", "g2^20", "wide", "diag", "one", "cancel"])
@pytest.mark.parametrize("N", [2, 64, 128, 129, 191, 192, 193, 320, 700])
def test_storage_and_energies(api, kind, N):
    Q = _q(kind, N)
    W = Q.astype(np.int64) + Q.T.astype(np.int64)
    np.fill_diagonal(W, 0)
    g = int(np.gcd.reduce(np.abs(W).reshape(-1))) or 1
    top = int(np.abs(W).max()) // g
    ctx = api.da_create(Q)
    info = ctx.info()
    assert info["wscale"] == g
    assert info["dtype"] == (1 if top <= 127 else 2 if top <= 32767 else 4)
    rng = np.random.Generator(np.random.PCG64(7))
    x = rng.integers(0, 2, size=(9, N), dtype=np.uint8)
    xi = x.astype(np.int64)
    want = ((xi @ W) * xi).sum(axis=1) // 2 + xi @ np.diag(Q).astype(np.int64)
    assert np.array_equal(api.da_energy(ctx, x), want)


@pytest.mark.parametrize("N", [64, 300])
def test_refused(api, N):
    Q = np.zeros((N, N), np.int32)
    Q[0, N - 1] = 2**30
    api.da_create(Q)                          # |b| + sum |W| = 2^30: the bound
    Q[0, 0] = 1
    with pytest.raises(api.DaError) as e:
        api.da_create(Q)
    assert "2^30" in str(e.value)
    Q = np.full((N, N), 100, np.int32)
    Q[0, 1] = 101
    with pytest.raises(api.DaError) as e:
        api.da_create(Q, 1)
    assert "requested type" in str(e.value)


def test_beside_a_running_anneal(api):
    """An instance made while another context's anneal runs does not wait for it."""
    import torch
    Q = _q("g1", 300)
    api.da_create(Q)
    big = api.da_create(_q("g1", 1024))
    sch = api.schedule(300.0, 3.0, "geometric", 16, 1)
    out, stream, done = api.device_outputs(8, 1024), torch.cuda.Stream(), torch.cuda.Event()
    api.da_anneal_async(big, sch, 0, 8, 1000, 1, None, out, stream)
    torch.cuda.synchronize()
    api.da_anneal_async(big, sch, 0, 8, 1_000_000, 1, None, out, stream)   # about half a second
    done.record(stream)
    ctx = api.da_create(Q)
    assert not done.query()
    torch.cuda.synchronize()
    x = np.ones((1, 300), np.uint8)
    assert api.da_energy(ctx, x)[0] == Q.astype(np.int64).sum()


@pytest.mark.parametrize("kind", ["g1", "g6", "g2^20", "wide", "diag", "one", "cancel"])
@pytest.mark.parametrize("N", [224, 225, 255, 256, 257, 449])
def test_storage_and_energies_past_the_host_sizes(api, kind, N):
    """Up to 224 variables the host derives the instance, past them the device."""
    test_storage_and_energies(api, kind, N)
