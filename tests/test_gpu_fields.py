"""Fields and energies on the matrix cores (byte planes of every coupling type)
against numpy in 64 bits: edges of the 32- and 128-row tiles and of the reduction
splits, both forms (one wave per tile, tiled), states at any alignment and with
any nonzero byte for a one.  Integer work: bit-exact."""
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


def _want(Q, x):
    xd = (x != 0).astype(np.float64)          # whole numbers below 2^53
    return ((xd @ Q.astype(np.float64)) * xd).sum(axis=1).astype(np.int64)


# lim 60: int8; 16000: int16 up to 32000 in size; 10^5: int32 in three planes;
# 'top': a few couplings up to 2^29 (four planes)
@pytest.mark.parametrize("lim", [60, 16000, 10**5, "top"])
@pytest.mark.parametrize("N,count", [(1, 1), (33, 31), (64, 33), (257, 129), (320, 3),
                                     (1000, 1100), (1000, 1153), (2048, 600), (4097, 270),
                                     (8191, 2)])
def test_energies(api, N, count, lim):
    import torch
    g = np.random.Generator(np.random.PCG64(N))
    if lim == "top":
        Q = np.zeros((N, N), np.int32)
        i = np.arange(N - 1)
        Q[i, i + 1] = g.integers(-2**28, 2**28, size=N - 1)
        Q[i, i] = g.integers(-2**28, 2**28, size=N - 1)
    else:
        Q = g.integers(-lim, lim + 1, size=(N, N), dtype=np.int32)
        Q[0, 0] = lim
    x = g.integers(0, 2, size=(count, N), dtype=np.uint8) * g.integers(1, 256, size=(count, N)).astype(np.uint8)
    x[0], x[-1] = 255, g.integers(0, 2, size=N)
    ctx = api.da_create(Q)
    want = _want(Q, x)
    assert np.array_equal(api.da_energy(ctx, x), want)
    # device states starting at an odd address, the last byte of their buffer
    # the last of the states
    buf = torch.zeros(x.size + 3, dtype=torch.uint8, device="cuda")
    buf[3:] = torch.from_numpy(x.reshape(-1)).cuda()
    E = torch.zeros(count, dtype=torch.int64, device="cuda")
    api.da_energy_noalloc(ctx, buf[3:].view(count, N), E, torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert np.array_equal(E.cpu().numpy(), want)


@pytest.mark.parametrize("lim", [60, 16000, 10**5])
@pytest.mark.parametrize("N,R", [(70, 33), (1000, 130), (1000, 1200)])
def test_random_start_fields(api, N, R, lim):
    """Fields and energies of random starts, read back through a snapshot."""
    g = np.random.Generator(np.random.PCG64(N + R))
    Q = g.integers(-lim, lim + 1, size=(N, N), dtype=np.int32)
    ctx = api.da_create(Q)
    sch = api.schedule(100.0, 1.0, "geometric", 4, init="random")
    out = api.da_anneal_steps(ctx, sch, 0, R, 64, 0, 0, 5)
    buf = api.da_state_save(ctx, R)
    x = buf[32:32 + R * N].reshape(R, N)
    h = buf[32 + 2 * R * N:32 + 6 * R * N].view(np.int32).reshape(R, N)
    W = (Q.astype(np.int64) + Q.T.astype(np.int64))
    W[np.arange(N), np.arange(N)] = 0
    want = (x.astype(np.float64) @ W.astype(np.float64)).astype(np.int64) + np.diag(Q)
    assert np.array_equal(out["final_x"], x)
    assert np.array_equal(h.astype(np.int64), want)
    assert np.array_equal(out["final_E"], _want(Q, x))
