"""gcp_mttkrp over every order that has kernels of its own and two that have not,
against the oracle within the rounding bound of its sums: lane groups of 8 to 64
lanes with one, two and four columns a lane, hardware atomics, LDS-private and
row-bucketed modes together, mixed-radix keys, sample counts at the edges of the
kernel's chunks, accumulation with a scale, and coordinates out of range."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_20353_amd import _lib as G
from paper_2605_20353_amd import synth
from parity_util import SAFETY, frob_rel_errs

pytestmark = pytest.mark.gpu

TOL = {torch.float64: 1e-12, torch.float32: 1e-5}
# dims, ranks, modes LDS-private and row-bucketed in the mixed form (the others are atomic)
CASES = [([90, 70], (6, 33), 2, 1), ([60, 50, 40], (6, 16, 50), 4, 2), ([60, 50, 40], (100, 200), 0, 3),
         ([30, 25, 20, 15], (6, 32, 63), 8, 5), ([20, 18, 16, 14, 12], (7, 24), 16, 3),
         ([9, 8, 7, 6, 5, 10], (5, 32), 32, 7), ([40000, 40000, 40000, 40000], (4,), 0, 2),
         ([4200, 4500, 4600, 4300, 4700], (6,), 0, 16)]      # the last two: 64- and 65-bit keys


def bound(dims, R, A64, coords, y, u):
    """d - 1 products per contribution, count - 1 additions per element in any order."""
    gamma = lambda n: np.asarray(n, dtype=np.float64) * u / (1 - np.asarray(n, dtype=np.float64) * u)  # noqa: E731
    count = np.concatenate([np.bincount(coords[:, k], minlength=dims[k]) for k in range(len(dims))])
    absG = oracle.mttkrp(dims, R, np.abs(A64), coords, np.abs(y))
    return SAFETY * (gamma(len(dims)) + gamma(np.repeat(np.maximum(count - 1, 0), R))) * absG * (1 + oracle.U_F64 / u)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("dims,ranks,lds,bucket", CASES)
def test_mttkrp_orders(gpu, dtype, dims, ranks, lds, bucket):
    rng = np.random.default_rng(len(dims) * 1000 + ranks[0])
    big = sum(dims) > 10**4
    data = synth.count_tensor(dims, 3, 200, seed=2605)
    t = G.SparseTensor(dims, data.coords.to(gpu), data.vals.to(dtype).to(gpu))
    u = oracle.U_F32 if dtype == torch.float32 else oracle.U_F64
    for R in ranks:
        A = (0.2 + 0.8 * synth.init_model(dims, R, 5, dtype=torch.float64)).to(dtype).to(gpu)
        A64 = A.double().cpu().numpy().reshape(-1)
        for n in (1, 63, 4097) if big else (1, 63, 4097, 33001, 140003):
            coords = np.stack([rng.integers(0, m, n) for m in dims], axis=1)
            coords[: n // 2] %= np.minimum(dims, 50)          # rows with many samples in every mode
            y = rng.normal(size=n).astype(np.float32).astype(np.float64)
            Go = oracle.mttkrp(dims, R, A64, coords, y)
            b = bound(dims, R, A64, coords, y, u)
            t.reserve(n, R)
            c, v = torch.from_numpy(coords).to(gpu), torch.from_numpy(y).to(dtype).to(gpu)
            print(f"mttkrp {dims} R={R} {dtype} n={n}", flush=True)
            for tile in (None, G.Tile(lds_modes=0, bucket_modes=0), G.Tile(lds_modes=lds, bucket_modes=bucket)):
                g = G.gcp_mttkrp(t, c, v, A, R, tile=tile)
                t.status()
                g = g.double().cpu().numpy().reshape(-1)
                bad = np.nonzero(~(np.abs(g - Go) <= b))[0]
                assert bad.size == 0, (tile, n, bad[:5], g[bad[:5]], Go[bad[:5]], b[bad[:5]])
        # scaled and added to what is there; the last sample list
        g = torch.full_like(A, 0.25)
        G.gcp_mttkrp(t, c, v, A, R, G=g, accumulate=True, scale=torch.tensor([-0.5], dtype=dtype, device=gpu))
        got = g.double().cpu().numpy().reshape(-1) - 0.25
        err = np.abs(got + 0.5 * Go)
        assert np.all(err <= b + 4 * u * (0.25 + np.abs(Go)) * (1 + n)), err.max()
        if not big:
            assert max(frob_rel_errs(got, -0.5 * Go, dims, R)) <= 8 * TOL[dtype]


@pytest.mark.parametrize("dims", [[60, 50, 40], [30, 25, 20, 15], [9, 8, 7, 6, 5, 10]])
def test_out_of_range_coordinates_add_nothing(gpu, dims):
    rng = np.random.default_rng(3)
    R, n = 8, 500
    data = synth.count_tensor(dims, 3, 200, seed=2605)
    t = G.SparseTensor(dims, data.coords.to(gpu), data.vals.to(torch.float64).to(gpu))
    A = 0.2 + 0.8 * synth.init_model(dims, R, 5, dtype=torch.float64)
    coords = np.stack([rng.integers(0, m, n) for m in dims], axis=1)
    y = rng.normal(size=n)
    keep = np.ones(n, dtype=bool)
    wrong = coords.copy()
    for s, value in ((7, -1), (130, dims[1]), (499, 2**33)):
        wrong[s, 1] = value
        keep[s] = False
    t.reserve(n, R)
    g = G.gcp_mttkrp(t, torch.from_numpy(wrong).to(gpu), torch.from_numpy(y).to(gpu), A.to(gpu), R)
    with pytest.raises(G.GCPError):
        t.status()
    Go = oracle.mttkrp(dims, R, A.numpy().reshape(-1), coords[keep], y[keep])
    assert max(frob_rel_errs(g.cpu().numpy(), Go, dims, R)) <= 1e-12
