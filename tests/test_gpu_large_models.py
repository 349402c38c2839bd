"""Models around 4 GiB, against the oracle: the last model whose rows have 32-bit
byte offsets (top bit set for half of its rows), the first one of 2^32 bytes,
and one well above.  Half of the nonzeros lie in the first and last rows of each
mode.  The oracle works on the touched rows alone, renumbered; all other rows of
the gradient have to be zero.  Every form of the call: hardware atomics,
LDS-private and row-bucketed modes, objective only, materialised samples, the
sampled tensor and its MTTKRP, bit-reproducible."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_20353_amd import _lib as G
from parity_util import assert_grad_close

pytestmark = pytest.mark.gpu

TOL = {torch.float64: 1e-12, torch.float32: 1e-5}
EDGE = 1 << 22        # rows of 1 KiB in 4 GiB


def tensor(dims, dtype, gpu, nnz=3000):
    rng = np.random.default_rng(sum(dims))
    c = np.stack([rng.integers(0, n, nnz) for n in dims], axis=1)
    ends = np.stack([rng.choice([0, 1, n - 2, n - 1], nnz // 2) for n in dims], axis=1)
    c = np.unique(np.concatenate([c[: nnz // 2], ends]), axis=0)
    vals = rng.integers(1, 9, len(c)).astype(np.float64)
    return G.SparseTensor(dims, torch.from_numpy(c).to(gpu), torch.from_numpy(vals).to(dtype).to(gpu))


class Touched:
    """The rows that the samples touch, as a small problem for the oracle."""

    def __init__(self, dims, R, A, coords):
        off = torch.tensor(np.concatenate([[0], np.cumsum(dims)[:-1]]), device=coords.device)
        self.rows, self.dims, small = [], [], []
        for k in range(len(dims)):
            u, inv = torch.unique(coords[:, k], return_inverse=True)
            self.rows.append(u + off[k])
            self.dims.append(int(u.numel()))
            small.append(inv)
        self.rows = torch.cat(self.rows)
        self.coords = torch.stack(small, dim=1).cpu().numpy()
        self.A = A.view(-1, R)[self.rows].double().cpu().numpy().reshape(-1)

    def of(self, g, R, what):
        """The touched rows of g; every other row is zero."""
        g = g.view(-1, R)
        part = g[self.rows].clone()
        g[self.rows] = 0
        assert torch.count_nonzero(g).item() == 0, f"{what}: rows without samples hold a gradient"
        return part.double().cpu().numpy()


# (dims, LDS-private modes, row-bucketed modes): the tall mode is atomic
SHAPES = [([1500000, 1400000], 0, 0), ([40, 900], 1, 2), ([500, 40, 900], 2, 5), ([500, 900], 0, 3), ([700, 40, 600], 0, 7),
          ([60, 50, 40, 30], 0, 15)]


@pytest.mark.parametrize("rows", [EDGE - 1, EDGE, EDGE + 900000])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("short,lds,bucket", SHAPES)
def test_models_around_4_gib(gpu, dtype, rows, short, lds, bucket):
    R = 1024 // dtype.itemsize
    dims = short + [rows - sum(short)]
    t = tensor(dims, dtype, gpu)
    gen = torch.Generator(device=gpu).manual_seed(7)
    A = torch.rand(rows * R, generator=gen, device=gpu, dtype=dtype).mul_(0.02).add_(0.9)
    sp = G.SampleParams("stratified", 1500, 700, seed=20353, step=5)
    t.reserve(sp.n, R)
    coords, x, w = G.gcp_sample(t, sp)
    T = Touched(dims, R, A, coords)
    smp = (T.coords, x.double().cpu().numpy(), w.double().cpu().numpy())
    Go, Fo = oracle.loss_grad(T.dims, R, T.A, *smp, "poisson")
    print(f"model of {rows} rows x 1 KiB, dims {dims}, {dtype}", flush=True)

    def check(g, f, what):
        t.status()
        assert_grad_close(T.of(g, R, what), Go, T.dims, R, T.A, *smp, "poisson", dtype, what=what)
        if f is not None:
            assert abs(f.item() - Fo) <= TOL[dtype] * abs(Fo), what

    g = torch.full_like(A, 3.0)
    tile = G.Tile(lds_modes=lds, bucket_modes=bucket, bucket_block_samples=512)
    check(*G.gcp_loss_grad(t, sp, A, R, "poisson", G=g, tile=tile), "scatter of each mode")
    if short[0] == 500 or lds == 0 and bucket == 0:
        check(*G.gcp_loss_grad(t, sp, A, R, "poisson", G=g, tile=G.Tile(lds_modes=0, bucket_modes=0)), "atomics")
        check(*G.gcp_loss_grad(t, sp, A, R, "poisson", G=g, samples=(coords, x, w)), "materialised")
        _, f = G.gcp_loss_grad(t, sp, A, R, "poisson", loss_only=True)
        assert abs(f.item() - Fo) <= TOL[dtype] * abs(Fo)
        c2, y, _ = G.gcp_sample_y(t, sp, A, R, "poisson")
        assert torch.equal(c2, coords)
        check(G.gcp_mttkrp(t, coords, y, A, R, G=g), None, "non-fused")
        check(*G.gcp_loss_grad(t, sp, A, R, "poisson", G=g, deterministic=True), "bit-reproducible")
