"""Edges of the row-bucketed scatter and of the bit-reproducible form, against
the oracle: streams of more than 64 segments per wavefront, batches that end
inside a segment and empty segments, at every way an entry reaches its lane
group (DPP row, half-row and quad broadcasts, bpermute); sorted blocks taken in
turn by workgroups with LDS-private modes; gradients that are not 16-byte
aligned; rows with and without pairs, listed and not."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_20353_amd import _lib as G
from paper_2605_20353_amd import synth
from parity_util import assert_grad_close

pytestmark = pytest.mark.gpu


class Case:
    def __init__(self, gpu, dtype, dims, R, p, q, nnz=20000):
        self.dims, self.R, self.dtype = dims, R, dtype
        data = synth.count_tensor(dims, 3, nnz, seed=2681)
        self.t = G.SparseTensor(dims, data.coords.to(gpu), data.vals.to(dtype).to(gpu))
        to = oracle.SparseTensor(dims, data.coords.numpy(), data.vals.to(dtype).double().numpy())
        self.sp = G.SampleParams("stratified", p, q, seed=20353, step=3)
        self.t.reserve(self.sp.n, R)
        self.A = (0.2 + 0.8 * synth.init_model(dims, R, 9, dtype=torch.float64)).to(dtype).to(gpu)
        self.A64 = self.A.double().cpu().numpy().reshape(-1)
        self.samples = oracle.sample_stratified(to, p, q, self.sp.seed, self.sp.step)
        self.G, self.F = oracle.loss_grad(dims, R, self.A64, *self.samples, "poisson")

    def check(self, g, what):
        self.t.status()
        assert_grad_close(g.double().cpu().numpy(), self.G, self.dims, self.R, self.A64, *self.samples, "poisson",
                          self.dtype, what=what)


# (dtype, rank): 4, 8 and 16 lanes (DPP), 32 and 64 (lane reads), 2 (bpermute)
SHAPES = [(torch.float32, 8), (torch.float32, 16), (torch.float32, 32), (torch.float32, 20), (torch.float32, 64),
          (torch.float32, 96), (torch.float32, 33), (torch.float64, 6), (torch.float64, 24), (torch.float64, 48),
          (torch.float64, 5)]


@pytest.mark.parametrize("dtype,R", SHAPES)
def test_owner_streams(gpu, dtype, R):
    c = Case(gpu, dtype, [700, 450, 90], R, 40001, 30011)
    for bblock, splits, spb in ((64, 1, 512), (1024, 3, 512), (0, 0, 0), (256, 40, 1024)):
        tile = G.Tile(lds_modes=0, bucket_modes=7, bucket_block=bblock, bucket_splits=splits, bucket_block_samples=spb)
        print(f"owner {dtype} R={R} block={bblock} splits={splits} spb={spb}", flush=True)
        g, _ = G.gcp_loss_grad(c.t, c.sp, c.A, R, "poisson", tile=tile)
        c.check(g, f"block={bblock} splits={splits}")


@pytest.mark.parametrize("dims,R,lds", [([700, 450, 60], 32, 4), ([60, 50, 40, 300], 16, 3), ([40, 30, 20, 10, 600], 12, 15)])
def test_sorted_blocks_in_turn(gpu, dims, R, lds):
    # 391 sorted blocks for the workgroups that fit at once
    c = Case(gpu, torch.float32, dims, R, 120001, 80003)
    tile = G.Tile(lds_modes=lds, bucket_modes=(1 << len(dims)) - 1, bucket_block_samples=512)
    for block in (256, 1024):
        tile.block = block
        g, f = G.gcp_loss_grad(c.t, c.sp, c.A, R, "poisson", tile=tile)
        c.check(g, f"block={block}")
        assert abs(f.item() - c.F) <= 1e-5 * abs(c.F)


def test_gradient_not_16_byte_aligned(gpu):
    c = Case(gpu, torch.float32, [700, 450, 90], 32, 40001, 30011)
    buf = torch.full((c.A.numel() + 1,), 7.0, dtype=torch.float32, device=gpu)
    g, _ = G.gcp_loss_grad(c.t, c.sp, c.A, 32, "poisson", G=buf[1:])
    c.check(g, "unaligned G")
    assert buf[0].item() == 7.0


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("R", [32, 10, 7])
@pytest.mark.parametrize("n", [300, 40007])
def test_reproducible_rows(gpu, dtype, R, n):
    # 5400 rows: 300 samples list the rows with pairs, 40007 visit every row
    c = Case(gpu, dtype, [3000, 2000, 400], R, n // 2, n - n // 2)
    g = torch.full_like(c.A, 3.0)
    G.gcp_loss_grad(c.t, c.sp, c.A, R, "poisson", G=g, deterministic=True)
    c.check(g, "overwrite")
    base = torch.rand_like(c.A)
    acc = base.clone()
    G.gcp_loss_grad(c.t, c.sp, c.A, R, "poisson", G=acc, accumulate=True, deterministic=True)
    assert torch.equal(acc, base + g)
