"""Bit-reproducible gradient where rows have long runs of samples, which a
workgroup shares: runs on both sides of the 512 pairs from which it does, runs
of tens of thousands, slices that are empty, every row visited and only the
listed ones (more rows than pairs), accumulation, one to four passes over the
columns.  Repeated calls are bit-identical and the gradient is the oracle's
within the rounding bound of its sums."""
import pytest
import torch

import oracle
from paper_2605_20353_amd import _lib as G
from paper_2605_20353_amd import synth
from parity_util import assert_grad_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("dims,R,p,q", [
    ([2, 40, 700], 8, 12000, 8500),           # runs of ~10000, ~512 and ~30
    ([2, 40, 700], 5, 511, 512),              # one column per lane; runs of about 512
    ([3, 300000, 4], 32, 1500, 1200),         # rows listed, two modes with long runs
    ([40, 6, 300, 5], 100, 3000, 2000),       # 32 lanes a row, two rows a wavefront
    ([20, 30, 40], 200, 9000, 9000),          # 64 lanes a row (f64: two passes over the columns)
    ([12, 10, 8, 6, 9], 6, 3000, 1500),       # general order, short modes only
])
def test_long_runs(gpu, dtype, dims, R, p, q):
    data = synth.count_tensor(dims, 3, 4000, seed=2671)
    t = G.SparseTensor(dims, data.coords.to(gpu), data.vals.to(dtype).to(gpu))
    to = oracle.SparseTensor(dims, data.coords.numpy(), data.vals.to(dtype).double().numpy())
    A = (0.2 + 0.8 * synth.init_model(dims, R, 13, dtype=torch.float64)).to(dtype).to(gpu)
    sp = G.SampleParams("stratified", p, q, seed=20353, step=3)
    t.reserve(sp.n, R)
    print(f"long runs dims={dims} R={R} {dtype}", flush=True)
    G1, L1 = G.gcp_loss_grad(t, sp, A, R, "poisson", deterministic=True)
    G2, L2 = G.gcp_loss_grad(t, sp, A, R, "poisson", deterministic=True)
    G3, _ = G.gcp_loss_grad(t, sp, A, R, "poisson", G=G1.clone(), loss_out=L1.clone(), accumulate=True,
                            deterministic=True)
    t.status()
    assert torch.equal(G1, G2) and torch.equal(L1, L2), "deterministic runs differ"
    assert torch.equal(G3, G1 + G1), "accumulated: one sum per row added to what was there"
    sc, sx, sw = oracle.sample_stratified(to, sp.p, sp.q, sp.seed, sp.step)
    A64 = A.double().cpu().numpy().reshape(-1)
    Go, _ = oracle.loss_grad(dims, R, A64, sc, sx, sw, "poisson")
    assert_grad_close(G1.cpu().numpy(), Go, dims, R, A64, sc, sx, sw, "poisson", dtype,
                      what=f"long runs dims={dims} R={R}")
