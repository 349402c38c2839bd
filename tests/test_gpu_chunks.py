"""Sample counts at the edges of the sampled-gradient kernel's chunks, against
the oracle: a call with few samples cuts its chunks from 64 samples down to
what a lane group keeps in flight, so that the counts below reach every chunk
size, full and ragged, in the forms that scatter in the sampling loop (hardware
atomics, LDS-private) and the one that does not (objective only), for the
order-specific kernels and the any-order one."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_20353_amd import _lib as G
from paper_2605_20353_amd import synth
from parity_util import assert_grad_close

pytestmark = pytest.mark.gpu

TOL = {torch.float64: 1e-12, torch.float32: 1e-5}
COUNTS = [1, 63, 4097, 8191, 16385, 33001, 65537, 140003]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("dims,R", [([90, 70, 50], 32), ([90, 70, 50], 5), ([40, 30, 20, 10], 16),
                                    ([12, 10, 9, 8, 7], 8), ([200, 150], 6)])
def test_sample_counts_at_chunk_edges(gpu, dtype, dims, R):
    data = synth.count_tensor(dims, 3, min(2000, int(np.prod(dims)) // 10), seed=2671)
    t = G.SparseTensor(dims, data.coords.to(gpu), data.vals.to(dtype).to(gpu))
    to = oracle.SparseTensor(dims, data.coords.numpy(), data.vals.to(dtype).double().numpy())
    A = (0.2 + 0.8 * synth.init_model(dims, R, 9, dtype=torch.float64)).to(dtype).to(gpu)
    A64 = A.double().cpu().numpy().reshape(-1)
    for n in COUNTS:
        sp = G.SampleParams("stratified", n // 2, n - n // 2, seed=20353, step=n)
        sc, sx, sw = oracle.sample_stratified(to, sp.p, sp.q, sp.seed, sp.step)
        Go, Fo = oracle.loss_grad(dims, R, A64, sc, sx, sw, "poisson")
        print(f"chunks {dims} R={R} {dtype} n={n}", flush=True)
        for tile in (None, G.Tile(lds_modes=0, bucket_modes=0)):
            Gg, Lg = G.gcp_loss_grad(t, sp, A, R, "poisson", tile=tile)
            t.status()
            assert_grad_close(Gg.double().cpu().numpy(), Go, dims, R, A64, sc, sx, sw, "poisson", dtype, what=f"n={n}")
            assert abs(Lg.item() - Fo) <= TOL[dtype] * abs(Fo)
        _, Lg = G.gcp_loss_grad(t, sp, A, R, "poisson", loss_only=True)
        assert abs(Lg.item() - Fo) <= TOL[dtype] * abs(Fo)
