"""Drawn samples of every order that has its own sampling kernel and of one that
has not, bit for bit against the oracle: bit-packed and mixed-radix keys, dense
enough for repeated rejections, several passes of the launch's grid, stratified,
semi-stratified and uniform; and the gradient of the mixed-radix 5-way samples."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_20353_amd import _lib as G
from paper_2605_20353_amd import synth
from parity_util import assert_grad_close

pytestmark = pytest.mark.gpu

# name: dims, stored cells
SPARSE = {
    "2way": ([90, 70], 2000),
    "3way": ([30, 20, 14], 2000),
    "4way": ([12, 10, 9, 8], 2000),
    "5way": ([7, 6, 5, 8, 6], 3000),
    "6way": ([4, 5, 6, 3, 5, 4], 2000),
    "5way_65bit": ([4200, 4500, 4600, 4300, 4700], 3000),     # 5 x 13 bits: mixed-radix keys
}


def case(name, dtype, gpu):
    dims, nnz = SPARSE[name]
    data = synth.count_tensor(dims, 3, nnz, seed=2605)
    t = G.SparseTensor(dims, data.coords.to(gpu), data.vals.to(dtype).to(gpu))
    return t, oracle.SparseTensor(dims, data.coords.numpy(), data.vals.to(dtype).double().numpy()), dims


def assert_same(drawn, expected, dtype):
    for got, want in zip(drawn, expected):
        got = got.cpu().numpy()
        np.testing.assert_array_equal(got, np.asarray(want).astype(got.dtype))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("name", list(SPARSE))
def test_orders_bit_exact(gpu, dtype, name):
    t, to, _ = case(name, dtype, gpu)
    for kind, p, q in (("stratified", 700001, 600007), ("semi_stratified", 300, 4099), ("stratified", 1, 63)):
        print(f"sample {name} {dtype} {kind} {p}+{q}", flush=True)
        drawn = G.gcp_sample(t, G.SampleParams(kind, p, q, seed=2**63 + 5, step=7, client=2))
        t.status()
        assert_same(drawn, oracle.sample_stratified(to, p, q, 2**63 + 5, 7, 2, semi=kind == "semi_stratified"), dtype)


@pytest.mark.parametrize("dims", [[90, 70], [12, 10, 9, 8, 7]])
def test_uniform_orders_bit_exact(gpu, dims):
    x = torch.rand(*dims, dtype=torch.float64, generator=torch.Generator().manual_seed(3))
    t = G.DenseTensor(dims, x.to(gpu))
    c, xs, w = G.gcp_sample(t, G.SampleParams("uniform", 5003, 0, seed=20353, step=9))
    assert_same((c, xs, w), oracle.sample_uniform(dims, x.numpy(), 5003, 20353, 9), torch.float64)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_mixed_radix_5way_gradient(gpu, dtype):
    t, to, dims = case("5way_65bit", dtype, gpu)
    R = 6
    A = (0.2 + 0.8 * synth.init_model(dims, R, 9, dtype=torch.float64)).to(dtype).to(gpu)
    A64 = A.double().cpu().numpy().reshape(-1)
    sp = G.SampleParams("stratified", 2000, 1500, seed=20353, step=3)
    t.reserve(sp.n, R)
    smp = oracle.sample_stratified(to, sp.p, sp.q, sp.seed, sp.step)
    Go, _ = oracle.loss_grad(dims, R, A64, *smp, "poisson")
    for what, kw in (("atomics", dict(tile=G.Tile(lds_modes=0, bucket_modes=0))),
                     ("bucketed", dict(tile=G.Tile(lds_modes=0, bucket_modes=31))), ("reproducible", dict(deterministic=True))):
        g, _ = G.gcp_loss_grad(t, sp, A, R, "poisson", **kw)
        t.status()
        assert_grad_close(g.double().cpu().numpy(), Go, dims, R, A64, *smp, "poisson", dtype, what=what)
