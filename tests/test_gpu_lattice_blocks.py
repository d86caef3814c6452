"""The lattice transform of few and many slabs, on both sides of every line of the rule for slabs per block.

Lines (mesh side times slabs, or side squared times slabs on a cube) under and over 200; one to several slabs per block,
full and partly filled last blocks, up to blocks filled to their limit.  Against torch's FFT in FP64.  An output is a sum
of N_k terms; the passes along the axes leave at most d (n + 4) + 2 roundings on a path for d axes of side n, so its error
is at most (d (n + 4) + 2) u sum |x|.
"""
import numpy as np
import pytest
import torch

from paper_2604_22223_amd import qgw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n", [(2, 2), (2, 9), (2, 15), (2, 24), (2, 36), (3, 2), (3, 6), (3, 8)])
@pytest.mark.parametrize("batch", [1, 4, 13, 25, 255, 256, 257, 625, 1025, 4099])
@pytest.mark.parametrize("precision", [qgw.F64, qgw.F32], ids=["f64", "f32"])
def test_transform_of_any_batch(dim, n, batch, precision):
    nodes = dict(omega=np.array([0.5]), tau_t=np.array([0.5]), n_f=np.array([0]), n_b=np.array([0]))
    p = qgw.Plan.from_nodes(n, [1], 1.0, nodes, precision=precision, dim=dim)
    c = torch.complex128 if precision == qgw.F64 else torch.complex64
    u = 2.0 ** -53 if precision == qgw.F64 else 2.0 ** -24
    g = torch.Generator().manual_seed(batch)
    x = torch.randn((batch,) + (n,) * dim, dtype=torch.complex128, generator=g).to("cuda:0").to(c)
    x64 = x.to(torch.complex128)
    axes = tuple(range(1, dim + 1))
    bar = (dim * (n + 4) + 2) * u * x64.abs().sum(dim=axes, keepdim=True)
    y = torch.full_like(x, float("nan"))
    p.lattice_fft(qgw.R_TO_K, x.view(batch, -1), y.view(batch, -1))
    assert bool(((y.to(torch.complex128) - torch.fft.fftn(x64, dim=axes)).abs() <= bar).all())
    y.fill_(float("nan"))
    p.lattice_fft(qgw.K_TO_R, x.view(batch, -1), y.view(batch, -1))
    assert bool(((y.to(torch.complex128) - torch.fft.ifftn(x64, dim=axes)).abs() <= bar / n ** dim).all())
    p.close()
