"""The bubble over all pairs at output sizes on both sides of the lines between plain and streamed stores (30 MB, 128 MiB).

Five orbitals on 24 x 24: an output node takes 5.76 MB in FP64 and 2.88 MB in FP32.  Against the product and the
transform in FP64 with torch.  An output is a sum of 576 products; two passes of length 24 and the product leave less than
2 (24 + 4) + 8 = 64 roundings on any path through them, so its error is at most 64 u sum_R |P(R)|, u = 2^-53 or 2^-24.
"""
import numpy as np
import pytest
import torch

from paper_2604_22223_amd import qgw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,rank", [(qgw.F64, 5), (qgw.F64, 6), (qgw.F64, 23), (qgw.F64, 24), (qgw.F32, 10),
                                            (qgw.F32, 11), (qgw.F32, 46), (qgw.F32, 47)])
def test_bubble_by_output_size(precision, rank):
    n, no = 24, 5
    nodes = dict(omega=np.linspace(-1.0, 1.0, rank), tau_t=np.linspace(0.1, 0.9, rank), n_f=np.arange(rank) - rank // 2,
                 n_b=np.arange(rank) - rank // 2)
    p = qgw.Plan.from_nodes(n, [no], 3.0, nodes, precision=precision)
    c = torch.complex128 if precision == qgw.F64 else torch.complex64
    rng = np.random.default_rng(rank)
    gt, gr = (torch.from_numpy(rng.standard_normal((rank, no, no, n, n)) + 1j * rng.standard_normal((rank, no, no, n, n)))
              .to("cuda:0").to(c) for _ in range(2))
    out = torch.full((rank, no * no, no * no, n, n), float("nan"), dtype=c, device="cuda:0")
    p.bubble(gt.view(rank, no, no, n * n), gr.view(rank, no, no, n * n), out.view(rank, no * no, no * no, n * n))
    i = (-torch.arange(n, device="cuda:0")) % n
    u = 2.0 ** -53 if precision == qgw.F64 else 2.0 ** -24
    for t in sorted({0, rank // 2, rank - 1}):
        a = gt[t].to(torch.complex128)                           # [l, j]
        b = gr[t].to(torch.complex128)[:, :, i][:, :, :, i]      # [k, i] at -R
        # P_{(il),(jk)}(R) = -2 G_lj(R) G_ki(-R)
        x = -2.0 * a[None, :, :, None] * b.permute(1, 0, 2, 3)[:, None, None, :]
        x = x.reshape(no * no, no * no, n, n)
        bar = 64.0 * u * x.abs().sum(dim=(2, 3), keepdim=True)
        assert bool(((out[t].to(torch.complex128) - torch.fft.fft2(x)).abs() <= bar).all())
    p.close()
