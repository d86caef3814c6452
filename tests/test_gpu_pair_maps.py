"""The pair maps with a layout change at the sizes where their kernels change or leave remainders.

Every result is held to the map as a dense product in FP64 (the plan's own map, qgw_plan_get_map): each output is a sum
of r products, so its rounding stays within 2 (r + 4) u sum |T| |x| with u = 2^-53 or 2^-24 (in FP32 the map is rounded
once more, which the same bound holds).
"""
import numpy as np
import pytest
import torch

from paper_2604_22223_amd import qgw

pytestmark = pytest.mark.gpu


def nodes(rank):
    x = np.linspace(-4.0, 4.0, rank) if rank > 1 else np.array([0.5])
    return dict(omega=x, tau_t=(np.arange(rank) + 0.5) / rank, n_f=np.arange(rank) - rank // 2,
                n_b=np.arange(rank) - rank // 2)


# ranks around the 4-deep slices and 16-row tiles; columns of one strip, ragged strips, and on both sides of the
# 24,576 columns (96 per CU of 256) up to which the small-column kernel runs (N_b = 16, 9 x 9 and 10 x 10)
@pytest.mark.parametrize("rank", [1, 4, 5, 15, 16, 17, 33, 48, 49, 53, 63, 64])
@pytest.mark.parametrize("site_norb,n", [([1], 1), ([1, 1], 3), ([2, 1], 5), ([4], 9), ([4], 10), ([3], 20)], ids=str)
@pytest.mark.parametrize("precision", [qgw.F64, qgw.F32], ids=["f64", "f32"])
def test_pair_maps_are_the_dense_product(rank, site_norb, n, precision):
    rng = np.random.default_rng(rank)
    p = qgw.Plan.from_nodes(n, site_norb, 1.0, nodes(rank), precision=precision)
    c = torch.complex128 if precision == qgw.F64 else torch.complex64
    na, nk = p.n_b * p.n_b, p.n_k
    x = torch.from_numpy(rng.standard_normal((rank, na, nk)) + 1j * rng.standard_normal((rank, na, nk))).to("cuda:0").to(c)
    print("\n[pair maps] r = %d, %s, %d x %d" % (rank, site_norb, n, n), flush=True)
    u = 2.0 ** -53 if precision == qgw.F64 else 2.0 ** -24
    for which in (qgw.B_TAU2IW, qgw.B_IW2TAU):
        T = torch.from_numpy(p.get_map(which)).to("cuda:0")
        x64 = x.to(torch.complex128)
        ref = (T @ x64.reshape(rank, -1)).reshape(rank, na, nk)
        # Re and Im are sums of r products each of |T| |x| at most
        bar = 4.0 * (rank + 4) * u * (T.abs() @ x64.abs().reshape(rank, -1)).reshape(rank, na, nk)
        y = torch.full((rank, nk, na), float("nan"), dtype=c, device="cuda:0")
        p.dlr_transform_pairs(which, qgw.LAYOUT_SLAB, qgw.LAYOUT_MATRIX, x, y)
        assert bool(((y.to(torch.complex128).transpose(1, 2) - ref).abs() <= bar).all())
        z = torch.full((rank, na, nk), float("nan"), dtype=c, device="cuda:0")
        p.dlr_transform_pairs(which, qgw.LAYOUT_MATRIX, qgw.LAYOUT_SLAB, x.transpose(1, 2).contiguous(), z)
        assert bool(((z.to(torch.complex128) - ref).abs() <= bar).all())
    p.close()


# on both sides of the lines between the kernels in FP64 (44 columns per CU of 256 with up to two row tiles, 60 with
# more) and of the line for wave priority (512 columns per block of 512 blocks)
@pytest.mark.parametrize("rank,site_norb,n", [(r, s, n) for r in (16, 32, 33, 64)
                                              for s, n in (([2], 24), ([3], 12), ([2], 30), ([4], 8))]
                         + [(33, [5], 18), (33, [5], 24)], ids=str)
@pytest.mark.parametrize("precision", [qgw.F64, qgw.F32], ids=["f64", "f32"])
def test_pair_maps_between_kernels(rank, site_norb, n, precision):
    test_pair_maps_are_the_dense_product(rank, site_norb, n, precision)
