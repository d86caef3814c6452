"""The folded pair basis of a state (classes of (i, l) and (l, i)) against the oracle.

A state whose V(R) does not change under i <-> l of either pair index keeps its pair arrays per class; one whose V(R)
does change keeps the full basis.  Both are held to the oracle's iteration at 1e-10 in every output, P and W^C (which
come back in the full basis) among them.
"""
import numpy as np
import pytest
import torch

from oracle import gw
from oracle.dlr import DLR
from paper_2604_22223_amd import qgw
from paper_2604_22223_amd import workloads as wl

pytestmark = pytest.mark.gpu
TOL = 1e-10


def flat(x, d):
    return np.ascontiguousarray(x.reshape(x.shape[:x.ndim - d] + (-1,)))


def dev(x):
    return torch.from_numpy(x.astype(np.complex128)).to("cuda:0")


def rel_err(a, b):
    return np.abs(a - b).max() / np.abs(b).max()


def matrix(x, d):  # oracle [m, A, B, *mesh] -> [m, k, A, B]
    return np.moveaxis(flat(x, d), -1, 1)


# N_b -> classes: 4 -> 3, 5 -> 4, 8 -> 6, 9 -> 6, 9 -> 7, 16 -> 10, 16 -> 12, 25 -> 15, 25 -> 16
@pytest.mark.parametrize("site_norb", [[2], [2, 1], [2, 2], [3], [2, 2, 1], [4], [3, 2, 1, 1, 1], [5], [4, 3]], ids=str)
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("symmetric", [True, False], ids=["folded", "full"])
def test_state_in_the_folded_basis(site_norb, dim, symmetric):
    n = 3
    make = wl.random_model if dim == 2 else wl.random_model_3d
    w = make((n,) * dim, site_norb, seed=11, U=1.0, J=0.1, Vnn=0.1, beta=8.0, omega_max=16.0, eps=1e-9)
    if not symmetric:  # an exchange element of one ordered pair only
        w["V_R"][(1, 1) + (0,) * dim] += 0.05
    print("\n[fold] %s, %d-D, %s" % (site_norb, dim, "folded" if symmetric else "full"), flush=True)
    d = DLR(w["beta"], w["omega_max"], w["eps"])
    m = gw.Model(w["mesh"], w["site_norb"], w["H_R"], w["V_R"], w["beta"], w["n_target"])
    s1 = gw.gw_iteration(m, d, gw.initial_state(m, d), keep=True)
    p = qgw.Plan.from_nodes(n, site_norb, w["beta"], d.nodes(), dim=dim)
    st = qgw.State(p, dev(flat(w["H_R"], dim)), dev(flat(w["V_R"], dim)), n_target=w["n_target"])
    st.init_g0()
    _, _, mu = st.iterate(1)
    host = lambda k: st.array(k).cpu().numpy()  # noqa: E731
    assert abs(mu - s1["mu"]) < TOL * max(1.0, abs(mu))
    assert rel_err(host(1), flat(s1["sig_iw"], dim)) < TOL
    assert rel_err(host(0), flat(s1["G_iw"], dim)) < TOL
    # P and W^C; P a second time, after another stopped iteration has queued its next step
    assert rel_err(host(3), matrix(s1["intermediates"]["P_nu_q"], dim)) < TOL
    assert rel_err(host(4), matrix(s1["intermediates"]["Wc_nu_q"], dim)) < TOL
    s2 = gw.gw_iteration(m, d, s1, keep=True)
    assert st.iterate(5, tol=1e6)[0] == 1
    assert rel_err(host(3), matrix(s2["intermediates"]["P_nu_q"], dim)) < TOL
    assert rel_err(host(1), flat(s2["sig_iw"], dim)) < TOL
