"""The chemical-potential search in one launch against the oracle's bisection.

One block takes the whole search where n_o <= 2 and the points r N_k fit its registers (16384 / n_o) or where n_o >= 3
and r N_k n_o^3 is at most 50000, and the rest is taken by launches; the sizes here lie on both sides of each line and
leave partly filled blocks.  The bar is the FP64 parity bar, 1e-10.
"""
import numpy as np
import pytest

from conftest import rel_err
from oracle import gw
from oracle.dlr import DLR
from paper_2604_22223_amd import qgw
from paper_2604_22223_amd import workloads as wl

pytestmark = pytest.mark.gpu

TOL = 1e-10
BETA = 12.0


def _torch():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    return torch


@pytest.fixture(scope="module")
def dlr():
    return DLR(BETA, 8.0, 1e-10)


def dev(x):
    return _torch().from_numpy(np.ascontiguousarray(x.reshape(x.shape[:-2] + (-1,)))).to("cuda:0")


@pytest.mark.parametrize("sigma", [False, True])
@pytest.mark.parametrize("n_o,n", [(1, 1), (1, 2), (1, 16), (1, 20), (1, 24), (1, 25), (2, 1), (2, 6), (2, 15), (2, 16),
                                   (2, 18), (3, 3), (3, 6), (3, 8), (4, 4), (4, 5), (4, 6), (5, 3), (5, 4), (8, 1),
                                   (8, 2)])
def test_search_against_oracle(dlr, n_o, n, sigma):
    torch = _torch()
    r = len(dlr.iw)
    rng = np.random.default_rng(100 * n_o + n)
    x = rng.standard_normal((n_o, n_o, n, n)) + 1j * rng.standard_normal((n_o, n_o, n, n))
    h = x + np.conj(np.swapaxes(x, 0, 1))
    sig = None
    if sigma:  # poles at +-0.7 with positive weights that differ per orbital pair and k
        c = 0.3 * (rng.standard_normal((n_o, n_o, n, n)) + 1j * rng.standard_normal((n_o, n_o, n, n)))
        w = np.einsum("ac...,bc...->ab...", c, np.conj(c))
        sig = np.stack([w * (0.5 / (z - 0.7) + 0.5 / (z + 0.7)) for z in dlr.iw])
    nt = 0.8 * n_o
    mu_ref, g_ref, _ = gw.solve_mu(h, np.zeros_like(h), sig, dlr, nt)
    sites = {3: [3], 6: [2, 1, 1, 1, 1], 7: [2, 1, 1, 1, 1, 1]}.get(n_o, [1] * n_o)
    plan = qgw.Plan.from_nodes(n, sites, BETA, dlr.nodes())
    out = torch.empty((r, n_o, n_o, n * n), dtype=torch.complex128, device="cuda:0")
    hd, sd = dev(h), None if sig is None else dev(sig)
    for start in (0.0, mu_ref + 0.3, -6.0):
        mu = plan.dyson_G(hd, sd, out, n_target=nt, mu=start)
        assert abs(mu - mu_ref) <= TOL * max(1.0, abs(mu_ref))
        assert rel_err(out.cpu().numpy(), g_ref.reshape(out.shape)) < TOL
    plan.close()


@pytest.mark.parametrize("seed", [6, 7])
def test_late_evaluations_of_a_batch(seed):
    """A chain of 64 evaluations: ten launches and one more for the rest (r N_k n_o^3 = 43 * 64 * 27 or so), against the
    eager search's launches.  An almost full band at low temperature, whose search takes more than ten evaluations."""
    w = wl.random_model((8, 8), [2, 1], seed=seed, beta=500.0, omega_max=12.0, eps=1e-8, U=6.0, J=0.3, Vnn=0.5,
                        n_target=4.0 - 1e-7)
    d = DLR(w["beta"], w["omega_max"], w["eps"])
    plan = qgw.Plan.from_nodes(8, w["site_norb"], w["beta"], d.nodes())
    states = [qgw.State(plan, dev(w["H_R"]), dev(w["V_R"]), n_target=w["n_target"]) for _ in range(2)]
    for st in states:
        st.init_g0()
    b = qgw.Batch([states[0]], mu_steps=64)
    b.launch()
    ds, mu, status, evals = b.read(with_evals=True)
    _, ds_ref, mu_ref = states[1].iterate(1)
    assert status[0] == 0 and evals[0] > 10
    assert abs(mu[0] - mu_ref) <= TOL * abs(mu_ref)
    assert abs(ds[0] - ds_ref) <= TOL * ds_ref
    assert rel_err(states[0].array(0).cpu().numpy(), states[1].array(0).cpu().numpy()) < TOL
    b.close()
    for st in states:
        st.close()
    plan.close()


@pytest.mark.parametrize("sigma", [False, True])
@pytest.mark.parametrize("n_o,n", [(1, 2), (1, 16), (2, 1), (2, 6), (3, 3)])
def test_search_from_afar(n_o, n, sigma):
    """Starts of tens to hundreds of eV from the solution (as far as a search from there ends at all), and levels with a
    common offset of 1000 eV.  Where the search began must not show: it ends at a filling error of 1e-13 or a step of
    1e-13, so the filling of the returned mu, taken from inverses in NumPy, is within 1e-13 max(1, dN/dmu) and the
    rounding of the two evaluations, together at most twice that; at the offset the parity bar holds."""
    torch = _torch()
    d = DLR(100.0, 20.0, 1e-10)
    r = len(d.iw)
    rng = np.random.default_rng(10 * n_o + n)
    x = rng.standard_normal((n_o, n_o, n, n)) + 1j * rng.standard_normal((n_o, n_o, n, n))
    h = x + np.conj(np.swapaxes(x, 0, 1))
    sig = np.zeros((r, n_o, n_o, n, n), dtype=complex)
    if sigma:
        c = 0.3 * (rng.standard_normal((n_o, n_o, n, n)) + 1j * rng.standard_normal((n_o, n_o, n, n)))
        w = np.einsum("ac...,bc...->ab...", c, np.conj(c))
        sig = np.stack([w * (0.5 / (z - 0.7) + 0.5 / (z + 0.7)) for z in d.iw])
    nt = 0.8 * n_o
    rho = np.asarray(d.F_iw2beta).reshape(-1)
    base = np.moveaxis(-h[None] - sig, (1, 2), (3, 4))

    def filling(mu):  # N_e and dN_e/dmu
        g = np.linalg.inv(base + (np.asarray(d.iw)[:, None, None, None, None] + mu) * np.eye(n_o))
        t1, t2 = np.einsum("mxyaa->m", g), np.einsum("mxyab,mxyba->m", g, g)
        return -2.0 * (rho @ t1).real / n ** 2, 2.0 * (rho @ t2).real / n ** 2

    plan = qgw.Plan.from_nodes(n, [3] if n_o == 3 else [1] * n_o, 100.0, d.nodes())
    out = torch.empty((r, n_o, n_o, n * n), dtype=torch.complex128, device="cuda:0")
    hd, sd = dev(h), dev(sig) if sigma else None
    for start in (0.0, -30.0, 30.0, 100.0, -300.0):
        mu = plan.dyson_G(hd, sd, out, n_target=nt, mu=start)
        ne, dne = filling(mu)
        assert abs(ne - nt) <= 2e-13 * max(1.0, dne), (start, ne - nt)
    mu_ref, far = mu, dev(h + 1000.0 * np.eye(n_o)[:, :, None, None])
    for start in (1000.0, 970.0, 1030.0):
        mu = plan.dyson_G(far, sd, out, n_target=nt, mu=start)
        assert abs(mu - 1000.0 - mu_ref) <= TOL
    plan.close()


@pytest.mark.parametrize("sites,n", [([2, 1], 24), ([2, 1, 1, 1, 1], 9), ([4, 3], 6), ([2, 2, 2, 2], 6)], ids=str)
def test_late_evaluations_in_several_blocks(sites, n):
    """As above on larger systems, whose late evaluations several blocks share, against the
    eager search's launches: the first two iterations of almost full bands, the first with more than ten evaluations
    except at [2, 1] (nine)."""
    full = 2.0 * sum(sites)
    w = wl.random_model((n, n), sites, seed=7, beta=300.0, omega_max=12.0, eps=1e-8, U=4.0, J=0.3, Vnn=0.5,
                        n_target=full - 1e-6)
    nodes = qgw.dlr_build(w["beta"] * w["omega_max"], w["eps"])
    nodes["omega"] = nodes["x"] / w["beta"]
    plan = qgw.Plan.from_nodes(n, sites, w["beta"], nodes)
    states = [qgw.State(plan, dev(w["H_R"]), dev(w["V_R"]), n_target=w["n_target"], mixing=0.5) for _ in range(2)]
    for st in states:
        st.init_g0()
    b = qgw.Batch([states[0]], mu_steps=64)
    for it in range(2):
        b.launch()
        ds, mu, status, evals = b.read(with_evals=True)
        _, ds_ref, mu_ref = states[1].iterate(1)
        assert status[0] == 0 and evals[0] == states[1].mu_evals()
        assert it > 0 or evals[0] > (8 if sites == [2, 1] else 10)
        assert abs(mu[0] - mu_ref) <= TOL * abs(mu_ref)
        assert abs(ds[0] - ds_ref) <= TOL * ds_ref
        assert rel_err(states[0].array(0).cpu().numpy(), states[1].array(0).cpu().numpy()) < TOL
    b.close()
    for st in states:
        st.close()
    plan.close()
