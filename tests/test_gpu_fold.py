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


def fold_v(rng, nk, site_norb):
    """Hermitian V(q) unchanged under i <-> l of either index (random values per class pair)."""
    first, second, off = [], [], 0
    for n in site_norb:
        for i in range(n):
            for l in range(n):
                first.append(off + min(i, l))
                second.append(off + max(i, l))
        off += n
    cls = {}
    idx = np.array([cls.setdefault(k, len(cls)) for k in zip(first, second)])
    v = rng.standard_normal((nk, len(cls), len(cls))) + 1j * rng.standard_normal((nk, len(cls), len(cls)))
    v = 0.1 * (v + np.conj(np.swapaxes(v, 1, 2))) + 0.5 * np.eye(len(cls))
    return np.ascontiguousarray(v[:, idx][:, :, idx])


# every compiled (N_b, classes) pair of the folded solver; ranks of every remainder modulo four nodes per wavefront, on
# a mesh that puts the matrices above the 4,096 from which the folded solver runs
@pytest.mark.parametrize("site_norb", [[5], [4, 3], [4], [2, 2, 2, 2], [3], [2, 2, 1]], ids=str)
@pytest.mark.parametrize("rank", [4, 5, 6, 7])
@pytest.mark.parametrize("mixed", [False, True], ids=["symmetric", "some_q_not"])
def test_dyson_w_of_a_foldable_interaction(site_norb, rank, mixed):
    n = 32
    nk = n * n
    rng = np.random.default_rng(5 + rank)
    nodes = dict(omega=np.linspace(-1.0, 1.0, rank), tau_t=np.linspace(0.1, 0.9, rank), n_f=np.arange(rank) - rank // 2,
                 n_b=np.arange(rank) - rank // 2)
    p = qgw.Plan.from_nodes(n, site_norb, 3.0, nodes)
    nb = p.n_b
    v = fold_v(rng, nk, site_norb)
    if mixed:  # one entry of one index at some q
        v[1, 1, 0] += 0.1
        v[4, 0, 1] += 0.1
    pnu = 0.05 * (rng.standard_normal((rank, nk, nb, nb)) + 1j * rng.standard_normal((rank, nk, nb, nb)))
    vd, pd = dev(v), dev(pnu)
    out = torch.empty_like(pd)
    print("\n[fold] Dyson W %s, rank %d" % (site_norb, rank), flush=True)
    p.dyson_W(vd, pd, out)
    p.sync_status()
    some = np.unique(np.concatenate([[0, 1, 4, nk - 1], rng.integers(0, nk, 40)]))  # the q compared
    v64, p64 = v[some], pnu[:, some]
    ref = np.linalg.solve(np.eye(nb) - v64[None] @ p64, np.broadcast_to(v64[None], p64.shape)) - v64[None]
    assert rel_err(out.cpu().numpy()[:, some], ref) < TOL
    p.dyson_W(vd, pd, pd)  # the output over P: the general kernel alone
    assert rel_err(pd.cpu().numpy()[:, some], ref) < TOL
    p.close()


@pytest.mark.parametrize("site_norb", [[5], [4], [3]], ids=str)
def test_singular_system_of_a_foldable_interaction_is_reported(site_norb):
    """I - V P with a zero row and column in the folded basis: the status word, and non-finite entries there only."""
    n, rank = 32, 5
    nodes = dict(omega=np.linspace(-1.0, 1.0, rank), tau_t=np.linspace(0.1, 0.9, rank), n_f=np.arange(rank) - 2,
                 n_b=np.arange(rank) - 2)
    p = qgw.Plan.from_nodes(n, site_norb, 3.0, nodes)
    nb, nk = p.n_b, p.n_k
    v = np.zeros((nk, nb, nb), dtype=complex)
    v[:, 0, 0] = 2.0
    pnu = np.zeros((rank, nk, nb, nb), dtype=complex)
    pnu[3, 1, 0, 0] = 0.5
    out = torch.empty((rank, nk, nb, nb), dtype=torch.complex128, device="cuda:0")
    p.dyson_W(dev(v), dev(pnu), out)
    with pytest.raises(qgw.QGWError) as e:
        p.sync_status()
    assert e.value.status == qgw.QGW_ERR_SINGULAR
    got = out.cpu().numpy()
    assert not np.all(np.isfinite(got[3, 1]))
    got[3, 1] = 0.0
    assert np.all(got == 0.0)
    p.close()


# N_b = 9 with 8 classes: a state folds it, the call on full matrices has no folded solver and takes the general one
NINE_EIGHT = [2, 1, 1, 1, 1, 1]


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("symmetric", [True, False], ids=["folded", "full"])
def test_state_of_nine_pairs_in_eight_classes(dim, symmetric):
    test_state_in_the_folded_basis(NINE_EIGHT, dim, symmetric)


@pytest.mark.parametrize("mixed", [False, True], ids=["symmetric", "some_q_not"])
def test_dyson_w_of_nine_pairs_in_eight_classes(mixed):
    test_dyson_w_of_a_foldable_interaction(NINE_EIGHT, 5, mixed)


def test_adjoint_of_nine_pairs_in_eight_classes():
    """The adjoint's forward solve at the same size (5 x 32^2 matrices), against dense solves at some q."""
    n, rank = 32, 5
    nodes = dict(omega=np.linspace(-1.0, 1.0, rank), tau_t=np.linspace(0.1, 0.9, rank), n_f=np.arange(rank) - 2,
                 n_b=np.arange(rank) - 2)
    rng = np.random.default_rng(3)
    p = qgw.Plan.from_nodes(n, NINE_EIGHT, 3.0, nodes)
    nb, nk = p.n_b, p.n_k
    v = fold_v(rng, nk, NINE_EIGHT)
    pnu, b = (rng.standard_normal((rank, nk, nb, nb)) + 1j * rng.standard_normal((rank, nk, nb, nb)) for _ in range(2))
    pnu *= 0.05
    pd = dev(pnu)
    pbar, vbar = torch.zeros_like(pd), torch.zeros_like(dev(v))
    p.dyson_W_bwd(dev(v), pd, dev(b), pbar, vbar)
    p.sync_status()
    some = np.array([0, 1, 31, 32, 500, nk - 1])
    vs, ps, bs = v[some][None], pnu[:, some], b[:, some]
    a = np.eye(nb) - vs @ ps
    w = np.linalg.solve(a, np.broadcast_to(vs, ps.shape))
    h = lambda x: np.conj(np.swapaxes(x, -1, -2))  # noqa: E731
    x = np.linalg.solve(h(a), bs)
    assert rel_err(pbar.cpu().numpy()[:, some], h(w) @ bs @ h(w)) < TOL
    assert rel_err(vbar.cpu().numpy()[some], (x + x @ h(w) @ h(ps) - bs).sum(axis=0)) < TOL
    p.close()


@pytest.mark.parametrize("dim,n,grid,eps", [(2, 5, "dlr", 1e-9), (3, 3, "dlr", 1e-9), (2, 3, "dlr", 1e-13), (2, 4, "mf", 0)])
def test_p_of_a_folded_state_on_every_grid(dim, n, grid, eps):
    """P of a folded state on the grids and ranks its map has (a rank above 64 among them), against the bubble and map of
    G(i w) as the step calls make them; nothing past the end of dst."""
    make = wl.random_model if dim == 2 else wl.random_model_3d
    w = make((n,) * dim, [2, 1], seed=5, U=1.0, J=0.1, Vnn=0.1, beta=8.0 if eps != 1e-13 else 400.0, omega_max=16.0, eps=1e-9)
    if grid == "mf":
        p = qgw.Plan.uniform(n, w["site_norb"], w["beta"], 128, dim=dim)
    else:
        nodes = qgw.dlr_build(w["beta"] * w["omega_max"], eps)
        nodes["omega"] = nodes["x"] / w["beta"]
        p = qgw.Plan.from_nodes(n, w["site_norb"], w["beta"], nodes, dim=dim)
    assert (p.r > 64) == (eps == 1e-13 or grid == "mf")
    st = qgw.State(p, dev(flat(w["H_R"], dim)), dev(flat(w["V_R"], dim)), n_target=w["n_target"])
    st.init_g0()
    g0 = st.array(0)
    st.iterate(1)
    c = torch.complex128
    gt, gr = (torch.empty((p.r, p.n_o, p.n_o, p.n_k), dtype=c, device="cuda:0") for _ in range(2))
    p.dlr_transform(qgw.F_IW2TAU, g0, gt)
    p.dlr_transform(qgw.F_IW2TAUR, g0, gr)
    for x in (gt, gr):
        p.lattice_fft(qgw.K_TO_R, x, x)
    pq = torch.empty((p.r, p.n_b, p.n_b, p.n_k), dtype=c, device="cuda:0")
    ref = torch.empty((p.r, p.n_k, p.n_b, p.n_b), dtype=c, device="cuda:0")
    p.bubble(gt, gr, pq)
    p.dlr_transform_pairs(qgw.B_TAU2IW, qgw.LAYOUT_SLAB, qgw.LAYOUT_MATRIX, pq, ref)
    big = torch.full((ref.numel() + 64,), -7.0, dtype=c, device="cuda:0")
    qgw._check(qgw.lib().qgw_state_copy(st.handle, 3, qgw._ptr(big), None, qgw._stream()))
    assert bool((big[ref.numel():] == -7.0).all())
    assert rel_err(big[:ref.numel()].cpu().numpy(), ref.reshape(-1).cpu().numpy()) < TOL
    st.close()
    p.close()


def test_copies_of_p_do_not_disturb_iterations():
    """Copies of P on one stream while the state iterates on another: the iterations end as without them."""
    w = wl.five_orbital(n=12, U=1.0, J=0.1, Vnn=0.2, beta=20.0, omega_max=25.0, eps=1e-8, scale_mesh=12)
    nodes = qgw.dlr_build(w["beta"] * w["omega_max"], w["eps"])
    nodes["omega"] = nodes["x"] / w["beta"]
    p = qgw.Plan.from_nodes(12, w["site_norb"], w["beta"], nodes)
    sig = []
    for copies in (0, 40):
        st = qgw.State(p, dev(flat(w["H_R"], 2)), dev(flat(w["V_R"], 2)), n_target=w["n_target"])
        st.init_g0()
        b = qgw.Batch([st], n_iter=8)
        other = torch.cuda.Stream()
        torch.cuda.synchronize()
        b.launch()
        with torch.cuda.stream(other):
            for _ in range(copies):
                st.array(3)
        b.launch()
        torch.cuda.synchronize()
        assert b.read()[2][0] == 0
        sig.append(st.array(1).cpu().numpy())
        b.close()
        st.close()
    assert np.array_equal(sig[0], sig[1])
    p.close()


@pytest.mark.parametrize("site_norb", [[3], [2, 2, 1], NINE_EIGHT], ids=str)
@pytest.mark.parametrize("n,rank", [(1, 1), (3, 5), (6, 61), (6, 62)])
@pytest.mark.parametrize("precision", [qgw.F64, qgw.F32], ids=["f64", "f32"])
def test_dyson_w_of_few_nine_pair_matrices(site_norb, n, rank, precision):
    """N_b = 9 on both sides of the 2,200 FP64 matrices from which a wavefront takes four, down to one matrix.  FP32: each
    of the 9 elimination steps and the product V P leave an error of a few u relative to the entries; 4 N_b^2 u of the
    largest entry holds at the condition these matrices have (below 4)."""
    nk = n * n
    rng = np.random.default_rng(rank)
    nodes = dict(omega=np.linspace(-1.0, 1.0, rank), tau_t=np.linspace(0.1, 0.9, rank), n_f=np.arange(rank) - rank // 2,
                 n_b=np.arange(rank) - rank // 2)
    p = qgw.Plan.from_nodes(n, site_norb, 3.0, nodes, precision=precision)
    nb = p.n_b
    v = fold_v(rng, nk, site_norb) + 0.01 * rng.standard_normal((nk, nb, nb))
    pnu = 0.02 * (rng.standard_normal((rank, nk, nb, nb)) + 1j * rng.standard_normal((rank, nk, nb, nb)))
    c = torch.complex128 if precision == qgw.F64 else torch.complex64
    vd, pd = dev(v).to(c), dev(pnu).to(c)
    v, pnu = vd.cpu().numpy().astype(complex), pd.cpu().numpy().astype(complex)
    a = np.eye(nb) - v[None] @ pnu
    assert np.linalg.cond(a).max() < 4.0
    out = torch.full_like(pd, float("nan"))
    p.dyson_W(vd, pd, out)
    p.sync_status()
    ref = np.linalg.solve(a, np.broadcast_to(v[None], pnu.shape)) - v[None]
    err = np.abs(out.cpu().numpy() - ref).max()
    if precision == qgw.F64:
        assert err < TOL * np.abs(ref).max()
    else:
        assert err < 4 * nb ** 2 * 2.0 ** -24 * np.abs(ref + v[None]).max()
    p.close()


@pytest.mark.parametrize("site_norb", [[2], [2, 1], [2, 2], [3], [2, 2, 1], NINE_EIGHT, [4], [2, 2, 2, 2], [3, 2, 1, 1, 1],
                                       [5], [4, 3]], ids=str)
@pytest.mark.parametrize("n", [3, 16])
@pytest.mark.parametrize("symmetric", [True, False], ids=["folded", "full"])
def test_single_precision_iteration_in_every_basis(site_norb, n, symmetric):
    """One FP32 iteration from G0 in every number of classes, with few matrices and with more than the 6,000 from which all
    sizes take four to a wavefront, against the FP64 iteration of the same state (held to the oracle above).  The bar is
    that of the FP32 iteration elsewhere, 2e-4 of the largest entry: rounding 2^-24, amplified up to 56 times by the map
    i nu -> tau, in sums of up to 64 nodes."""
    w = wl.random_model((n, n), site_norb, seed=11, U=1.0, J=0.1, Vnn=0.1, beta=8.0, omega_max=16.0, eps=1e-9)
    if not symmetric:
        w["V_R"][(1, 1, 0, 0)] += 0.05
    nodes = qgw.dlr_build(w["beta"] * w["omega_max"], w["eps"])
    nodes["omega"] = nodes["x"] / w["beta"]
    p = qgw.Plan.from_nodes(n, site_norb, w["beta"], nodes)
    assert (p.r * p.n_k >= 6000) == (n == 16)
    st = qgw.State(p, dev(flat(w["H_R"], 2)), dev(flat(w["V_R"], 2)), n_target=w["n_target"])
    sig = []
    for mode in (0, 2):
        st.set_precision(mode)
        st.init_g0()
        st.iterate(1)
        sig.append(st.array(1).cpu().numpy())
    assert 0.0 < rel_err(sig[1], sig[0]) < 2e-4
    st.close()
    p.close()
