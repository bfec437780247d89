"""GPU parity of the Chapman-Enskog viscosity path: transport cross-section
and viscosity against hard-sphere closed forms and against the FP64 oracle
for the Jager form."""
import math

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_21244_amd import _lib
    _lib.load()
    return torch.device("cuda:0")


@pytest.fixture(scope="module")
def api(dev):
    from paper_2602_21244_amd import api as A
    return A


def test_hard_sphere_closed_forms(dev, api):
    say("CE hard sphere")
    d = 3.0
    pot = api.potential_hs(d)
    E = torch.tensor([50.0, 500.0, 5e4], dtype=torch.float64, device=dev)
    Q = api.transport_q2(E, 4e-10, pot, n_panels=64, n_gl=8).cpu().numpy()
    np.testing.assert_allclose(Q, 2.0 / 3.0 * math.pi * (d * 1e-10) ** 2, rtol=1e-12)
    T = torch.tensor([300.0, 3000.0], dtype=torch.float64, device=dev)
    om, mu = api.viscosity_ce(T, W.AR_MASS, 4e-10, pot, n_panels=64, n_gl=8, n_lag=8)
    np.testing.assert_allclose(om.cpu().numpy(), math.pi * (d * 1e-10) ** 2, rtol=1e-12)
    want = 5.0 / 16.0 * np.sqrt(math.pi * W.AR_MASS * W.KB * T.cpu().numpy()) / (math.pi * (d * 1e-10) ** 2)
    np.testing.assert_allclose(mu.cpu().numpy(), want, rtol=1e-12)
    om_p, _ = api.viscosity_ce(T, W.AR_MASS, 4e-10, pot, n_panels=64, n_gl=8, n_lag=8,
                               mode=api.L.CE_AS_PRINTED)
    np.testing.assert_allclose(om_p.cpu().numpy(), Q[0], rtol=1e-12)


def test_jager_cross_section_and_viscosity_match_oracle(orc, dev, api):
    say("CE Jager")
    pot = api.potential_jager(W.JAGER_PLACEHOLDER)
    P = orc.potential_jager(W.JAGER_PLACEHOLDER)
    b_cut = 2.5e-9
    E = np.array([20.0, 150.0, 1000.0, 3e4])
    Qg = api.transport_q2(torch.as_tensor(E, device=dev), b_cut, pot, n_panels=256,
                          n_gl=8).cpu().numpy()
    Qo = orc.transport_q2(P, E, b_cut, n_panels=256, n_gl=8)
    say("  Q2 rel err", np.abs(Qg - Qo) / Qo)
    np.testing.assert_allclose(Qg, Qo, rtol=1e-6)
    T = np.array([1500.0, 3000.0, 6000.0])
    om, mu = api.viscosity_ce(torch.as_tensor(T, device=dev), W.AR_MASS, b_cut, pot,
                              n_panels=256, n_gl=8, n_lag=16)
    oo = orc.collision_integral(P, T, b_cut, n_lag=16, n_panels=256, n_gl=8)
    mo = orc.viscosity_ce(oo, T, W.AR_MASS)
    say("  mu (Pa s)", mu.cpu().numpy(), "oracle", mo)
    np.testing.assert_allclose(om.cpu().numpy(), oo, rtol=1e-6)
    np.testing.assert_allclose(mu.cpu().numpy(), mo, rtol=1e-6)


def test_cross_section_routes_agree(dev, api):
    """Rules of up to 32 nodes a panel take the potential's table, longer ones
    the direct kernel: the same integral by 64 panels of 32 nodes and by 32 of
    64 (2 048 nodes each) agrees to the b rule's own convergence, which 48 of
    32 against 64 of 32 bounds."""
    E = torch.tensor([150.0, 300.0, 1000.0, 20000.0], dtype=torch.float64, device=dev)
    pot = api.potential_jager(W.JAGER_PLACEHOLDER)
    a = api.transport_q2(E, 2.5e-9, pot, n_panels=64, n_gl=32).cpu().numpy()
    b = api.transport_q2(E, 2.5e-9, pot, n_panels=32, n_gl=64).cpu().numpy()
    c = api.transport_q2(E, 2.5e-9, pot, n_panels=48, n_gl=32).cpu().numpy()
    say("  Q2 routes: rel", np.abs(b / a - 1).max(), "48 panels:", np.abs(c / a - 1).max())
    assert np.all(np.abs(b / a - 1) <= 1e-9 + 4 * np.abs(c / a - 1))


@pytest.mark.parametrize("n_gl", [2, 7, 8, 31, 32, 33])
def test_cross_section_is_its_rules_sum(dev, api, n_gl):
    """Q2 against the sum over the same panels and nodes of the batch entry point's
    angles: rules of an even and an odd number of nodes on the table route and one
    on the direct route, to 1e-10 (the angles' own bound is 1e-9 to 1e-7, of which
    a node has a hundredth of the sum at most)."""
    say("Q2 node by node", n_gl)
    E = np.array([150.0, 300.0, 1000.0, 20000.0, 5e5])
    pot, b_cut, n_panels = api.potential_jager(W.JAGER_PLACEHOLDER), 2.5e-9, 24
    x, w = np.polynomial.legendre.leggauss(n_gl)
    h = b_cut / n_panels
    b = (h * (np.arange(n_panels)[:, None] + 0.5 * (1.0 + x))).ravel()
    wb = np.tile(0.5 * h * w, n_panels) * b
    g = np.sqrt(2.0 * W.KB * E / (W.AR_MASS / 2))
    chi = api.deflect_jager(torch.as_tensor(np.tile(b, len(E)), device=dev),
                            torch.as_tensor(np.repeat(g, b.size), device=dev), W.AR_MASS / 2, pot)
    chi = chi.cpu().numpy().reshape(len(E), -1)
    want = 2.0 * math.pi * np.sum(np.sin(chi) ** 2 * wb, axis=1)
    Q = api.transport_q2(torch.as_tensor(E, device=dev), b_cut, pot, n_panels=n_panels, n_gl=n_gl)
    err = np.abs(Q.cpu().numpy() / want - 1.0)
    say("  rel", err)
    assert err.max() < 1e-10
