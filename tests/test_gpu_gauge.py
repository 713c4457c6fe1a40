"""GPU parity of the Wilson gauge force and action (the force whose spectra section 2 measures)
against the oracle, the gauge-force power spectrum pipeline of Fig. 1 on synthetic links, and
finite differences of the GPU's own action."""
import numpy as np
import pytest
import torch
from scipy.linalg import expm

from gpu_helpers import announce, dev, rel_max, setup
from oracle import chebyshev as och
from oracle import gauge as og
from oracle import su3
from paper_2112_04556_amd import api, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,kind,beta", [((4, 4, 6, 5), "eps", 6.4), ((4, 4, 6, 5), "haar", 10.0),
                                         ((2, 3, 2, 2), "haar", 2.5), ((16, 16, 16, 16), "eps", 6.4)])
def test_gauge_force_parity(L, kind, beta):
    announce(f"gauge force parity {L} {kind}")
    U, _, Ud, _ = setup(L, kind, 0.6, 71)
    F, S = api.wilson_gauge_force(L, Ud, beta)
    assert rel_max(F.cpu().numpy(), og.gauge_force(U, L, beta)) <= 1e-12
    So = og.wilson_action(U, L, beta)
    assert abs(S - So) <= 1e-12 * abs(So)


@pytest.mark.parametrize("L", [(64, 2, 2, 2), (70, 2, 3, 2), (33, 3, 2, 2), (2, 2, 2, 2)])
def test_gauge_force_block_edges(L):
    """Rows of a block's 64 sites, longer and odd ones, and a lattice within one block: links read from the
    block's own in LDS and from memory, in the same wave."""
    announce(f"gauge force block edges {L}")
    U, _, Ud, _ = setup(L, "haar", 0.0, 75)
    F, S = api.wilson_gauge_force(L, Ud, 5.5)
    assert rel_max(F.cpu().numpy(), og.gauge_force(U, L, 5.5)) <= 1e-12
    So = og.wilson_action(U, L, 5.5)
    # a sum of 6 V terms of order 1 that may cancel: bounded by the terms, not by the sum
    assert abs(S - So) <= 1e-12 * 5.5 * 6 * np.prod(L)


@pytest.mark.parametrize("L", [(7, 6, 8, 5), (33, 16, 8, 4), (8, 8, 4, 4)])
def test_gauge_force_small_and_large_grids(L):
    """Rows across block ends on a grid of one block per CU at most, where every link comes from memory, on a larger
    one, and whole rows on a small one, where the block's own come from LDS."""
    announce(f"gauge force grids {L}")
    U, _, Ud, _ = setup(L, "haar", 0.0, 76)
    F, S = api.wilson_gauge_force(L, Ud, 5.5)
    assert rel_max(F.cpu().numpy(), og.gauge_force(U, L, 5.5)) <= 1e-12
    # a sum of 6 V terms of order 1 that may cancel: bounded by the terms, not by the sum
    assert abs(S - og.wilson_action(U, L, 5.5)) <= 1e-12 * 5.5 * 6 * np.prod(L)


def test_gauge_force_unit_links():
    L = (6, 4, 4, 4)
    _, _, Ud, _ = setup(L, "unit", 0.0, 72)
    F, S = api.wilson_gauge_force(L, Ud, 6.0)
    assert float(torch.abs(F).max()) == 0.0 and S == 0.0


def test_gauge_force_spectrum_pipeline():
    """Fig. 1 workload on synthetic links: the power spectrum of the gauge force, GPU force into the
    GPU spectrum against the oracle's force into the oracle's spectrum."""
    L = (6, 6, 6, 6)
    announce("gauge force spectrum 6^4")
    U, _, Ud, _ = setup(L, "eps", 0.5, 73)
    F, _ = api.wilson_gauge_force(L, Ud, 6.4, want_action=False)
    mom, pw = api.power_spectrum(L, Ud, F[None].contiguous(), 48, 12)
    Fo = og.gauge_force(U, L, 6.4)
    mref, pref = och.power_spectrum(U, Fo[None], L, 48, och.equal_windows(12))
    assert np.abs(mom - mref).max() <= 1e-12 * mref[0, 0]
    assert np.abs(pw - pref).max() <= 1e-12 * mref[0, 0]


def test_gauge_action_finite_differences_16():
    """Central differences (h = 1e-5) of the GPU action against the GPU force at 16^4: rounding of
    S ~ 1e-16 x 4e5 terms over 2h gives ~ 1e-6 absolute against forces of order 1-10."""
    L = (16, 16, 16, 16)
    announce("gauge action FD 16^4")
    Ua = inputs.random_links(L, "eps", 0.5, seed=74)
    Ud = api.pack_links(L, Ua.to(dev()))
    F, _ = api.wilson_gauge_force(L, Ud, 6.4, want_action=False)
    F = F.cpu().numpy()
    rng = np.random.default_rng(74)
    h = 1e-5
    worst = 0.0
    for _ in range(24):
        mu, c, s = int(rng.integers(4)), int(rng.integers(8)), int(rng.integers(api.volume(L)))
        vals = []
        for sign in (1, -1):
            U2 = Ua.clone()
            U2[mu, s] = torch.from_numpy(expm(1j * sign * h * su3.T[c]) @ Ua[mu, s].numpy())
            vals.append(api.wilson_gauge_force(L, api.pack_links(L, U2.to(dev())), 6.4)[1])
        fd = -(vals[0] - vals[1]) / (2 * h)
        worst = max(worst, abs(fd - F[mu, c, s]) / np.abs(F).max())
    assert worst <= 1e-5
