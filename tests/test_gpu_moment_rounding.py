"""Rounding of a snapshot's moment sums over the workgroups."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed", range(6))
def test_sums_of_identical_tiles_do_not_round(seed):
    """u_y = A cos(n x / 4 + phi): its gradient takes four values in turn along
    every row, and its transforms multiply by 1, -1, i and -i only.  With the
    same four values at every n (the wavenumber is a power of two), every
    tile's sums are the same numbers, and the tree that adds 4, 32 and 256 of
    them is exact, so the mean moments of the three members are the same in
    every bit.  (32 equal sums added one after another round at 3, 5, 6, ...
    times the sum.)"""
    import torch
    import paper_2506_23712_amd as ens
    rng = np.random.default_rng(seed)
    c = complex(*rng.uniform(0.5, 2.0, 2))
    E = ens.Ensemble(hist=ens.HistSpec(qr_bins=64, eps_ref=1.0, nu_ref=1.0))
    mean = []
    for n in (16, 32, 64):
        u = np.zeros((3, n, n, n // 2 + 1), dtype=np.complex128)
        u[1, 0, 0, n // 4] = c * (4.0 / n)
        m = E.add_member(ens.MemberSpec(n=n, nu=0.5, box=2 * math.pi, dt=0.01, seed=n))
        m.set_state(torch.from_numpy(u))
        E.accumulate_stats([m])
        mean.append(m.stats()[1].numpy()[:26] / n ** 3)
    E.close()
    even = [7, 9, 11, *range(12, 20), 22]              # A_T^2, ^4, ^6; eps and Omega to 1..4; S^2: all terms >= 0
    x = 2.0 * np.array([c.real, c.imag])               # the values are +-2 Re c, +-2 Im c
    assert np.isclose(mean[0][7], np.mean(x ** 2), rtol=1e-14)
    for other in mean[1:]:
        assert np.array_equal(other[even], mean[0][even]), (other[even] - mean[0][even]) / mean[0][even] / 2.0 ** -53
