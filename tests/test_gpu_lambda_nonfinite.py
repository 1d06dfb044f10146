"""The lambda density of a characteristic function with infinities, NaN or
values near the largest double, against the sum of its terms."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def by_terms(phi, lam0, h):
    """Re sum_k phi_k e^(-i omega_k (lam0 + j h)) / (M h): real and imaginary part
    of each phi_k times the cosine and sine of its whole phase."""
    M = len(phi)
    k = np.arange(M)
    omega = 2 * math.pi * np.where(k < M // 2, k, k - M) / (M * h)
    out = np.zeros(M)
    with np.errstate(all="ignore"):
        for j in range(M):
            th = -(omega * lam0) - 2 * math.pi * (k * j % M) / M
            out[j] = np.sum(phi.real * np.cos(th) - phi.imag * np.sin(th)) / (M * h)
    return out


# odd M: no phase is a multiple of a right angle but phase 0, so that no term's sign rests on rounding
@pytest.mark.parametrize("M", [7, 1031, 2049])
@pytest.mark.parametrize("what", ["inf_at_0", "inf", "inf_im", "nan", "large"])
def test_terms_that_are_not_finite(M, what):
    import torch
    import paper_2506_23712_amd as ens
    rng = np.random.default_rng(M)
    phi = rng.standard_normal(M) + 1j * rng.standard_normal(M)
    h, lam0 = 0.37, 0.0
    at = M - 2
    if what == "inf_at_0":
        phi[0] = math.inf
    elif what == "inf":
        phi[at] = complex(-math.inf, 1.0)
    elif what == "inf_im":                             # sample 0 is inf * sin 0
        phi[at] = complex(0.5, math.inf)
    elif what == "nan":
        phi[at] = complex(math.nan, 0.0)
    else:                                              # |phi| beyond the largest double, its terms up to 1.98e308
        phi[at] = 1.4e308 * (1 + 1j)
        lam0 = 0.3 * h
    got = ens.lambda_pdf_from_cf(torch.from_numpy(phi).cuda(), lam0, h).cpu().numpy()
    ref = by_terms(phi, lam0, h)
    if what == "large":
        # samples whose large term is within its rounding of the largest double aside
        top = np.finfo(np.float64).max / (M * h)
        clear = np.abs(np.abs(ref) / top - 1.0) > 1e-12
        ok = np.isfinite(ref) & clear
        assert ok.sum() > M // 2
        assert np.array_equal(np.isfinite(got)[clear], np.isfinite(ref)[clear])
        # relative to the largest term: the phase's rounding (a few eps of up to 2 pi M) and the sum's
        assert np.max(np.abs(got[ok] - ref[ok])) <= 1e-15 * (8 + M) * 1.1 * top
    else:
        assert np.array_equal(np.isnan(got), np.isnan(ref))
        assert np.array_equal(got[~np.isnan(ref)], ref[~np.isnan(ref)])
