"""RK steps of fields with energy in every retained mode, and of forcing bands
of thousands of modes, against a plain torch FP64 pseudo-spectral step (itself
held against the oracle)."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

A, B, H = (0.0, -5 / 9, -153 / 128), (1 / 3, 15 / 16, 8 / 15), (1 / 3, 5 / 12, 1 / 4)


def modes(n):
    import torch
    f = torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device="cuda")
    h = torch.arange(n // 2 + 1, dtype=torch.float64, device="cuda")
    return h.view(1, 1, -1), f.view(1, -1, 1), f.view(-1, 1, 1)


def kept(k, n):
    return (k[0] <= n // 3) & (k[1].abs() <= n // 3) & (k[2].abs() <= n // 3)


def white(n, seed):
    """Solenoidal velocity with the same mean energy in every retained mode; the
    real field it stands for has unit mean square per component or so."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    k = modes(n)
    k2 = k[0] ** 2 + k[1] ** 2 + k[2] ** 2
    keep = kept(k, n) & (k2 > 0)
    k2[0, 0, 0] = 1.0
    u = torch.stack([torch.fft.rfftn(torch.randn((n, n, n), generator=g, dtype=torch.float64, device="cuda"),
                                     norm="forward") * keep for _ in range(3)])
    div = (u[0] * k[0] + u[1] * k[1] + u[2] * k[2]) / k2
    for c in range(3):
        u[c] -= div * k[c]
    return u


def largest_speed(u, n):
    import torch
    return float(sum(torch.fft.irfftn(u[c], s=(n, n, n), norm="forward").abs() for c in range(3)).max())


def rhs(u, n, eps, kf_hi):
    """(projected u x omega plus linear band forcing, E_f)"""
    import torch
    k = modes(n)
    k2 = k[0] ** 2 + k[1] ** 2 + k[2] ** 2
    keep = kept(k, n) & (k2 > 0)
    band = keep & (k2 <= kf_hi ** 2)
    weight = torch.full((n // 2 + 1,), 1.0, dtype=torch.float64, device="cuda")
    weight[0] = 0.5
    ef = float(sum(((u[c].real ** 2 + u[c].imag ** 2) * weight * band).sum() for c in range(3)))
    k2[0, 0, 0] = 1.0
    real = lambda x: torch.fft.irfftn(x, s=(n, n, n), norm="forward")
    v = [real(u[c]) for c in range(3)]
    w = [real(1j * (k[a] * u[b] - k[b] * u[a])) for a, b in ((1, 2), (2, 0), (0, 1))]
    G = torch.empty_like(u)
    for c, (a, b) in enumerate(((1, 2), (2, 0), (0, 1))):
        G[c] = torch.fft.rfftn(v[a] * w[b] - v[b] * w[a], norm="forward") * keep
        G[c] += eps / (2 * ef) * u[c] * band
    div = (G[0] * k[0] + G[1] * k[1] + G[2] * k[2]) / k2
    for c in range(3):
        G[c] -= div * k[c]
    return G, ef


def reference(u, n, nu, eps, kf_hi, dt, steps):
    """(velocity after `steps` steps, E_f at the start of the last one)"""
    import torch
    k = modes(n)
    k2 = k[0] ** 2 + k[1] ** 2 + k[2] ** 2
    u = u.clone()
    for _ in range(steps):
        q = torch.zeros_like(u)
        for s in range(3):
            G, ef = rhs(u, n, eps, kf_hi)
            first = ef if s == 0 else first
            e = torch.exp(-nu * k2 * H[s] * dt)
            q = e * (A[s] * q + dt * G)
            u = e * u + B[s] * q
    return u, first


def err(a, b):
    return float((a - b).abs().square().sum().sqrt() / b.abs().square().sum().sqrt())


def test_the_reference_steps_as_the_oracle(orc):
    n, nu, eps, kf_hi = 32, 0.02, 0.5, 9.5
    u = white(n, 1)
    dt = 0.5 * 2 * math.pi / n / largest_speed(u, n)
    got, ef = reference(u, n, nu, eps, kf_hi, dt, 2)
    ref, _ = orc.run(orc.Member(n=n, nu=nu, eps=eps, kf_hi=kf_hi, dt=dt), u.cpu().numpy(), 2)
    assert np.linalg.norm(got.cpu().numpy() - ref) <= 1e-12 * np.linalg.norm(ref)


def library(u, n, prec, nu, eps, kf_hi, dt, steps, zvariant=None):
    import torch
    import paper_2506_23712_amd as ens
    E = ens.Ensemble()
    m = E.add_member(ens.MemberSpec(n=n, nu=nu, eps_ref=eps, kf_hi=kf_hi, dt=dt, precision=prec, seed=1))
    m.set_state(u)
    if zvariant is not None:
        E.set_variant("zfwd_update", n, prec, zvariant)
    E.step(steps)
    out, d = m.state(), m.diag()
    torch.cuda.synchronize()
    E.close()
    return out, d


# the tolerances of the one-step comparisons with the oracle at these sizes
TOL = {"fp64": 1e-12, "fp32": 2e-5}


@pytest.mark.parametrize("n,prec", [(128, "fp64"), (256, "fp64"), (512, "fp64"), (256, "fp32"), (512, "fp32")])
@pytest.mark.parametrize("zvariant", [0, 1])
def test_two_steps_of_a_field_in_every_mode(n, prec, zvariant):
    """Two steps of one call, so that every kernel of the z forward runs: each
    stage's, with and without the next z inverse; a step of half a CFL length
    turns a large part of the high modes' values over."""
    import torch
    print(f"case n={n} {prec} z forward {zvariant}", flush=True)
    nu, eps, kf_hi = 1e-3, 0.5, 2.5
    u = white(n, n)
    dt = 0.5 * 2 * math.pi / n / largest_speed(u, n)
    got, d = library(u, n, prec, nu, eps, kf_hi, dt, 2, zvariant)
    ref, _ = reference(u, n, nu, eps, kf_hi, dt, 2)
    assert err(u, ref) > 0.1
    e = err(got, ref)
    print(f"{n} {prec}: rel L2 {e:.2e}")
    del got, ref, u
    torch.cuda.empty_cache()
    assert e <= TOL[prec] and d["step"] == 2 and d["flags"] == 0


@pytest.mark.parametrize("n,kf_hi", [(16, 4.9), (64, 20.5), (128, 41.5), (256, 60.0)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_a_band_of_thousands_of_modes(n, kf_hi, prec):
    """The band step's workgroup over bands up to the truncation: in the plane
    pass (n = 16 with 128 threads, 64) and in the y inverse (128, 256)."""
    print(f"case n={n} {prec} band to {kf_hi}", flush=True)
    nu, eps = 1e-3, 50.0
    u = white(n, n + 1)
    dt = 0.25 * 2 * math.pi / n / largest_speed(u, n)
    got, d = library(u, n, prec, nu, eps, kf_hi, dt, 2)
    ref, ef = reference(u, n, nu, eps, kf_hi, dt, 2)
    assert err(got, ref) <= TOL[prec]
    assert abs(d["E_f"] - ef) <= 2 * TOL[prec] * ef and d["inj"] == eps and d["flags"] == 0
