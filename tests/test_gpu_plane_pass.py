"""The plane pass (n <= 64: y inverse, x pass, y forward and band step in one
launch) against the separate passes, from one member to a batch, with the z
inverse fused and not, and as the only passes of a captured and a direct step."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def advance(n, prec, count, xvariant, zvariant, graphs):
    import paper_2506_23712_amd as ens
    E = ens.Ensemble(graphs=graphs)
    E.set_variant("xpass", n, prec, xvariant)
    E.set_variant("zfwd_update", n, prec, zvariant)
    ms = [E.add_member(ens.MemberSpec(n=n, nu=0.02, eps_ref=0.1, lam=0.3 * i, kf_hi=2.0, dt=0.0, cfl=0.5, seed=7 + i,
                                      precision=prec)) for i in range(count)]
    E.step(1)
    E.step(2)
    out = [(m.state().cpu().numpy(), m.diag()) for m in ms]
    E.close()
    return out


@pytest.mark.parametrize("n", [16, 32, 64])
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-13), ("fp32", 2e-6)])
@pytest.mark.parametrize("count,zvariant,graphs", [(1, 1, True), (5, 0, False), (9, 1, False)])
def test_plane_pass_matches_separate_passes(n, prec, tol, count, zvariant, graphs):
    # nine stages of transforms whose rounding is a few eps each, in a field of
    # order one: 1e-13 and 2e-6 are 450 eps (FP64) and 17 eps (FP32) of the norm
    a = advance(n, prec, count, 5, zvariant, graphs)
    b = advance(n, prec, count, 0, zvariant, graphs)
    for (u, du), (v, dv) in zip(a, b):
        assert np.linalg.norm(u - v) <= tol * np.linalg.norm(v)
        for k in ("t", "dt", "E", "D", "E_f", "inj", "umax"):
            assert abs(du[k] - dv[k]) <= 40 * tol * abs(dv[k]), k
        assert du["step"] == dv["step"] == 3 and du["flags"] == dv["flags"] == 0


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_plane_pass_steps_as_the_oracle(orc, prec):
    import paper_2506_23712_amd as ens
    E = ens.Ensemble()
    m = E.add_member(ens.MemberSpec(n=64, nu=0.02, eps_ref=0.1, kf_hi=2.0, dt=0.0, cfl=0.5, seed=3, precision=prec))
    assert E.variants()[f"xpass:64:{prec}"] == 5
    u0 = orc.init_field(64, 3, k_peak=2.0, e0=0.5)
    E.step(4)
    got = m.state().cpu().numpy()
    ref, _ = orc.run(orc.Member(n=64, nu=0.02, eps=0.1, kf_hi=2.0, dt=0.0, cfl=0.5), u0, 4)
    E.close()
    assert np.linalg.norm(got - ref) <= (1e-11 if prec == "fp64" else 2e-5) * np.linalg.norm(ref)
