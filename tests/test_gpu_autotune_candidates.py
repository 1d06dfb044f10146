"""What the autotuner times: every kernel once, the x pass beside tuned y passes."""
import pytest

pytestmark = pytest.mark.gpu

RUNS = 2 + 3 * 5                                   # warm-up launches and three timed runs of five


def tuned(n, prec):
    """Kernels in the order the autotuner launched them (names without arguments)."""
    import torch
    import paper_2506_23712_amd as ens
    E = ens.Ensemble()
    E.add_member(ens.MemberSpec(n=n, nu=0.02, kf_hi=2.0, dt=0.01, seed=1, precision=prec))
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as p:
        E.autotune()
        torch.cuda.synchronize()
    E.close()
    ev = sorted((e.time_range.start, e.name) for e in p.events() if "ens::k_" in e.name)
    return [name.split("(")[0].replace("void ", "").replace("ens::", "") for _, name in ev]


@pytest.mark.parametrize("n,prec", [(16, "fp64"), (32, "fp32"), (64, "fp64"), (64, "fp32"), (128, "fp64"), (128, "fp32")])
def test_every_x_pass_kernel_is_timed_once(n, prec):
    """Variants that run another variant's kernel are left out: a kernel timed
    several times would be compared by the best of more runs."""
    names = tuned(n, prec)
    x = [k for k in names if k.startswith(("k_xpass", "k_plane"))]
    assert {k: x.count(k) for k in x} == {k: RUNS for k in x}
    # 8 and 16 values per thread, streamed (two of them in FP32 from n = 128), wave-private, plane pass
    assert len(set(x)) == 2 + (n >= 64) + (n >= 128 and prec == "fp32") + (n >= 64) + (n <= 64)


@pytest.mark.parametrize("n,prec", [(32, "fp64"), (64, "fp32"), (128, "fp64")])
def test_the_y_passes_are_tuned_before_the_x_pass(n, prec):
    """The plane pass stands for the y inverse, an x pass and the y forward; the
    separate passes it is compared with are the tuned ones."""
    names = tuned(n, prec)
    first = next(i for i, k in enumerate(names) if k.startswith(("k_xpass", "k_plane")))
    for p in ("k_yinv", "k_yfwd"):
        kinds = {k for k in names if k.startswith(p + "<")}
        assert len(kinds) == 4 and kinds == {k for k in names[:first] if k.startswith(p + "<")}
