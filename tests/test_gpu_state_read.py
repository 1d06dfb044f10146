"""The state read into a caller's array of doubles at any 8-byte address."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec", [(16, "fp64"), (32, "fp32"), (64, "fp64"), (128, "fp32")])
@pytest.mark.parametrize("shift", [0, 1])
def test_state_into_an_array_of_doubles(n, prec, shift):
    """`shift` doubles past the allocation's (256-byte aligned) start: the same
    values in the same places, and nothing written beside them."""
    import torch
    import paper_2506_23712_amd as ens
    from paper_2506_23712_amd import _lib
    E = ens.Ensemble()
    m = E.add_member(ens.MemberSpec(n=n, nu=0.02, kf_hi=2.0, dt=0.01, seed=n, precision=prec))
    E.step(1)
    ref = torch.view_as_real(m.state()).reshape(-1)
    buf = torch.full((ref.numel() + 3,), 7.0, dtype=torch.float64, device="cuda")
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    _lib.check(_lib.lib().ens_member_get_state(E.ctx, m.id, ctypes.c_void_p(buf.data_ptr() + 8 * shift), stream))
    torch.cuda.synchronize()
    assert torch.equal(buf[shift:shift + ref.numel()], ref)
    assert (buf[:shift] == 7.0).all() and (buf[shift + ref.numel():] == 7.0).all()
    E.close()
