"""Strain and stress of one solve written to the device: from one pass over the
stress they must hold, bit for bit, what each holds when asked for alone, and what
the state's own fields hold in double; where the two outputs overlap, the stress
is written after the strain."""
import numpy as np
import pytest

from paper_2403_09158_amd import inputs

pytestmark = pytest.mark.gpu


def _case(n, prec, frame, bc):
    h = inputs.H_VOXEL
    prob = inputs.Problem(n, n * h, *inputs.CUBIC_FE, prec=prec, bc=bc, frame=inputs.FRAME_111 if frame else ())
    b = 0.5 * inputs.A_FE * np.array([1.0, 1.0, 1.0])
    c = np.array([0.4, 0.5, 0.3]) * n * h
    d = np.concatenate([inputs.loop(c, 0.2 * n * h, b, b), inputs.sphere(c + h, 0.15 * n * h, 0.012)])
    return prob, d


@pytest.mark.parametrize("n", [16, 45])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("frame, bc", [(False, 0), (True, 1)])
def test_both_outputs(n, prec, frame, bc):
    import torch

    from paper_2403_09158_amd import ec

    prob, d = _case(n, prec, frame, bc)
    dt = torch.float32 if prec else torch.float64
    st = ec.State(ec.Context(), prob)
    eps, sig, eps1, sig1 = (torch.full((6, n, n, n), np.nan, dtype=dt, device="cuda") for _ in range(4))
    st.solve(d, eps_out=eps1)
    st.solve(d, sig_out=sig1)
    st.solve(d, eps_out=eps, sig_out=sig)
    assert torch.equal(eps, eps1) and torch.equal(sig, sig1)
    assert np.array_equal(eps.cpu().numpy(), st.field("eps").astype(eps.cpu().numpy().dtype))
    assert np.array_equal(sig.cpu().numpy(), st.field("sigma").astype(sig.cpu().numpy().dtype))
    assert not torch.equal(eps, sig)
    st.close()


@pytest.mark.parametrize("shift", [0, 3, -3])
def test_overlapping_outputs(shift):
    import torch

    from paper_2403_09158_amd import ec

    n = 32
    prob, d = _case(n, 1, False, 0)
    st = ec.State(ec.Context(), prob)
    buf = torch.zeros((12, n, n, n), dtype=torch.float32, device="cuda")
    eps, sig = buf[3:9], buf[3 + shift : 9 + shift]
    st.solve(d, eps_out=eps, sig_out=sig)
    ref = torch.zeros_like(buf)
    ref[3:9] = torch.from_numpy(st.field("eps").astype(np.float32)).cuda()
    ref[3 + shift : 9 + shift] = torch.from_numpy(st.field("sigma").astype(np.float32)).cuda()
    assert torch.equal(buf, ref)
    st.close()
