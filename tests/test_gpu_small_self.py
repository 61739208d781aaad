"""Self terms of small cells, which run beside the whole solve: every call that may
follow a solve while they still run gives what it gives after a wait for the
device (energies, the no-allocation energies under graph capture and replayed, a
hop, another solve of another list, jump energies), and short lists' pair sums
(more, smaller work items) agree with the oracle's self terms."""
import numpy as np
import pytest

from helpers import energy_ok_fp64
from oracle import energy
from paper_2403_09158_amd import inputs

pytestmark = pytest.mark.gpu


def _case(n, ndef, seed):
    h = inputs.H_VOXEL
    prob = inputs.Problem(n, n * h, *inputs.CUBIC_FE)
    rng = np.random.default_rng(seed)
    return prob, inputs.mixed_population(rng, ndef, n * h, h, r111=(0.5, 0.4 * n * h), r100=(1.0, 0.4 * n * h))


def _after_solve(call, wait):
    import torch

    from paper_2403_09158_amd import ec

    prob, d = _case(64, 300, 5)
    st = ec.State(ec.Context(), prob)
    st.solve(d[:100])
    st.energies()
    st.solve(d)
    if wait:
        torch.cuda.synchronize()
    out = np.array(call(st, d))
    st.close()
    return out


def _hop(st, d):
    moved = d[7:8].copy()
    moved["c"] += np.array([1.0, -1.0, 1.0]) * inputs.H_VOXEL
    return st.update(7, moved)


def _again(st, d):
    st.solve(d[50:250])
    return st.energies()


def _captured(st, d):
    import torch

    out = torch.zeros(len(d), dtype=torch.float64, device="cuda")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        st.energies_noalloc(out, stream=s)
    res = []
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        res.append(out.cpu().numpy())
    assert np.array_equal(res[0], res[1]) and np.array_equal(res[0], res[2])
    return res[0]


@pytest.mark.parametrize(
    "call",
    [lambda st, d: st.energies(), _hop, _again, lambda st, d: st.jump_energies(inputs.glide_jumps(d)), _captured],
    ids=["energies", "hop", "solve", "jumps", "capture"],
)
def test_calls_while_the_self_terms_run(call):
    assert np.array_equal(_after_solve(call, False), _after_solve(call, True))


@pytest.mark.parametrize("n, ndef", [(16, 3), (32, 12)])
def test_short_lists_against_oracle(n, ndef):
    from paper_2403_09158_amd import ec

    prob, d = _case(n, ndef, n)
    st = ec.State(ec.Context(), prob)
    st.solve(d)
    assert energy_ok_fp64(st.energies(), energy.energies_fast(prob, d))
    st.close()
