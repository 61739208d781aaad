"""A device allocation that the runtime refuses is reported by the call that asked
for it, and by no later one: the state's next solve, whose launches ask for the
last error, succeeds and gives what it gave before."""
import numpy as np
import pytest

from paper_2403_09158_amd import inputs

pytestmark = pytest.mark.gpu


def test_next_call_after_a_refused_allocation():
    from paper_2403_09158_amd import ec

    n, h = 128, inputs.H_VOXEL
    d = inputs.mixed_population(np.random.default_rng(4), 40, n * h, h)
    ctx = ec.Context(0, budget_bytes=1 << 50, allocator="hip")  # the ledger admits what the card does not hold
    st = ec.State(ctx, inputs.Problem(n, n * h, *inputs.CUBIC_FE, prec=1))
    st.solve(d)
    ref = st.energies()
    many = np.repeat(inputs.sphere(np.full(3, 0.5 * n * h), 0.49 * n * h, 0.01), 60000)  # footprint slots: 470 GB
    with pytest.raises(ec.EcError) as err:
        st.solve(many)
    assert "allocation" in str(err.value)
    st.solve(d)
    assert np.array_equal(st.energies(), ref)
    st.close()
    ctx.close()
