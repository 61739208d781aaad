"""The membership lists of a moved defect at footprints of one to tens of thousands
of voxels: after hops and changes of size and place among overlapping defects, the
footprints and the eigenstrain read through the lists are those of a fresh solve
of the list, bit for bit, and so is the stress to rounding (tolerance rel L2
1e-12, that of FP64 fields)."""
import numpy as np
import pytest

from helpers import rel_l2
from paper_2403_09158_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, r", [(16, 0.6), (32, 5.3), (64, 12.6), (96, 28.0)])
def test_moves_against_fresh_solve(n, r):
    from paper_2403_09158_amd import ec

    h = inputs.H_VOXEL
    prob = inputs.Problem(n, n * h, *inputs.CUBIC_FE)
    b = 0.5 * inputs.A_FE * np.array([1.0, 1.0, 1.0])
    c = np.full(3, 0.5 * n * h)
    d = np.concatenate(
        [
            inputs.sphere(c, r * h, 0.01),
            inputs.sphere(c + 0.6 * h, max(0.5 * r, 0.7) * h, 0.012),  # inside the first
            inputs.loop(c + h, max(r, 1.5) * h, b, b),  # through both
        ]
    )
    ctx = ec.Context()
    st, ref = ec.State(ctx, prob), ec.State(ctx, prob)
    st.solve(d)
    for i, lam, size in ((0, (1, 0, 0), 1.0), (2, (0, -1, 1), 1.0), (1, (0, 1, 0), 1.0), (0, (0.3, 0, 0.4), 1.03),
                         (0, (-1, n // 2 - 1, 0), 1.0), (2, (0.2, 0, 0), 0.9)):
        d[i]["c"] = d[i]["c"] + np.asarray(lam) * h
        d[i]["radius"] *= size
        st.update(i, d[i], energies=False)
        ref.solve(d)
        for a, e in zip(st.footprints(), ref.footprints()):
            assert np.array_equal(np.sort(a), e)
        assert np.array_equal(st.field("eps_star"), ref.field("eps_star"))
    assert rel_l2(st.field("sigma"), ref.field("sigma")) < 1e-12
    st.close()
    ref.close()
