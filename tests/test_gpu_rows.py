"""The x forward pass by direct row sums (lists that fill a small part of the
cell) against the oracle: the stress of a list whose rows hold nothing, single
voxels, runs across the 64-voxel pieces and the cell faces, and voxels of several
defects, at every kind of length (one piece or several, a ragged last piece, odd,
fewer columns than lanes).  FP64 storage; tolerance rel L2 1e-12, that of the
solve's fields."""
import numpy as np
import pytest

from helpers import rel_l2, to6
from oracle import elastic, raster, solve
from paper_2403_09158_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8, 16, 24, 45, 64, 96, 129])
def test_row_sums_against_oracle(n):
    from paper_2403_09158_amd import ec

    h = inputs.H_VOXEL
    L = n * h
    prob = inputs.Problem(n, L, *inputs.CUBIC_FE, prec=0)
    b100 = np.array([0.0, 0.0, inputs.A_FE])
    b111 = 0.5 * inputs.A_FE * np.array([1.0, 1.0, 1.0])
    r = min(0.3 * L, 6.0)
    d = np.concatenate(
        [
            inputs.loop(np.array([0.5 * n, 0.4 * n, 0.5 * n]) * h, r, b100, b100),  # long rows in its plane
            inputs.loop(np.array([0.5 * n + 1, 0.4 * n, 0.5 * n]) * h, 0.5 * r, b111, b111),  # shares voxels with it
            inputs.sphere(np.array([0.2, 0.3, n - 0.4]) * h, 1.4 * h, 0.01),  # across three faces
            inputs.sphere(np.array([n - 1.1, 0.7 * n, 0.2 * n]) * h, 1.1 * h, 0.015),
        ]
    )
    fps, Es = raster.rasterise(prob, d)
    _, sig, _ = solve.solve_field(elastic.stiffness_of(prob), L, raster.eigenstrain_field(n, fps, Es), 0)
    st = ec.State(ec.Context(), prob)
    st.solve(d)
    assert rel_l2(st.field("sigma"), to6(sig)) < 1e-12
    st.close()
