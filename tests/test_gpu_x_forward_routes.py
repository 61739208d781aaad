"""FP64 solves by either x forward pass, against the oracle: lists that fill more of
the cell than the direct row sums' limit (the transforms), lists just below and
just above the limit, and the smallest length's row sums. Which pass ran is read
from the kernels' names. Tolerance rel L2 1e-12, that of FP64 fields."""
import numpy as np
import pytest

from helpers import kernels_of, rel_l2, to6
from oracle import elastic, raster, solve
from paper_2403_09158_amd import inputs

pytestmark = pytest.mark.gpu

ROWS, TRANSFORMS = "k_x_forward_rows<", "k_x_forward<"


# (length, ball radii in voxels, pass): the limit is 4 % of the cell (8^3: 20.5
# voxels, 64^3: 10486), 50 % at 129
@pytest.mark.parametrize(
    "n, radii, route",
    [
        (8, (1.6,), ROWS),  # 17 voxels
        (16, (4.8,), TRANSFORMS),  # 463
        (45, (13.5, 4.0), TRANSFORMS),
        (64, (13.5,), ROWS),  # 10306
        (64, (13.65,), TRANSFORMS),  # 10653
        (64, (19.0, 12.0, 9.0), TRANSFORMS),
        (129, (24.5,) * 16, ROWS),  # 46 %
        (129, (24.5,) * 20, TRANSFORMS),  # 57 %, nearly all of it twenty times over
        (160, (24.5,) * 4, TRANSFORMS),  # 6 %
    ],
)
def test_solve_against_oracle(n, radii, route):
    from paper_2403_09158_amd import ec

    h = inputs.H_VOXEL
    prob = inputs.Problem(n, n * h, *inputs.CUBIC_FE)
    c = np.array([0.52, 0.47, 0.05]) * n * h  # across the z faces
    d = np.concatenate([inputs.sphere(c + 0.3 * k * h, r * h, 0.01 / (k + 1)) for k, r in enumerate(radii)])
    st = ec.State(ec.Context(), prob)
    st.solve(d)  # the kernel window's own solves
    names = kernels_of(lambda: st.solve(d))
    assert route in names
    assert (TRANSFORMS if route == ROWS else ROWS) not in names
    fps, Es = raster.rasterise(prob, d)
    _, sig, _ = solve.solve_field(elastic.stiffness_of(prob), prob.L, raster.eigenstrain_field(n, fps, Es), 0)
    assert rel_l2(st.field("sigma"), to6(sig)) < 1e-12
    st.close()
