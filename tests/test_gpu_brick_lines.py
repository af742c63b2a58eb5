"""The matrix-free element kernel (a lane per line of points, 7 Q2 or 16 Q1
elements per wavefront, 28 or 64 per workgroup): element counts around a full
wavefront, a full workgroup and more groups than workgroups."""
import numpy as np
import pytest

import basin
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# elements: 1; 6, 7, 8 and 27, 28, 30 (Q2's wavefront and workgroup); 15, 16, 18
# and 63, 64, 66 (Q1's); 14,400 (more than 512 workgroups of 28)
GRIDS = [(1, 1, 1), (6, 1, 1), (7, 1, 1), (2, 2, 2), (9, 3, 1), (7, 2, 2), (5, 3, 2), (5, 3, 1),
         (4, 2, 2), (3, 3, 2), (7, 3, 3), (8, 4, 2), (11, 3, 2), (60, 40, 6)]


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("grid", GRIDS, ids=["x".join(map(str, g)) for g in GRIDS])
def test_product_at_group_edges(order, grid):
    """Every row against the oracle's assembled operator to rounding: a row sums
    fewer than 200 products through at most three contractions of three terms."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1207_0486_amd.hns import Operator
    m = basin.basin_hex_mesh(*grid, order=order, seed=5)
    op = Operator(m, 1e3, 1e-2, 3600.0, kind="helmholtz", matrix_free=True)
    x = np.random.default_rng(3).standard_normal(m.n)
    y = op.apply(torch.as_tensor(x, device="cuda:0")).cpu().numpy()
    op.close()
    ref = oracle.hex_helmholtz(m, 1e3, 1e-2, 3600.0).matvec(x)
    assert np.linalg.norm(y - ref) <= 1e-12 * np.linalg.norm(ref)
