"""Small FP64 solves in one launch (csrc/small_solve.hip): every number of rows
per thread it is compiled for, at the edges of its row groups, against the
launch-per-phase solve and the oracle; caps, zero and non-finite right-hand
sides, an indefinite operator, and sessions that advance it piecewise."""
import numpy as np
import pytest

import basin
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

NU = (1e3, 1e-2)
DT = 3600.0


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1207_0486_amd import hns  # noqa: F401
    return torch.device("cuda", 0)


def _case(grid, bit, seed, dev):
    from paper_1207_0486_amd.hns import Operator
    m = basin.basin_mesh(*grid, seed=3)
    op = Operator(m, *NU, DT, kind="poisson" if bit < 0 else "helmholtz", keep_fp32=True)
    d = None if bit < 0 else ((m.bc >> bit) & 1) == 1
    b = basin.normal_rhs(m.n, seed, zero_mean=False, dirichlet=d)   # Neumann: the mean is removed
    return m, op, d, b, torch.as_tensor(b, device=dev)


# rows: 18; 510; 512; 520; 1020; 1024; 1440; 1536; 1980; 2048; 2400; 2560, and
# 2574 beyond it
GRIDS = [(2, 2, 1), (4, 16, 5), (7, 7, 7), (4, 7, 12), (16, 11, 4), (7, 15, 7), (15, 14, 5),
         (11, 15, 7), (14, 10, 11), (15, 15, 7), (23, 19, 4), (19, 15, 7), (21, 12, 8)]


@pytest.mark.parametrize("bit", [-1, 1])
@pytest.mark.parametrize("grid", GRIDS, ids=["x".join(map(str, g)) for g in GRIDS])
def test_solve_equals_launches_and_oracle(dev, grid, bit):
    m, op, d, b, bg = _case(grid, bit, 3, dev)
    # (an O(1) guess of the pressure problem, whose entries are 1e9 apart, leaves
    # no digits of b in the residual: from rest there)
    x0 = np.random.default_rng(5).standard_normal(m.n) * (bit >= 0)
    got = {}
    for small in (4096, 0):
        op.set_param("small_n", small)
        got[small] = op.solve(bg, torch.as_tensor(x0, device=dev), tol=1e-10, mask_bit=bit)
        capped, info = op.solve(bg, torch.as_tensor(x0, device=dev), tol=1e-14, max_iter=5,
                                mask_bit=bit, check=False)
        got[small, "cap"] = capped, info
    op.close()
    (x, i), (y, j) = got[4096], got[0]
    assert i.status == j.status == 0 and i.relres_true <= 1e-10 and i.outer_iterations == 1
    assert abs(i.iterations - j.iterations) <= max(1, 0.02 * j.iterations)
    assert abs(i.removed_mean - j.removed_mean) <= 1e-14 * np.abs(b).max()
    (xc, ic), (yc, jc) = got[4096, "cap"], got[0, "cap"]
    if d is not None and (~d).sum() <= 5:   # CG ends within the cap, at rounding
        return
    assert ic.status == jc.status and ic.iterations == jc.iterations
    assert float((xc - yc).norm() / yc.norm()) <= 1e-12
    A = oracle.stiffness(m, *NU) if bit < 0 else oracle.helmholtz(m, *NU, DT)
    r = b - A.matvec(x.cpu().numpy())
    if bit < 0:
        r -= b.mean()
        bb = b - b.mean()
    else:
        r[d] = 0.0
        bb = b
        assert np.all(x.cpu().numpy()[d] == 0.0)
    assert np.linalg.norm(r) <= 1.01e-10 * np.linalg.norm(bb)


def test_edges(dev):
    from paper_1207_0486_amd.hns import HNSError, Operator
    m, op, d, b, bg = _case((15, 14, 5), 0, 4, dev)
    x, info = op.solve(torch.zeros_like(bg), torch.ones_like(bg), mask_bit=0)
    assert info.status == 0 and info.iterations == 0 and float(x.abs().max()) == 0.0
    bad = bg.clone()
    bad[int(np.flatnonzero(~d)[0])] = float("nan")
    with pytest.raises(HNSError, match="non-finite"):
        op.solve(bad, mask_bit=0)
    bad = bg.clone()
    bad[int(np.flatnonzero(d)[0])] = float("inf")      # ignored: a Dirichlet entry
    y, info = op.solve(bad, mask_bit=0)
    x, _ = op.solve(bg, mask_bit=0)
    assert info.status == 0 and torch.equal(x, y)
    x, info = op.solve(bg, mask_bit=0, max_iter=0, check=False)
    assert info.status == 1 and info.iterations == 0 and float(x.abs().max()) == 0.0
    # below the rounding floor: ends not converged, as the launches do
    x, info = op.solve(bg, mask_bit=0, tol=1e-19, check=False)
    assert info.status == 1 and info.relres_true < 1e-14
    op.close()
    op = Operator(m, *NU, -1e9, kind="helmholtz")       # M - c K: indefinite
    with pytest.raises(HNSError):
        op.solve(bg, mask_bit=0)
    op.close()


@pytest.mark.parametrize("bit", [-1, 2])
def test_session_advances_it_piecewise(dev, bit):
    from paper_1207_0486_amd.hns import BatchSession
    m, op, d, b, bg = _case((15, 14, 5), bit, 6, dev)
    x, info = op.solve(bg, tol=1e-10, mask_bit=bit)
    s = BatchSession(op, 2)
    s.add([1], [bit], [bg], [1e-10], [100000])
    for n in (1, 2, 7, 3) + (400,) * 10:
        if s.advance(n) == 0:
            break
    y, got = s.take(1)
    s.close()
    op.close()
    assert got.status == 0 and got.iterations == info.iterations and torch.equal(x, y)
