"""Jacobi-scaled CG chunks in one cooperative launch (csrc/cg_grid.hip): every
tiling the planner takes (one plane, few planes, ragged last tiles, one to many
row groups per wavefront, vectors and diagonals partly read from memory)
against the launch-per-phase iterations and the oracle's iterates."""
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


def _operator(m, bit, keep_fp32=False):
    from paper_1207_0486_amd.hns import Operator
    op = Operator(m, NU[0], NU[1], DT, kind="poisson" if bit < 0 else "helmholtz",
                  keep_fp32=keep_fp32, gpu_assembly=True)
    op.set_param("small_n", 0)
    return op


def _rhs(m, bit, seed, dev):
    d = None if bit < 0 else ((m.bc >> bit) & 1) == 1
    b = basin.normal_rhs(m.n, seed, zero_mean=bit < 0, dirichlet=d)
    return d, b, torch.as_tensor(b, device=dev)


def _rel(x, y):
    return float((x - y).norm() / y.norm())


# (Nx, Ny, Nz): 18 rows; a plane of 8 rows; two planes; one group of 64 places
# that ends a row short and one that begins a row over; several groups
SMALL = [(2, 2, 1), (40, 1, 1), (1, 60, 3), (9, 8, 6), (9, 15, 7), (33, 47, 13)]


@pytest.mark.parametrize("bit", [-1, 0, 2])
@pytest.mark.parametrize("grid", SMALL, ids=["x".join(map(str, g)) for g in SMALL])
def test_iterate_is_the_oracles(dev, grid, bit):
    """Seven iterations (or fewer, to the answer): the oracle's Jacobi-PCG
    iterate to rounding, and the launch-per-phase one's."""
    m = basin.basin_mesh(*grid, seed=3)
    if bit >= 0 and ((m.bc >> bit) & 1).all():
        pytest.skip("no free node")
    d, b, bg = _rhs(m, bit, 11, dev)
    A = oracle.stiffness(m, *NU) if bit < 0 else oracle.helmholtz(m, *NU, DT)
    w = oracle.mass(m).matvec(np.ones(m.n)) if bit < 0 else None
    op = _operator(m, bit)
    got = {}
    for one in (-1, 0):
        op.set_param("one_launch", one)
        got[one] = op.solve(bg, tol=1e-9, max_iter=7, mask_bit=bit, check=False)
    op.close()
    (x, i), (y, j) = got[-1], got[0]
    assert i.iterations == j.iterations and i.status == j.status
    assert _rel(x, y) <= 1e-12
    ref = oracle.pcg(A, b, dirichlet=d, singular=bit < 0, weights=w, tol=1e-9,
                     maxit=i.iterations)
    assert np.linalg.norm(x.cpu().numpy() - ref.x) <= 1e-11 * np.linalg.norm(ref.x)


# one mesh per compiled form: rows per wavefront 1, 2, 4, 6, 8, 12 (FP64) and
# 1, 2, 4, 8, 12 (FP32), below and above 64 and 128 workgroups
FORMS = [(30, 28, 7), (61, 47, 13), (90, 80, 11), (128, 128, 16), (160, 140, 20), (180, 190, 21),
         (250, 200, 22), (255, 201, 24)]


@pytest.mark.parametrize("grid", FORMS, ids=["x".join(map(str, g)) for g in FORMS])
def test_every_form_equals_the_launches(dev, grid):
    """40 FP64 iterations equal those of a launch per phase to rounding (the
    dot products' order differs); a mixed velocity solve meets its tolerance in
    the same number of iterations."""
    m = basin.basin_mesh(*grid, seed=5)
    d, b, bg = _rhs(m, -1, 21, dev)
    op = _operator(m, -1)
    xs = {}
    for one in (-1, 0):
        op.set_param("one_launch", one)
        xs[one], info = op.solve(bg, tol=1e-12, max_iter=40, check=False)
        assert info.iterations == 40
    op.close()
    assert _rel(xs[-1], xs[0]) <= 1e-11
    d, b, bg = _rhs(m, 1, 22, dev)
    op = _operator(m, 1, keep_fp32=True)
    it = {}
    for one in (-1, 0):
        op.set_param("one_launch", one)
        x, info = op.solve(bg, tol=1e-11, mask_bit=1, mode="mixed")
        assert info.status == 0 and info.relres_true <= 1e-11
        it[one] = info.iterations
    op.close()
    assert abs(it[-1] - it[0]) <= 1


def test_chunks_join(dev):
    """A session advancing 1, 2, 13, ... iterations at a time (its chunks start
    and end anywhere) takes the whole solve's iterates, bit for bit."""
    from paper_1207_0486_amd.hns import BatchSession
    m = basin.basin_mesh(40, 36, 6, seed=5)
    d, b, bg = _rhs(m, 0, 31, dev)
    for mode in ("fp64", "mixed"):
        op = _operator(m, 0, keep_fp32=True)
        x, info = op.solve(bg, tol=1e-10, mask_bit=0, mode=mode)
        s = BatchSession(op, 1, mode)
        s.add([0], [0], [bg], [1e-10], [1000])
        for n in (1, 2, 13, 5, 100, 100):
            s.advance(n)
        y, got = s.take(0)
        s.close()
        op.close()
        assert got.iterations == info.iterations and torch.equal(x, y)


def test_a_missed_meeting_falls_back(dev):
    """Workgroups that give up waiting at once (a bound of no polls): the solve
    goes on with a launch per phase, from the same x, to the same bits."""
    m = basin.basin_mesh(40, 36, 6, seed=5)
    for bit, mode in ((-1, "fp64"), (1, "fp64"), (1, "mixed")):
        d, b, bg = _rhs(m, bit, 41, dev)
        op = _operator(m, bit, keep_fp32=True)
        x0 = torch.as_tensor(np.random.default_rng(1).standard_normal(m.n), device=dev)
        op.set_param("one_launch", 0)
        x, i = op.solve(bg, x0.clone(), tol=1e-10, mask_bit=bit, mode=mode)
        op.set_param("one_launch", -1)
        op.set_param("meet_polls", 0)
        y, j = op.solve(bg, x0.clone(), tol=1e-10, mask_bit=bit, mode=mode)
        op.close()
        assert j.status == 0 and i.iterations == j.iterations and torch.equal(x, y)


def test_bad_values_refused(dev):
    from paper_1207_0486_amd.hns import HNSError
    op = _operator(basin.box_mesh(4, 4, 2), -1)
    for name, bad in (("one_launch", 1), ("one_launch", -2), ("meet_polls", -1),
                      ("meet_polls", 1 << 30), ("meet_polls", 0.5)):
        with pytest.raises(HNSError):
            op.set_param(name, bad)
    op.close()
